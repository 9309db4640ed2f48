// LR-shared attention, decode (one query token per request, or a chunk of a few
// whose (token, head) pairs per KV head fit 16 columns), gfx950.
//
// Reuse step of PreLRShared (Sec. 3.1): the current agent attends over the
// shared base cache plus its own rank-r LR cache.  Keys are rebuilt on chip,
// K = K_base + RoPE(L_k B_k), with the rank-r expansion done before RoPE
// (App. D.2).  Values use the associativity of App. D.2:
//     P (V_base + L_v B_v) = P V_base + (P L_v) B_v,
// so only an r-wide accumulator is carried per head and B_v is applied once,
// in the merge.
//
// Work split (flash-decoding): one workgroup per (request, KV-range split,
// group of up to 8 KV heads); one wavefront per KV head.  The waves of a
// workgroup walk the same tokens, so the RoPE cos/sin table of each 32-token
// tile is built once in LDS for all heads, and the per-token LR rows are read
// through shared L1 lines.  A second kernel merges the split partials with
// log-sum-exp weights.
//
// Per 16-token sub-block, each wave (lane l: query head l%16 of the group,
// q = l/16):
//   1. scores S^T = K Q^T on 16x16x32 MFMAs in two parts: the raw bf16
//      K_base rows (no rounding) plus bf16(RoPE(E)), where E^T = B_k^T L_k^T
//      comes from 16x16 MFMAs (16x16x32 over 32-rank chunks for ranks 32 and
//      64, 16x16x16 below) whose result layout holds both halves of every
//      RoPE pair in one lane;
//   2. online softmax per head (lane l%16), exp2 domain, lazily rescaled;
//   3. O^T += V^T P^T and (P L_v)^T += L_v^T P^T on 16x16x16 MFMAs.  V and
//      L_v rows pass through a wave-private LDS tile and come back through
//      the transposing LDS read (ds_read_b64_tr_b16), so P, already in B
//      operand layout, needs no shuffles and the softmax rescale is a
//      per-lane scalar.
// The loads of the next sub-block (the next two in the 4-wave rank-64
// kernel) are in flight while the current one is consumed.  The direct form of
// the rank-64 kernel at d = 128 (contiguous calls and long paged ones, one query
// token) sends its V rows straight to LDS (direct global->LDS loads into a
// two-buffer ring) instead of through registers.
#include "common.hpp"
#include "kernels.hpp"
#include "rebuild.hpp"

namespace prc {
namespace {

constexpr int TK = 32;        // tokens per KV tile (one LDS table, one barrier)
constexpr int NSB = TK / 16;  // 16-token sub-blocks per tile
constexpr float kRescaleLog2 = 8.f;  // lazy-rescale threshold (log2 domain)
constexpr int kMaxSplits = 1024;     // the merge holds one split per thread
// Waves per workgroup (one KV head each).  Rank 64 keeps its B_k^T
// fragments (64 VGPRs) in registers; with V staged in registers that needs
// one wave per SIMD (the whole register file, architected plus accumulation
// registers) to avoid spilling.
constexpr int dec_waves(int rank) { return rank >= 64 ? 4 : 8; }
// Sub-blocks whose loads are in flight ahead of the one being consumed.  With
// one wave per SIMD (rank 64) no other wave hides a wave's load latency, and
// the whole register file leaves room for one more staged sub-block; at two
// waves per SIMD the extra stage spills and loses.
constexpr int dec_prefetch(int rank) { return rank >= 64 ? 2 : 1; }
// Rank-64 decode at d = 128 instead stages its V rows by direct global->LDS
// loads, which frees the registers the V stages take: with one sub-block in
// flight it then fits in 256 registers (251), so it runs 8-wave workgroups,
// two waves per SIMD, like the lower ranks (64k, 8 requests: 467 -> 440 us).
// Paged calls take it too where it pays (decode_direct_paged) while their block
// tables are short enough for the split's entries to wait in LDS (a table read
// from memory between the stages would upset the fixed load count of the V wait
// below); the others, and several query tokens, keep the register-staged 4-wave
// form (`staged`).
// Eight paged requests of 65.5k tokens: 462 -> 426 us; of 36.8k-65.5k: 369 us,
// 410 with equal splits for each request, 345 with balanced ones (below); four
// of 3000: 43.8 -> 34.0 us.
constexpr bool dec_vdma(int d, int rank, bool staged) { return d == 128 && rank == 64 && !staged; }
constexpr int dec_nw(int d, int rank, bool staged) { return dec_vdma(d, rank, staged) ? 8 : dec_waves(rank); }
// Waves per SIMD the kernel is compiled for: two, except the register-staged
// rank-64 form at d = 128, which takes the whole register file for one.  At d =
// 64 it needs 256 registers, all of a wave's share at two: without the bound the
// compiler took 258, and eleven paged requests of 30000 tokens, one KV head, 98 us
// instead of 67.  (With several query tokens it needs more, and plans one
// workgroup per CU.)
constexpr int dec_occ(int d, int rank, bool staged, bool mt) {
  return rank >= 64 && (d == 128 || mt) && !dec_vdma(d, rank, staged) ? 1 : 2;
}
constexpr int kLdsBlocks = 2048;  // block-table entries of a split the direct paged form holds in LDS
constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }

template <int D, int R, bool VD = false>
struct Dec {
  static constexpr int NW = VD ? 8 : dec_waves(R);  // waves per workgroup (KV heads)
  static constexpr int NT = NW * 64;         // threads per workgroup
  static constexpr int HALF = D / 2;
  static constexpr int NB = D / 32;           // 16-dim blocks per RoPE half
  static constexpr int NBLK = D / 16;         // 16-dim blocks
  static constexpr int NCH = D / 32;          // 8-dim chunks per lane
  static constexpr int QPG = D / 8;           // dims per lane group per half
  static constexpr int RC = RCH(R);           // 16-wide rank chunks
  // float2 per table row.  A lane reads row l%16 at frequencies from
  // (l/16)*QPG; with an odd row length (d = 128) the 32 lanes of each
  // half-wave pass then cover all 64 banks once.
  static constexpr int CS_ROW = D == 128 ? HALF + 1 : HALF + 2;
  static constexpr int EPT = TK * HALF / NT;  // table entries per thread
  // Row strides of the tiles read with ds_read_b64_tr_b16: the two 16-lane
  // groups serviced together read 8 consecutive rows of 32 bytes, which land
  // on disjoint banks when the stride is an odd multiple of 8 dwords mod 64.
  static constexpr int V_ROW = D + 16;                          // 72 / 40 dwords
  static constexpr int LV_ROW = RC == 1 ? 16 : (RC == 2 ? 48 : 80);  // 8 / 24 / 40 dwords
  static constexpr int LPR = D / 8;           // lanes per V row (16 bytes each)
  static constexpr int RPL = 64 / LPR;        // V rows per wave load
  static constexpr int NVL = 16 / RPL;        // V loads per sub-block
  static constexpr int PS = 4 + D + R;        // floats per split partial
  static constexpr int PF = VD ? 1 : dec_prefetch(R);  // sub-blocks loaded ahead
  static constexpr int NST = PF + 1;          // staged sub-blocks (a ring)
  static constexpr int TPR = NST / gcd_c(NST, NSB);  // tiles per whole number of turns of the ring
  // Direct-to-LDS V staging: a stage is the 16 V rows at the padded row
  // stride V_ROW, written by NVD 1 KB loads (lane i of load k lands at byte
  // 1024 k + 16 i; lanes that fall in a row's padding or past the last row
  // load nothing).  VST: bf16 per stage buffer.
  static constexpr int NVD = (16 * V_ROW * 2 + 1023) / 1024;
  static constexpr int VST = NVD * 512;
};

// Keys request r's query may see: t < kv_len (clamped into the buffer) and
// t <= the query's position.
__device__ __forceinline__ int visible_keys(const AttnArgs& a, int r) {
  int64_t kvl = a.kv_len[r];
  kvl = kvl < 0 ? 0 : (kvl > a.s_cap ? a.s_cap : kvl);
  const int64_t pos = a.positions[(int64_t)r * a.n_tok];
  const int64_t vis = pos + 1 < kvl ? pos + 1 : kvl;
  return vis < 0 ? 0 : (int)vis;
}
// The same for a request of several query tokens (at most 16): lane l reads its
// own column's token; returns the furthest end, `mine` this lane's.
__device__ __forceinline__ int request_visible_keys(const AttnArgs& a, int b, int tok, int& mine) {
  int64_t kvl = a.kv_len[b];
  kvl = kvl < 0 ? 0 : (kvl > a.s_cap ? a.s_cap : kvl);
  const int64_t pos = a.positions[(int64_t)b * a.n_tok + tok];
  const int64_t v = pos + 1 < kvl ? pos + 1 : kvl;
  mine = v < 0 ? 0 : (int)v;
  int vis = mine;
#pragma unroll
  for (int x = 1; x < 16; x <<= 1) vis = max(vis, __shfl_xor(vis, x, 64));
  return __builtin_amdgcn_readfirstlane(vis);
}
// KV tiles per split over `vis` visible keys.  The host plan sizes the grid
// and the workspace for the caches' capacity (it cannot read kv_len); the
// splits themselves divide the keys in use, so a cache reserved far beyond
// its current length still spreads over all the planned workgroups.  Splits
// at or past the end have no work and write no partial.  (One request, 12345
// of 65920 tokens, 8 KV heads, rank 16: kernel 31.0 us with splits of the
// capacity, which leave 43 of 229 workgroups with work, 14.7 us with these.)
__device__ __forceinline__ int tiles_per_split(int vis, int n_splits) {
  const int st = ((vis + TK - 1) / TK + n_splits - 1) / n_splits;
  return st < 1 ? 1 : st;
}
// The furthest end among the requests whose splits cover the same ranges
// (one request, or the dec_group <= kMaxGroup requests of a shared-base
// workgroup).  Lane i reads request i's length and position, so the reads run
// side by side; `mine` receives its visible keys (0 past the group or the batch).
constexpr int kMaxGroup = 8;  // a power of two: the lanes the maximum is taken over
__device__ __forceinline__ int group_visible_keys(const AttnArgs& a, int b, int grp, int lane, int& mine) {
  const int r = b / grp * grp + lane;
  mine = lane < grp && r < a.batch ? visible_keys(a, r) : 0;
  int vis = mine;
#pragma unroll
  for (int x = 1; x < kMaxGroup; x <<= 1) vis = max(vis, __shfl_xor(vis, x, 64));
  return __builtin_amdgcn_readfirstlane(vis);
}

// Splits of one length over all requests of a batch (at most 64: lane r holds
// request r), so that requests of different lengths take workgroups in
// proportion to their keys: the smallest tiles-per-split for which all splits
// fit a.wg_total workgroups and each request's fit its a.n_splits places in the
// workspace.  Every workgroup, and the merge, derive the same cut from the
// lengths.  Returns tiles per split; `mine` is lane r's number of splits.
// (Eight requests of 36.8k-65.5k tokens, rank 64, one round of workgroups:
// 409 us with as many splits for each request, 342 us so; sixteen of 5k-20k,
// paged: 273 -> 187 us; equal lengths are cut as before.)
__device__ __forceinline__ int balanced_splits(const AttnArgs& a, int lane, int& mine) {
  // Over the lanes that hold requests (the next power of two of them).
  auto sum64 = [&](int v) {
    for (int x = 1; x < a.batch; x <<= 1) v += __shfl_xor(v, x, 64);
    return __builtin_amdgcn_readfirstlane(v);
  };
  const int tiles = lane < a.batch ? max(1, (visible_keys(a, lane) + TK - 1) / TK) : 0;
  int longest = tiles;
  for (int x = 1; x < a.batch; x <<= 1) longest = max(longest, __shfl_xor(longest, x, 64));
  longest = __builtin_amdgcn_readfirstlane(longest);
  const int total = sum64(tiles);
  int st = max((total + a.wg_total - 1) / a.wg_total, (longest + a.n_splits - 1) / a.n_splits);
  // Rounding up leaves at most one split per request too many: a step of 1/32
  // reaches a fit within a few turns (wg_total is at least twice the batch).
  for (;;) {
    mine = (tiles + st - 1) / st;
    if (sum64(mine) <= a.wg_total) break;
    st += st < 64 ? 1 : st / 32;
  }
  return st;
}

// Transposing LDS read: lane j of each 16-lane group points at 4 consecutive
// bf16; lane i receives element i%4 of lanes i/4, i/4+4, i/4+8, i/4+12.
__device__ __forceinline__ i16x4 lds_read_tr(const uint16_t* p) {
  typedef short v4s __attribute__((ext_vector_type(4)));
  v4s v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((v4s __attribute__((address_space(3)))*)(p));
  return __builtin_bit_cast(i16x4, v);
}

template <int D, int R>
struct Stage {
  u32x4 kb[D / 32];                         // K_base chunks of token l%16
  typename Ex<R>::Frag lk[Ex<R>::NC];       // L_k row fragments of token l%16 (expansion B operand)
  u32x4 v[Dec<D, R>::NVL];                  // V rows, natural layout
  u32x2 lv[RCH(R)];                         // L_v row fragment of token l%16
};

// Buffer resource over `bytes` bytes from `base` (raw, stride 0): loads at
// offsets at or past the end return zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const uint16_t* base, int32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), (short)0, bytes, 0x00020000);
}

// Per-lane byte offsets of one 16-token sub-block's data (constant over the
// kernel): the sub-block itself is addressed by resources built per
// sub-block, whose range check zero-fills tokens at or past the split end.
// The loads are branch-free, so the compiler can keep the next sub-block's
// loads in flight while the current one is consumed.
template <int D, int R>
struct StageOffsets {
  int32_t kb[D / 32], lk[Ex<R>::NC], lr[RCH(R)], v[Dec<D, R>::NVL], vd[Dec<D, R>::NVD];
};

template <int D, int R, bool VD>
__device__ __forceinline__ StageOffsets<D, R> stage_offsets(int64_t row, int lane) {
  using C = Dec<D, R>;
  StageOffsets<D, R> o;
  const int c16 = lane & 15, q = lane >> 4;
#pragma unroll
  for (int kk = 0; kk < C::NCH; ++kk) o.kb[kk] = c16 * (int32_t)(row * 2) + chunk_dim<D>(kk, q) * 2;
#pragma unroll
  for (int rc = 0; rc < C::RC; ++rc) {
    const int r0 = rc * 16 + q * 4;
    o.lr[rc] = r0 < R ? c16 * R * 2 + r0 * 2 : INT32_MIN;  // ranks past r read as zeros
  }
#pragma unroll
  for (int c = 0; c < Ex<R>::NC; ++c) {
    const int r0 = Ex<R>::rank0(c, q);
    o.lk[c] = r0 < R ? c16 * R * 2 + r0 * 2 : INT32_MIN;
  }
  const int vrow = lane / C::LPR, vdim = (lane % C::LPR) * 8;
  if constexpr (VD) {
#pragma unroll
    for (int k = 0; k < C::NVD; ++k) {
      const int byte = 1024 * k + 16 * lane, t = byte / (2 * C::V_ROW), in_row = byte % (2 * C::V_ROW);
      o.vd[k] = (t < 16 && in_row < 2 * D) ? t * (int32_t)(row * 2) + in_row : INT32_MIN;
    }
  } else {
#pragma unroll
    for (int iv = 0; iv < C::NVL; ++iv) o.v[iv] = (vrow + C::RPL * iv) * (int32_t)(row * 2) + vdim * 2;
  }
  return o;
}

// One expansion fragment of an LR row through a buffer resource.
template <int R>
__device__ __forceinline__ typename Ex<R>::Frag lr_frag_load(__amdgpu_buffer_rsrc_t r, int32_t off) {
  if constexpr (Ex<R>::WIDE)
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
  else
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}

// VD: V goes straight to the stage buffer `vdst` in LDS (its rows at stride
// V_ROW), issued after the stage's other loads.
template <int D, int R, bool VD>
__device__ __forceinline__ void stage_load(Stage<D, R>& s, const StageOffsets<D, R>& o, const uint16_t* Kb,
                                           const uint16_t* Vb, const uint16_t* Lk, const uint16_t* Lv,
                                           int64_t kv_row, int64_t lr_row, int64_t row, int64_t t0,
                                           int64_t t_end, uint16_t* vdst) {
  using C = Dec<D, R>;
  // Valid tokens of the sub-block (none past the end: every load reads zeros).
  const int64_t n = t_end - t0 < 0 ? 0 : (t_end - t0 < 16 ? t_end - t0 : 16);
  const int32_t kv_bytes = n > 0 ? (int32_t)((n - 1) * row * 2 + D * 2) : 0;
  // kv_row / lr_row: cache rows of token t0 (t0 itself unless paged).
  const auto rk = make_rsrc(Kb + kv_row * row, kv_bytes);
  const auto rv = make_rsrc(Vb + kv_row * row, kv_bytes);
  // Absent LR caches get empty resources (loads read zeros, touch nothing).
  const auto rlk = make_rsrc(Lk != nullptr ? Lk + lr_row * R : Kb, Lk != nullptr ? (int32_t)(n * R * 2) : 0);
  const auto rlv = make_rsrc(Lv != nullptr ? Lv + lr_row * R : Kb, Lv != nullptr ? (int32_t)(n * R * 2) : 0);
#pragma unroll
  for (int kk = 0; kk < C::NCH; ++kk)
    s.kb[kk] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, o.kb[kk], 0, 0));
#pragma unroll
  for (int c = 0; c < Ex<R>::NC; ++c) s.lk[c] = lr_frag_load<R>(rlk, o.lk[c]);
#pragma unroll
  for (int rc = 0; rc < C::RC; ++rc)
    s.lv[rc] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rlv, o.lr[rc], 0, 0));
  if constexpr (VD) {
#ifdef __HIP_DEVICE_COMPILE__  // the host pass does not know the 16-byte form
#pragma unroll
    for (int k = 0; k < C::NVD; ++k)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (__attribute__((address_space(3))) void*)(vdst + 512 * k), 16,
                                               o.vd[k], 0, 0, 0);
#endif
  } else {
#pragma unroll
    for (int iv = 0; iv < C::NVL; ++iv)
      s.v[iv] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rv, o.v[iv], 0, 0));
  }
}

// The paged walk over block-table entries in LDS: the entries of the block
// after the current one are read a block ahead.  Entries are clamped into the
// pools, indexes into the split's entries (past its end nothing is loaded).
struct LdsWalk {
  const int32_t *kv, *lr;
  int n, blk, kv_nblk, lr_nblk, q, rem;
  int ek, el;            // current block (wave-uniform)
  int32_t nk, nl;        // entries of the next
  __device__ __forceinline__ void enter() {
    ek = __builtin_amdgcn_readfirstlane(nk);
    el = __builtin_amdgcn_readfirstlane(nl);
    ek = ek < 0 ? 0 : (ek >= kv_nblk ? kv_nblk - 1 : ek);
    el = el < 0 ? 0 : (el >= lr_nblk ? lr_nblk - 1 : el);
    const int i = q + 1 < n ? q + 1 : 0;
    nk = kv[i];
    nl = lr[i];
  }
  __device__ __forceinline__ void start(const int32_t* kv_, const int32_t* lr_, int n_, int blk_, int kvn, int lrn, int rem_) {
    kv = kv_;
    lr = lr_;
    n = n_;
    blk = blk_;
    kv_nblk = kvn;
    lr_nblk = lrn;
    q = 0;
    rem = rem_;
    nk = nl = 0;
    if (n > 0) {
      nk = kv[0];
      nl = lr[0];
    }
    enter();
  }
  // Pool rows (base, LR) of the next sub-block's first token; then step on.
  __device__ __forceinline__ void next(int step, int64_t& kv_row, int64_t& lr_row) {
    kv_row = (int64_t)ek * blk + rem;
    lr_row = (int64_t)el * blk + rem;
    rem += step;
    if (rem == blk) {
      rem = 0;
      ++q;
      enter();
    }
  }
};

// s_waitcnt with vmcnt(n) and no wait on the other counters.
constexpr int vmcnt_imm(int n) { return (n & 0xF) | ((n >> 4) << 14) | 0x0F70; }
// Vector memory instructions one VD stage issues (K_base chunks, L_k
// fragments, L_v fragments, then the direct V loads).
template <int D, int R>
constexpr int kStageLoads = D / 32 + Ex<R>::NC + RCH(R) + Dec<D, R>::NVD;

// PAGED: the caches are pools reached through block tables (a separate
// instantiation, so the contiguous kernel carries none of the walk's state).
// MT: several query tokens per request, n_tok * G <= 16: column c of the score
// result is head c % G of token c / G, each with its own last visible key.
// (It always takes the register-staged form, so that contiguous and paged
// calls cut the same splits and agree bit for bit.)
template <int D, int R, bool PAGED, bool MT, bool STAGED = PAGED || MT>
__global__ void __launch_bounds__(dec_nw(D, R, STAGED) * 64, dec_occ(D, R, STAGED, MT))
lrsa_decode_kernel(const AttnArgs a) {
  constexpr bool VD = dec_vdma(D, R, STAGED);
  constexpr bool LW = PAGED && VD;  // the table walk reads LDS
  using C = Dec<D, R, VD>;
  constexpr int NW = C::NW, NT = C::NT;
  __shared__ float2 cs_lds[2][TK * C::CS_ROW];
  __shared__ float2 base_lds[2][C::HALF];
  // Per wave: the V tile written from registers, or (VD) the two V stage
  // buffers the direct loads fill, as separate arrays so that the compiler
  // can tell the LDS reads of one from the direct loads into the other.
  static_assert(!VD || C::NST == 2, "two V stage buffers");
  __shared__ __attribute__((aligned(16))) uint16_t v_lds[NW][VD ? C::VST : 16 * C::V_ROW];
  __shared__ __attribute__((aligned(16))) uint16_t v_lds1[VD ? NW : 1][VD ? C::VST : 8];
  __shared__ __attribute__((aligned(16))) uint16_t lv_lds[NW][16 * C::LV_ROW];
  __shared__ int32_t tbl_lds[2][LW ? kLdsBlocks : 1];  // this split's base and LR block-table entries

  // The wave index is made visibly wave-uniform, so that everything derived
  // from it (the KV head and its buffer resources) lives in scalar registers.
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int split = blockIdx.x, b = blockIdx.z, st_bal = 0;
  if (VD && a.wg_total > 0) {
    // Workgroup x takes the x-th split of the batch, request by request.
    int mine;
    st_bal = balanced_splits(a, lane, mine);
    int end = mine;  // splits of requests 0 .. lane
    for (int x = 1; x < a.batch; x <<= 1) {
      const int o = __shfl_up(end, x, 64);
      if (lane >= x) end += o;
    }
    const uint64_t past = __ballot(lane < a.batch && end <= (int)blockIdx.x);  // requests wholly before this workgroup
    b = __builtin_popcountll(past);
    if (b >= a.batch) return;  // uniform over the workgroup
    split = (int)blockIdx.x - (__builtin_amdgcn_readlane(end, b) - __builtin_amdgcn_readlane(mine, b));
  }
  const int g = blockIdx.y * NW + w;
  const bool active = g < a.n_kv;
  const int G = a.group;
  const int q = lane >> 4, c16 = lane & 15;
  const bool has_lk = a.Lk != nullptr, has_lv = a.Lv != nullptr;
  // The one-time loads go out first, then (below) the first stages' rows: a
  // split of a small batch covers only a few tiles, and each of these reads
  // behind another adds a memory latency to it.
  BtStage<D, R> bts;
  bts.issue(has_lk ? a.Bk + (int64_t)b * a.b_stride + (int64_t)g * D : nullptr, (int64_t)a.n_kv * D,
            has_lk && active, lane);

  const int n_col = MT ? a.n_tok * G : G;       // columns in use
  const int tok = MT && c16 < n_col ? c16 / G : 0;  // this lane's query token
  // Q^T of the group as the B operand (cols = q heads, zero past G).
  bf16x8 qf[C::NCH];
  {
    const bool ok = active && c16 < n_col;
    const uint16_t* qp = a.Q + (((int64_t)b * a.n_tok + tok) * a.n_q + (int64_t)g * G + (MT ? c16 - tok * G : c16)) * D;
#pragma unroll
    for (int kk = 0; kk < C::NCH; ++kk) qf[kk] = as_bf16x8(ld16(qp + chunk_dim<D>(kk, q), ok));
  }
  // This thread's frequency: of its table entries and of the base angles.
  static_assert(NT % C::HALF == 0, "one frequency per thread");
  const double w2pi_t = a.w2pi[tid % C::HALF];
  // This split's share of the keys the request may see.
  int vis_col = 0;                              // keys this lane's column may see (MT)
  const int vis = MT ? request_visible_keys(a, b, tok, vis_col) : visible_keys(a, b);
  const int st_tiles = VD && a.wg_total > 0 ? st_bal : tiles_per_split(vis, a.n_splits);
  const int64_t t_begin = (int64_t)split * st_tiles * TK;
  if (split > 0 && t_begin >= vis) return;  // past the end (uniform over the workgroup)
  int64_t t_end = t_begin + (int64_t)st_tiles * TK;
  if (t_end > vis) t_end = vis;
  const int64_t t_end_col = MT && vis_col < t_end ? vis_col : t_end;
  const int n_tiles = t_end > t_begin ? (int)((t_end - t_begin + TK - 1) / TK) : 0;

  const int64_t row = (int64_t)a.n_kv * D;  // elements between tokens
  // This request's caches (or pools, paged through its rows of the block
  // tables).
  const uint16_t* Kb = a.Kb + (int64_t)b * a.kv_stride + (int64_t)g * D;
  const uint16_t* Vb = a.Vb + (int64_t)b * a.kv_stride + (int64_t)g * D;
  const uint16_t* Lk = has_lk ? a.Lk + (int64_t)b * a.l_stride : nullptr;
  const uint16_t* Lv = has_lv ? a.Lv + (int64_t)b * a.l_stride : nullptr;
  const int64_t t_end_w = active ? t_end : t_begin;  // inactive waves load nothing

  uint16_t* vl = v_lds[w];
  uint16_t* lvl = lv_lds[w];
  const StageOffsets<D, R> so = stage_offsets<D, R, VD>(row, lane);
  Stage<D, R> st[C::NST];
  // Sub-blocks are loaded in token order, so paged caches are walked with them.
  PageWalk walk;
  LdsWalk lwalk;
  if constexpr (LW) {
    const int q0 = (int)(t_begin / a.blk), nq = t_end > t_begin ? (int)((t_end - 1) / a.blk) - q0 + 1 : 0;
    for (int i = tid; i < nq; i += NT) {
      tbl_lds[0][i] = a.kv_tbl[(int64_t)b * a.max_blk + q0 + i];
      tbl_lds[1][i] = a.lr_tbl[(int64_t)b * a.max_blk + q0 + i];
    }
    __syncthreads();
    lwalk.start(tbl_lds[0], tbl_lds[1], nq, a.blk, a.kv_nblk, a.lr_nblk, (int)(t_begin - (int64_t)q0 * a.blk));
  } else if constexpr (PAGED) {
    walk.start(a.kv_tbl + (int64_t)b * a.max_blk, a.lr_tbl + (int64_t)b * a.max_blk, a.max_blk, a.blk, a.kv_nblk,
               a.lr_nblk, t_begin, t_end_w);
  }
  // Stage `slot` of the ring (VD: also its V buffer in LDS).
  auto load = [&](Stage<D, R>& s, int64_t t, int slot) {
    int64_t kr = t, lr = t;
    if constexpr (LW) lwalk.next(16, kr, lr);
    else if constexpr (PAGED) walk.next(16, t_end_w, kr, lr);
    stage_load<D, R, VD>(s, so, Kb, Vb, Lk, Lv, kr, lr, row, t, t_end_w, slot == 0 ? vl : v_lds1[VD ? w : 0]);
  };
  if constexpr (!VD) {  // (direct V loads wait until their buffers are free and zeroed)
#pragma unroll
    for (int p = 0; p < C::PF; ++p) load(st[p], t_begin + 16 * p, p);
    __builtin_amdgcn_sched_barrier(0);
  }

  // RoPE table entries this thread builds every tile, by angle addition from
  // the exact base angle of the tile and exact per-entry offset angles.
  float cdl[C::EPT], sdl[C::EPT];
  int ej[C::EPT], eidx[C::EPT];
#pragma unroll
  for (int k = 0; k < C::EPT; ++k) {
    const int e = tid + NT * k, tok = e / C::HALF;
    ej[k] = e - tok * C::HALF;
    eidx[k] = tok * C::CS_ROW + ej[k];
    cdl[k] = 1.f;
    sdl[k] = 0.f;
    if (has_lk) rope_cs(tok, w2pi_t, cdl[k], sdl[k]);
  }
  if (has_lk && tid < C::HALF && n_tiles > 0) {
    float c, s;
    rope_cs((int)t_begin, w2pi_t, c, s);
    base_lds[0][tid] = make_float2(c, s);
  }
  // L_v tile columns past the rank stay zero (rank 8 pads to 16).
  for (int i = lane; i < 16 * C::LV_ROW; i += 64) lv_lds[w][i] = 0;

  typename Ex<R>::Frag bkf[C::NBLK][Ex<R>::NC];
  bts.finish(bkf, v_lds[w], lane);
  if constexpr (VD) {
    // The stage buffers start as zeros (finite rows for tokens past the end,
    // whatever the direct loads do at out-of-range offsets), written before
    // the first direct load is issued.
    for (int i = lane; i < C::VST / 8; i += 64) {
      *reinterpret_cast<u32x4*>(v_lds[w] + 8 * i) = u32x4{0u, 0u, 0u, 0u};
      *reinterpret_cast<u32x4*>(v_lds1[VD ? w : 0] + 8 * i) = u32x4{0u, 0u, 0u, 0u};
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  }

  float m_run = -INFINITY, l_part = 0.f;
  f32x4 acc[C::NBLK];   // O^T: dims blk*16 + 4q + i, head l%16
  f32x4 accl[C::RC];    // (P L_v)^T: rank rc*16 + 4q + i, head l%16
#pragma unroll
  for (int blk = 0; blk < C::NBLK; ++blk) acc[blk] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int rc = 0; rc < C::RC; ++rc) accl[rc] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int vrow = lane / C::LPR, vdim = (lane % C::LPR) * 8;
  // Transposing-read addresses: lane j of group l/16 reads row
  // 4*(l/16) + (j/4), columns 4*(j%4) .. +3 of a 16-column block.
  const int tr_row = 4 * q + (c16 >> 2), tr_col = 4 * (c16 & 3);

  if constexpr (VD) {
#pragma unroll
    for (int p = 0; p < C::PF; ++p) load(st[p], t_begin + 16 * p, p);
  }

  __syncthreads();  // base angles of the first tile, zeroed L_v tiles

  // RoPE table of tile k (from its base angles in base_lds[k & 1]) into
  // cs_lds[k & 1], and the base angles of tile k + 1 into base_lds[(k + 1) & 1].
  // Tile 0's here; each later one while the tile before it runs, beside that
  // tile's first loads, so that the barrier at the head of a tile has no
  // table work in front of it.
  auto build_table = [&](int k) {
    float2* csk = cs_lds[k & 1];
    const float2* base = base_lds[k & 1];
#pragma unroll
    for (int e = 0; e < C::EPT; ++e) {
      const float2 bc = base[ej[e]];
      csk[eidx[e]] = make_float2(bc.x * cdl[e] - bc.y * sdl[e], bc.y * cdl[e] + bc.x * sdl[e]);
    }
    if (tid < C::HALF && k + 1 < n_tiles) {
      float c, sn;
      rope_cs((int)(t_begin + (int64_t)(k + 1) * TK), w2pi_t, c, sn);
      base_lds[(k + 1) & 1][tid] = make_float2(c, sn);
    }
  };
  if (has_lk && n_tiles > 0) build_table(0);

  // The tile loop is unrolled by the tiles of one turn of the stage ring, so
  // that every stage index is a constant.  Inside it every path issues the
  // same loads (inactive waves and sub-blocks past the split end load zeros
  // and compute on them), and the only early exit leaves the loop for good:
  // the compiler's load counting then sees the same loads in flight on every
  // path and waits for no stage before it is needed.
  for (int tile0 = 0; tile0 < n_tiles; tile0 += C::TPR)
#pragma unroll
  for (int tt = 0; tt < C::TPR; ++tt) {
    const int tile = tile0 + tt;
    if (tile >= n_tiles) goto tiles_done;  // uniform over the workgroup
    const int64_t t0 = t_begin + (int64_t)tile * TK;
    float2* cs = cs_lds[tile & 1];
    __syncthreads();  // this tile's table and the next tile's base angles are
                      // ready, and every wave is done with the previous tile
                      // (whose table buffer the next table goes into).

#pragma unroll
    for (int sb = 0; sb < NSB; ++sb) {
      const int cslot = (tt * NSB + sb) % C::NST, nslot = (tt * NSB + sb + C::PF) % C::NST;
      Stage<D, R>& cur = st[cslot];
      Stage<D, R>& nxt = st[nslot];
      // A sub-block past the split end (only in its last tile) holds zeros
      // and no visible key: all its weights are exactly 0 and the running
      // maximum does not move, so it changes nothing.
      const int64_t ts = t0 + sb * 16;
      // Issue the loads of the sub-block PF ahead before consuming this one
      // (past the split end they read zeros and touch no memory).
      load(nxt, ts + 16 * C::PF, nslot);
      // Keep the loads ahead of this sub-block's work: the scheduler would
      // otherwise sink them to shorten their registers' live ranges, and the
      // wait for this stage would then also wait for the next one.
      __builtin_amdgcn_sched_barrier(0);
      // The next tile's table, while this sub-block's data is still landing.
      if (sb == 0 && has_lk && tile + 1 < n_tiles) build_table(tile + 1);

      // ---- V and L_v rows into the wave's LDS tile ------------------------
      if constexpr (!VD) {
#pragma unroll
        for (int iv = 0; iv < C::NVL; ++iv)
          *reinterpret_cast<u32x4*>(vl + (vrow + C::RPL * iv) * C::V_ROW + vdim) = cur.v[iv];
      }
      if (has_lv) {
#pragma unroll
        for (int rc = 0; rc < C::RC; ++rc)
          if (rc * 16 + q * 4 < R) *reinterpret_cast<u32x2*>(lvl + c16 * C::LV_ROW + rc * 16 + q * 4) = cur.lv[rc];
      }

      // ---- scores S^T = K_base Q^T + bf16(RoPE(E)) Q^T --------------------
      f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < C::NCH; ++kk) sc = mfma16x16x32(as_bf16x8(cur.kb[kk]), qf[kk], sc);
      if (has_lk) {
        const float2* csr = cs + (sb * 16 + c16) * C::CS_ROW + q * C::QPG;
        u32x4 ek[C::NCH];
#pragma unroll
        for (int blk = 0; blk < C::NB; ++blk) {
          f32x4 elo = {0.f, 0.f, 0.f, 0.f}, ehi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < Ex<R>::NC; ++c) {
            elo = Ex<R>::mma(bkf[blk][c], cur.lk[c], elo);
            ehi = Ex<R>::mma(bkf[blk + C::NB][c], cur.lk[c], ehi);
          }
          float rlo[4], rhi[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float2 r = csr[blk * 4 + i];
            rlo[i] = elo[i] * r.x - ehi[i] * r.y;
            rhi[i] = ehi[i] * r.x + elo[i] * r.y;
          }
          const int klo = blk >> 1, khi = (blk + C::NB) >> 1, w0 = (blk & 1) * 2;
          ek[klo][w0] = pack_bf16(rlo[0], rlo[1]);
          ek[klo][w0 + 1] = pack_bf16(rlo[2], rlo[3]);
          ek[khi][w0] = pack_bf16(rhi[0], rhi[1]);
          ek[khi][w0 + 1] = pack_bf16(rhi[2], rhi[3]);
        }
#pragma unroll
        for (int kk = 0; kk < C::NCH; ++kk) sc = mfma16x16x32(as_bf16x8(ek[kk]), qf[kk], sc);
      }

      // ---- online softmax: lane l%16 is a head, 4 tokens per lane ---------
      float s2[4];
      float mx = -INFINITY;
      const int64_t left = t_end_col - ts;  // visible tokens from ts on
      const int n_vis = left < 0 ? 0 : (left < 16 ? (int)left : 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s2[i] = (q * 4 + i < n_vis) ? sc[i] * a.scale_log2 : -INFINITY;
        mx = fmaxf(mx, s2[i]);
      }
      mx = max_xor32(max_xor16(mx));
      // Lazy rescale: a head's reference maximum m_run only moves when a
      // score exceeds it by more than 2^8 (P stays below 256), so the
      // accumulators are rescaled a few times per split, not per sub-block.
      if (__ballot(mx > m_run + kRescaleLog2)) {
        const float mn = fmaxf(m_run, mx);
        const float alpha = fast_exp2(m_run - (mn == -INFINITY ? 0.f : mn));
#pragma unroll
        for (int blk = 0; blk < C::NBLK; ++blk) acc[blk] *= alpha;
#pragma unroll
        for (int rc = 0; rc < C::RC; ++rc) accl[rc] *= alpha;
        l_part *= alpha;
        m_run = mn;
      }
      const float ms = (m_run == -INFINITY) ? 0.f : m_run;
      float p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = fast_exp2(s2[i] - ms);
      l_part += (p[0] + p[1]) + (p[2] + p[3]);
      u32x2 pw;
      pw[0] = pack_bf16(p[0], p[1]);
      pw[1] = pack_bf16(p[2], p[3]);
      const i16x4 pb = as_i16x4(pw);
      __builtin_amdgcn_wave_barrier();

      // ---- O^T += V^T P^T, (P L_v)^T += L_v^T P^T -----------------------
      const uint16_t* vcur = vl;
      if constexpr (VD) {
        // This stage's direct V loads have landed once at most the loads of
        // the next stage, issued after them, are still in flight (the
        // counter drains in issue order; the sched barrier keeps the LDS
        // reads below the wait).
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(kStageLoads<D, R>));
        __builtin_amdgcn_sched_barrier(0);
        vcur = cslot == 0 ? vl : v_lds1[VD ? w : 0];
      }
#pragma unroll
      for (int blk = 0; blk < C::NBLK; ++blk)
        acc[blk] = mfma16x16x16(lds_read_tr(vcur + tr_row * C::V_ROW + blk * 16 + tr_col), pb, acc[blk]);
      if (has_lv) {
#pragma unroll
        for (int rc = 0; rc < C::RC; ++rc)
          accl[rc] = mfma16x16x16(lds_read_tr(lvl + tr_row * C::LV_ROW + rc * 16 + tr_col), pb, accl[rc]);
      }
      __builtin_amdgcn_wave_barrier();
    }
  }

tiles_done:
  // Direct loads past the split end may still be in flight: let them land
  // before the wave (and with the last wave, the workgroup's LDS) retires.
  if constexpr (VD) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  if (!active) return;
  // One partial per (request, q head, split): lane l%16 is the head; lanes
  // l, l^16, l^32, l^48 share it and hold different dims of O^T.
  l_part += shfl_xor(l_part, 16);
  l_part += shfl_xor(l_part, 32);
  if (c16 >= n_col) return;
  const int64_t hstride = (int64_t)a.n_splits * C::PS;
  float* wsb = a.ws + (((int64_t)b * a.n_tok + tok) * a.n_q + (int64_t)g * G + (MT ? c16 - tok * G : c16)) * hstride +
               (int64_t)split * C::PS;
  if (q == 0) {
    wsb[0] = m_run;
    wsb[1] = l_part;
  }
#pragma unroll
  for (int blk = 0; blk < C::NBLK; ++blk)
    *reinterpret_cast<f32x4*>(wsb + 4 + blk * 16 + q * 4) = acc[blk];
  if (has_lv) {
#pragma unroll
    for (int rc = 0; rc < C::RC; ++rc)
      if (rc * 16 + q * 4 < R) *reinterpret_cast<f32x4*>(wsb + 4 + D + rc * 16 + q * 4) = accl[rc];
  }
}

// Splits of request b that wrote partials: decode splits past the request's
// (shared base: its group's) last key do not exist; a prefill writes them all.
__device__ __forceinline__ int splits_written(const AttnArgs& a, int b) {
  if (a.dec_group == 0) return a.n_splits;
  int mine;
  const int lane = threadIdx.x & 63;
  if (a.wg_total > 0) {
    balanced_splits(a, lane, mine);
    return __builtin_amdgcn_readlane(mine, b);
  }
  const int vis = a.n_tok > 1      ? request_visible_keys(a, b, (lane & 15) < a.n_tok ? lane & 15 : 0, mine)
                  : a.dec_group == 1 ? visible_keys(a, b)
                                     : group_visible_keys(a, b, a.dec_group, lane, mine);
  const int tiles = (vis + TK - 1) / TK, st = tiles_per_split(vis, a.n_splits);
  const int ns = (tiles + st - 1) / st;
  return ns < 1 ? 1 : ns;
}

// Merge the split partials of one (request, query token, q head):
// log-sum-exp weights, then the deferred up-projection
// O += (sum_s w_s P_s L_v) B_v, then 1/l.  Decode has one query token per
// request; a split prefill has n_tok.
// A row's partials are n_splits x (d + r) fp32 beside their maxima and sums.
// Thread s holds split s's maximum and sum (loaded before the number of
// splits in use is known: that read runs beside it) and leaves its weight in
// LDS.  Thread t owns float4 column t % NV of the d + r accumulators for the
// splits congruent to t / NV modulo the number of such groups, so a
// workgroup keeps one independent 16-byte load per thread and split group
// in flight; the groups' sums then meet in LDS.  Rows with many splits
// (small decode batches) take 16-wave workgroups, rows with few 4-wave ones.
// The chain of dependent reads bounds it: the up-projection column of each
// output dim is read at the start, beside the partials.
template <int D, int R, int MW>
__global__ void __launch_bounds__(64 * MW)
lrsa_merge_kernel(const AttnArgs a) {
  constexpr int PS = 4 + D + R, NT = 64 * MW;
  constexpr int NV = (D + R) / 4;  // float4 columns of the accumulators
  constexpr int NG = NT / NV;      // split groups
  static_assert(NT >= D, "one thread per head dim");
  __shared__ float red[NG][D + R];
  __shared__ float red_w[MW][2];
  __shared__ float wgt[NT];
  __shared__ float fin[D + R];
  const int h = blockIdx.x, bi = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int b = bi / a.n_tok;  // bi = request * n_tok + query token
  const int g = h / a.group;
  const bool has_lv = a.Lv != nullptr;
  const int64_t orow = (int64_t)bi * a.n_q + h;  // (request, token, head) row of O
  const float* base = a.ws + orow * (int64_t)a.n_splits * PS;

  // One split per thread (n_splits <= NT by the launch rule).
  f32x2 ml = {-INFINITY, 0.f};
  if (tid < a.n_splits) ml = *reinterpret_cast<const f32x2*>(base + (int64_t)tid * PS);
  uint16_t bv[R];
  if (has_lv && tid < D) {
    // B_v [r, n_kv*d]: rank j of this thread's head dim, coalesced over the threads.
    const uint16_t* bp = a.Bv + (int64_t)b * a.b_stride + (int64_t)g * D + tid;
    const int64_t ldb = (int64_t)a.n_kv * D;
#pragma unroll
    for (int j = 0; j < R; ++j) bv[j] = bp[j * ldb];
  }
  const int ns = splits_written(a, b);
  if (tid >= ns) ml = f32x2{-INFINITY, 0.f};

  // Global maximum over the splits, then each split's weight and the row sum
  // L = sum_s w_s l_s.
  float M = ml[0];
#pragma unroll
  for (int x = 1; x < 64; x <<= 1) M = fmaxf(M, shfl_xor(M, x));
  if (lane == 0) red_w[w][0] = M;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MW; ++i) M = fmaxf(M, red_w[i][0]);
  const float Ms = (M == -INFINITY) ? 0.f : M;
  const float w_s = fast_exp2(ml[0] - Ms);
  wgt[tid] = w_s;
  float L = w_s * ml[1];
#pragma unroll
  for (int x = 1; x < 64; x <<= 1) L += shfl_xor(L, x);
  if (lane == 0) red_w[w][1] = L;
  __syncthreads();

  // Weighted accumulators (d of P V, r of P L_v), one float4 column per thread.
  const int grp = tid / NV, v = tid - grp * NV;
  const int nv_used = has_lv ? NV : D / 4;
  if (grp < NG && v < nv_used) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int s = grp; s < ns; s += NG) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(base + (int64_t)s * PS + 4 + 4 * v);
      const float ww = wgt[s];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] += ww * x[c];
    }
    *reinterpret_cast<f32x4*>(&red[grp][4 * v]) = acc;
  }
  __syncthreads();
  for (int c = tid; c < D + R; c += NT) {
    float t = 0.f;
    if (c < D || has_lv)
      for (int i = 0; i < NG; ++i) t += red[i][c];
    fin[c] = t;
  }
  L = 0.f;
#pragma unroll
  for (int i = 0; i < MW; ++i) L += red_w[i][1];
  __syncthreads();

  // O = (acc + (sum_s w_s P_s L_v) B_v) / L, one head dim per thread.
  const float inv = L > 0.f ? 1.f / L : 0.f;
  uint16_t* o = a.O + orow * D;
  if (tid < D) {
    float sum = fin[tid];
    if (has_lv) {
#pragma unroll
      for (int j = 0; j < R; ++j) sum += fin[D + j] * __uint_as_float((uint32_t)bv[j] << 16);
    }
    const uint32_t pk = pack_bf16(sum * inv, 0.f);
    o[tid] = (uint16_t)(pk & 0xffffu);
  }
  if (a.lse != nullptr && tid == 0)
    a.lse[orow] = L > 0.f ? (M + __log2f(L)) * kLn2 : -INFINITY;
}

// ---------------------------------------------------------------------------
// Decode over one base cache shared by every request (kv_req_stride == 0):
// several agents' queries over the same trajectory, each with its own LR
// plane, up-projections, query and position.  The heads of RPB requests fill
// the 16 columns of one MFMA result (column c: request c / G, head c % G), so
// a wave scores, softmaxes and weights each 16-token sub-block of the base
// once for all of them; only the key expansion RoPE(L_k B_k) and P L_v run
// per request.
//
// One workgroup per (split, KV head, up to sh_groups(R) groups of RPB
// requests): each group has SH_W / n_grp waves, which take the split's
// sub-blocks in turn (stream s: sub-blocks s, s + n_str, ...), keep their own
// running softmax and combine through LDS at the end, so nothing in the loop
// waits for another wave.  The B_k^T fragments of all the workgroup's requests
// wait in LDS.  The partials go to the same workspace and the same merge.
//
// Eight agents over 32k tokens, 8 KV heads, rank 16: 90 us per call with one
// request per wave (12 of 16 columns empty, softmax and P V repeated per
// request), 66 us with four.  What is left is vector work: about 510 vector
// instructions per sub-block of four requests, 336 of them the rotation of
// the expansions, at two waves per SIMD half of the cycles.  Measured and no
// better: two sub-blocks of loads in flight (256 registers; 72 us), base rows
// shared by the groups through LDS with a barrier per sub-block (75 us,
// though without key LR, where memory bounds it, 55 -> 48 us), two rounds of
// workgroups (84 us: the fixed cost of a workgroup, about 8 us of dependent
// reads at its start and the combine at its end, is paid twice).
constexpr int SH_W = 8;                                           // waves per workgroup
constexpr int sh_groups(int rank) { return rank >= 64 ? 1 : 2; }  // request groups per workgroup (B_k in LDS: 64 KB at most)
// Requests whose heads share the 16 columns: what fits, but at most 4 (more
// would only lengthen the per-request part of a sub-block), and no more than it
// takes for as few workgroups: the empty slots of a last one cost the others
// their time (8 requests, group 5, 14123 tokens, two workgroups of two groups of 3
// / 2: rank 16 47.3 / 40.2 us, values only 34.7 / 32.2; 6 of 32768, group 4, one
// workgroup of two groups of 4 / 3: 60.7 / 53.6).
constexpr int sh_rpb_most(int group) { return group <= 4 ? 4 : (group == 5 ? 3 : 2); }
inline int sh_rpb(int64_t batch, int group, int rank) {
  const int most = sh_rpb_most(group);
  const auto wgs = [&](int rpb) {
    const int64_t rq = rpb * (batch > rpb ? sh_groups(rank) : 1);
    return (batch + rq - 1) / rq;
  };
  for (int r = batch < most ? (int)batch : 2; r < most; ++r)
    if (wgs(r) == wgs(most) && (batch > most || batch <= r)) return r;
  return most;
}

template <int D, int R, int RPB>
__global__ void __launch_bounds__(SH_W * 64, 2)
lrsa_decode_shared_kernel(const AttnArgs a, int n_grp) {
  using C = Dec<D, R>;
  using Frag = typename Ex<R>::Frag;
  constexpr int SB = 16, NTH = SH_W * 64, NC = Ex<R>::NC;
  constexpr int NBF = C::NBLK * NC * 64;  // B_k^T fragments of one request
  // LDS: B_k^T fragments, V and L_v tiles, RoPE offsets and base angles; the
  // streams' partials reuse it after the loop.
  constexpr int kBk = sh_groups(R) * RPB * NBF * (int)sizeof(Frag);
  // L_v tiles: one per request up to rank 16, so that all are written with V
  // at the head of a sub-block; above, one that the requests use in turn.
  constexpr int NLT = R <= 16 ? RPB : 1, LVT = 16 * C::LV_ROW;
  // P L_v of every column with each request's L_v, of which a column keeps its
  // own request's: an accumulator per request up to rank 32, selected at the
  // end; above, one, selected at every sub-block (the registers end there).
  constexpr int NLA = C::RC <= 2 ? RPB : 1;
  constexpr int kV = SH_W * 16 * C::V_ROW * 2, kLv = SH_W * NLT * LVT * 2;
  constexpr int kOff = SB * C::CS_ROW * 8 + (SB * C::CS_ROW % 2) * 8, kBase = SH_W * 2 * C::HALF * 8;
  constexpr int kLoop = kBk + kV + kLv + kOff + kBase;
  constexpr int PR = D + R + 4, kPart = SH_W * 16 * PR * 4;  // [wave][column][acc, accl, m, l]
  static_assert(kBk % 16 == 0 && kV % 16 == 0 && kLv % 16 == 0 && kOff % 16 == 0, "16-byte aligned areas");
  __shared__ __attribute__((aligned(16))) char smem[kLoop > kPart ? kLoop : kPart];
  Frag* bk_lds = reinterpret_cast<Frag*>(smem);
  float2* off_lds = reinterpret_cast<float2*>(smem + kBk + kV + kLv);

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_str = SH_W / n_grp, grp = w / n_str, stream = w - grp * n_str;
  const int split = blockIdx.x, g = blockIdx.y, G = a.group;
  const int b_wg = blockIdx.z * n_grp * RPB, b0 = b_wg + grp * RPB;  // first request of the workgroup, of this wave
  const int q = lane >> 4, c16 = lane & 15;
  const bool has_lk = a.Lk != nullptr, has_lv = a.Lv != nullptr;
  // The split's range divides the furthest end among the workgroup's
  // requests; each request stops at its own.
  static_assert(sh_groups(R) * RPB <= kMaxGroup, "one reduction over the lanes of a group");
  int vis_lane;
  const int vis_wg = group_visible_keys(a, b_wg, n_grp * RPB, lane, vis_lane);
  const int st_tiles = __builtin_amdgcn_readfirstlane(tiles_per_split(vis_wg, a.n_splits));
  if (split > 0 && (int64_t)split * st_tiles * TK >= vis_wg) return;  // past the end (uniform over the workgroup)
  const int t_begin = split * st_tiles * TK;
  auto clip = [&](int end) { return end < t_begin ? t_begin : (end - t_begin < st_tiles * TK ? end : t_begin + st_tiles * TK); };
  const int t_end_wg = __builtin_amdgcn_readfirstlane(clip(vis_wg));
  int t_end_r[RPB];  // per request of this wave (uniform)
#pragma unroll
  for (int i = 0; i < RPB; ++i) t_end_r[i] = clip(__builtin_amdgcn_readlane(vis_lane, grp * RPB + i));
  int t_end_min = t_end_wg;  // up to here every request of this wave has keys
#pragma unroll
  for (int i = 0; i < RPB; ++i) t_end_min = b0 + i < a.batch ? min(t_end_min, t_end_r[i]) : t_end_min;
  t_end_min = __builtin_amdgcn_readfirstlane(t_end_min);
  // This lane's column: request slot, head, end.
  const int slot = c16 / G, b_l = b0 + slot;
  const bool col_ok = slot < RPB && b_l < a.batch;
  int t_end_l = t_begin;
#pragma unroll
  for (int i = 0; i < RPB; ++i) t_end_l = slot == i ? t_end_r[i] : t_end_l;

  // Q^T of the columns as the B operand (zero where there is no head).
  bf16x8 qf[C::NCH];
  {
    const uint16_t* qp =
        a.Q + ((int64_t)(col_ok ? b_l : 0) * a.n_tok * a.n_q + (int64_t)g * G + (col_ok ? c16 - slot * G : 0)) * D;
#pragma unroll
    for (int kk = 0; kk < C::NCH; ++kk) qf[kk] = as_bf16x8(ld16(qp + chunk_dim<D>(kk, q), col_ok));
  }

  const double w2pi_l = a.w2pi[lane % C::HALF];

  // One-time loads first (all of them older than the staged rows, so the
  // loop's waits count staged loads only): a wave per request reads its B_k.
  BtStage<D, R> bts;
  {
    const bool ok = has_lk && w < n_grp * RPB && b_wg + w < a.batch;
    bts.issue(ok ? a.Bk + (int64_t)(b_wg + w) * a.b_stride + (int64_t)g * D : nullptr, (int64_t)a.n_kv * D, ok, lane);
  }

  const int64_t row = (int64_t)a.n_kv * D;
  const uint16_t* Kb = a.Kb + (int64_t)g * D;
  const uint16_t* Vb = a.Vb + (int64_t)g * D;
  const int vrow = lane / C::LPR, vdim = (lane % C::LPR) * 8;
  int32_t voff[C::NVL], lvoff[C::RC], lkoff[NC];
  const int32_t koff = c16 * (int32_t)(row * 2) + chunk_dim<D>(0, q) * 2;
#pragma unroll
  for (int iv = 0; iv < C::NVL; ++iv) voff[iv] = (vrow + C::RPL * iv) * (int32_t)(row * 2) + vdim * 2;
#pragma unroll
  for (int rc = 0; rc < C::RC; ++rc) {
    const int r0 = rc * 16 + q * 4;
    lvoff[rc] = r0 < R ? c16 * R * 2 + r0 * 2 : INT32_MIN;
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int r0 = Ex<R>::rank0(c, q);
    lkoff[c] = r0 < R ? c16 * R * 2 + r0 * 2 : INT32_MIN;
  }
  // Staged rows of the next sub-block.  Rows past an end read as zeros and
  // touch no memory.
  u32x4 kst[C::NCH], vst[C::NVL];
  Frag lkst[RPB][NC];
  u32x2 lvst[RPB][C::RC];
  // Every path issues the same loads in the same order, without branches, so
  // that the compiler's load counting waits only for what it needs (a load
  // behind a branch made each sub-block wait for the last load issued: the
  // whole memory latency).
  // (readfirstlane: the clamp would otherwise be done on the vector ALU, and
  // resources in vector registers cost a loop around each load.)
  auto valid = [&](int end, int t0) { return __builtin_amdgcn_readfirstlane(max(0, min(end - t0, SB))); };
  auto load_base = [&](int t0) {
    const int n = valid(t_end_wg, t0);
    const int32_t bytes = n > 0 ? (n - 1) * (int32_t)(row * 2) + D * 2 : 0;
    const auto rk = make_rsrc(Kb + t0 * row, bytes), rv = make_rsrc(Vb + t0 * row, bytes);
#pragma unroll
    for (int kk = 0; kk < C::NCH; ++kk)
      kst[kk] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rk, koff + chunk_dim<D>(kk, 0) * 2, 0, 0));
#pragma unroll
    for (int iv = 0; iv < C::NVL; ++iv)
      vst[iv] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rv, voff[iv], 0, 0));
  };
  // Absent LR caches read the base through empty resources: zeros.
  const uint16_t* Lk = has_lk ? a.Lk + (int64_t)b0 * a.l_stride : Kb;
  const uint16_t* Lv = has_lv ? a.Lv + (int64_t)b0 * a.l_stride : Kb;
  const int lk_row = has_lk ? R * 2 : 0, lv_row = has_lv ? R * 2 : 0;
  auto load_lk = [&](int t0) {
#pragma unroll
    for (int i = 0; i < RPB; ++i) {
      const auto r = make_rsrc(Lk + i * a.l_stride + (int64_t)t0 * R, valid(t_end_r[i], t0) * lk_row);
#pragma unroll
      for (int c = 0; c < NC; ++c) lkst[i][c] = lr_frag_load<R>(r, lkoff[c]);
    }
  };
  auto load_lv = [&](int t0) {
#pragma unroll
    for (int i = 0; i < RPB; ++i) {
      const auto r = make_rsrc(Lv + i * a.l_stride + (int64_t)t0 * R, valid(t_end_r[i], t0) * lv_row);
#pragma unroll
      for (int rc = 0; rc < C::RC; ++rc)
        lvst[i][rc] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, lvoff[rc], 0, 0));
    }
  };

  const int n_sb = (t_end_wg - t_begin + SB - 1) / SB;
  load_base(t_begin + stream * SB);
  load_lk(t_begin + stream * SB);
  load_lv(t_begin + stream * SB);

  // B_k^T fragments of every request of the workgroup, fragment order: a
  // wave per request, read with coalesced loads and transposed through its V
  // tile.
  if (has_lk) {
    const int r = w;
    if (r < n_grp * RPB) {
      Frag f[C::NBLK][NC];
      bts.finish(f, reinterpret_cast<uint16_t*>(smem + kBk) + w * 16 * C::V_ROW, lane);
#pragma unroll
      for (int blk = 0; blk < C::NBLK; ++blk)
#pragma unroll
        for (int c = 0; c < NC; ++c) bk_lds[r * NBF + (blk * NC + c) * 64 + lane] = f[blk][c];
    }
    // In-tile offsets of this lane's frequency (read above: a load here would
    // wait for the staged rows, which were issued before it).
    constexpr int TPW = 64 / C::HALF;  // tokens per wave and step
    for (int tok = w * TPW + lane / C::HALF; tok < SB; tok += SH_W * TPW) {
      float c, s;
      rope_cs(tok, w2pi_l, c, s);
      off_lds[tok * C::CS_ROW + lane % C::HALF] = make_float2(c, s);
    }
  }
  uint16_t* vl = reinterpret_cast<uint16_t*>(smem + kBk) + w * 16 * C::V_ROW;
  uint16_t* lvl = reinterpret_cast<uint16_t*>(smem + kBk + kV) + w * NLT * LVT;
  float2* base = reinterpret_cast<float2*>(smem + kBk + kV + kLv + kOff) + w * 2 * C::HALF;  // [2][HALF]
  for (int i = lane; i < NLT * LVT; i += 64) lvl[i] = 0;

  float m_run = -INFINITY, l_part = 0.f;
  f32x4 acc[C::NBLK], accl[NLA][C::RC];
#pragma unroll
  for (int blk = 0; blk < C::NBLK; ++blk) acc[blk] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < NLA; ++r)
#pragma unroll
    for (int rc = 0; rc < C::RC; ++rc) accl[r][rc] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int tr_row = 4 * q + (c16 >> 2), tr_col = 4 * (c16 & 3);

  // Exact angles of a sub-block's first token, a sub-block ahead.
  auto base_angles = [&](int t0, int buf) {
    float c, s;
    rope_cs(t0, w2pi_l, c, s);
    if (lane < C::HALF) base[buf * C::HALF + lane] = make_float2(c, s);
  };
  auto lv_store = [&](int r) {
#pragma unroll
    for (int rc = 0; rc < C::RC; ++rc)
      if (rc * 16 + q * 4 < R)
        *reinterpret_cast<u32x2*>(lvl + (r % NLT) * LVT + c16 * C::LV_ROW + rc * 16 + q * 4) = lvst[r][rc];
  };
  base_angles(t_begin + stream * SB, 0);
  __syncthreads();  // B_k^T fragments and offsets in LDS

  int buf = 0;
  for (int sb = stream; sb < n_sb; sb += n_str, buf ^= 1) {
    const int ts = t_begin + sb * SB, tn = ts + n_str * SB;
    // The two waves of a SIMD (w, w + 4) take turns at the higher issue
    // priority: left alone the older one always issues first, finishes early
    // and leaves the other without a partner (74 -> 71 us).
    if ((buf ^ (w >> 2)) & 1) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
    // ---- base scores, V (and L_v) rows to LDS; the next sub-block's loads ------
#pragma unroll
    for (int iv = 0; iv < C::NVL; ++iv)
      *reinterpret_cast<u32x4*>(vl + (vrow + C::RPL * iv) * C::V_ROW + vdim) = vst[iv];
    f32x4 sc0 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < C::NCH; ++kk) sc0 = mfma16x16x32(as_bf16x8(kst[kk]), qf[kk], sc0);
    load_base(tn);
    if constexpr (NLT == RPB) {
      if (has_lv) {
#pragma unroll
        for (int r = 0; r < RPB; ++r) lv_store(r);
      }
      load_lv(tn);
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- key expansion of each request, into its columns' scores -------------
    f32x4 sc = sc0;
    if (has_lk) {
      // Two 16-dim blocks of each RoPE half at a time (one 8-dim chunk of the
      // low half and its partner): the angles of four blocks at once would
      // cost 16 more registers.
      f32x4 sr[RPB];
#pragma unroll
      for (int r = 0; r < RPB; ++r) sr[r] = sc0;
#pragma unroll
      for (int hb = 0; hb < C::NB / 2; ++hb) {
        float cc[2][4], ss[2][4];
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int j = q * C::QPG + (2 * hb + b2) * 4 + i;
            const float2 o = off_lds[c16 * C::CS_ROW + j], bs = base[buf * C::HALF + j];
            cc[b2][i] = bs.x * o.x - bs.y * o.y;
            ss[b2][i] = bs.y * o.x + bs.x * o.y;
          }
#pragma unroll
        for (int r = 0; r < RPB; ++r) {
          const Frag* bk = bk_lds + (grp * RPB + r) * NBF + lane;
          u32x4 elc, ehc;  // chunks hb and hb + NB / 2 of the rotated expansion
#pragma unroll
          for (int b2 = 0; b2 < 2; ++b2) {
            const int blk = 2 * hb + b2;
            f32x4 elo = {0.f, 0.f, 0.f, 0.f}, ehi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < NC; ++c) {
              elo = Ex<R>::mma(bk[(blk * NC + c) * 64], lkst[r][c], elo);
              ehi = Ex<R>::mma(bk[((blk + C::NB) * NC + c) * 64], lkst[r][c], ehi);
            }
            float rlo[4], rhi[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              rlo[i] = elo[i] * cc[b2][i] - ehi[i] * ss[b2][i];
              rhi[i] = ehi[i] * cc[b2][i] + elo[i] * ss[b2][i];
            }
            elc[2 * b2] = pack_bf16(rlo[0], rlo[1]);
            elc[2 * b2 + 1] = pack_bf16(rlo[2], rlo[3]);
            ehc[2 * b2] = pack_bf16(rhi[0], rhi[1]);
            ehc[2 * b2 + 1] = pack_bf16(rhi[2], rhi[3]);
          }
          sr[r] = mfma16x16x32(as_bf16x8(elc), qf[hb], sr[r]);
          sr[r] = mfma16x16x32(as_bf16x8(ehc), qf[hb + C::NB / 2], sr[r]);
        }
      }
#pragma unroll
      for (int r = 0; r < RPB; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) sc[i] = slot == r ? sr[r][i] : sc[i];
    }
    load_lk(tn);
    __builtin_amdgcn_sched_barrier(0);
    base_angles(tn, buf ^ 1);
    // ---- online softmax: one column per lane, 4 tokens -----------------------
    float s2[4];
    float mx = -INFINITY;
    const int n_vis = max(0, min(t_end_l - ts, SB));  // visible tokens of the sub-block
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s2[i] = (q * 4 + i < n_vis) ? sc[i] * a.scale_log2 : -INFINITY;
      mx = fmaxf(mx, s2[i]);
    }
    mx = max_xor32(max_xor16(mx));
    if (__ballot(mx > m_run + kRescaleLog2)) {  // lazy rescale, as above
      const float mn = fmaxf(m_run, mx);
      const float alpha = fast_exp2(m_run - (mn == -INFINITY ? 0.f : mn));
#pragma unroll
      for (int blk = 0; blk < C::NBLK; ++blk) acc[blk] *= alpha;
#pragma unroll
      for (int r = 0; r < NLA; ++r)
#pragma unroll
        for (int rc = 0; rc < C::RC; ++rc) accl[r][rc] *= alpha;
      l_part *= alpha;
      m_run = mn;
    }
    const float ms = (m_run == -INFINITY) ? 0.f : m_run;
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = fast_exp2(s2[i] - ms);
    l_part += (p[0] + p[1]) + (p[2] + p[3]);
    const u32x2 pw = {pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3])};
    const i16x4 pb = as_i16x4(pw);
    __builtin_amdgcn_wave_barrier();
    // ---- O^T += V^T P^T; (P L_v)^T += L_v^T P^T, each request its columns ------
    // A weight of zero does not keep an infinity or a NaN out (0 x Inf is NaN),
    // so rows that are not a column's own are kept out by selection: base rows
    // past a shorter request's end here, every other request's L_v below.
    if (ts < t_end_min) {
#pragma unroll
      for (int blk = 0; blk < C::NBLK; ++blk)
        acc[blk] = mfma16x16x16(lds_read_tr(vl + tr_row * C::V_ROW + blk * 16 + tr_col), pb, acc[blk]);
    } else {
#pragma unroll
      for (int blk = 0; blk < C::NBLK; ++blk) {
        const f32x4 x = mfma16x16x16(lds_read_tr(vl + tr_row * C::V_ROW + blk * 16 + tr_col), pb, acc[blk]);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[blk][i] = n_vis > 0 ? x[i] : acc[blk][i];
      }
    }
    if (has_lv) {
      f32x4 own[C::RC];
#pragma unroll
      for (int r = 0; r < RPB; ++r) {
        if constexpr (NLT == 1) lv_store(r);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int rc = 0; rc < C::RC; ++rc) {
          f32x4& acl = accl[r % NLA][rc];
          const f32x4 x = mfma16x16x16(lds_read_tr(lvl + (r % NLT) * LVT + tr_row * C::LV_ROW + rc * 16 + tr_col), pb, acl);
          if constexpr (NLA == RPB) acl = x;
          else
#pragma unroll
            for (int i = 0; i < 4; ++i) own[rc][i] = r == 0 || slot == r ? x[i] : own[rc][i];
        }
        __builtin_amdgcn_wave_barrier();
      }
      if constexpr (NLA == 1)
#pragma unroll
        for (int rc = 0; rc < C::RC; ++rc) accl[0][rc] = own[rc];
    }
    if constexpr (NLT == 1) {
      load_lv(tn);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- combine the streams of each group, one partial per (request, head) ----
  l_part += shfl_xor(l_part, 16);
  l_part += shfl_xor(l_part, 32);
  __syncthreads();  // every wave is done with the loop's LDS
  float* part = reinterpret_cast<float*>(smem);
  {
    float* pr = part + (w * 16 + c16) * PR;
#pragma unroll
    for (int blk = 0; blk < C::NBLK; ++blk) *reinterpret_cast<f32x4*>(pr + blk * 16 + q * 4) = acc[blk];
#pragma unroll
    for (int rc = 0; rc < C::RC; ++rc) {
      f32x4 own = accl[0][rc];
#pragma unroll
      for (int r = 1; r < NLA; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) own[i] = slot == r ? accl[r][rc][i] : own[i];
      if (rc * 16 + q * 4 < R) *reinterpret_cast<f32x4*>(pr + D + rc * 16 + q * 4) = own;
    }
    if (q == 0) {
      pr[D + R] = m_run;
      pr[D + R + 1] = l_part;
    }
  }
  __syncthreads();
  constexpr int NV = (D + R) / 4;  // float4 columns of a partial's accumulators
  const int n_col = RPB * G;
  auto combine = [&](auto n) {  // compile-time stream count: all reads of an item in flight at once
    constexpr int NS = decltype(n)::value;
    for (int e = tid; e < n_grp * n_col * NV; e += NTH) {
      const int v = e % NV, col = (e / NV) % n_col, gi = e / (NV * n_col);
      const int rs = col / G, bb = b_wg + gi * RPB + rs;
      if (bb >= a.batch || (v >= D / 4 && !has_lv)) continue;
      const float* p0 = part + (gi * NS * 16 + col) * PR;
      f32x4 x[NS];
      f32x2 ml[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        x[s] = *reinterpret_cast<const f32x4*>(p0 + s * 16 * PR + 4 * v);
        ml[s] = *reinterpret_cast<const f32x2*>(p0 + s * 16 * PR + D + R);
      }
      float M = ml[0][0];
#pragma unroll
      for (int s = 1; s < NS; ++s) M = fmaxf(M, ml[s][0]);
      const float Ms = M == -INFINITY ? 0.f : M;
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
      float L = 0.f;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const float wt = fast_exp2(ml[s][0] - Ms);
        L += wt * ml[s][1];
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] += wt * x[s][i];
      }
      float* wsb = a.ws + (((int64_t)bb * a.n_q + (int64_t)g * G + (col - rs * G)) * a.n_splits + split) * C::PS;
      *reinterpret_cast<f32x4*>(wsb + 4 + 4 * v) = sum;
      if (v == 0) {
        wsb[0] = M;
        wsb[1] = L;
      }
    }
  };
  if (n_grp == 1) combine(std::integral_constant<int, SH_W>{});
  else combine(std::integral_constant<int, SH_W / 2>{});
}

// The same merge for many rows with at most 16 splits (split prefill, longer
// decode splits): one wave per row and four rows per workgroup.  Lane s < ns
// reads split s's maximum and sum; lane v < (d + r)/4 owns float4 column v of
// the accumulators and folds every split into it (all loads of the row in
// flight at once); the row's (d + r) sums then pass through LDS for the
// B_v product.
constexpr int MR_ROWS = 4;

template <int D, int R>
__global__ void __launch_bounds__(64 * MR_ROWS) lrsa_merge_rows_kernel(const AttnArgs a, int64_t n_rows) {
  constexpr int PS = 4 + D + R, NV = (D + R) / 4;
  static_assert(NV <= 64, "one lane per float4 column");
  __shared__ __attribute__((aligned(16))) float fin[MR_ROWS][D + R];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t orow = (int64_t)blockIdx.x * MR_ROWS + w;  // (request, token, head) row of O
  if (orow >= n_rows) return;
  const int h = (int)(orow % a.n_q);
  const int b = (int)(orow / a.n_q / a.n_tok);
  const int g = h / a.group;
  const bool has_lv = a.Lv != nullptr;
  const float* base = a.ws + orow * (int64_t)a.n_splits * PS;
  const int ns = splits_written(a, b);

  const float m_s = lane < ns ? base[(int64_t)lane * PS] : -INFINITY;
  const float l_s = lane < ns ? base[(int64_t)lane * PS + 1] : 0.f;
  float M = m_s;
#pragma unroll
  for (int x = 1; x < 64; x <<= 1) M = fmaxf(M, shfl_xor(M, x));
  const float Ms = (M == -INFINITY) ? 0.f : M;
  const float w_s = lane < ns ? fast_exp2(m_s - Ms) : 0.f;
  float L = w_s * l_s;
#pragma unroll
  for (int x = 1; x < 64; x <<= 1) L += shfl_xor(L, x);

  const int nv_used = has_lv ? NV : D / 4;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  const int v = lane < nv_used ? lane : 0;
#pragma unroll 4
  for (int s = 0; s < ns; ++s) {
    const float wgt = __shfl(w_s, s, 64);
    const f32x4 x = *reinterpret_cast<const f32x4*>(base + (int64_t)s * PS + 4 + 4 * v);
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] += wgt * x[c];
  }
  if (lane < nv_used) *reinterpret_cast<f32x4*>(&fin[w][4 * lane]) = acc;
  __builtin_amdgcn_wave_barrier();

  const float inv = L > 0.f ? 1.f / L : 0.f;
  uint16_t* o = a.O + orow * D;
#pragma unroll
  for (int dd = 0; dd < D / 64; ++dd) {
    const int dim = lane + 64 * dd;
    float sum = fin[w][dim];
    if (has_lv) {
      const int64_t ldb = (int64_t)a.n_kv * D;
      const uint16_t* bv = a.Bv + (int64_t)b * a.b_stride + (int64_t)g * D + dim;
#pragma unroll 8
      for (int j = 0; j < R; ++j) sum += fin[w][D + j] * __uint_as_float((uint32_t)bv[j * ldb] << 16);
    }
    const uint32_t pk = pack_bf16(sum * inv, 0.f);
    o[dim] = (uint16_t)(pk & 0xffffu);
  }
  if (a.lse != nullptr && lane == 0)
    a.lse[orow] = L > 0.f ? (M + __log2f(L)) * kLn2 : -INFINITY;
}

template <int D, int R>
hipError_t launch_merge_t(const AttnArgs& a, hipStream_t st) {
  const int64_t n_rows = (int64_t)a.batch * a.n_tok * a.n_q;
  // Chunks, shared-base calls and paged rank-64 ones of few rows take a workgroup
  // per row with few splits too: one wave's reads of B_v and of the splits are a chain as long as
  // the rank, and too few rows run side by side to hide it (4 tokens of 4
  // requests over 512 keys, dim 128, one wave / four: rank 16 19.9 / 15.7 us, 32
  // 23.5 / 18.5; 8 requests over one base, rank 64, of 500 tokens 26.2 / 20.5,
  // of 64, two splits, 20.7 / 18.3; 8 paged requests of 2048 tokens, rank 64, 41.7
  // / 30.0).  Not more rows: 100 requests, 1600 rows of 5
  // splits 11.0 / 12.1; 2560 rows of 6 splits, rank 64, 23.9 / 26.7.
  // (Paged: the register-staged form at d = 128 only; the others are to sum as the
  // contiguous calls do.)
  const bool staged64 = D == 128 && R == 64 && a.kv_tbl != nullptr && !a.dec_direct;
  const bool few_rows = a.dec_group != 0 && (a.n_tok > 1 || a.dec_shared || staged64) &&
                        n_rows <= (a.n_splits >= 8 ? 2048 : 1024);
  if (a.n_splits <= 16 && !few_rows) {
    hipLaunchKernelGGL((lrsa_merge_rows_kernel<D, R>), dim3((unsigned)((n_rows + MR_ROWS - 1) / MR_ROWS)),
                       dim3(64 * MR_ROWS), 0, st, a, n_rows);
    return hipGetLastError();
  }
  const dim3 grid(a.n_q, a.batch * a.n_tok);
  // The wider merge holds one split per thread (decode_plan keeps n_splits
  // within 1024); rows of at most 64 splits take four waves.
  if (a.n_splits > 64)
    hipLaunchKernelGGL((lrsa_merge_kernel<D, R, 16>), grid, dim3(64 * 16), 0, st, a);
  else
    hipLaunchKernelGGL((lrsa_merge_kernel<D, R, 4>), grid, dim3(64 * 4), 0, st, a);
  return hipGetLastError();
}

template <int D, int R>
hipError_t launch_t(AttnArgs a, hipStream_t st) {
  a.dec_group = 1;
  const unsigned gx = a.wg_total > 0 ? a.wg_total : a.n_splits, gz = a.wg_total > 0 ? 1 : a.batch;
  const auto go = [&](auto paged, auto mt) {
    constexpr bool P = decltype(paged)::value, M = decltype(mt)::value;
    if constexpr (P && !M && dec_vdma(D, R, false)) {
      if (a.dec_direct) {
        constexpr int nw = dec_nw(D, R, false);
        const dim3 grid(gx, (a.n_kv + nw - 1) / nw, gz);
        hipLaunchKernelGGL((lrsa_decode_kernel<D, R, P, M, false>), grid, dim3(64 * nw), 0, st, a);
        return;
      }
    }
    constexpr int nw = dec_nw(D, R, P || M);
    const dim3 grid(gx, (a.n_kv + nw - 1) / nw, gz);
    hipLaunchKernelGGL((lrsa_decode_kernel<D, R, P, M>), grid, dim3(64 * nw), 0, st, a);
  };
  const std::true_type yes{};
  const std::false_type no{};
  if (a.kv_tbl != nullptr) a.n_tok > 1 ? go(yes, yes) : go(yes, no);
  else a.n_tok > 1 ? go(no, yes) : go(no, no);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_merge_t<D, R>(a, st);
}

template <int D, int R, int RPB>
hipError_t launch_shared_rpb(AttnArgs a, hipStream_t st) {
  // One group of requests needs all eight waves as streams; more go two to a
  // workgroup where their B_k fits.
  const int n_grp = a.batch > RPB ? sh_groups(R) : 1;
  static_assert(sh_groups(R) * RPB <= kMaxGroup, "group_visible_keys covers it");
  a.dec_group = n_grp * RPB;
  const dim3 grid(a.n_splits, a.n_kv, (a.batch + a.dec_group - 1) / a.dec_group);
  hipLaunchKernelGGL((lrsa_decode_shared_kernel<D, R, RPB>), grid, dim3(SH_W * 64), 0, st, a, n_grp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_merge_t<D, R>(a, st);
}

template <int D, int R>
hipError_t launch_shared_t(const AttnArgs& a, hipStream_t st) {
  switch (sh_rpb(a.batch, a.group, R)) {
    case 4: return launch_shared_rpb<D, R, 4>(a, st);
    case 3: return launch_shared_rpb<D, R, 3>(a, st);
    default: return launch_shared_rpb<D, R, 2>(a, st);
  }
}

template <int D>
hipError_t launch_merge_r(const AttnArgs& a, hipStream_t st) {
  switch (a.rank) {
    case 8: return launch_merge_t<D, 8>(a, st);
    case 16: return launch_merge_t<D, 16>(a, st);
    case 32: return launch_merge_t<D, 32>(a, st);
    case 64: return launch_merge_t<D, 64>(a, st);
    default: return hipErrorInvalidValue;
  }
}

template <int D>
hipError_t launch_r(const AttnArgs& a, hipStream_t st, bool shared) {
  switch (a.rank) {
    case 8: return shared ? launch_shared_t<D, 8>(a, st) : launch_t<D, 8>(a, st);
    case 16: return shared ? launch_shared_t<D, 16>(a, st) : launch_t<D, 16>(a, st);
    case 32: return shared ? launch_shared_t<D, 32>(a, st) : launch_t<D, 32>(a, st);
    case 64: return shared ? launch_shared_t<D, 64>(a, st) : launch_t<D, 64>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int decode_tile_tokens() { return TK; }

// Workgroups of the shared-base kernel for one split.
static int64_t shared_workgroups(int64_t batch, int n_kv, int group, int rank) {
  const int rpb = sh_rpb(batch, group, rank);
  const int64_t rq = rpb * (batch > rpb ? sh_groups(rank) : 1);
  return (int64_t)n_kv * ((batch + rq - 1) / rq);
}

// Below 2048 tokens the base tiles stay in the L2 whoever reads them, and the
// shared-base kernel's longer start costs more than its one read saves (8 / 2 /
// 16 requests of 300 tokens: 19.3 / 16.5 / 21.4 us shared, 16.6 / 14.9 / 18.4
// each by itself; of 1200: 19.0 / 14.8 / 25.9 and 17.9 / 13.9 / 25.6; 8 of 2400:
// 21.9 and 23.0).  The line is on the capacity, as the host does not know the
// lengths; a short context in a large cache stays near its own size's time,
// since its splits divide the keys in use (rank 16, 300 of 65920 tokens, 2 / 8 /
// 16 requests: 13.0 / 15.5 / 16.5 us).
bool decode_can_share_base(int batch, int64_t kv_req_stride) { return batch > 1 && kv_req_stride == 0; }
bool decode_base_is_short(int64_t s_cap, int batch, int64_t kv_req_stride) {
  return decode_can_share_base(batch, kv_req_stride) && s_cap < 2048;
}
// At rank 64, dim 128, the per-request kernel's own start is the longer one (its
// heads' 64 KB of B_k): there the shared kernel runs at every size where one
// round of its workgroups holds the call (2 / 8 / 16 requests of 300 tokens, 32
// / 8 heads: 26.3 / 27.0 / 30.3 us each by itself, 17.2 / 19.3 / 20.8 shared; 8
// of 700 with 40 / 8 heads: 24.7 and 20.1).
bool decode_shares_base(int64_t s_cap, int batch, int64_t kv_req_stride, int n_kv, int group, int head_dim, int rank, int cus) {
  if (!decode_can_share_base(batch, kv_req_stride)) return false;
  if (!decode_base_is_short(s_cap, batch, kv_req_stride)) return true;
  if (!dec_vdma(head_dim, rank, false)) return false;
  int ns;
  decode_plan(s_cap, batch, n_kv, group, head_dim, rank, true, false, cus, &ns);
  return ns * shared_workgroups(batch, n_kv, group, rank) <= cus;
}

// The one-round kernel has nothing left to even out requests of different
// lengths with, so batches of 2 to 64 of them cut their splits by length (a
// request may then take up to twice its even share).  Not where splits are
// short anyway: the lengths are read before anything else, about 1.5 us in the
// kernel and the merge.  The two-round kernels gain nothing from it (16
// requests of 10k-32k tokens, rank 16: 262 us either way).
bool decode_balances(int64_t s_cap, int batch, int n_tok, int head_dim, int rank, int n_splits, bool shared_base, bool staged) {
  return dec_vdma(head_dim, rank, staged) && batch > 1 && batch <= 64 && n_tok == 1 && !shared_base && n_splits >= 2 &&
         2 * n_splits <= kMaxSplits && s_cap / n_splits >= 8 * TK;
}

void decode_plan(int64_t s_cap, int batch, int n_kv, int group, int head_dim, int rank, bool shared_base, bool staged,
                 int cus, int* n_splits) {
  const int64_t tiles = (s_cap + TK - 1) / TK;
  const int nw = shared_base ? SH_W : dec_waves(rank);
  const int64_t nb = batch > 0 ? batch : 1;
  // Workgroups per split: (request, group of nw KV heads) for the per-request
  // kernel, (KV head, groups of requests) when the base cache is shared.
  const int64_t groups = shared_base ? shared_workgroups(nb, n_kv, group, rank) : nb * ((n_kv + nw - 1) / nw);
  // Splits for a target of `rounds` 8-wave workgroups per CU.
  auto plan = [&](int64_t rounds, int64_t* ns_out, int64_t* st_out) {
    const int64_t target_wgs = rounds * (cus > 0 ? cus : 1) * 8 / nw;
    int64_t ns = (target_wgs + groups - 1) / groups;
    // Rounded down where splits are long: a split more for each request starts
    // a few workgroups after all others have (per call, rounded up / down: 14
    // requests of 31.6k tokens, dim 64, 518 / 504 workgroups: 134 / 109 us; 11
    // of 45.7k, dim 128: 455 / 370 us; 3 of 30k: 111 / 77 us).  Short splits
    // lose more by a longer one.
    if (target_wgs / groups >= 4 && tiles >= 8 * ns) ns = target_wgs / groups;
    if (ns < 1) ns = 1;
    if (ns > kMaxSplits) ns = kMaxSplits;
    if (ns > tiles) ns = tiles > 0 ? tiles : 1;
    int64_t st = (tiles + ns - 1) / ns;
    if (st < 1) st = 1;
    ns = (tiles + st - 1) / st;
    // One round is kept to one: workgroups past it wait for a whole round as soon
    // as their XCD has no CU left for them, which is up to the lengths (12 paged
    // requests of 4736 tokens of capacity, rank 8, 264 / 252 workgroups: of 3100
    // tokens each 37.4 / 37.3 us, of 3100, 3036, .. 46.4 / 35.6, of 4736 72.5 /
    // 49.6).  The splits in use may then be a tile longer (24 requests of 1320,
    // 1280, .. of 2000 tokens: 32.1 / 34.5).
    if (rounds == 1 && groups * ns > target_wgs && groups <= target_wgs) ns = target_wgs / groups;
    *ns_out = ns < 1 ? 1 : ns;
    *st_out = st;
  };
  // About two rounds of one workgroup per CU (measured best for large
  // batches) while splits stay at least 8 tiles long; otherwise one round:
  // small batches then get longer splits, each CU at most one workgroup,
  // and half the partials to merge (batch 1 at 36k: 46 -> 38 us per call).
  // The rank-64 kernel that stages V by direct global->LDS loads holds its
  // workgroup's whole register file per CU and keeps one sub-block in flight
  // per wave: one round of longer splits measured faster there (64k, 8
  // requests: 426 -> 419 us; two, three and four rounds 426, 442, 446 us).
  // The shared-base kernel takes one round too: its workgroups' start and
  // combine cost as much as many sub-blocks (see its comment).
  int64_t ns, st;
  plan(2, &ns, &st);
  if (st < 8 || shared_base || dec_vdma(head_dim, rank, staged)) plan(1, &ns, &st);
  // The form that holds the whole register file runs one four-wave workgroup per
  // CU, and one round of them: a second costs its start again, with or without
  // keys (paged, rank 64, 8 KV heads, splits for two / one: one request of 5955 of
  // 9024 tokens 24.5 / 21.3 us, five of 2256 of 9024 31.0 / 24.4).
  if (staged && !shared_base && dec_occ(head_dim, rank, true, false) == 1 && groups <= cus && ns > cus / groups)
    ns = cus / groups;
  *n_splits = (int)ns;
}

// A chunk's splits are a decode's in the register-staged form, at rank 64 one
// workgroup per CU for either head dim.  (4 tokens of 6 requests, 32 / 8 heads of
// dim 128, 64 of 65920 tokens: 19.7 us as a prefill, 30.3 with four rounds, 18.2
// so; 8192 of 8192: 73, 81 and 56.)
void decode_chunk_plan(int64_t s_cap, int batch, int n_kv, int group, int head_dim, int rank, int cus, int* n_splits) {
  decode_plan(s_cap, batch, n_kv, group, head_dim, rank, false, true, cus, n_splits);
  if (dec_occ(head_dim, rank, true, true) > 1) return;
  const int nw = dec_waves(rank);
  const int64_t tiles = (s_cap + TK - 1) / TK, groups = (int64_t)(batch > 0 ? batch : 1) * ((n_kv + nw - 1) / nw);
  const int64_t most = cus / groups > 1 ? cus / groups : 1, n = *n_splits < most ? *n_splits : most;
  const int64_t st = (tiles + n - 1) / n;
  *n_splits = (int)((tiles + st - 1) / st);
}

// A paged rank-64 call takes the direct-V form, eight KV heads a workgroup,
// - where it leaves no more waves idle than the register-staged one, four heads a
//   workgroup (30000 tokens, six / twenty requests, 4 KV heads: 98.8 / 288 us
//   staged, 143 / 377 direct; 10 KV heads, six: 272 and 341), and
// - where the staged splits would be longer than 24 tiles: shorter ones lose more
//   by the direct form's longer start than its second wave per SIMD brings (8 KV
//   heads, staged / direct: one request of 5955 of 9024 tokens 21.2 / 29.2 us,
//   eight of 2048 of 2048 30.0 / 34.3, of 9024 of 9024 75.4 / 80.1; past it, eight
//   of 10813, 10475, .. of 16384 86.9 / 85.4, of 16384 121.8 / 124.0; 24 and 32 are
//   alike over 354 shapes, 64 is slower for some).
// With more staged workgroups than CUs it is the direct form's one round against
// two.  The line is on the capacity; the splits of both divide the keys in use.
bool decode_direct_paged(int64_t s_cap, int batch, int n_tok, int n_kv, int head_dim, int rank, int max_blk, int cus) {
  if (!dec_vdma(head_dim, rank, false) || n_tok != 1 || max_blk > kLdsBlocks) return false;
  const int nw = dec_nw(head_dim, rank, true), per_req = (n_kv + nw - 1) / nw;
  if (per_req % 2) return false;
  const int64_t tiles = (s_cap + TK - 1) / TK, groups = (int64_t)batch * per_req;
  return groups > cus ? tiles > 2 : tiles > 24 * (cus / groups);
}

// A chunk of a few query tokens whose (token, head) pairs per KV head fit the
// decode's 16 columns runs as a decode: split over the keys as far as the chip
// is wide, where a prefill would give one workgroup per KV head (times at most
// eight splits) 256 rows to fill with 16.  (16 tokens over 528 keys, 4 heads of
// dim 64, rank 8: 20.9 us as a prefill, 10.8 us so, 6.4 of them the decode.)
// Not below 512 tokens, where a prefill has few tiles to walk and needs no
// merge (3 tokens, group 4, rank 32, over 128 / 256 / 512 / 1024 keys: 12.6 /
// 16.4 / 23.9 / 27.6 us as a prefill, 17.5 / 18.9 / 21.3 / 17.5 us so).
// Several requests at ranks 32 and 64, dim 128, only from 1024 tokens on, unless
// a prefill would take more than one round of the CUs: their splits are one or
// two tiles long and start with 32 or 64 KB of B_k (4 tokens of 12 requests, 512
// tokens: rank 32, 64 / 256 / 512 keys 16.7 / 17.1 / 25.2 us as a prefill, 20.6
// / 22.8 / 23.9 so; rank 64 17.2 / 18.5 / 28.2 and 23.3 / 25.0 / 27.7).  Where
// few tokens of a small cache are in use the others lose a little too (12
// requests, 64 / 256 / 512 of 512, rank 16: 16.8 / 17.1 / 23.8 and 16.6 / 18.6
// / 19.1); the host does not know the lengths.
bool decode_takes_chunk(int64_t s_cap, int batch, int n_tok, int n_kv, int group, int head_dim, int rank, int cus) {
  if (n_tok < 2 || n_tok * group > 16) return false;
  const bool several = (int64_t)batch * ((n_kv + 7) / 8) > 4 && (int64_t)batch * n_kv <= cus;
  return s_cap >= (head_dim == 128 && rank >= 32 && several ? 1024 : 512);
}

size_t decode_workspace_bytes(int batch, int n_q, int n_splits, int head_dim, int rank) {
  return (size_t)batch * n_q * n_splits * (4 + head_dim + rank) * sizeof(float);
}

hipError_t launch_split_merge(const AttnArgs& a, hipStream_t st) {
  if (a.head_dim == 64) return launch_merge_r<64>(a, st);
  if (a.head_dim == 128) return launch_merge_r<128>(a, st);
  return hipErrorInvalidValue;
}

hipError_t launch_decode(const AttnArgs& a, hipStream_t st) {
  if (a.head_dim == 64) return launch_r<64>(a, st, a.dec_shared);
  if (a.head_dim == 128) return launch_r<128>(a, st, a.dec_shared);
  return hipErrorInvalidValue;
}

}  // namespace prc
