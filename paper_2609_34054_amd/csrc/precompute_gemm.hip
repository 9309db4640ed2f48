// LR-cache precompute GEMM (PreLRShared, Sec. 3.1, Fig. 1 A1-A3), optionally
// joined with the base K/V projection of the same segment, gfx950.
//
// When a segment of T hidden states is first processed, every agent's LoRA
// down-projection is applied to it at once:
//     L[p][a][tok_offset + t][j] = sum_k X[t][k] * A_stack[k][(p*N + a)*r + j]
// i.e. one GEMM  X[T x d_in] . A_stack[d_in x n_cols]  whose n_cols = n_proj*N*r
// output columns are scattered into per-agent planes [s_cap][r].  With the
// base projection joined (Sec. 2.2 base cache), the same GEMM also produces
// K_base = RoPE(X W_k) and V_base = X W_v: X is read once for all of it.
// The weights come in the orientation of Eq. 1, [d_in, d_out] row-major.
//
// The kernel computes the transposed product C^T = W^T X^T.  X tiles are
// staged in LDS k-contiguous, so each lane's B fragment (8 consecutive k of
// one token) is one 16-byte read.  Weight tiles are staged as they lie in
// memory, k rows of output columns, and the A fragments (8 consecutive k of
// one column) come out of the transposing LDS read ds_read_b64_tr_b16 (two
// per fragment).  A workgroup owns TB columns x TB tokens and has 4 compute
// waves, each accumulating a 64 x 64 block on 32x32x16 MFMAs (four 16-byte
// fragment reads per four MFMAs), and 8 loader waves filling a 4-stage ring of
// 32 KB stages with direct global->LDS buffer loads.  For the narrow LR-only
// GEMM (TB = 64) the four compute waves split every stage's k steps between
// them and sum their 64 x 64 partials through LDS at the end, in a fixed
// order; for the wide joined GEMM (TB = 128) each owns a quarter of the tile.
// Inside a stage, 16-byte chunks are XOR-swizzled by row so that both kinds
// of fragment read are free of bank conflicts; with direct-to-LDS loads the
// swizzle is applied by choosing which global chunk each lane fetches.
// Tokens past T, k past d_in and LR columns past n_cols read as zeros.  The
// result layout gives each lane 4 consecutive output columns of one token: one
// 8-byte store.  Calls of 1 to 4 rows, LR precompute too narrow to fill the chip
// with such tiles, and wide problems have kernels of their own below; the
// launch picks by a model of the rounds each takes.
// Block order is XCD-aware: the column tiles that share rows of
// X run on the same XCD, so X is fetched into each L2 once.
#include "common.hpp"
#include "kernels.hpp"

namespace prc {
namespace {

constexpr int NPW = 8;          // loader waves
constexpr int NCW = 4;          // compute waves
constexpr int NST = 4;          // stages in the LDS ring
constexpr int AHEAD = NST - 2;  // stages in flight beyond the one awaited
constexpr int NXCD = 8;         // XCDs of an MI355X

template <int TB>
struct Tile {
  static constexpr bool SPLITK = TB == 64;        // compute waves split k (narrow GEMM)
  static constexpr int KST = TB == 64 ? 128 : 64;  // k per stage: 2 x TB x KST x 2 B = 32 KB
  // X tile: TB token rows of KST k (XCPR 16-byte chunks per row).
  static constexpr int XCPR = KST / 8;
  static constexpr int XRPI = 64 / XCPR;           // rows per load instruction (1 KB)
  static constexpr int XRPW = TB / NPW;            // rows per loader wave
  static constexpr int NIX = XRPW / XRPI;          // X load instructions per wave and stage
  // Weight tile: KST k rows of TB columns (WCPR chunks per row).
  static constexpr int WCPR = TB / 8;
  static constexpr int WRPI = 64 / WCPR;
  static constexpr int WRPW = KST / NPW;
  static constexpr int NIW = WRPW / WRPI;
  // Physical chunk of logical chunk c in row r.  X rows: the 16 rows one
  // fragment read touches hit distinct banks.  Weight rows: the 4 k rows x 64
  // bytes a half-wave of transposing reads touches hit distinct banks.
  static __device__ __forceinline__ int swx(int r, int c) { return XCPR == 16 ? c ^ (r & 15) : c ^ ((r >> 1) & 7); }
  static __device__ __forceinline__ int sww(int r, int c) {
    return WCPR == 8 ? c ^ (((r >> 1) & 1) << 2) : c ^ ((r & 3) << 2);
  }
};

// s_waitcnt vmcnt(n) for a wave-uniform n in {0, 4, ..., 24}, other
// counters not waited on.  gfx9 encoding: vmcnt bits [3:0] and [15:14],
// expcnt [6:4] = 7, lgkmcnt [11:8] = 15.  The immediate must be a constant,
// so the cases are spelled out.
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
__device__ __forceinline__ void wait_vmcnt_le(int n) {
  switch (n) {
    case 24: __builtin_amdgcn_s_waitcnt(vmcnt_imm(24)); break;
    case 20: __builtin_amdgcn_s_waitcnt(vmcnt_imm(20)); break;
    case 16: __builtin_amdgcn_s_waitcnt(vmcnt_imm(16)); break;
    case 12: __builtin_amdgcn_s_waitcnt(vmcnt_imm(12)); break;
    case 8: __builtin_amdgcn_s_waitcnt(vmcnt_imm(8)); break;
    case 4: __builtin_amdgcn_s_waitcnt(vmcnt_imm(4)); break;
    default: __builtin_amdgcn_s_waitcnt(vmcnt_imm(0)); break;
  }
}

// Transposing LDS read of 4 bf16 per lane: lane j of each 16-lane group
// points at 4 consecutive bf16; lane i receives element i%4 of lanes i/4,
// i/4+4, i/4+8, i/4+12 of its group.
__device__ __forceinline__ u32x2 lds_read_tr(const uint16_t* p) {
  typedef short v4s __attribute__((ext_vector_type(4)));
  v4s v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((v4s __attribute__((address_space(3)))*)(p));
  return __builtin_bit_cast(u32x2, v);
}

// First W column (within the [d_in, 2 nkv] key/value weights) of the 8
// output columns starting at key column vc (a multiple of 8).  Key tiles
// permute the columns of each head so that every RoPE pair (dims j and
// j + d/2) lands in one lane of the result: local column e of a head (32-column
// block e / 32) holds dim (e / 32) * 16 + e % 16 + (e % 32 >= 16 ? d / 2 : 0).
__device__ __forceinline__ int key_wcol(int vc, int head_dim) {
  const int hd = vc / head_dim, e = vc - hd * head_dim;
  return hd * head_dim + (e / 32) * 16 + (e % 16) + ((e % 32) / 16) * (head_dim / 2);
}

// Row of the caches (or pools) that holds absolute position trow.
__device__ __forceinline__ int64_t cache_row(const PrecomputeArgs& a, int64_t trow) {
  if (a.tbl == nullptr) return trow;
  const int qb = (int)(trow / a.blk);
  int32_t e = a.tbl[qb];
  e = e < 0 ? 0 : (e >= a.nblk ? a.nblk - 1 : e);
  return (int64_t)e * a.blk + (trow - (int64_t)qb * a.blk);
}

// Writes one 32 x 32 block of C^T in the 32x32x16 result layout: r[j] is
// output column cb + (j / 4) * 8 + h * 4 + j % 4 of token t (h = lane / 32).
// Keys are rotated at the token's position as they are written; every token
// goes to its cache row (its position, or its row in the paged pools).
__device__ __forceinline__ void store_block(const PrecomputeArgs& a, const f32x16& r, int region, int cb, int64_t t,
                                            int h) {
  if (t >= a.T) return;
  const int64_t trow = a.tok_offset + t;  // absolute position of the token
  const int64_t row = cache_row(a, trow);
  if (region == 0) {
    // Keys: registers j and j + 8 hold dims j0 + i and j0 + i + d/2 of one
    // head (the column order of key tiles); rotate-half RoPE at position trow.
#pragma unroll
    for (int jg = 0; jg < 2; ++jg) {
      const int vc = cb + jg * 8 + h * 4;
      const int hd = vc / a.head_dim, e = vc - hd * a.head_dim;
      const int j0 = (e / 32) * 16 + (e % 16);
      float lo[4], hi[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float cs, sn;
        rope_cs((int)trow, a.w2pi[j0 + i], cs, sn);
        const float x = r[4 * jg + i], y = r[4 * jg + 8 + i];
        lo[i] = x * cs - y * sn;
        hi[i] = y * cs + x * sn;
      }
      uint16_t* kp = a.Kout + row * a.nkv + hd * a.head_dim + j0;
      *reinterpret_cast<u32x2*>(kp) = u32x2{pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3])};
      *reinterpret_cast<u32x2*>(kp + a.head_dim / 2) = u32x2{pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
    }
    return;
  }
#pragma unroll
  for (int jg = 0; jg < 4; ++jg) {
    const int c = cb + jg * 8 + h * 4;
    u32x2 o;
    o[0] = pack_bf16(r[4 * jg + 0], r[4 * jg + 1]);
    o[1] = pack_bf16(r[4 * jg + 2], r[4 * jg + 3]);
    if (region == 1) {
      *reinterpret_cast<u32x2*>(a.Vout + row * a.nkv + (c - a.nkv)) = o;
    } else {
      const int lc = c - 2 * a.nkv;
      if (lc >= a.n_cols) continue;
      const int plane = lc / a.rank, jr = lc - plane * a.rank;
      *reinterpret_cast<u32x2*>(a.L + ((int64_t)plane * a.s_cap + row) * a.rank + jr) = o;
    }
  }
}

template <int TB>
__global__ void __launch_bounds__((NCW + NPW) * 64) precompute_kernel(const PrecomputeArgs a, int n_ct, int n_tt) {
  using C = Tile<TB>;
  constexpr int KST = C::KST;
  static_assert((C::NIX + C::NIW) * AHEAD <= 24 && (C::NIX + C::NIW) % 2 == 0 && C::NIX >= 1 && C::NIW >= 1,
                "vmcnt cases");
  static_assert(NST * 2 * TB * KST * 2 >= NCW * 4 * 16 * 64 * 4, "ring holds the split-k partials");
  static_assert(!C::SPLITK || (KST / 16) % NCW == 0, "k steps per stage split evenly");
  // [stage][X tile, weight tile][TB x KST]
  __shared__ __attribute__((aligned(1024))) uint16_t tiles[NST][2][TB * KST];
  // Waves 0..NCW-1 compute, the others fill the LDS ring, so loading and
  // computing overlap.
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool producer = wv >= NCW;
  const int w = producer ? wv - NCW : wv;
  // XCD-aware tile order: workgroup L runs on XCD L % 8, and each XCD takes a
  // contiguous eighth of the tiles, column tiles fastest: the column tiles
  // that share rows of X run on one XCD, and few token tiles still spread
  // over all of them (16 tokens x 2304 columns: 31.6 us with all column tiles
  // of a token tile on one XCD, 19.1 us so; 4096 tokens: 109 -> 102 us).
  const int n_tiles = n_ct * n_tt, per = (n_tiles + NXCD - 1) / NXCD;
  const int tile = (int)(blockIdx.x % NXCD) * per + (int)(blockIdx.x / NXCD);
  if ((int)(blockIdx.x / NXCD) >= per || tile >= n_tiles) return;  // padding of the grid (uniform over the workgroup)
  const int ct = tile % n_ct, tt = tile / n_ct;
  const int col0 = ct * TB;
  const int64_t tok0 = (int64_t)tt * TB;
  // Column regions (tiles never straddle them: nkv is a multiple of TB):
  // keys, values, then LR columns.
  const int region = col0 < a.nkv ? 0 : (col0 < 2 * a.nkv ? 1 : 2);
  const int lcol0 = col0 - 2 * a.nkv;  // first LR column of an LR tile
  const int cols = region < 2 ? TB : (a.n_cols - lcol0 < TB ? a.n_cols - lcol0 : TB);  // valid columns
  const int toks = (int)(a.T - tok0 < TB ? a.T - tok0 : (int64_t)TB);  // valid rows of the X tile
  const int64_t ldw = region < 2 ? 2 * (int64_t)a.nkv : (int64_t)a.n_cols;  // weight row stride (elements)
  const i32x4 rw = buffer_rsrc(region < 2 ? a.W : a.A, (int32_t)(a.d_in * ldw * 2));
  const i32x4 rx = buffer_rsrc(a.X + tok0 * a.ld_x, (int32_t)((toks - 1) * a.ld_x * 2 + a.d_in * 2));

  // Loader: each instruction writes 1 KB (whole rows) at consecutive LDS
  // positions.  Lane i of an X instruction holds physical chunk i % XCPR of
  // token row XRPW w + XRPI j + i / XCPR, i.e. logical chunk swx(row, i % XCPR);
  // lane i of a weight instruction physical chunk i % WCPR of k row
  // WRPW w + WRPI j + i / WCPR.
  int32_t offx[C::NIX], kch[C::NIX], offw[C::NIW], krow[C::NIW];
#pragma unroll
  for (int j = 0; j < C::NIX; ++j) {
    const int row = C::XRPW * w + C::XRPI * j + lane / C::XCPR;
    const int c = C::swx(row, lane % C::XCPR);
    kch[j] = c * 8;  // first k of this lane's chunk within a stage
    offx[j] = row * (int32_t)(a.ld_x * 2) + c * 16;
  }
#pragma unroll
  for (int j = 0; j < C::NIW; ++j) {
    const int row = C::WRPW * w + C::WRPI * j + lane / C::WCPR;
    const int c = C::sww(row, lane % C::WCPR);
    int wcol;
    if (region == 0) wcol = key_wcol(col0 + 8 * c, a.head_dim);
    else if (region == 1) wcol = col0 + 8 * c;  // W_v columns follow W_k's
    else wcol = lcol0 + 8 * c;
    krow[j] = row;
    offw[j] = 8 * c < cols ? row * (int32_t)(ldw * 2) + wcol * 2 : INT32_MIN;  // LR columns past n_cols: zeros
  }
  const int nstage = (int)((a.d_in + KST - 1) / KST);
  // Each token tile walks the k stages from its own starting point (the
  // column tiles that share its X rows use the same one), so that at any
  // moment the workgroups read rows at different k offsets: with row strides
  // that are multiples of 4 KB, equal offsets would all hit the same few L2
  // channels.
  const int rot = (int)(((int64_t)tt * nstage) / n_tt);
  auto issue = [&](int s) {
    const int sl = s % NST;
    const int ks = s + rot < nstage ? s + rot : s + rot - nstage;
    const int32_t k0 = ks * KST;
#pragma unroll
    for (int j = 0; j < C::NIX; ++j) {
      // Chunks wholly past d_in (d_in is a multiple of 8) read as zeros.
      const int32_t ox = k0 + kch[j] < a.d_in ? offx[j] : INT32_MIN;
      lds_dma16(rx, &tiles[sl][0][(C::XRPW * w + C::XRPI * j) * KST], ox, k0 * 2);
    }
#pragma unroll
    for (int j = 0; j < C::NIW; ++j) {
      // k rows past d_in read as zeros; the whole offset is range-checked.
      const int32_t ow =
          (k0 + krow[j] < a.d_in && offw[j] != INT32_MIN) ? offw[j] + k0 * (int32_t)(ldw * 2) : INT32_MIN;
      lds_dma16(rw, &tiles[sl][1][(C::WRPW * w + C::WRPI * j) * TB], ow, 0);
    }
  };

  f32x16 acc[2][2];
  if (producer) {
    // Stage s + AHEAD goes into the slot of stage s - 2, which the compute
    // waves finished before the previous barrier, so it is issued before
    // waiting for stage s: issuing overlaps the wait.
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
      if (s < nstage) issue(s);
    for (int s = 0; s < nstage; ++s) {
      if (s + AHEAD < nstage) issue(s + AHEAD);
      // Stage s has landed once at most the loads of the stages after it (up
      // to AHEAD of them, NIX + NIW instructions each) are still in flight.
      const int ahead = nstage - 1 - s < AHEAD ? nstage - 1 - s : AHEAD;
      wait_vmcnt_le((C::NIX + C::NIW) * ahead);
      __syncthreads();  // stage s visible to all waves
    }
  } else {
    // Compute: a 64 x 64 block of columns cw0 .. and tokens tw0 ..
    // (split k: the whole tile, k steps kk with kk % 4 == w).
    const int l32 = lane & 31, h = lane >> 5, grp = lane >> 4, i16 = lane & 15;
    const int cw0 = C::SPLITK ? 0 : 64 * (w & 1), tw0 = C::SPLITK ? 0 : 64 * (w >> 1);
#pragma unroll
    for (int bc = 0; bc < 2; ++bc)
#pragma unroll
      for (int bt = 0; bt < 2; ++bt)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[bc][bt][j] = 0.f;
    // Transposing-read address of this lane within a k16 step: k row
    // 8 (grp / 2) + i16 / 4 (+4 for the second read), columns
    // (grp % 2) * 16 + 4 (i16 % 4) .. + 3 of each 32-column block.
    const int tr_k = 8 * (grp >> 1) + (i16 >> 2);
    const int tr_c = (grp & 1) * 16 + 4 * (i16 & 3);
    auto wfrag = [&](const uint16_t* tw, int kr, int col) {
      const int ch = col >> 3;
      return tw + kr * TB + C::sww(kr, ch) * 8 + (col & 7);
    };
    constexpr int KK = KST / 16;
    for (int s = 0; s < nstage; ++s) {
      __syncthreads();  // stage s visible to all waves; stage s - 1 consumed by all
      const uint16_t* tx = tiles[s % NST][0];
      const uint16_t* tw = tiles[s % NST][1];
#pragma unroll
      for (int ki = 0; ki < (C::SPLITK ? KK / NCW : KK); ++ki) {
        const int kk = C::SPLITK ? ki * NCW + w : ki;
        bf16x8 fa[2], fx[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int kr = 16 * kk + tr_k, col = cw0 + 32 * b + tr_c;
          const u32x2 lo = lds_read_tr(wfrag(tw, kr, col)), hi = lds_read_tr(wfrag(tw, kr + 4, col));
          fa[b] = as_bf16x8(u32x4{lo[0], lo[1], hi[0], hi[1]});
          const int xr = tw0 + 32 * b + l32, c = 2 * kk + h;
          fx[b] = as_bf16x8(*reinterpret_cast<const u32x4*>(tx + xr * KST + C::swx(xr, c) * 8));
        }
#pragma unroll
        for (int bc = 0; bc < 2; ++bc)
#pragma unroll
          for (int bt = 0; bt < 2; ++bt) acc[bc][bt] = mfma32x32x16(fa[bc], fx[bt], acc[bc][bt]);
      }
    }
  }

  // Which 32 x 32 blocks this wave writes: split k sums the four waves'
  // partials through LDS (the ring is free once every wave is past the last
  // stage) in a fixed order, and wave w writes block (w & 1, w >> 1).
  if constexpr (C::SPLITK) {
    float* part = reinterpret_cast<float*>(&tiles[0][0][0]);  // [wave][bc][bt][16][64]
    __syncthreads();  // every wave is past the last stage
    if (!producer) {
#pragma unroll
      for (int bc = 0; bc < 2; ++bc)
#pragma unroll
        for (int bt = 0; bt < 2; ++bt)
#pragma unroll
          for (int j = 0; j < 16; ++j) part[(((w * 2 + bc) * 2 + bt) * 16 + j) * 64 + lane] = acc[bc][bt][j];
    }
    __syncthreads();
    if (producer) return;
    const int bc = w & 1, bt = w >> 1;
    f32x16 sum;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      float v = 0.f;
#pragma unroll
      for (int ww = 0; ww < NCW; ++ww) v += part[(((ww * 2 + bc) * 2 + bt) * 16 + j) * 64 + lane];
      sum[j] = v;
    }
    acc[0][0] = sum;
  } else {
    if (producer) return;
  }

  // acc[bc][bt][j]: column cw + 32 bc + (j / 4) * 8 + h * 4 + j % 4, token
  // tw + 32 bt + l32 (split k: the one block acc[0][0] at (32 (w & 1), 32 (w >> 1))).
  const int l32 = lane & 31, h = lane >> 5;
  const int cw = C::SPLITK ? 32 * (w & 1) : 64 * (w & 1), tw = C::SPLITK ? 32 * (w >> 1) : 64 * (w >> 1);
  constexpr int NBLK = C::SPLITK ? 1 : 2;
#pragma unroll
  for (int bt = 0; bt < NBLK; ++bt)
#pragma unroll
    for (int bc = 0; bc < NBLK; ++bc)
      store_block(a, acc[bc][bt], region, col0 + cw + 32 * bc, tok0 + tw + 32 * bt + l32, h);
}

template <int TB>
hipError_t launch_tb(const PrecomputeArgs& a, hipStream_t st) {
  const int n_ct = 2 * a.nkv / TB + (a.n_cols + TB - 1) / TB;
  const int n_tt = (int)((a.T + TB - 1) / TB);
  const int grid = (n_ct * n_tt + NXCD - 1) / NXCD * NXCD;
  hipLaunchKernelGGL((precompute_kernel<TB>), dim3(grid), dim3((NCW + NPW) * 64), 0, st, a, n_ct, n_tt);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Wide problems (the joined projection of a long segment).  A CU streams its
// tile's operands at a fixed rate (about 30 bytes a clock here), so a 128 x 128
// tile is bound by its 256 rows of loads, and 576 such tiles (4096 x 2304) are
// 2.25 rounds of the CUs besides.  This kernel takes 256 tokens x 16 NB columns
// per workgroup: 1.5 times the flops per byte, and the launch picks NB so that
// the tiles come out near a whole number of rounds.
// Four compute waves (2 x 2, each 128 tokens x 8 NB columns on 16x16x32 MFMAs)
// and four loader waves filling a three-stage LDS ring of 64 k with direct
// global->LDS loads.  X rows are XOR-swizzled in 16-byte chunks; weight rows
// lie as in memory, in 16-column units, rotated by row so that the eight rows
// a transposing read serves together (two groups of four, 8 rows apart) hit
// different banks.  A unit holds 16 value or LR columns, or 8 key dims and
// their 8 RoPE partners (which land in lanes l and l ^ 32 of the result).
// 4096 x 2304, d_in 4096: 107 us with 128 x 128 tiles, 69 us (1.12 PFLOP/s)
// with 256 x 160; alone on its CU a 256 x 160 tile takes 56 us, 33 of them
// MFMAs at their full rate and about 10 before the first stage and after the
// last.  Measured and slower (against 71 then): fragments read at the head of
// each stage instead of between the MFMAs of the step before (77 us); the compute waves issuing
// the weight loads (80 us: a full load queue stalls their MFMAs too).
constexpr int WD_TT = 256;  // tokens per workgroup
constexpr int WD_KS = 64;   // k per stage
constexpr int WD_NST = 3;   // stages
constexpr int WD_NL = 4;    // loader waves

template <int NB>
struct Wide {
  static constexpr int UW = NB / 2;  // units per compute wave
  static constexpr int XB = WD_TT * WD_KS * 2, WB = WD_KS * NB * 32, SB = XB + WB;  // bytes per stage
  static constexpr int NXI = XB / 1024, NWI = WB / 1024, NI = (NXI + NWI) / WD_NL;  // 1 KB loads; per loader wave
  static_assert(NB % 2 == 0 && (NXI + NWI) % WD_NL == 0 && WB % 1024 == 0, "even shares");
  // Units by which row r of the weight tile is rotated: the bank of unit u is
  // (r NB + u) mod 8 groups of 8 banks.
  static __device__ __forceinline__ int rot(int r) { return NB % 8 == 0 ? (r & 3) + 4 * ((r >> 3) & 1) : (r >> 3) & 1; }
};

template <int NB>
__global__ void __launch_bounds__((4 + WD_NL) * 64, 2) project_wide_kernel(const PrecomputeArgs a, int n_wt, int n_ct, int n_tt) {
  using C = Wide<NB>;
  __shared__ __attribute__((aligned(1024))) char ring[WD_NST * C::SB];
  __shared__ double w2pi_lds[kMaxHalfDim];  // the epilogue's RoPE frequencies
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Each XCD takes a contiguous eighth of the tiles, column tiles fastest.
  const int n_tiles = n_ct * n_tt, per = (n_tiles + NXCD - 1) / NXCD;
  const int tile = (int)(blockIdx.x % NXCD) * per + (int)(blockIdx.x / NXCD);
  if ((int)(blockIdx.x / NXCD) >= per || tile >= n_tiles) return;  // uniform over the workgroup
  const int ct = tile % n_ct, tt = tile / n_ct;
  const int64_t tok0 = (int64_t)tt * WD_TT;
  const int toks = (int)(a.T - tok0 < WD_TT ? a.T - tok0 : (int64_t)WD_TT);
  // Column tiles 0 .. n_wt - 1 are units of W (n_ku key units, then as many of
  // values), the others of A.
  const bool lr = ct >= n_wt;
  const int half = a.head_dim / 2, n_ku = a.nkv / 16;
  const int u0 = (lr ? ct - n_wt : ct) * NB, n_un = lr ? (a.n_cols + 15) / 16 : 2 * n_ku;  // first unit; units of the matrix
  const int d_in = (int)a.d_in, nstage = (d_in + WD_KS - 1) / WD_KS;
  // First column of 8-column chunk hc of unit U within its weight matrix.
  auto unit_col = [&](int U, int hc) {
    if (lr || U >= n_ku) return U * 16 + hc * 8;  // value units follow the key units' nkv columns
    const int hd = U * 8 / half;
    return hd * a.head_dim + (U * 8 - hd * half) + hc * half;
  };

  if (wv >= 4) {
    // ---- loaders ---------------------------------------------------------------
    const int w = wv - 4;
    const int32_t ldw = lr ? a.n_cols * 2 : a.nkv * 4;  // weight row stride (bytes)
    const i32x4 rx = buffer_rsrc(a.X + tok0 * a.ld_x, (int32_t)((toks - 1) * a.ld_x * 2 + a.d_in * 2));
    const i32x4 rw = buffer_rsrc(lr ? a.A : a.W, d_in * ldw);
    // Instruction j of this wave is load j WD_NL + w of the stage: X rows
    // first, then weight rows.  Offsets at k = 0 (INT32_MIN: columns past the
    // matrix, read as zeros) and each lane's first k.
    int32_t off[C::NI], kof[C::NI];
#pragma unroll
    for (int j = 0; j < C::NI; ++j) {
      const int li = j * WD_NL + w;
      if (j * WD_NL < C::NXI) {
        const int r = li * 8 + lane / 8, c = (lane % 8) ^ ((r >> 1) & 7);
        kof[j] = c * 8;
        off[j] = r * (int32_t)(a.ld_x * 2) + c * 16;
      } else {
        const int b = (li - C::NXI) * 1024 + lane * 16, r = b / (NB * 32), pc = (b % (NB * 32)) / 16;
        const int U = u0 + (pc / 2 + NB - C::rot(r)) % NB, hc = pc % 2;  // the unit stored here
        const int col = unit_col(U, hc);
        kof[j] = r;
        off[j] = U < n_un && (!lr || col < a.n_cols) ? r * ldw + col * 2 : INT32_MIN;
      }
    }
    auto issue = [&](int s) {
      char* st = ring + (s % WD_NST) * C::SB;
      const int k0 = s * WD_KS;
      if (k0 + WD_KS <= d_in) {  // whole stage: the k offset is scalar
#pragma unroll
        for (int j = 0; j < C::NI; ++j) {
          const int li = j * WD_NL + w;
          if (j * WD_NL < C::NXI) lds_dma16(rx, st + li * 1024, off[j], k0 * 2);
          else lds_dma16(rw, st + C::XB + (li - C::NXI) * 1024, off[j], k0 * ldw);
        }
        return;
      }
#pragma unroll
      for (int j = 0; j < C::NI; ++j) {
        const int li = j * WD_NL + w;
        const bool ok = k0 + kof[j] < d_in && off[j] != INT32_MIN;
        if (j * WD_NL < C::NXI)
          lds_dma16(rx, st + li * 1024, ok ? off[j] + k0 * 2 : INT32_MIN, 0);
        else
          lds_dma16(rw, st + C::XB + (li - C::NXI) * 1024, ok ? off[j] + k0 * ldw : INT32_MIN, 0);
      }
    };
    static_assert(C::NXI % WD_NL == 0 && C::NI < 64, "X and weight loads are separate instructions of every wave");
    issue(0);
    if (nstage > 1) issue(1);
    for (int s = 0; s < nstage; ++s) {
      // Stage s has landed once only stage s + 1's loads are still in flight.
      if (s + 1 < nstage) __builtin_amdgcn_s_waitcnt(vmcnt_imm(C::NI));
      else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __syncthreads();  // stage s visible to all; stage s - 1 consumed by all
      if (s + 2 < nstage) issue(s + 2);  // into the slot of stage s - 1
    }
    return;
  }

  if (!lr && tid < half) w2pi_lds[tid] = a.w2pi[tid];
  // ---- compute waves -------------------------------------------------------------
  const int q = lane >> 4, c16 = lane & 15, wr = wv >> 1, wc = wv & 1;
  f32x4 acc[C::UW][8];
#pragma unroll
  for (int u = 0; u < C::UW; ++u)
#pragma unroll
    for (int m = 0; m < 8; ++m) acc[u][m] = f32x4{0.f, 0.f, 0.f, 0.f};
  // LDS byte offsets of this lane within a stage: X rows 128 wr + 16 m + c16,
  // chunk 4 kk + q; weight rows 32 kk + 8 q + c16 / 4 (+ 4), columns
  // 4 (c16 % 4) .. + 3 of each unit.
  const int xo = (128 * wr + c16) * (WD_KS * 2), xs = (c16 >> 1) & 7;
  const int kr = 8 * q + (c16 >> 2), rt = C::rot(kr);  // rows kr + 32 kk and kr + 4 rotate alike
  int wo[C::UW];
#pragma unroll
  for (int u = 0; u < C::UW; ++u)
    wo[u] = C::XB + kr * (NB * 32) + ((wc * C::UW + u + rt) % NB) * 32 + (c16 & 3) * 8;
  // Software pipeline over k32 steps: the weight fragments of the next step and
  // the X fragments four token blocks ahead are read between the MFMAs of this
  // one (a second full set of X fragments would not fit the registers).  The barrier that publishes
  // stage s + 1 sits in the middle of the last step of stage s, after its last
  // read, so that the MFMAs of four token blocks cover the first reads of the
  // next stage (one compute wave per SIMD: nothing else does).
  u32x2 fwl[2][C::UW], fwh[2][C::UW];
  u32x4 fx[4];
  auto read_w = [&](int set, int u, const char* st, int kk) {
    const char* p = st + wo[u] + 32 * kk * (NB * 32);
    fwl[set][u] = lds_read_tr(reinterpret_cast<const uint16_t*>(p));
    fwh[set][u] = lds_read_tr(reinterpret_cast<const uint16_t*>(p + 4 * (NB * 32)));
  };
  auto read_x = [&](int m, const char* st, int kk) {
    fx[m % 4] = *reinterpret_cast<const u32x4*>(st + xo + m * (16 * WD_KS * 2) + (((4 * kk + q) ^ xs) * 16));
  };
  __syncthreads();  // stage 0 visible
#pragma unroll
  for (int u = 0; u < C::UW; ++u) read_w(0, u, ring, 0);
#pragma unroll
  for (int m = 0; m < 4; ++m) read_x(m, ring, 0);
  const char* st = ring;
  int slot = 0;
  for (int s = 0; s < nstage; ++s) {
    slot = slot + 1 == WD_NST ? 0 : slot + 1;
    const char* stn = ring + slot * C::SB;  // stage s + 1 (past the last: stale rows, unused)
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        if (kk == 1 && m == 4) {
          __builtin_amdgcn_sched_barrier(0);
          if (s + 1 < nstage) __syncthreads();  // stage s + 1 visible; stage s consumed
          __builtin_amdgcn_sched_barrier(0);
        }
        const bf16x8 x = as_bf16x8(fx[m % 4]);
#pragma unroll
        for (int u = 0; u < C::UW; ++u)
          acc[u][m] = mfma16x16x32(
              as_bf16x8(u32x4{fwl[kk][u][0], fwl[kk][u][1], fwh[kk][u][0], fwh[kk][u][1]}), x, acc[u][m]);
        if (m < 4) read_x(m + 4, st, kk);
        else read_x(m - 4, kk == 0 ? st : stn, kk ^ 1);
        // Weight fragments of the next step, spread over this one's blocks
        // (the second step's only after the barrier).
#pragma unroll
        for (int u = 0; u < C::UW; ++u)
          if (kk == 0 ? u == m : u * 4 / C::UW == m - 4) read_w(kk ^ 1, u, kk == 0 ? st : stn, kk ^ 1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    st = stn;
  }

  // acc[u][m][i]: column 4 q + i of unit u0 + wc UW + u, token 128 wr + 16 m + c16.
  int64_t rowm[8];  // cache row of each token block's token of this lane
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int64_t trow = a.tok_offset + tok0 + 128 * wr + 16 * m + c16;
    rowm[m] = 128 * wr + 16 * m + c16 < toks ? cache_row(a, trow) : 0;
  }
#pragma unroll
  for (int u = 0; u < C::UW; ++u) {
    const int U = u0 + wc * C::UW + u;
    if (U >= n_un) break;  // uniform over the wave
    if (!lr && U < n_ku) {
      // Keys: lanes q < 2 hold dims j .. j + 3, lanes q + 2 their partners.
      const int hd = U * 8 / half, j0 = U * 8 - hd * half + 4 * (q & 1);
      const int pos0 = (int)(a.tok_offset + tok0) + 128 * wr + c16;
      uint16_t* kp = a.Kout + hd * a.head_dim + j0 + (q >= 2 ? half : 0);
      double wj[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) wj[i] = w2pi_lds[j0 + i];
#pragma unroll
      for (int m = 0; m < 8; m += 2) {
        // Lanes l and l ^ 32 need the same angles, each reduced in fp64: one
        // forms those of token block m, the other those of m + 1, and they swap.
        float cs[2][4], sn[2][4], o[2][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float c, sw;
          rope_cs(pos0 + 16 * m + (q < 2 ? 0 : 16), wj[i], c, sw);
          const auto rc = __builtin_amdgcn_permlane32_swap(__float_as_uint(c), __float_as_uint(c), false, false);
          const auto rs = __builtin_amdgcn_permlane32_swap(__float_as_uint(sw), __float_as_uint(sw), false, false);
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            cs[e][i] = __uint_as_float(rc[e]);
            sn[e][i] = __uint_as_float(rs[e]);
          }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t v = __float_as_uint(acc[u][m + e][i]);
            const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
            const float x = __uint_as_float(r[0]), y = __uint_as_float(r[1]);  // lanes l % 32 and l % 32 + 32
            o[e][i] = q < 2 ? x * cs[e][i] - y * sn[e][i] : y * cs[e][i] + x * sn[e][i];
          }
          if (128 * wr + 16 * (m + e) + c16 < toks)
            *reinterpret_cast<u32x2*>(kp + rowm[m + e] * a.nkv) = u32x2{pack_bf16(o[e][0], o[e][1]), pack_bf16(o[e][2], o[e][3])};
        }
      }
      continue;
    }
    uint16_t* op;
    int64_t ld;
    const int c = U * 16 + 4 * q;
    if (lr) {
      if (c >= a.n_cols) continue;
      const int64_t plane = c / a.rank;
      op = a.L + plane * a.s_cap * a.rank + (c - plane * a.rank);
      ld = a.rank;
    } else {
      op = a.Vout + (c - a.nkv);
      ld = a.nkv;
    }
#pragma unroll
    for (int m = 0; m < 8; ++m)
      if (128 * wr + 16 * m + c16 < toks)
        *reinterpret_cast<u32x2*>(op + rowm[m] * ld) =
            u32x2{pack_bf16(acc[u][m][0], acc[u][m][1]), pack_bf16(acc[u][m][2], acc[u][m][3])};
  }
}

template <int NB>
int64_t wide_tiles(const PrecomputeArgs& a, int* n_wt, int* n_ct) {
  *n_wt = (a.nkv / 8 + NB - 1) / NB;
  *n_ct = *n_wt + ((a.n_cols + 15) / 16 + NB - 1) / NB;
  return (int64_t)*n_ct * ((a.T + WD_TT - 1) / WD_TT);
}

template <int NB>
hipError_t launch_wide(const PrecomputeArgs& a, hipStream_t st) {
  int n_wt, n_ct;
  const int64_t tiles = wide_tiles<NB>(a, &n_wt, &n_ct);
  hipLaunchKernelGGL((project_wide_kernel<NB>), dim3((unsigned)((tiles + NXCD - 1) / NXCD * NXCD)), dim3((4 + WD_NL) * 64), 0,
                     st, a, n_wt, n_ct, (int)((a.T + WD_TT - 1) / WD_TT));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// LR precompute of few rows or few columns: not enough 64 x 64 tiles to occupy
// the chip (512 rows x 128 columns make 16).  A CU streams its operands at a
// fixed rate, so what counts is the bytes of one workgroup's tile: 16 tokens x
// 32 columns here, 48 rows of k against 128, over eight times the workgroups.
// The eight waves each take a slice of k and are summed through LDS in a fixed
// order.  Nothing is staged in LDS: a lane loads 16 bytes of a token row of X
// (the MFMA B operand as it is) and two columns of eight weight rows, which it
// transposes in registers (v_perm_b32) into two A fragments: fragment j holds
// columns 2 c + j, c = lane % 16.
// Measured, d_in 4096, against 64 x 64 tiles: 512 x 128 17.6 -> 12.3 us, 64 x
// 256 17.3 -> 9.8 us, 1000 x 128 17.6 -> 13.0 us, 512 x 256 (one workgroup per
// CU) 17.8 -> 13.8 us; 1500 x 256 (three per CU) 18.0 -> 30.9 us.  Larger tiles
// of this form (32 x 32, 16 x 64, 32 x 64) and deeper rings measured slower.
constexpr int SM_W = 8;   // waves per workgroup (k slices)
constexpr int SM_U = 4;   // 32-k steps in flight per wave
constexpr int SM_TC = 32, SM_TT = 16;  // columns and tokens per workgroup

__global__ void __launch_bounds__(SM_W * 64) precompute_small_kernel(const PrecomputeArgs a) {
  __shared__ float part[SM_W][8][64];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, c16 = lane & 15;
  const int c0 = blockIdx.x * SM_TC;
  const int64_t tok0 = (int64_t)blockIdx.y * SM_TT;
  const int toks = (int)(a.T - tok0 < SM_TT ? a.T - tok0 : (int64_t)SM_TT);
  const int32_t ldw2 = a.n_cols * 2, ldx2 = (int32_t)(a.ld_x * 2), d_in = (int32_t)a.d_in;
  const auto rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.A), (short)0, d_in * ldw2, 0x00020000);
  const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.X + tok0 * a.ld_x), (short)0,
                                                    (toks - 1) * ldx2 + d_in * 2, 0x00020000);
  const int nk = (d_in + 31) / 32;  // 32-k steps; this wave's slice of them
  const int s_lo = nk * w / SM_W, s_hi = nk * (w + 1) / SM_W;
  // Per-lane byte offsets; a step adds uniform strides.  Columns past n_cols,
  // chunks of X past d_in and steps past the slice are pointed out of range,
  // weight rows past d_in fall outside their resource: all read as zeros.
  const bool col_ok = c0 + 2 * c16 < a.n_cols;  // n_cols is a multiple of 8
  const int32_t woff = 8 * q * ldw2 + (c0 + 2 * c16) * 2, xoff = c16 * ldx2 + 16 * q;
  struct Step {
    uint32_t w[8];  // two columns of rows 32 s + 8 q + i
    u32x4 x;        // X of token c16, k = 32 s + 8 q ..
  };
  auto load = [&](Step& st, int s) {
    const int32_t wo = s < s_hi && col_ok ? woff + s * 32 * ldw2 : INT32_MIN;
    const int32_t xo = s < s_hi && 32 * s + 8 * q < d_in ? xoff + 64 * s : INT32_MIN;  // d_in is a multiple of 8
#pragma unroll
    for (int i = 0; i < 8; ++i) st.w[i] = __builtin_amdgcn_raw_buffer_load_b32(rw, wo + i * ldw2, 0, 0);
    st.x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, xo, 0, 0));
  };
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  Step ring[SM_U];
#pragma unroll
  for (int u = 0; u < SM_U; ++u) load(ring[u], s_lo + u);
  for (int s = s_lo; s < s_hi; s += SM_U) {
#pragma unroll
    for (int u = 0; u < SM_U; ++u) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        u32x4 f;
#pragma unroll
        for (int p = 0; p < 4; ++p)
          f[p] = __builtin_amdgcn_perm(ring[u].w[2 * p + 1], ring[u].w[2 * p], j ? 0x07060302u : 0x05040100u);
        acc[j] = mfma16x16x32(as_bf16x8(f), as_bf16x8(ring[u].x), acc[j]);
      }
      load(ring[u], s + SM_U + u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) part[w][4 * j + i][lane] = acc[j][i];
  __syncthreads();
  // Columns 2 c, 2 c + 1 of token t, one thread each: lane 16 (c / 4) + t of
  // rows c % 4 and 4 + c % 4.
  if (tid >= SM_TT * SM_TC / 2) return;
  const int t = tid / (SM_TC / 2), c = tid % (SM_TC / 2), col = c0 + 2 * c;
  if (t >= toks || col >= a.n_cols) return;
  float v[2] = {0.f, 0.f};
#pragma unroll
  for (int ww = 0; ww < SM_W; ++ww)
#pragma unroll
    for (int j = 0; j < 2; ++j) v[j] += part[ww][4 * j + c % 4][16 * (c / 4) + t];
  const int64_t plane = col / a.rank, jr = col - plane * a.rank;
  *reinterpret_cast<uint32_t*>(a.L + (plane * a.s_cap + cache_row(a, a.tok_offset + tok0 + t)) * a.rank + jr) =
      pack_bf16(v[0], v[1]);
}

// A handful of rows (the K/V and LR rows of newly decoded tokens) is a
// matrix-vector product.  One workgroup per 8 output columns (a key
// workgroup: 8 dims of a head and their RoPE partners d/2 further on), so the
// weights are spread over many workgroups.  Thread t takes the k rows
// 8t .. 8t + 7 (+ 4096 per round, so a 4096-wide hidden state is one round
// with all of a thread's loads in flight at once): one 16-byte load of each
// of the T <= GV_T rows of X, and one 16-byte load (8 columns) of each weight
// row.  The partial sums are reduced over the lanes by shuffles and over the
// waves in LDS.
constexpr int GV_T = 4;
constexpr int GV_W = 8;  // waves per workgroup

__global__ void __launch_bounds__(64 * GV_W) project_gemv_kernel(const PrecomputeArgs a, int n_units) {
  __shared__ float red[GV_W][2][GV_T][8];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // The 8 workgroups whose columns share 128-byte lines of the weight rows run
  // on one XCD (workgroup L runs on XCD L % 8), so each line is fetched into
  // one L2 only.
  const int L = blockIdx.x, slot = L / NXCD;
  const int u = 8 * ((slot / 8) * NXCD + L % NXCD) + slot % 8;
  if (u >= n_units) return;
  const int half = a.head_dim / 2;
  const int n_pair = a.nkv / 16;  // key workgroups (8 pair columns each)
  const int n_val = a.nkv / 8;
  // Region of this workgroup: 0 keys (dims j0 .. j0+7 and their partners), 1
  // values, 2 LR.
  int region, c0;
  const uint16_t* w0;
  const uint16_t* w1 = nullptr;
  int64_t ldw;
  if (u < n_pair) {
    region = 0;
    const int hd = (u * 8) / half, j0 = u * 8 - hd * half;
    c0 = hd * a.head_dim + j0;  // first dim (column of W_k) of the low half
    ldw = 2 * (int64_t)a.nkv;
    w0 = a.W + c0;
    w1 = w0 + half;
  } else if (u < n_pair + n_val) {
    region = 1;
    c0 = (u - n_pair) * 8;
    ldw = 2 * (int64_t)a.nkv;
    w0 = a.W + a.nkv + c0;
  } else {
    region = 2;
    c0 = (u - n_pair - n_val) * 8;
    ldw = a.n_cols;
    w0 = a.A + c0;
  }
  const int T = (int)a.T;
  float acc0[GV_T][8], acc1[GV_T][8];
#pragma unroll
  for (int t = 0; t < GV_T; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc0[t][e] = acc1[t][e] = 0.f;
  for (int64_t k0 = (int64_t)tid * 8; k0 < a.d_in; k0 += 64 * GV_W * 8) {
    float x[GV_T][8];
#pragma unroll
    for (int t = 0; t < GV_T; ++t) {
      const u32x4 xv = ld16(a.X + t * a.ld_x + k0, t < T);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[t][2 * e] = bf_lo(xv[e]);
        x[t][2 * e + 1] = bf_hi(xv[e]);
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t k = k0 + i;  // d_in is a multiple of 8: k < d_in
      const u32x4 wv = *reinterpret_cast<const u32x4*>(w0 + k * ldw);
      float wf[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        wf[2 * e] = bf_lo(wv[e]);
        wf[2 * e + 1] = bf_hi(wv[e]);
      }
#pragma unroll
      for (int t = 0; t < GV_T; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc0[t][e] += x[t][i] * wf[e];
      if (region == 0) {  // uniform over the workgroup
        const u32x4 wv1 = *reinterpret_cast<const u32x4*>(w1 + k * ldw);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          wf[2 * e] = bf_lo(wv1[e]);
          wf[2 * e + 1] = bf_hi(wv1[e]);
        }
#pragma unroll
        for (int t = 0; t < GV_T; ++t)
#pragma unroll
          for (int e = 0; e < 8; ++e) acc1[t][e] += x[t][i] * wf[e];
      }
    }
  }
  // Sum each of the 32 (token, column) partials over the wave's lanes with a
  // transposing reduction: every step hands half of a lane's values to its
  // partner and adds the half it keeps, so after five steps lane l holds one
  // value, index (l >> 1) & 31, summed over the 32 lanes that share lane bit 0
  // (32 shuffles instead of 6 per value).
  auto reduce = [&](float (&acc)[GV_T][8]) -> float {
    float v[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = acc[i / 8][i % 8];
#pragma unroll
    for (int st = 0; st < 5; ++st) {
      const int m = 32 >> st, half = 16 >> st;
      const bool up = (lane & m) != 0;
#pragma unroll
      for (int i = 0; i < half; ++i) {
        const float send = up ? v[i] : v[i + half];
        const float keep = up ? v[i + half] : v[i];
        v[i] = keep + shfl_xor(send, m);
      }
    }
    return v[0] + shfl_xor(v[0], 1);
  };
  static_assert(GV_T * 8 == 32, "32 partials per lane");
  const float r0 = reduce(acc0);
  const float r1 = region == 0 ? reduce(acc1) : 0.f;  // uniform over the workgroup
  if ((lane & 1) == 0) {
    const int vi = (lane >> 1) & 31;
    red[w][0][vi / 8][vi % 8] = r0;
    red[w][1][vi / 8][vi % 8] = r1;
  }
  __syncthreads();
  if (tid >= T * 8) return;
  const int t = tid / 8, e = tid % 8;
  float x = 0.f, y = 0.f;
#pragma unroll
  for (int i = 0; i < GV_W; ++i) {
    x += red[i][0][t][e];
    y += red[i][1][t][e];
  }
  const int64_t pos = a.tok_offset + t;  // absolute position
  const int64_t row = cache_row(a, pos);
  if (region == 0) {
    const int hd = c0 / a.head_dim, j = c0 - hd * a.head_dim + e;
    float cs, sn;
    rope_cs((int)pos, a.w2pi[j], cs, sn);
    uint16_t* kp = a.Kout + row * a.nkv + hd * a.head_dim + j;
    kp[0] = (uint16_t)(pack_bf16(x * cs - y * sn, 0.f) & 0xffffu);
    kp[half] = (uint16_t)(pack_bf16(y * cs + x * sn, 0.f) & 0xffffu);
  } else if (region == 1) {
    a.Vout[row * a.nkv + c0 + e] = (uint16_t)(pack_bf16(x, 0.f) & 0xffffu);
  } else {
    const int c = c0 + e;
    const int64_t plane = c / a.rank, jr = c - plane * a.rank;
    a.L[(plane * a.s_cap + row) * a.rank + jr] = (uint16_t)(pack_bf16(x, 0.f) & 0xffffu);
  }
}

}  // namespace

hipError_t launch_precompute(const PrecomputeArgs& a, hipStream_t st) {
  const int64_t cus = a.cus;
  if (a.T <= GV_T) {
    const int units = a.nkv / 16 + a.nkv / 8 + a.n_cols / 8;
    hipLaunchKernelGGL(project_gemv_kernel, dim3(64 * ((units + 63) / 64)), dim3(64 * GV_W), 0, st, a, units);
    return hipGetLastError();
  }
  const auto cdiv = [](int64_t x, int64_t y) { return (x + y - 1) / y; };
  // LR rows alone: small tiles while they make at most one workgroup per CU
  // (beyond that they move more bytes per CU than 64 x 64 tiles do).
  const int64_t sm_x = cdiv(a.n_cols, SM_TC), sm_y = cdiv(a.T, SM_TT);
  if (a.nkv == 0 && sm_x * sm_y <= cus) {
    hipLaunchKernelGGL(precompute_small_kernel, dim3((unsigned)sm_x, (unsigned)sm_y), dim3(SM_W * 64), 0, st, a);
    return hipGetLastError();
  }
  // A CU takes one workgroup at a time, so a launch takes its rounds of the CUs
  // times the time of one tile: a fixed part and one that goes with d_in
  // (microseconds, the latter at 4096; measured at 256, 4096 and 5120 from 1 to
  // 600 tiles).  64 x 64 and 128 x 128 tiles are bound by the CU's load rate,
  // the 256-token ones by their MFMAs.  Over rounds that are nearly empty the
  // smaller tile wins (1000 tokens x 2304 columns: 57, 35, 48, 56, 65 us in
  // this order), over full ones the larger (4096 x 2304: 188, 107, 93, 97, 69
  // us; 2048 x 2816, d_in 5120: 148, 86, 67, 60, 71 us).  128-wide tiles need
  // the K/V boundary on a tile edge; 256-token tiles need their rows of X within
  // the 31 bits of their byte offsets (INT32_MIN, past them, marks what is not read).
  const bool wide_ok = a.ld_x * 2 * WD_TT <= (1LL << 31) - 2;
  int n_wt, n_ct;
  const double kd = (double)a.d_in / 4096.0;
  const auto model = [&](double fixed, double per_k, int64_t tiles) { return (fixed + per_k * kd) * (double)cdiv(tiles, cus); };
  const double t[5] = {
      model(2.7, 15.8, (2 * a.nkv / 64 + cdiv(a.n_cols, 64)) * cdiv(a.T, 64)),
      a.nkv % 128 == 0 ? model(5.0, 31.0, (2 * a.nkv / 128 + cdiv(a.n_cols, 128)) * cdiv(a.T, 128)) : 1e30,
      wide_ok ? model(5.0, 45.0, wide_tiles<6>(a, &n_wt, &n_ct)) : 1e30,
      wide_ok ? model(6.6, 42.4, wide_tiles<8>(a, &n_wt, &n_ct)) : 1e30,
      wide_ok ? model(8.4, 49.6, wide_tiles<10>(a, &n_wt, &n_ct)) : 1e30,
  };
  int best = 0;
  for (int i = 1; i < 5; ++i)
    if (t[i] < t[best]) best = i;
  switch (best) {
    case 0: return launch_tb<64>(a, st);
    case 1: return launch_tb<128>(a, st);
    case 2: return launch_wide<6>(a, st);
    case 3: return launch_wide<8>(a, st);
    default: return launch_wide<10>(a, st);
  }
}

}  // namespace prc
