// Tiled attention on the CDNA4 matrix cores, used for (a) the sparse attention stage of
// sea_forward when the mask has column structure (Sec. 3.1.1 rho, sigma, A* V with the mask of
// Sec. 3.1 "Linear Sparse Attention Mask Generation") and (b) the dense baseline
// softmax(QK^T)V (Sec. 3 "Preliminaries").
//
// Why tiles: every query row that selects compressed column c attends to the same r keys of
// that column, so the keys any row of a head can use form one fixed "compact" list of U = K r
// keys (all T keys when whole columns are emitted).  A wavefront takes 32 consecutive query
// rows and walks that list in chunks of 32 keys; a chunk no row of the tile selected is
// skipped, otherwise S^T = K_chunk Q_tile^T and O^T += V_chunk^T P^T run as
// v_mfma_f32_32x32x16_bf16 with per-(row, column) mask bits applied to S in registers.  K/V
// rows are thus read once per 32 query rows instead of once per row, and no T x T or T x L
// buffer exists.  The softmax is the streaming form; each lane owns one query (the MFMA
// output column), so row maxima and sums need a single cross-lane exchange.
//
// Operand layouts (32x32x16 bf16): A lane l = row l%32, contraction elems 8(l/32)..+7;
// B lane l = col l%32, same elems; C reg i = row 8(i/4) + 4(l/32) + i%4, col l%32.
// P leaves the first product in C layout (lane = query, regs = keys) and is fed back as the B
// operand of the second product; its register order fixes which key each contraction slot
// means, and the V^T fragments are fetched in that same order from LDS, where the value rows of a
// step are parked as they lie in memory and transposed on the way out by the LDS transpose read
// (the key and value rows themselves are gathered from K and V by position, so no compact or
// transposed copy exists in HBM).
#include "sea_columns.h"
#include "sea_gather.h"
#include "sea_internal.h"
#include "sea_tile.h"

#include <algorithm>
#include <type_traits>

namespace sea {
namespace {

struct TileArgs {
  const uint16_t* Q;    // [N][T][64]
  const uint16_t* K;    // [N][T][64]
  const uint16_t* V;    // [N][T][64]
  const uint32_t* mbits;  // [N][T][KW] selected-column bits, nullptr for dense
  uint16_t* O;          // [N][T][64]
  const int32_t* seq_len;
  int32_t N, H, T;
  int32_t U;            // compact keys per head: K r (all T keys when whole columns are emitted)
  int32_t KW;           // mask words per row
  int32_t rlog;         // log2(keys per column r)
  int32_t w;            // column width in keys
  int32_t causal;
  int32_t group_heads;  // heads per scheduling group (a multiple of 8 unless it is N)
  float c;              // scale * log2(e)
  // bucket mode (one selected column per row): rows grouped by their column
  const int32_t* perm;      // [N][entries] row id | slot << 24, bucket after bucket
  const int32_t* bstart;    // [N][K + 1] first perm slot of each column's bucket
  const int32_t* chunk_col; // [N][max_chunks] column of each 128-row chunk, -1 past the last
  const int32_t* cstart;    // [N][K + 1] first chunk of each column
  int32_t max_chunks, Kcols;
  int64_t perm_stride;  // entries per head in perm
  // several columns per row (2 <= k^ <= 8): each (row, selected column) pair is one bucket entry
  // whose normalised partial output and (reference maximum, sum) go here, merged per row later
  uint16_t* part_o;   // [N][T][slots][64] bf16, nullptr when k^ = 1
  float* part_ml;     // [N][T][slots][2]
  int32_t slots;
};

// position in the sequence of compact key u
__device__ __forceinline__ int32_t pos_of(int32_t u, int32_t rlog, int32_t w) {
  const int32_t col = u >> rlog, i = u & ((1 << rlog) - 1);
  return col * w + ((i * w) >> rlog);
}

// number of compact keys with position <= jmax (positions ascend with u)
__device__ __forceinline__ int32_t compact_count(int32_t jmax, int32_t rlog, int32_t w) {
  if (jmax < 0) return 0;
  const int32_t col = jmax / w, delta = jmax - col * w;
  const int32_t r = 1 << rlog;
  const int32_t inside = min(r, ((delta + 1) * r + w - 1) / w);
  return col * r + inside;
}

// Staged rows are 128 bytes without padding, two of them as wide as the banks.  K: the 16-byte part p of row r lies at
// slot p ^ (r / 2 & 7), so that the sixteen rows of sixteen neighbouring lanes' reads hit distinct banks (with r & 7
// only eight do: 0.41 against 0.19 conflict cycles per active one, the layers 0.3 % slower); V: the 64-byte halves of
// rows 2, 3 (mod 4) are exchanged, which does the same for the four rows of a transpose read.
constexpr int kRow = kHeadDim;

// waves per SIMD that a kernel's registers have to leave room for
constexpr int tile_waves(int RW, int NS, bool odd) { return NS > 1 ? 4 : (RW == 4 && odd ? 3 : 16 / RW); }

// Block = 4 waves = 128 consecutive query rows of one head (32 per wave); other splits below.  The block
// walks the compact key list in steps of 64 keys (two 32-key sub-chunks); each step's K and V rows are fetched
// once, straight to LDS as they lie in memory (double buffered, one barrier per step), and read by all four waves as
// MFMA fragments, those of V through the transpose read.
// RLOG = log2(keys per column) for 1..16 keys per column, 5 for 32 or more (then a 32-key
// sub-chunk lies inside one column and the actual shift is a.rlog).
//
// MODE 0: rows in sequence order, per-(row, column) mask bits.  MODE 1: dense baseline (no mask
// bits).  MODE 2: "bucket" form for k^ = 1 -- every row selected exactly one column, rows are
// grouped by that column, and a block takes 128 rows of one bucket against the r keys of its
// column, so every visited tile is fully used no matter how scattered the choices are.
// ODD: K or V starts between two 4-byte words, so a step's pieces wait in registers.
template <int RLOG, int MODE, int RW = 4, int NS = 1, int SC = 2, bool ODD = false>
__global__ __launch_bounds__(64 * RW * NS, tile_waves(RW, NS, ODD)) void tile_attn_kernel(TileArgs a) {
  // RW = waves side by side: 32 RW query rows share every staged key step (8 instead of 4 halve the bytes a
  // head's keys and values travel from the L2s to LDS; two blocks per CU).
  // NS = sets of RW waves that share the block's rows: each takes every NS-th SC sub-chunks of the list, and
  // the partial results are merged through LDS at the end.
  static_assert(MODE != 2 || (RW == 4 && NS == 1), "bucket chunks are 128 rows");
  static_assert(NS > 1 || SC == 2, "one set takes whole chunks");
  constexpr int kRows = 32 * RW, kThreads = 64 * RW * NS;
  constexpr int kStep = 32 * SC * NS;        // keys per step
  constexpr bool kTwo = 8 * kStep == 2 * kThreads;  // K and V pieces per thread and step: two or one
  static_assert(kTwo || 8 * kStep == kThreads, "one or two pieces");
  constexpr bool DENSE = MODE == 1 || MODE == 2;  // no per-column bits to look up
  constexpr bool BUCKET = MODE == 2;
  // MODE 3: one bit per (row, key) in HBM ([N][T][KW] words); a lane reads its row's two words of a
  // step straight from memory one step ahead, nothing of the mask is parked in LDS
  constexpr bool STREAM = MODE == 3;
  __shared__ __attribute__((aligned(16))) uint16_t KVs[2][2][kStep * kRow];  // [place][K, V]
  // selected-column bits of the block's rows, KW words per row (K <= 1024: at most 16 KB)
  extern __shared__ uint32_t Ms[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wall = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, keep it scalar
  const int wid = NS > 1 ? wall % RW : wall, set = NS > 1 ? wall / RW : 0;
  const int ql = lane & 31, g = lane >> 5;
  const uint32_t wgs = (a.T + kRows - 1) / kRows;  // blocks per head
  int64_t head;
  int32_t wg_tile = 0, q0 = 0, t, eslot = 0, col = 0, chunk = 0;
  int32_t ubase = 0, ulim = a.U;  // compact keys this block may touch: [ubase, ulim)
  if (BUCKET) {
    head = blockIdx.x / static_cast<uint32_t>(a.max_chunks);
    chunk = static_cast<int32_t>(blockIdx.x % static_cast<uint32_t>(a.max_chunks));
    col = a.chunk_col[head * a.max_chunks + chunk];
    if (col < 0) return;  // past the last chunk of this head (block-uniform)
    ubase = col << a.rlog;
    ulim = ubase + (1 << a.rlog);
  } else {
    // Launch order = longest first: heads are taken in groups (group_heads_for);
    // inside a group the row tiles go from the last (most keys, causal) to the first, heads
    // fastest.  Blocks are dealt round-robin to the 8 XCDs, so with 8 | group size a head stays on
    // one XCD, and blocks that start late are the short ones that fill the gaps.
    const uint32_t per_group = static_cast<uint32_t>(a.group_heads) * wgs;
    const uint32_t place_b = dealt_in_turn(blockIdx.x, gridDim.x, 16 / (RW * NS), a.causal);
    const uint32_t grp = place_b / per_group, rem = place_b - grp * per_group;
    const uint32_t nh = min(static_cast<uint32_t>(a.group_heads), static_cast<uint32_t>(a.N) - grp * a.group_heads);
    head = static_cast<int64_t>(grp) * a.group_heads + rem % nh;
    wg_tile = static_cast<int32_t>(wgs - 1 - rem / nh);
    q0 = wg_tile * kRows + 32 * wid;  // first row of this wave
  }
  const uint16_t* Kh = a.K + head * static_cast<int64_t>(a.T) * kHeadDim;
  const uint16_t* Vh = a.V + head * static_cast<int64_t>(a.T) * kHeadDim;

  // The first step's rows and the mask words are requested ahead of everything else: they go straight to LDS, so
  // their latency runs beside that of the rows' own loads.  Against rows that pass through registers (16 of them,
  // four LDS stores and a wait per step), us per layer: c2 71.2 -> 66.2, c4 at T = 32768 763 -> 758, c5 76.6 -> 74.0,
  // per-row widths at c2 171 -> 165.
  // Staging roles: slot tid & 7 of the K and V rows (tid >> 3) and, with four waves, (tid >> 3) + 32 of the step
  // (eight waves cover the 64 rows in one go).  The rows go from memory to LDS without a register between; a wave's
  // 64 pieces are eight rows, one after the other.  The slots past the list re-read its last key; their scores are
  // masked.
  const int srow = tid >> 3;
  const uint32_t kpart = 16 * ((tid & 7) ^ ((srow >> 1) & 7)), vpart = 16 * ((tid & 7) ^ (((srow >> 1) & 1) << 2));
  // With at most 64 keys per column a step of 64 compact keys advances every slot's position by
  // the same amount, so the four row offsets (bytes inside the head, 32 bits) just step by a
  // constant; they are clamped to the last row, since slots past the list only need an address
  // that is in bounds.  Steps are fetched in order, one fetch() per step.
  const bool linear = a.rlog <= 6;
  const uint32_t row_bytes = kHeadDim * 2, off_max = static_cast<uint32_t>(a.T - 1) * row_bytes;
  const uint32_t off_step = linear ? static_cast<uint32_t>((kStep >> a.rlog) * a.w) * row_bytes : 0u;
  uint32_t offa = static_cast<uint32_t>(pos_of(ubase + srow, a.rlog, a.w)) * row_bytes;
  uint32_t offb = static_cast<uint32_t>(pos_of(ubase + srow + kThreads / 8, a.rlog, a.w)) * row_bytes;
  // The head's keys and values as buffer resources (base in scalar registers, 32-bit byte offset
  // per lane): a staging load then needs no 64-bit address arithmetic on the vector pipe.
  const uint32_t head_bytes = static_cast<uint32_t>(a.T) * row_bytes;
  const u32x4 Kres = buffer_words(Kh, head_bytes), Vres = buffer_words(Vh, head_bytes);
  auto slot_off = [&](int32_t step, int32_t slot) {
    return static_cast<uint32_t>(pos_of(min(ubase + step * kStep + slot, a.U - 1), a.rlog, a.w)) * row_bytes;
  };
  u32x4 odd[4];
  auto fetch = [&](int32_t step, int place) __attribute__((always_inline)) {
    if (!linear) {
      offa = slot_off(step, srow);
      if (kTwo) offb = slot_off(step, srow + kThreads / 8);
    }
    const uint32_t oa = min(offa, off_max), ob = min(offb, off_max);
    if constexpr (ODD) {
      odd[0] = load16_odd(Kres, oa + kpart);
      if (kTwo) odd[1] = load16_odd(Kres, ob + kpart);
      odd[2] = load16_odd(Vres, oa + vpart);
      if (kTwo) odd[3] = load16_odd(Vres, ob + vpart);
    } else {
      uint16_t* const at = &KVs[place][0][wall * 8 * kRow];
      if (kTwo) {
        buffer_load_lds16(Kres, at, oa + kpart, at + kThreads / 8 * kRow, ob + kpart);
        buffer_load_lds16(Vres, at + kStep * kRow, oa + vpart, at + (kStep + kThreads / 8) * kRow, ob + vpart);
      } else {
        buffer_load_lds16(Kres, at, oa + kpart);
        buffer_load_lds16(Vres, at + kStep * kRow, oa + vpart);
      }
    }
    offa += off_step;
    offb += off_step;
  };
  auto park = [&](int place) __attribute__((always_inline)) {
    if constexpr (ODD) {
      uint16_t* const at = &KVs[place][0][wall * 8 * kRow];
      park16(at, odd[0]);
      if (kTwo) park16(at + kThreads / 8 * kRow, odd[1]);
      park16(at + kStep * kRow, odd[2]);
      if (kTwo) park16(at + (kStep + kThreads / 8) * kRow, odd[3]);
    }
  };
  fetch(0, 0);
  // mask words of the block's rows -> LDS, KW words a row (words past the last row repeat the last one)
  if (!DENSE && !STREAM) {
    const int32_t row0 = wg_tile * kRows, nwords = min(kRows, a.T - row0) * a.KW;
    const u32x4 Mres = buffer_words(a.mbits + (head * a.T + row0) * a.KW, static_cast<uint32_t>(nwords) * 4u);
    for (int32_t x = 0; x < kRows * a.KW; x += kThreads)
      buffer_load_lds4(Mres, &Ms[x + 64 * wall], static_cast<uint32_t>(min(x + tid, nwords - 1)) * 4u);
  }
  if (BUCKET) {
    const int32_t* bs = a.bstart + head * (a.Kcols + 1);
    const int32_t slot = bs[col] + (chunk - a.cstart[head * (a.Kcols + 1) + col]) * 128 + 32 * wid + ql;
    const int32_t entry = slot < bs[col + 1] ? a.perm[head * a.perm_stride + slot] : -1;
    t = entry < 0 ? -1 : (entry & 0xffffff);
    eslot = entry < 0 ? 0 : (entry >> 24);
  } else {
    t = q0 + ql;
  }
  const int32_t b = static_cast<int32_t>(head / a.H);
  const int32_t len = a.seq_len ? min(max(a.seq_len[b], 0), a.T) : a.T;
  const bool row_active = t >= 0 && t < len;
  const int32_t tq = min(max(t, 0), a.T - 1);

  const uint16_t* Qr = a.Q + (head * a.T + tq) * kHeadDim + 8 * g;
  bf16x8 bq[4];
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) bq[kc] = *reinterpret_cast<const bf16x8*>(Qr + 16 * kc);
  // Nothing but padding: no keys are walked for it.  (Decided behind the first loads, as in the rows kernel: ahead of them
  // it cost 32 sequences of 512 tokens 2 %.)
  if (!BUCKET && wg_tile * kRows >= len && padding_returns(gridDim.x, 16 / (RW * NS), a.causal)) {
    lds_loads_done();
    zero_rows<kThreads>(a.O + (head * a.T + wg_tile * kRows) * kHeadDim, min(kRows, a.T - wg_tile * kRows));
    return;
  }
  // Re-define the fragments through an empty asm: inside the loop they then count as plain
  // register values, not as results of memory loads the loop's own prefetch could be queued behind.
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) asm volatile("" : "+v"(bq[kc]));

  const uint32_t* mrow = (DENSE || STREAM) ? nullptr : &Ms[(32 * wid + ql) * a.KW];
  const uint32_t* krow = STREAM ? a.mbits + (head * a.T + tq) * a.KW : nullptr;
  uint32_t mw0 = 0u, mw1 = 0u, mn0 = 0u, mn1 = 0u;  // the row's words of this step and of the next
  auto fetch_words = [&](int32_t step_, uint32_t& w0, uint32_t& w1) {
    const int32_t wi = SC * (step_ * NS + set);
    w0 = (row_active && wi < a.KW) ? krow[wi] : 0u;
    w1 = (SC == 2 && row_active && wi + 1 < a.KW) ? krow[wi + 1] : 0u;
  };

  // keys the block / this wave can see: position <= min(last row, len - 1) when causal
  int32_t u_end_wg, u_end, u_free;  // below u_free every entry is admissible for every active row of the wave
  if (BUCKET) {
    u_end_wg = u_end = ulim;
    // rows of a bucket come from anywhere in the sequence: positions are compared only in the
    // sub-chunks that reach past the earliest limit among the wave's rows
    int32_t jm = row_active ? (a.causal ? min(t, len - 1) : len - 1) : 0x7fffffff;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) jm = min(jm, __shfl_xor(jm, off, 64));
    u_free = min(u_end, compact_count(jm, a.rlog, a.w));
  } else {
    const int32_t wg_hi = min(wg_tile * kRows + kRows - 1, a.T - 1);
    u_end_wg = compact_count(a.causal ? min(wg_hi, len - 1) : len - 1, a.rlog, a.w);
    const int32_t t_hi = min(q0 + 31, a.T - 1);
    u_end = q0 < len ? compact_count(a.causal ? min(t_hi, len - 1) : len - 1, a.rlog, a.w) : 0;
    u_free = min(u_end, compact_count(a.causal ? min(q0, len - 1) : len - 1, a.rlog, a.w));
  }
  const int32_t my_jmax = a.causal ? min(t, len - 1) : len - 1;
  // compact keys this row may attend: those of the block's range whose position is <= my_jmax
  const int32_t my_ucount = min(ulim, compact_count(row_active ? my_jmax : -1, a.rlog, a.w));
  const int32_t nsteps = (u_end_wg - ubase + kStep - 1) / kStep;

  // this lane's pieces of a K row: slots 2 kc + g of row ql
  int kat[4];
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) kat[kc] = ql * kRow + 8 * ((2 * kc + g) ^ ((ql >> 1) & 7));

  floatx16 oacc[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) { oacc[0][i] = 0.f; oacc[1][i] = 0.f; }
  // Streaming softmax in the exponent's own units: a score enters as y = s c - m_ref (log2 units,
  // one fused multiply-add with the group's offset, -inf for a masked group), so the row maximum
  // is the plain maximum of y and no score is touched twice.
  // m_thr = how far a row's maximum may exceed its reference: -inf until the row has one.  Both
  // halves of a row (lanes l, l + 32) always hold the same m_ref and m_thr.
  float m_ref = 0.f, m_thr = -INFINITY, l_run = 0.f;

  if (STREAM && nsteps > 0) fetch_words(0, mn0, mn1);
  park(0);
  lds_loads_done();
  __syncthreads();
  // One step, its keys and values at a place that the compiler knows: all LDS addresses of the loop are then a
  // per-lane base and an immediate offset.
  auto walk = [&](int32_t step, auto stage_c) __attribute__((always_inline)) {
    constexpr int stage = decltype(stage_c)::value;
    if (step + 1 < nsteps) fetch(step + 1, stage ^ 1);
    if (STREAM) {
      mw0 = mn0;
      mw1 = mn1;
      if (step + 1 < nsteps) fetch_words(step + 1, mn0, mn1);
    }
    // With two or more keys per column the (at most 32) columns of a 64-key step lie in one mask
    // word: it is read once per step, unconditionally (every row of the block has its words in
    // LDS), ahead of both sub-chunks instead of in front of each one's first fragment read.
    constexpr bool kStepWord = !DENSE && !STREAM && RLOG >= 1;
    uint32_t wstep = 0u;
    if (kStepWord) {
      wstep = mrow[((step * kStep + 32 * SC * set) >> (RLOG < 5 ? RLOG : a.rlog)) >> 5];
      wstep = row_active ? wstep : 0u;
    }
#pragma unroll
    for (int sc = 0; sc < SC; ++sc) {
      const int32_t u0 = ubase + step * kStep + 32 * (SC * set + sc);
      if (u0 >= u_end) break;  // wave-uniform: beyond what this wave's rows can see
      if (BUCKET && __ballot(row_active) == 0ull) break;  // a wave past the end of its bucket
      uint32_t bits = 0xffffffffu;
      if (!DENSE) {
        const int32_t col0 = u0 >> (RLOG < 5 ? RLOG : a.rlog);  // first column of the sub-chunk
        const uint32_t word = STREAM ? (sc == 0 ? mw0 : mw1) : (kStepWord ? wstep : (row_active ? mrow[col0 >> 5] : 0u));
        bits = word >> (col0 & 31);
        constexpr uint32_t ncol = RLOG >= 5 ? 1u : (32u >> RLOG);
        constexpr uint32_t cmask = ncol >= 32 ? 0xffffffffu : ((1u << ncol) - 1u);
        if (__ballot((bits & cmask) != 0u) == 0ull) continue;  // no row of the wave uses it
      }
      // S^T sub-chunk = K (32 keys x 64) . Q_tile^T
      const uint16_t* Kr = &KVs[stage][0][32 * (SC * set + sc) * kRow];
      floatx16 sv;
#pragma unroll
      for (int i = 0; i < 16; ++i) sv[i] = 0.f;
#pragma unroll
      for (int kc = 0; kc < 4; ++kc)
        sv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(Kr + kat[kc]), bq[kc],
                                                     sv, 0, 0, 0);
      // admissibility of each (key, query) entry: reg i <-> key slot 8(i/4) + 4g + i%4.
      // Interior sub-chunks need only the column bits; the few that straddle the causal
      // diagonal or the end of the sequence also compare key positions.
      const bool boundary = u0 + 32 > u_free;
      // Registers of one lane fall into groups that share a column (and so a mask bit): 4 for 4
      // or 8 keys per column, 8 for 16, all 16 for 32 or more and for the dense kernel.  One
      // bit-select per group picks its offset (-m_ref or -inf).
      constexpr int kGroup = DENSE ? 16 : (RLOG >= 5 ? 16 : (RLOG == 4 ? 8 : (RLOG >= 2 ? 4 : 1)));
      constexpr int kGroups = 16 / kGroup;
      float y[16];
      if (!boundary && kGroup > 1) {
        const uint32_t ref_bits = __float_as_uint(-m_ref), inf_bits = 0xff800000u;
#pragma unroll
        for (int gi = 0; gi < kGroups; ++gi) {
          const int col = DENSE ? 0 : (RLOG >= 5 ? 0 : (RLOG == 2 ? 2 * gi + g : gi));  // column of the group
          // all ones where the group's column is selected
          const uint32_t sel = DENSE ? (row_active ? ~0u : 0u)
                                     : static_cast<uint32_t>(static_cast<int32_t>(bits << (31 - col)) >> 31);
          const float off = __uint_as_float((sel & ref_bits) | (~sel & inf_bits));
#pragma unroll
          for (int e = 0; e < kGroup; ++e) y[kGroup * gi + e] = fmaf(sv[kGroup * gi + e], a.c, off);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int32_t slot = 8 * (i >> 2) + 4 * g + (i & 3);
          uint32_t okb = DENSE ? (row_active ? 1u : 0u) : ((bits >> (RLOG >= 5 ? 0 : (slot >> RLOG))) & 1u);
          // positions ascend with the compact index, so "position <= the row's last admissible
          // key" is "index below the row's count of such keys", taken once per row.  The variants
          // with one key per column walk this per-element path in every sub-chunk and have no
          // register left for that count: they compare positions.
          if (boundary) {
            if (kGroup > 1) {
              okb &= (u0 + slot < my_ucount) ? 1u : 0u;
            } else {
              const int32_t u = u0 + slot;
              const int32_t pu = pos_of(min(u, a.U - 1), a.rlog, a.w);
              okb &= (u < ulim ? 1u : 0u) & (pu <= my_jmax ? 1u : 0u);
            }
          }
          y[i] = okb ? fmaf(sv[i], a.c, -m_ref) : -INFINITY;
        }
      }
      // The V^T fragments of the sub-chunk are requested here, into the registers the raw scores
      // just left, so that their LDS latency lies under the softmax arithmetic below instead of in
      // front of the products that use them.  The LDS transpose read hands lane i of a 16-lane
      // group element i % 4 of the 8 bytes that lanes 4 e + i / 4 (e = 0..3) of the group point at:
      // with lane r pointing at dims 4 (r % 4) .. + 3 of key r / 4, lane i receives dim i of keys
      // 0..3 -- four consecutive keys of one dimension.  Lanes 8..15 of a group point at rows 2, 3
      // (mod 4), whose halves are stored exchanged.
      // (With the per-key mask words of MODE 3 in registers as well there is no room for that:
      // there the fragments are requested just before their products.)
      bf16x8 av[2][2];
      auto request_v = [&]() {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          const uint16_t* Vr = &KVs[stage][1][(32 * (SC * set + sc) + 4 * g + ((ql & 15) >> 2)) * kRow +
                                          32 * (mt ^ ((ql >> 3) & 1)) + (ql & 16) + 4 * (ql & 3)];
#pragma unroll
          for (int c2 = 0; c2 < 2; ++c2) {
            const bf16x4 lo = lds_transpose4(Vr + (16 * c2) * kRow);
            const bf16x4 hi = lds_transpose4(Vr + (16 * c2 + 8) * kRow);
            av[mt][c2] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          }
        }
      };
      if (!STREAM) request_v();
      float ymax = max_of(y);
      // The reference only has to keep the exponentials in range: it is moved (and the accumulators
      // rescaled) when some row's maximum exceeds it by more than kRefSlack, or when the row has none yet.
      if (__ballot(ymax > m_thr) != 0ull) {
        // rows that did not ask keep their reference (factor exactly 1): a row's arithmetic
        // never depends on the other rows of its wave
        ymax = half_max(ymax);
        const bool refresh = ymax > m_thr;
        const float delta = refresh ? ymax : 0.f;
        const float corr = (refresh && m_thr > 0.f) ? __builtin_amdgcn_exp2f(-delta) : 1.f;
        l_run *= corr;
#pragma unroll
        for (int i = 0; i < 16; ++i) { oacc[0][i] *= corr; oacc[1][i] *= corr; }
        m_ref += delta;
        m_thr = refresh ? kRefSlack : m_thr;
#pragma unroll
        for (int i = 0; i < 16; ++i) y[i] -= delta;
      }
      // P to bf16 (exp2(-inf) = 0 for masked entries); the row sum is taken over the rounded
      // values, the ones the product uses
      bf16x2 h[8];
      const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const floatx2 f2 = {__builtin_amdgcn_exp2f(y[2 * e]), __builtin_amdgcn_exp2f(y[2 * e + 1])};
        h[e] = __builtin_convertvector(f2, bf16x2);
        l_run = __builtin_amdgcn_fdot2_f32_bf16(h[e], ones, l_run, false);
      }
      bf16x8 bp[2];
#pragma unroll
      for (int c2 = 0; c2 < 2; ++c2) {
        const bf16x4 lo = __builtin_shufflevector(h[4 * c2], h[4 * c2 + 1], 0, 1, 2, 3);
        const bf16x4 hi = __builtin_shufflevector(h[4 * c2 + 2], h[4 * c2 + 3], 0, 1, 2, 3);
        bp[c2] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
      // O^T += V^T P^T; V^T fragments in the key order of the P registers
      if (STREAM) request_v();
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2)
          oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[mt][c2], bp[c2], oacc[mt], 0, 0, 0);
    }
    if (step + 1 < nsteps) park(stage ^ 1);
    lds_loads_done();
    __syncthreads();
  };
  for (int32_t step = 0; step < nsteps; step += 2) {
    walk(step, std::integral_constant<int, 0>{});
    if (step + 1 < nsteps) walk(step + 1, std::integral_constant<int, 1>{});
  }
  if constexpr (NS > 1) {
    // log-sum-exp merge of the sets' partial results, halving the number of sets per round; the keys and
    // values of the last step are no longer needed (the loop ended with a barrier)
    static_assert(NS / 2 * 64 * RW * kPartFloats * 4 <= static_cast<int>(sizeof(KVs)), "partial results fit the keys' and values' place");
    float* const part = reinterpret_cast<float*>(&KVs[0][0][0]) + 64 * wid + lane;
    float m_own = m_thr > 0.f ? m_ref : -INFINITY;
#pragma unroll
    for (int half = NS / 2; half >= 1; half >>= 1) {
      float* const p = part + (set & (half - 1)) * 64 * RW * kPartFloats;
      if (set >= half && set < 2 * half) store_part<64 * RW>(p, oacc, l_run, m_own);
      __syncthreads();
      if (set < half) merge_part<64 * RW>(p, oacc, l_run, m_own);
      if (half > 1) __syncthreads();
    }
    if (set > 0) return;
  }
  l_run = half_sum(l_run);
  const float inv = (row_active && l_run > 0.f) ? 1.f / l_run : 0.f;
  if (BUCKET && a.part_o && t >= 0 && g == 0) {
    const int64_t e = (head * a.T + t) * a.slots + eslot;
    a.part_ml[2 * e] = m_thr > 0.f ? m_ref : -INFINITY;
    a.part_ml[2 * e + 1] = row_active ? l_run : 0.f;
  }
  // (behind the partial results of other waves, where there are such)
  constexpr int kPartBytes = NS > 1 ? NS / 2 * 64 * RW * kPartFloats * 4 : 0;
  static_assert(kPartBytes + RW * 32 * kRow * 2 <= static_cast<int>(sizeof(KVs)), "rows on their way out fit the keys' and values' place");
  if constexpr (RW == 2 && NS == 4) {
    // (blocks of the smallest launches, which wait for the trip through LDS: 7.5 against 7.1 us.  Two sets fill the chip: with this
    // store per-key bits, H = 12, T = 2048, B = 4 161.2 against 159.6, T = 1536, B = 3 97.2 / 96.4, columns, T = 512, B = 8 25.8 / 25.6)
    if (t < a.T) store_row(a.O + (head * a.T + t) * kHeadDim, oacc, inv);
    return;
  }
  store_rows(&KVs[0][0][0] + kPartBytes / 2 + wid * 32 * kRow, oacc, inv, 0u, [&](int r) -> uint16_t* {
    if (BUCKET) {
      const int32_t tr = __shfl(t, r, kWave), slot = __shfl(eslot, r, kWave);
      if (tr < 0) return nullptr;
      return a.part_o ? a.part_o + ((head * a.T + tr) * a.slots + slot) * kHeadDim : a.O + (head * a.T + tr) * kHeadDim;
    }
    return q0 + r < a.T ? a.O + (head * a.T + q0 + r) * kHeadDim : nullptr;
  });
}

// ---- few columns per row: group the rows of a head by the columns each selected (Sec. 3.1, App. A.5.3:
// the long-sequence regime where k K < T) ----
// A block takes 256 RPT rows of a head, RPT per thread, so that its counters meet memory once for all of
// them (one row per thread cost 675 K global atomics for 12 heads of 131072 rows: counting 23 us, scattering
// 32 us; with eight 10 and 15 us).  RPT S <= 8 entries of a thread wait in registers between ranking and
// scattering, S >= the columns a row may select.
constexpr int kMaxSlots = 8;

__global__ __launch_bounds__(256) void zero_i32_kernel(int32_t* __restrict__ p, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

// calls take(column) for the first `slots` set bits of a row's mask words (further bits of a foreign mask
// are ignored); rows of whole, aligned 16-byte pieces: one load per four words
template <typename F>
__device__ __forceinline__ void row_columns(const uint32_t* __restrict__ mw, int32_t KW, bool vec, int32_t slots, F&& take) {
  int n = 0;
  auto word = [&](uint32_t w, int32_t j) {
    while (w != 0u && n < slots) {
      take(n, 32 * j + __ffs(static_cast<int>(w)) - 1);
      w &= w - 1u;
      ++n;
    }
  };
  if (vec) {
    for (int32_t j = 0; j < KW; j += 4) {
      const uint4 w4 = *reinterpret_cast<const uint4*>(mw + j);
      word(w4.x, j); word(w4.y, j + 1); word(w4.z, j + 2); word(w4.w, j + 3);
    }
  } else {
    for (int32_t j = 0; j < KW; ++j) word(mw[j], j);
  }
}

// bucket sizes: every set mask bit of a row is one entry of that column's bucket
template <int RPT>
__global__ __launch_bounds__(256) void bucket_count_kernel(const uint32_t* __restrict__ mbits,
                                                           int32_t* __restrict__ cnt, int32_t T, int32_t KW,
                                                           int32_t Kc, int32_t slots) {
  extern __shared__ int32_t hist[];  // Kc counters
  const int64_t head = blockIdx.y;
  const bool vec = (KW & 3) == 0 && (reinterpret_cast<uintptr_t>(mbits) & 15) == 0;
  for (int c = threadIdx.x; c < Kc; c += 256) hist[c] = 0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int32_t row = (blockIdx.x * RPT + q) * 256 + threadIdx.x;
    if (row < T)
      row_columns(mbits + (head * T + row) * KW, KW, vec, slots, [&](int, int32_t col) { atomicAdd(&hist[col], 1); });
  }
  __syncthreads();
  for (int c = threadIdx.x; c < Kc; c += 256)
    if (hist[c] != 0) atomicAdd(&cnt[head * Kc + c], hist[c]);
}

// per head: bucket offsets, the 128-row chunks of each bucket, and which column each chunk is
__global__ __launch_bounds__(1024) void bucket_scan_kernel(const int32_t* __restrict__ cnt,
                                                           int32_t* __restrict__ bstart,
                                                           int32_t* __restrict__ cstart,
                                                           int32_t* __restrict__ cursor,
                                                           int32_t* __restrict__ chunk_col, int32_t Kc,
                                                           int32_t max_chunks) {
  __shared__ int32_t wrows[16], wchunks[16], first[1024];
  const int64_t head = blockIdx.x;
  const int c = threadIdx.x, lane = c & 63, wave = c >> 6;
  const int32_t n = c < Kc ? cnt[head * Kc + c] : 0;
  const int32_t nch = (n + 127) >> 7;
  int32_t r = n, k = nch;  // inclusive scans: inside the wave, then over the waves' totals
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t ar = __shfl_up(r, off, kWave), ak = __shfl_up(k, off, kWave);
    if (lane >= off) { r += ar; k += ak; }
  }
  if (lane == kWave - 1) { wrows[wave] = r; wchunks[wave] = k; }
  __syncthreads();
  int32_t total_rows = 0, total_chunks = 0, r0 = r - n, c0 = k - nch;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    if (w < wave) { r0 += wrows[w]; c0 += wchunks[w]; }
    total_rows += wrows[w];
    total_chunks += wchunks[w];
  }
  if (c < Kc) {
    bstart[head * (Kc + 1) + c] = r0;
    cstart[head * (Kc + 1) + c] = c0;
    cursor[head * Kc + c] = r0;
  }
  first[c] = c0;
  __syncthreads();
  if (c == 0) {
    bstart[head * (Kc + 1) + Kc] = total_rows;
    cstart[head * (Kc + 1) + Kc] = total_chunks;
  }
  // the column of chunk x: the last one whose first chunk is <= x (empty buckets share their successor's
  // first chunk, so that is the one that owns x); a thread per chunk, however the chunks are spread
  for (int32_t x = c; x < max_chunks; x += 1024) {
    int32_t lo = 0, hi = Kc - 1;
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (first[mid] <= x) lo = mid; else hi = mid - 1;
    }
    chunk_col[head * max_chunks + x] = x < total_chunks ? lo : -1;
  }
}

// entries into their buckets (order inside a bucket is whatever the atomics give: no result
// depends on it).  An entry is the row id with, above bit 24, its rank among the row's selected
// columns.  With one column per row, rows that selected nothing (padding, no admissible key) get
// their zero output here; with several, the merge kernel writes every row.
template <int S, int RPT>
__global__ __launch_bounds__(256) void bucket_scatter_kernel(const uint32_t* __restrict__ mbits,
                                                             int32_t* __restrict__ cursor, int32_t* __restrict__ perm,
                                                             uint16_t* __restrict__ O_zero, int32_t T, int32_t KW,
                                                             int32_t Kc, int64_t perm_stride, int32_t slots) {
  extern __shared__ int32_t hist[];  // Kc counters, then Kc bases
  int32_t* base = hist + Kc;
  const int64_t head = blockIdx.y;
  const bool vec = (KW & 3) == 0 && (reinterpret_cast<uintptr_t>(mbits) & 15) == 0;
  for (int c = threadIdx.x; c < Kc; c += 256) hist[c] = 0;
  __syncthreads();
  uint32_t entry[RPT][S];  // column | rank in the block's part of its bucket << 10, all ones: none
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
#pragma unroll
    for (int e = 0; e < S; ++e) entry[q][e] = 0xffffffffu;
    const int32_t row = (blockIdx.x * RPT + q) * 256 + threadIdx.x;
    if (row < T)
      row_columns(mbits + (head * T + row) * KW, KW, vec, slots, [&](int n, int32_t col) {
        const uint32_t v = static_cast<uint32_t>(col) | (static_cast<uint32_t>(atomicAdd(&hist[col], 1)) << 10);
#pragma unroll
        for (int e = 0; e < S; ++e)
          if (e == n) entry[q][e] = v;
      });
  }
  __syncthreads();
  for (int c = threadIdx.x; c < Kc; c += 256)
    base[c] = hist[c] != 0 ? atomicAdd(&cursor[head * Kc + c], hist[c]) : 0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int32_t row = (blockIdx.x * RPT + q) * 256 + threadIdx.x;
#pragma unroll
    for (int e = 0; e < S; ++e)
      if (entry[q][e] != 0xffffffffu)
        perm[head * perm_stride + base[entry[q][e] & 1023u] + static_cast<int32_t>(entry[q][e] >> 10)] = row | (e << 24);
    if (O_zero && row < T && entry[q][0] == 0xffffffffu) {
      uint4* o = reinterpret_cast<uint4*>(O_zero + (head * T + row) * kHeadDim);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = make_uint4(0u, 0u, 0u, 0u);
    }
  }
}

// Attention of buckets whose columns hold at most 64 keys: a block takes CH (see the launch) consecutive 128-row chunks of
// a head, so that a column's keys and values are staged once for the chunks of it that follow one another, and the next chunk's
// query rows are on their way while a chunk is computed.  All keys of a row are there at once: no running reference.
// Bound: memory (rows gathered and scattered).  Rows come and go as whole lines, eight lanes of 16 bytes each, through
// LDS: 12 heads of 131072 rows in 128 buckets, 64 keys each, 77 us (5.2 TB/s) against 118 with the one-chunk blocks of
// the kernel above, whose lanes each move 16 and 8 bytes of their own row per instruction; with CH chunks per block but
// rows moved like that 138.
template <int CH>
__global__ __launch_bounds__(256, 4) void bucket_attn_kernel(TileArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t KVs[2][64 * kRow];    // [K, V]
  __shared__ __attribute__((aligned(16))) uint16_t rows_s[4][32 * kRow];  // a wave's query rows on their way in, its results on their way out
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ql = lane & 31, g = lane >> 5;
  const uint32_t groups = (static_cast<uint32_t>(a.max_chunks) + CH - 1) / CH;
  const int64_t head = blockIdx.x / groups;
  const int32_t first = static_cast<int32_t>(blockIdx.x % groups) * CH;
  const int32_t* cols = a.chunk_col + head * a.max_chunks;
  int32_t col[CH], entry[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) col[i] = first + i < a.max_chunks ? cols[first + i] : -1;
  if (col[0] < 0) return;  // past the last chunk of this head (block-uniform)
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int32_t c = max(col[i], 0);
    const int32_t* bs = a.bstart + head * (a.Kcols + 1);
    const int32_t slot = bs[c] + (first + i - a.cstart[head * (a.Kcols + 1) + c]) * 128 + 32 * wid + ql;
    entry[i] = col[i] >= 0 && slot < bs[c + 1] ? a.perm[head * a.perm_stride + slot] : -1;
  }
  const int32_t r = 1 << a.rlog, subs = r > 32 ? 2 : 1;
  const int32_t b = static_cast<int32_t>(head / a.H);
  const int32_t len = a.seq_len ? min(max(a.seq_len[b], 0), a.T) : a.T;
  const uint32_t row_bytes = kHeadDim * 2, head_bytes = static_cast<uint32_t>(a.T) * row_bytes;
  const u32x4 Kres = buffer_words(a.K + head * static_cast<int64_t>(a.T) * kHeadDim, head_bytes);
  const u32x4 Vres = buffer_words(a.V + head * static_cast<int64_t>(a.T) * kHeadDim, head_bytes);
  const u32x4 Qres = buffer_words(a.Q + head * static_cast<int64_t>(a.T) * kHeadDim, head_bytes);
  auto stage = [&](int32_t c) {
    const int srow = tid >> 3;
    const uint32_t kpart = 16 * ((tid & 7) ^ (srow & 7)), vpart = 16 * ((tid & 7) ^ (((srow >> 1) & 1) << 2));
    for (int e = 0; e < subs; ++e) {
      const uint32_t at = static_cast<uint32_t>(pos_of((c << a.rlog) + min(srow + 32 * e, r - 1), a.rlog, a.w)) * row_bytes;
      buffer_load_lds16(Kres, &KVs[0][(8 * wid + 32 * e) * kRow], at + kpart);
      buffer_load_lds16(Vres, &KVs[1][(8 * wid + 32 * e) * kRow], at + vpart);
    }
  };
  // Rows move whole: eight lanes of 16 bytes each, piece p of row r at slot p ^ (r & 7) of the wave's place (and of
  // the staged keys here, so that both are read at the same offsets).
  uint16_t* const place = rows_s[wid];
  const int mrow = lane >> 3, mpart = lane & 7;
  auto ask_rows = [&](int32_t en) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int32_t e = __shfl(en, 8 * j + mrow, kWave);
      buffer_load_lds16(Qres, place + 8 * j * kRow, static_cast<uint32_t>(e < 0 ? 0 : (e & 0xffffff)) * row_bytes + 16 * (mpart ^ mrow));
    }
  };
  int kat[4];
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) kat[kc] = ql * kRow + 8 * ((2 * kc + g) ^ (ql & 7));
  bf16x8 bq[4];
  auto take_rows = [&]() {
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) bq[kc] = *reinterpret_cast<const bf16x8*>(place + kat[kc]);
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) asm volatile("" : "+v"(bq[kc])::"memory");  // (read before the place is used again)
  };
  ask_rows(entry[0]);
  int32_t staged = -1;
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    if (col[i] < 0) break;
    if (col[i] != staged) {
      if (i > 0) __syncthreads();  // every wave is done with the column before
      stage(col[i]);
      staged = col[i];
      lds_loads_done();
      __syncthreads();
    }
    if (i == 0) take_rows();
    const bool more = i + 1 < CH && col[i + 1 < CH ? i + 1 : i] >= 0;
    if (more) ask_rows(entry[i + 1 < CH ? i + 1 : i]);
    const int32_t t = entry[i] < 0 ? -1 : (entry[i] & 0xffffff);
    const bool active = t >= 0 && t < len;
    // keys of the column that the row may attend: the first mine
    const int32_t jmax = active ? (a.causal ? min(t, len - 1) : len - 1) : -1;
    const int32_t mine = max(min(compact_count(jmax, a.rlog, a.w) - (col[i] << a.rlog), r), 0);
    const bool whole = __ballot(mine < 32 * subs) == 0ull;
    float y[2][16];
#pragma unroll
    for (int sc = 0; sc < 2; ++sc) {
      floatx16 sv;
#pragma unroll
      for (int x = 0; x < 16; ++x) sv[x] = 0.f;
      if (sc < subs) {
#pragma unroll
        for (int kc = 0; kc < 4; ++kc)
          sv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(&KVs[0][32 * sc * kRow] + kat[kc]), bq[kc], sv, 0, 0, 0);
      }
#pragma unroll
      for (int x = 0; x < 16; ++x) y[sc][x] = sv[x] * a.c;
      if (!whole || sc >= subs) {
#pragma unroll
        for (int x = 0; x < 16; ++x) y[sc][x] = sc < subs && 32 * sc + 8 * (x >> 2) + 4 * g + (x & 3) < mine ? y[sc][x] : -INFINITY;
      }
    }
    const float m = half_max(fmaxf(max_of(y[0]), max_of(y[1]))), ref = m == -INFINITY ? 0.f : m;
    float l = 0.f;
    floatx16 oacc[2];
#pragma unroll
    for (int x = 0; x < 16; ++x) { oacc[0][x] = 0.f; oacc[1][x] = 0.f; }
    const bf16x2 ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
#pragma unroll
    for (int sc = 0; sc < 2; ++sc) {
      if (sc >= subs) break;
      bf16x2 h[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const floatx2 f2 = {__builtin_amdgcn_exp2f(y[sc][2 * e] - ref), __builtin_amdgcn_exp2f(y[sc][2 * e + 1] - ref)};
        h[e] = __builtin_convertvector(f2, bf16x2);
        l = __builtin_amdgcn_fdot2_f32_bf16(h[e], ones, l, false);
      }
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const uint16_t* Vr = &KVs[1][(32 * sc + 4 * g + ((ql & 15) >> 2)) * kRow + 32 * (mt ^ ((ql >> 3) & 1)) + (ql & 16) + 4 * (ql & 3)];
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2) {
          const bf16x4 lo = lds_transpose4(Vr + (16 * c2) * kRow), hi = lds_transpose4(Vr + (16 * c2 + 8) * kRow);
          oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7),
                                                             join_pairs(h + 4 * c2), oacc[mt], 0, 0, 0);
        }
      }
    }
    l = half_sum(l);
    const float inv = (active && l > 0.f) ? 1.f / l : 0.f;
    if (a.part_o && t >= 0 && g == 0) {
      const int64_t e = (head * a.T + t) * a.slots + (entry[i] >> 24);
      a.part_ml[2 * e] = m;
      a.part_ml[2 * e + 1] = active ? l : 0.f;
    }
    if (more) {
      lds_loads_done();
      take_rows();
    }
    store_rows(place, oacc, inv, 0u, [&](int rr) -> uint16_t* {
      const int32_t e = __shfl(entry[i], rr, kWave);
      if (e < 0) return nullptr;
      const int64_t row = head * a.T + (e & 0xffffff);
      return a.part_o ? a.part_o + (row * a.slots + (e >> 24)) * kHeadDim : a.O + row * kHeadDim;
    });
  }
}

// several columns per row: O[t] = sum_s w_s On_s / sum_s w_s with w_s = l_s 2^(m_s - M), over the
// row's entries (On_s normalised partial outputs, m_s references in log2 units, l_s sums)
__global__ __launch_bounds__(256) void bucket_merge_kernel(const uint32_t* __restrict__ mbits,
                                                           const uint16_t* __restrict__ part_o,
                                                           const float* __restrict__ part_ml,
                                                           uint16_t* __restrict__ O, int64_t rows, int32_t KW,
                                                           int32_t slots) {
  const int64_t gid = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t row = gid >> 3;
  const int part = static_cast<int>(gid & 7);
  if (row >= rows) return;
  int n = 0;
  for (int32_t j = 0; j < KW; ++j) n += __popc(mbits[row * KW + j]);
  n = min(n, slots);
  // all of the row's entries are requested before any is used
  float ms[kMaxSlots], ls[kMaxSlots];
  uint4 vs[kMaxSlots];
  float M = -INFINITY;
#pragma unroll
  for (int q = 0; q < kMaxSlots; ++q) {
    const int64_t e = row * slots + min(q, max(n - 1, 0));
    ms[q] = part_ml[2 * e];
    ls[q] = q < n ? part_ml[2 * e + 1] : 0.f;
    vs[q] = *reinterpret_cast<const uint4*>(part_o + e * kHeadDim + part * 8);
    if (q < n) M = fmaxf(M, ms[q]);
  }
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float wsum = 0.f;
#pragma unroll
  for (int q = 0; q < kMaxSlots; ++q) {
    if (!(ls[q] > 0.f)) continue;
    const float wq = ls[q] * __builtin_amdgcn_exp2f(ms[q] - M);
    const uint32_t wds[4] = {vs[q].x, vs[q].y, vs[q].z, vs[q].w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[2 * i] = fmaf(wq, bf16lo_to_f32(wds[i]), acc[2 * i]);
      acc[2 * i + 1] = fmaf(wq, bf16hi_to_f32(wds[i]), acc[2 * i + 1]);
    }
    wsum += wq;
  }
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  uint4 o;
  o.x = pack_bf16(acc[0] * inv, acc[1] * inv);
  o.y = pack_bf16(acc[2] * inv, acc[3] * inv);
  o.z = pack_bf16(acc[4] * inv, acc[5] * inv);
  o.w = pack_bf16(acc[6] * inv, acc[7] * inv);
  *reinterpret_cast<uint4*>(O + row * kHeadDim + part * 8) = o;
}

}  // namespace

// Heads per scheduling group: the keys and values (2 x U x 128 B per head) of the heads an
// XCD works on at one time should fit its 4 MB L2 with room to spare.
// Causal: inside a group the long tiles come first, so a launch ends evenly only if the last group has blocks of all
// lengths for every CU, and groups that fit the L2s (768 blocks at U = 2048, of 1024 that are resident) do not: a last
// group of a few heads starts with its longest tiles when the others are nearly done.  From two blocks per resident one on
// (2048) balance is worth more than the L2, whose misses the memory-side cache takes (twice the L2s' keys and values in
// flight).  Groups of at least 2048 blocks then, alike up to the rounding to eight heads, which leaves some launches a short
// last one (36 heads of 32768 rows 16, 16, 4; 17 of them 16 and 1).  Layer, us, groups that fit the L2s / these: H = 32, K = 256,
// k^ = 64, T = 2048, B = 8 (48 / 128 heads) 373 / 364, ragged T = 2000 559 / 538, with padding 467 / 438, T = 8192, B = 2, whole columns (8 / 32)
// 840 / 793; H = 12, K = 128, B = 8, T = 2048 (48 / 96) 112.4 / 107.5, T = 4096 (24 / 96) 334 / 319, B = 11 (24 / 72, 60) 460 / 442; 512 keys
// per row, T = 4096, B = 4 358 / 355, T = 8192, B = 2 364 / 362; short last groups 36 heads 466 / 468, 17 2999 / 2992.  Other sizes at the
// first of these: 32, 64, 96, 160, 256 heads 351, 350, 346, 348, 352 where 48 took 358 and 128 343.
int32_t group_heads_for(const Shape& s, int64_t U) {
  const int64_t per_head = 2 * U * kHeadDim * 2;
  int64_t g = 8 * std::max<int64_t>(1, (3 << 20) / std::max<int64_t>(per_head, 1));
  if (s.causal) {
    const int64_t groups = std::max<int64_t>(1, static_cast<int64_t>(s.N) * ((s.T + 127) / 128) / 2048);
    g = std::max(g, ((s.N + groups - 1) / groups + 7) / 8 * 8);
  }
  return static_cast<int32_t>(std::min<int64_t>(g, s.N));
}

#ifndef SEA_NW8_MIN_BLOCKS
#define SEA_NW8_MIN_BLOCKS 1024
#endif
// Dense baseline: eight-wave blocks (256 rows) when even those are at least two per block slot of
// the chip (2 per CU x 256 CUs); every staged key step then serves twice the rows (3-6 % at
// T = 32768).  The masked kernels keep four-wave blocks: interleaved on one box the wide form
// was within 1 % at T = 32768 and 4 % slower at T = 2048.
static bool wide_blocks(const Shape& s) {
  return static_cast<int64_t>(s.N) * ((s.T + 255) / 256) >= SEA_NW8_MIN_BLOCKS;
}

// How the waves of a block are split.  A launch that leaves the chip room takes as long as its longest list
// does, so sets of waves share the rows of a block and walk the list in parallel (the merge costs about one
// 64-key chunk).  kPairs: 64 rows, four sets of two waves, while the 128-row blocks number at most one per CU
// (half the rows halve a CU's longest work as well); per-key bits (MODE 3) cost more per step, so there a
// little longer.  kHalves: 64 rows, two sets of two waves, whose blocks are as many waves as kOne's 128 rows: half the list and
// half the rows per block, and two blocks end where one did, up to what is resident at once (its sets take alternate 32 keys, those
// of kTwo 64, so some weights round to bf16 against another reference: per-key bits, T = 2048, B = 4 differ by 1.8e-3, and both are off the
// 64-bit result by 1.846e-3, of which the result's own rounding is 1.632e-3).  kFour: 128 rows, four sets of
// four waves, where the last rows of a causal list have many times the keys of the first.  kTwo: 128 rows, two sets of four.
// Whole forward, K = 128, H = 12, us as kOne / kTwo / kHalves / kPairs (kFour): causal, k^ = 48, T = 1024, B = 2 (192 blocks of 128)
// 33.7 / 29.5 / 27.8 / 26.0, B = 3 (288) 35.3 / 31.4 / 28.8 / 31.1, B = 4 (384) 35.0 / 31.3 / 29.1 / 33.4, B = 6 (576) 39.8 / 39.8 / 39.1 / 44.0,
// B = 8 (768) 45.0 / 48.1 / 46.6 / 53.1; T = 2048, B = 2 (384) 49.4 / 41.1 / 38.3 / 41.1, B = 3 (576) 55.4 / 51.8 / 49.4 / 55.6, B = 4 (768)
// 60.9 / 62.3 / 60.8 / 66.9; H = 20, B = 1 (320) 49.2 / 41.1 / 37.5 / 38.2; T = 4096, B = 1 (384) 82.6 / 63.1 / 60.2 / 60.1 (57.8), H = 8, T = 8192
// (512) 149 / 113 / 112.5 / 114 (108); T = 512, K = 64, k^ = 16, B = 10 (480) 28.9 / 28.1 / 27.1 / 33.3, B = 12 (576) 31.3 / 35.3 / 32.7 / 38.2;
// T = 256, B = 18 (432) 24.7 / 25.4 / 25.0 / 30.6.  Bidirectional, T = 1024, B = 3 41.0 / 39.6 / 36.5 / 39.4, B = 4 40.9 / 39.5 / 37.2 / 39.5, B = 5 (480)
// 43.9 / 43.0 / 44.5 / 48.4, B = 6 52.7 / 55.1 / 52.7 / 56.4; T = 2048, B = 2 59.5 / 55.6 / 52.7 / 54.6; T = 512, K = 64, B = 8 (384) 29.4 / 29.8 / 28.1 / 33.3, B = 10
// 31.7 / 31.9 / 32.5 / 36.8.  Per-key bits, T = 2048, B = 1 94 / 78 / 77 / 68, B = 2 119 / 103 / 103 / 99, B = 3 149 / 134.4 / 133.9 / 142, B = 4 169 /
// 165.2 / 163.5 / 175, T = 1024, B = 6 107 / 102.5 / 100.8 / 111, B = 8 123.0 / 124.9 / 122.3 / 132, T = 4096, B = 2 (768) 263 / 247 / 247 / 257, H = 32,
// T = 3500 (896) 258 / 253 / 252 / 265.
enum WaveSplit { kOne, kTwo, kFour, kPairs, kHalves };
static WaveSplit wave_split(const Shape& s, int32_t U, bool key_bits) {
  const int64_t blocks = static_cast<int64_t>(s.N) * ((s.T + 127) / 128);
  if (U >= 256 && blocks <= (key_bits ? 384 : 256)) return kPairs;
  if (U >= 4096 && blocks <= 512 && s.causal) return kFour;
  if (key_bits) return U >= 1024 && blocks <= (U >= 2048 ? 896 : 768) ? kHalves : kOne;
  if (U >= 512 && blocks <= (!s.causal ? 384 : (U >= 1024 ? 576 : 512))) return kHalves;
  if (U >= 1024 && blocks <= 512) return kTwo;
  return kOne;
}

template <int RLOG, int MODE, int RW, int NS, int SC, bool ODD = false>
static void launch_tile(const Shape& s, const TileArgs& a, hipStream_t st) {
  if constexpr (!ODD) {
    if (starts_odd(a.K) || starts_odd(a.V)) return launch_tile<RLOG, MODE, RW, NS, SC, true>(s, a, st);
  }
  constexpr int kRows = 32 * RW, kThreads = 64 * RW * NS;  // (mask words arrive kThreads at a time)
  const size_t shm = MODE == 0 ? static_cast<size_t>((kRows * a.KW + kThreads - 1) / kThreads * kThreads) * sizeof(uint32_t) : 0;
  hipLaunchKernelGGL((tile_attn_kernel<RLOG, MODE, RW, NS, SC, ODD>), dim3(static_cast<uint32_t>(s.N) * ((s.T + kRows - 1) / kRows)),
                     dim3(64 * RW * NS), shm, st, a);
}

bool tile_attn_supported(const Shape& s, sea_dtype dt, int32_t* rlog_out) {
  if (dt != SEA_BF16 || s.T % s.K != 0) return false;
  if (s.geometry != 0) return false;  // a row's own column ranges: no structure shared between rows
  const int32_t w = s.T / s.K;
  const int32_t r = w < s.rep_cap ? w : s.rep_cap;
  if (r <= 0 || (r & (r - 1)) != 0) return false;
  int32_t rlog = 0;
  while ((1 << rlog) < r) ++rlog;
  if (static_cast<int64_t>(w) * r > (int64_t(1) << 30)) return false;
  if (s.T > (1 << 24)) return false;  // row offsets inside a head are 32-bit byte counts
  if (rlog_out) *rlog_out = rlog;
  return true;
}

namespace {
// Few columns per row under per-query grouping: rows (k^ = 1) or (row, column) entries (k^ <= 8,
// and no more than an eighth of the columns) are bucketed by column -- from the list length on where that
// pays.  A (row, column) entry costs the bucket form (counting, scattering, partial results, merge) as much
// as 450 list keys cost the tile walk, whose rows walk half the list when causal: B = 8, H = 12, T = 512,
// K = 64, k^ = 8 with 8 keys each 83 us in buckets, 34 us in tiles; B = 1, H = 12, T = 4096, K = 128,
// k^ = 4 with 32 keys each, causal, 64 and 74 us.  One column per row needs no merge: from 512 keys on.
bool bucket_mode(const Shape& s) {
  const int32_t w = s.T / s.K, r = w < s.rep_cap ? w : s.rep_cap;
  const int64_t U = static_cast<int64_t>(s.K) * r;
  if (s.grouping != 0) return false;
  if (s.k_hat == 1) return U >= 512;
  return s.k_hat <= kMaxSlots && 8 * s.k_hat <= s.K && (s.causal ? U / 2 : U) >= 450 * s.k_hat;
}
size_t al256(size_t b) { return (b + 255) & ~size_t(255); }
struct BucketWs {
  size_t perm, cnt, cursor, bstart, cstart, chunk_col, part_o, part_ml, total;
  int64_t entries;      // perm slots per head
  int32_t max_chunks;
};
BucketWs bucket_layout(const Shape& s) {
  BucketWs b{};
  const size_t N = static_cast<size_t>(s.N);
  b.entries = static_cast<int64_t>(s.T) * s.k_hat;
  b.max_chunks = static_cast<int32_t>((b.entries + 127) / 128) + s.K;
  size_t off = 0;
  b.perm = off; off += al256(N * b.entries * 4);
  b.cnt = off; off += al256(N * s.K * 4);
  b.cursor = off; off += al256(N * s.K * 4);
  b.bstart = off; off += al256(N * (s.K + 1) * 4);
  b.cstart = off; off += al256(N * (s.K + 1) * 4);
  b.chunk_col = off; off += al256(N * b.max_chunks * 4);
  b.part_o = off; if (s.k_hat > 1) off += al256(N * b.entries * kHeadDim * 2);
  b.part_ml = off; if (s.k_hat > 1) off += al256(N * b.entries * 2 * 4);
  b.total = off;
  return b;
}
}  // namespace

// the tiled path reads K and V in place; only the bucket form needs scratch: the permutation,
// per-column counters / offsets / cursors, the chunk table and (several columns per row) the
// partial results
size_t tile_attn_workspace(const Shape& s) {
  if (!tile_attn_supported(s, SEA_BF16, nullptr) || !bucket_mode(s)) return 0;
  return bucket_layout(s).total;
}

int32_t* bucket_counts(const Shape& s, void* ws) {
  if (!tile_attn_supported(s, SEA_BF16, nullptr) || !bucket_mode(s)) return nullptr;
  return reinterpret_cast<int32_t*>(static_cast<char*>(ws) + bucket_layout(s).cnt);
}

hipError_t launch_tile_attn(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                            const uint32_t* mbits, uint16_t* O, void* ws, hipStream_t st, BucketCounts have) {
  int32_t rlog = 0;
  if (!tile_attn_supported(s, SEA_BF16, &rlog)) return hipErrorNotSupported;
  const int32_t w = s.T / s.K, r = 1 << rlog;
  const int32_t U = s.K * r;
  if (bucket_mode(s)) {
    StageScope scope(SEA_STAGE_SPARSE, st);
    const BucketWs lay = bucket_layout(s);
    const int32_t KW = (s.K + 31) / 32;
    char* base = static_cast<char*>(ws);
    int32_t* perm = reinterpret_cast<int32_t*>(base + lay.perm);
    int32_t* cnt = reinterpret_cast<int32_t*>(base + lay.cnt);
    int32_t* cursor = reinterpret_cast<int32_t*>(base + lay.cursor);
    int32_t* bstart = reinterpret_cast<int32_t*>(base + lay.bstart);
    int32_t* cstart = reinterpret_cast<int32_t*>(base + lay.cstart);
    int32_t* chunk_col = reinterpret_cast<int32_t*>(base + lay.chunk_col);
    const bool multi = s.k_hat > 1;
    if (have == BucketCounts::none) {
      const int64_t n = static_cast<int64_t>(s.N) * s.K;
      hipLaunchKernelGGL(zero_i32_kernel, dim3(static_cast<uint32_t>((n + 255) / 256)), dim3(256), 0, st, cnt, n);
    }
    uint16_t* O_zero = multi ? nullptr : O;
    auto grid_of = [&](int rpt) { return dim3((s.T + 256 * rpt - 1) / (256 * rpt), static_cast<uint32_t>(s.N)); };
    // rows per thread: eight entries, fewer where that leaves less than two blocks per CU
    const int64_t rows256 = static_cast<int64_t>(s.N) * ((s.T + 255) / 256);
    const int rpt = rows256 >= 8 * 512 ? 8 : (rows256 >= 2 * 512 ? 2 : 1);
    if (have == BucketCounts::counted) {  // (by the kernel that selected the columns)
    } else if (rpt == 8) hipLaunchKernelGGL(bucket_count_kernel<8>, grid_of(8), dim3(256), s.K * sizeof(int32_t), st, mbits, cnt, s.T, KW, s.K, s.k_hat);
    else if (rpt == 2) hipLaunchKernelGGL(bucket_count_kernel<2>, grid_of(2), dim3(256), s.K * sizeof(int32_t), st, mbits, cnt, s.T, KW, s.K, s.k_hat);
    else hipLaunchKernelGGL(bucket_count_kernel<1>, grid_of(1), dim3(256), s.K * sizeof(int32_t), st, mbits, cnt, s.T, KW, s.K, s.k_hat);
    hipLaunchKernelGGL(bucket_scan_kernel, dim3(static_cast<uint32_t>(s.N)), dim3(1024), 0, st, cnt, bstart, cstart,
                       cursor, chunk_col, s.K, lay.max_chunks);
#define SEA_SCATTER(S_, RPT_)                                                                                    \
    hipLaunchKernelGGL((bucket_scatter_kernel<S_, RPT_>), grid_of(RPT_), dim3(256), 2 * s.K * sizeof(int32_t), st, mbits, cursor, \
                       perm, O_zero, s.T, KW, s.K, lay.entries, s.k_hat)
    if (s.k_hat == 1 && rpt == 8) SEA_SCATTER(1, 8);
    else if (s.k_hat == 1 && rpt == 2) SEA_SCATTER(1, 2);
    else if (s.k_hat == 1) SEA_SCATTER(1, 1);
    else if (s.k_hat <= 4 && rpt >= 2) SEA_SCATTER(4, 2);
    else SEA_SCATTER(8, 1);
#undef SEA_SCATTER
    TileArgs a{};
    a.Q = Q; a.K = K; a.V = V; a.mbits = nullptr; a.O = O; a.seq_len = s.seq_len;
    a.N = s.N; a.H = s.H; a.T = s.T; a.U = U; a.KW = 0; a.rlog = rlog; a.w = w; a.causal = s.causal;
    a.group_heads = s.N;
    a.c = s.scale * kLog2e;
    a.perm = perm; a.bstart = bstart; a.chunk_col = chunk_col; a.cstart = cstart;
    a.max_chunks = lay.max_chunks; a.Kcols = s.K; a.perm_stride = lay.entries;
    a.slots = s.k_hat;
    if (multi) {
      a.part_o = reinterpret_cast<uint16_t*>(base + lay.part_o);
      a.part_ml = reinterpret_cast<float*>(base + lay.part_ml);
    }
    const int32_t max_chunks = lay.max_chunks;
    const dim3 chunks(static_cast<uint32_t>(s.N) * max_chunks);
    const bool odd = starts_odd(K) || starts_odd(V);
    // Four chunks per block save staging where the launch is many times what is resident at once (1024 blocks); below, they
    // only make a block's chain longer.  Layers, us with one / four chunks a block: 1584 chunks (12 heads, T = 512, K = 128)
    // 26.9 / 32.0, 1536 (8, 8192) 40.2 / 44.9, 4608 (12, 32768) 98.5 / 102.7, 8192 (32, 16384) 148.6 / 150.3, 9216 (96, 2048,
    // two columns) 94.6 / 95.6, 13824 (12, 131072) 307 / 303.
    if (rlog <= 6 && !odd && !starts_odd(Q) && chunks.x <= 8192u)
      hipLaunchKernelGGL(bucket_attn_kernel<1>, chunks, dim3(256), 0, st, a);
    else if (rlog <= 6 && !odd && !starts_odd(Q))
      hipLaunchKernelGGL(bucket_attn_kernel<4>, dim3(static_cast<uint32_t>(s.N) * ((max_chunks + 3) / 4)), dim3(256), 0, st, a);
    else if (odd)
      hipLaunchKernelGGL((tile_attn_kernel<0, 2, 4, 1, 2, true>), chunks, dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL((tile_attn_kernel<0, 2>), chunks, dim3(256), 0, st, a);
    if (multi) {
      const int64_t rows = static_cast<int64_t>(s.N) * s.T;
      hipLaunchKernelGGL(bucket_merge_kernel, dim3(static_cast<uint32_t>((rows * 8 + 255) / 256)), dim3(256), 0, st,
                         mbits, a.part_o, a.part_ml, O, rows, KW, s.k_hat);
    }
    return hipGetLastError();
  }
  StageScope scope(SEA_STAGE_SPARSE, st);
  TileArgs a{};
  a.Q = Q; a.K = K; a.V = V; a.mbits = mbits; a.O = O; a.seq_len = s.seq_len;
  a.N = s.N; a.H = s.H; a.T = s.T; a.U = U; a.KW = (s.K + 31) / 32;
  a.rlog = rlog; a.w = w; a.causal = s.causal;
  a.group_heads = group_heads_for(s, U);
  a.c = s.scale * kLog2e;
  const WaveSplit split = wave_split(s, U, false);
#define SEA_TILE(R_)                                                                        \
  switch (split) {                                                                          \
    case kPairs: launch_tile<R_, 0, 2, 4, 1>(s, a, st); break;                              \
    case kHalves: launch_tile<R_, 0, 2, 2, 1>(s, a, st); break;                             \
    case kFour: launch_tile<R_, 0, 4, 4, 2>(s, a, st); break;                               \
    case kTwo: launch_tile<R_, 0, 4, 2, 2>(s, a, st); break;                                \
    default: launch_tile<R_, 0, 4, 1, 2>(s, a, st); break;                                  \
  }                                                                                         \
  break
  switch (rlog) {
    case 0: SEA_TILE(0);
    case 1: SEA_TILE(1);
    case 2: SEA_TILE(2);
    case 3: SEA_TILE(3);
    case 4: SEA_TILE(4);
    default: SEA_TILE(5);
  }
#undef SEA_TILE
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// fp32 tensors: the same walk over the compact key list on the fp64 / fp32 matrix cores.
// Block = 4 waves on the same 16 query rows; wave w takes the 16-key chunks c = w (mod 4) and the
// four partial results are merged through LDS (log-sum-exp weights).  Per chunk:
//   S^T (keys x queries) = K_c Q^T with v_mfma_f64_16x16x4_f64 (fp32 inputs widened, fp64 sums: the
//   precision contract of the fp32 mode), softmax weights in fp32 against a running reference,
//   O^T (dims x queries) += V_c^T P^T with v_mfma_f32_16x16x4_f32.
// Layouts: A lane l = A[row l % 16][k l / 16], B lane l = B[k l / 16][col l % 16]; the fp64 result
// register i is D[row 4 i + l / 16][col l % 16], the fp32 one D[row 4 (l / 16) + i][col l % 16].
// So a lane is one query (column); its four S^T registers are keys 4 i + g, g = l / 16, exactly the
// contraction slot (k = g of step i) the second product expects of P^T.  The contraction index of
// the first product is a free permutation of the 64 dims: step 4 j + e of lane group g is dim
// 16 j + 4 g + e, so Q and K rows are read as 16-byte pieces.  The rows of an output tile are free as
// well: row x of tile dt is dim 4 x + dt, so a lane's values of a key are one 16-byte piece too.
// Bound: a chunk's matrix instructions take 1536 cycles of a SIMD (16 fp64 of 64, 16 fp32 of 32), and fp64 and
// fp32 products do not run beside vector instructions as the bf16 ones do: 180 of those per chunk.  So they are
// what to save: two register sets in turn instead of copies, probes without branches, no rescaling while no
// maximum rises (257 -> 210 instructions; 12 heads of 1024 rows 38.9 -> 36.7 us, 4096 rows 418 -> 399 us).
// ------------------------------------------------------------------------------------------
typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

struct TileF32Args {
  const float* Q;
  const float* K;
  const float* V;
  const uint32_t* mbits;  // [N][T][KW]
  float* O;
  const int32_t* seq_len;
  int32_t N, H, T, U, KW, rlog, w, causal;
  double f;  // scale * log2(e)
  ColumnList g;  // columns of any width (ANYW)
};

__device__ __forceinline__ float rows_max_f(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum_f(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// ANYW: columns of any width, any number of keys per column (otherwise both as in the bf16 kernel).  These
// layers also have a per-row form, in which a key that is not selected is not read: a row whose result is not
// finite may have met such a key (a value that is not finite against a weight of zero) and is computed again
// from its own keys.  WIDE: columns of 2^24 keys and more.
template <bool ANYW, bool WIDE = false>
__global__ __launch_bounds__(256, 2) void tile_attn_f32_kernel(TileF32Args a) {
  __shared__ float m_s[4][16], l_s[4][16];
  __shared__ float o_s[4][kHeadDim][17];  // [wave][dim][query], padded
  __shared__ uint32_t mask_s[16 * 129];    // at most 128 mask words per row (K <= 1024 columns, or T <= 4096 keys)
  __shared__ uint32_t again_s;             // rows to compute again, a bit each
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qc = lane & 15, g = lane >> 4;
  const uint32_t tiles = (a.T + 15) / 16;
  // Longest first: the last row tiles of every head come first.  A launch that is resident as a whole (three blocks
  // per CU) is dealt to the 256 CUs in turn, so there the second round of 256 runs backwards: a CU that got a
  // longer tile gets a shorter one next (12 heads of 1024 rows 43 -> 39 us).  In longer launches a CU takes its
  // next block when it is done with one, and plain order is the better one (12 heads of 2048 rows 125 against
  // 120 us).
  uint32_t pos = blockIdx.x;
  if (gridDim.x <= 768 && ((pos >> 8) & 1)) {
    const uint32_t lo = pos & ~255u, n = min(256u, gridDim.x - lo);
    pos = lo + (n - 1 - (pos - lo));
  }
  const uint32_t tile = tiles - 1 - pos / static_cast<uint32_t>(a.N);
  const int64_t head = pos % static_cast<uint32_t>(a.N);
  const int32_t q0 = static_cast<int32_t>(tile) * 16;
  const int32_t t = q0 + qc;
  const int32_t b = static_cast<int32_t>(head / a.H);
  const int32_t len = a.seq_len ? min(max(a.seq_len[b], 0), a.T) : a.T;
  if (q0 >= len && gridDim.x > 768) {  // nothing but padding: no keys are walked for it (in a launch of several rounds)
    if (q0 + (tid >> 4) < a.T)
      *reinterpret_cast<float4*>(a.O + (head * a.T + q0 + (tid >> 4)) * kHeadDim + 4 * (tid & 15)) = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  const bool row_active = t < len;
  const int32_t tq = min(t, a.T - 1);
  const float* Kh = a.K + head * static_cast<int64_t>(a.T) * kHeadDim;
  const float* Vh = a.V + head * static_cast<int64_t>(a.T) * kHeadDim;
  // selected-column bits of the tile's 16 rows -> LDS (row stride KW + 1 words)
  {
    const uint32_t* msrc = a.mbits + (head * a.T + q0) * a.KW;
    const int32_t nwords = min(16, a.T - q0) * a.KW;
    for (int32_t x = tid; x < 16 * a.KW; x += 256) {
      const int32_t r = x / a.KW, wi = x - r * a.KW;
      mask_s[r * (a.KW + 1) + wi] = x < nwords ? msrc[x] : 0u;
    }
    if (ANYW && tid == 0) again_s = 0u;
  }
  __syncthreads();
  const uint32_t* mrow_s = &mask_s[qc * (a.KW + 1)];

  double qd[16];
  {
    const float* Qr = a.Q + (head * a.T + tq) * kHeadDim + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float4 v = *reinterpret_cast<const float4*>(Qr + 16 * j);
      qd[4 * j] = v.x; qd[4 * j + 1] = v.y; qd[4 * j + 2] = v.z; qd[4 * j + 3] = v.w;
    }
  }
  const int32_t my_jmax = a.causal ? min(t, len - 1) : len - 1;
  const int32_t t_hi = min(q0 + 15, a.T - 1);
  const int32_t j_end = a.causal ? min(t_hi, len - 1) : len - 1;
  const int32_t u_end = ANYW ? list_count(a.g, j_end) : compact_count(j_end, a.rlog, a.w);
  auto locate = [&](int32_t u, int32_t* col) -> int32_t {  // position and column of list entry u
    if (ANYW) {
      if (a.g.r == 0) {
        *col = column_of(a.g.cg, u);
        return u;
      }
      *col = div_small(u, a.g.invr);
      return entry_pos(a.g, *col, u - *col * a.g.r);
    }
    *col = u >> a.rlog;
    if (WIDE) return pos_of(u, a.rlog, a.w);
    // the same in two products at the full rate: columns, keys of a column and w lie below 2^24
    return static_cast<int32_t>(__umul24(*col, a.w) + (__umul24(u & ((1 << a.rlog) - 1), a.w) >> a.rlog));
  };
  const int32_t nchunks = (u_end + 15) / 16;

  float m_run = -INFINITY;
  float l_run = 0.f;
  floatx4 o[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) o[dt] = floatx4{0.f, 0.f, 0.f, 0.f};

  // one chunk's operands: K row of key 16 cc + qc (16-byte pieces at dims 16 j + 4 g), V entries of this lane's four
  // keys 16 cc + 4 i + g at dims 4 qc .. 4 qc + 3 (output tile dt = dims 4 x + dt), and which of the four count
  struct Chunk {
    float4 kf[4], vf[4];
    bool ok[4];
  };
  int32_t pv[4];
  // admissibility and positions of chunk cc's entries; false when no row of the tile uses the chunk
  auto probe = [&](int32_t cc, Chunk& x) -> bool {
    bool any = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int32_t u = 16 * cc + 4 * i + g;
      int32_t col;
      pv[i] = locate(min(u, a.U - 1), &col);
      const uint32_t bit = (mrow_s[col >> 5] >> (col & 31)) & 1u;
      x.ok[i] = static_cast<bool>(static_cast<int>(row_active) & static_cast<int>(u < a.U) & static_cast<int>(bit) &
                                  static_cast<int>(pv[i] <= my_jmax));
      if (ANYW) pv[i] = min(pv[i], len - 1);  // rows past the sequence end are not read
      any |= x.ok[i];
    }
    return __ballot(any) != 0ull;
  };
  auto request = [&](int32_t cc, Chunk& x) {
    int32_t col, pos_k = locate(min(16 * cc + qc, a.U - 1), &col);
    if (ANYW) pos_k = min(pos_k, len - 1);
    const float* Kr = Kh + static_cast<int64_t>(pos_k) * kHeadDim + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j) x.kf[j] = *reinterpret_cast<const float4*>(Kr + 16 * j);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      x.vf[i] = *reinterpret_cast<const float4*>(Vh + static_cast<int64_t>(pv[i]) * kHeadDim + 4 * qc);
  };
  // looks for the wave's next chunk after c and requests it: its number, or one past the last
  auto next = [&](int32_t c, Chunk& x) -> int32_t {
    do c += 4;
    while (c < nchunks && !probe(c, x));
    if (c < nchunks) request(c, x);
    return c;
  };
  auto compute = [&](const Chunk& x) {
    // two independent chains halve the latency of the 16 dependent products
    doublex4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
      const float4 k0 = x.kf[j], k1 = x.kf[j + 1];
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(k0.x), qd[4 * j], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(k1.x), qd[4 * j + 4], acc1, 0, 0, 0);
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(k0.y), qd[4 * j + 1], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(k1.y), qd[4 * j + 5], acc1, 0, 0, 0);
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(k0.z), qd[4 * j + 2], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(k1.z), qd[4 * j + 6], acc1, 0, 0, 0);
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(k0.w), qd[4 * j + 3], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(k1.w), qd[4 * j + 7], acc1, 0, 0, 0);
    }
    double y[4];
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      y[i] = x.ok[i] ? (acc0[i] + acc1[i]) * a.f : -INFINITY;
      mx = fmaxf(mx, static_cast<float>(y[i]));
    }
    // The reference only has to be common to the row's keys: an fp32 rounding of the maximum does.  While no
    // row's maximum rises, every factor is exactly 1.
    mx = rows_max_f(mx);
    if (__ballot(mx > m_run) != 0ull) {
      const float m_new = fmaxf(m_run, mx);
      const float corr = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= corr;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[dt][i] *= corr;
    }
    if (__ballot(m_run != -INFINITY) == 0ull) return;
    const double m_safe = (m_run == -INFINITY) ? 0.0 : static_cast<double>(m_run);
    float pw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      pw[i] = __builtin_amdgcn_exp2f(static_cast<float>(y[i] - m_safe));  // exp2(-inf) = 0 for masked entries
      l_run += pw[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.vf[i].x, pw[i], o[0], 0, 0, 0);
      o[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.vf[i].y, pw[i], o[1], 0, 0, 0);
      o[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.vf[i].z, pw[i], o[2], 0, 0, 0);
      o[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.vf[i].w, pw[i], o[3], 0, 0, 0);
    }
  };

  // one chunk is computed while the wave's next is on its way; two sets of registers take turns
  Chunk even, odd;
  int32_t c = next(wid - 4, even);
  while (c < nchunks) {
    c = next(c, odd);
    compute(even);
    if (c >= nchunks) break;
    c = next(c, even);
    compute(odd);
  }
  // merge the four waves: O = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w
  l_run = rows_sum_f(l_run);
  if (g == 0) {
    m_s[wid][qc] = m_run;
    l_s[wid][qc] = l_run;
  }
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int i = 0; i < 4; ++i) o_s[wid][4 * (4 * g + i) + dt][qc] = o[dt][i];
  __syncthreads();
  {
    const int q = tid & 15, dq = tid >> 4;  // query, quad of dims
    const int32_t tt = q0 + q;
    float M = fmaxf(fmaxf(m_s[0][q], m_s[1][q]), fmaxf(m_s[2][q], m_s[3][q]));
    float L = 0.f, acc4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float wgt = (m_s[w][q] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_s[w][q] - M);
      L = fmaf(wgt, l_s[w][q], L);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc4[e] = fmaf(wgt, o_s[w][4 * dq + e][q], acc4[e]);
    }
    if (ANYW) {
      float zero = 0.f * L;  // NaN if anything is not finite
#pragma unroll
      for (int e = 0; e < 4; ++e) zero = fmaf(0.f, acc4[e], zero);
      if (tt >= len) acc4[0] = acc4[1] = acc4[2] = acc4[3] = 0.f;  // zero times what it met need not be zero
      else if (zero != 0.f) atomicOr(&again_s, 1u << q);
      __syncthreads();  // (also: the mask words are no longer read)
    }
    // (a row to compute again is left alone: O may lie in the place of Q)
    if (tt < a.T && !(ANYW && ((again_s >> q) & 1u) != 0u)) {
      const float inv = (tt < len && L > 0.f) ? 1.f / L : 0.f;
      *reinterpret_cast<float4*>(a.O + (head * a.T + tt) * kHeadDim + 4 * dq) =
          make_float4(acc4[0] * inv, acc4[1] * inv, acc4[2] * inv, acc4[3] * inv);
    }
  }
  if constexpr (ANYW) {
    uint16_t* const place = reinterpret_cast<uint16_t*>(mask_s) + 1024 * wid;
    for (uint32_t rows = again_s; rows != 0u; rows &= rows - 1u) {
      const int r = __builtin_amdgcn_readfirstlane(__ffs(static_cast<int>(rows)) - 1);
      if ((r & 3) != wid) continue;
      const int64_t row = head * a.T + q0 + r;
      const ColumnKeys keys(a.g, a.mbits + row * a.KW, a.KW, a.causal ? min(q0 + r, len - 1) : len - 1, place);
      gather_row_f32(keys, a.f, a.Q + row * kHeadDim, Kh, Vh, a.O + row * kHeadDim);
    }
  }
}

namespace {
// the power-of-two form; log2(keys per column)
bool tile_attn_f32_pow2(const Shape& s, int32_t* rlog_out) {
  if (s.geometry != 0 || s.T % s.K != 0) return false;
  const int32_t w = s.T / s.K, r = w < s.rep_cap ? w : s.rep_cap;
  if (r <= 0 || (r & (r - 1)) != 0 || static_cast<int64_t>(w) * r > (int64_t(1) << 30)) return false;
  int32_t rlog = 0;
  while ((1 << rlog) < r) ++rlog;
  *rlog_out = rlog;
  return true;
}
}  // namespace

bool tile_attn_f32_supported(const Shape& s) {  // (a tile's mask words live in LDS: K <= 1024)
  int32_t rlog;
  return s.K <= 1024 && (tile_attn_f32_pow2(s, &rlog) || column_list_supported(s));
}
bool tile_attn_f32_structured(const Shape& s) {
  int32_t rlog;
  return s.K <= 1024 && tile_attn_f32_pow2(s, &rlog);
}

hipError_t launch_tile_attn_f32(const Shape& s, const float* Q, const float* K, const float* V,
                                const uint32_t* mbits, float* O, hipStream_t st) {
  if (!tile_attn_f32_supported(s)) return hipErrorNotSupported;
  int32_t rlog = 0;
  const bool pow2 = tile_attn_f32_pow2(s, &rlog);
  if (!pow2 && column_gather_pays(s, SEA_F32)) return launch_column_gather(s, SEA_F32, Q, K, V, mbits, O, st);
  StageScope scope(SEA_STAGE_SPARSE, st);
  TileF32Args a{};
  a.Q = Q; a.K = K; a.V = V; a.mbits = mbits; a.O = O; a.seq_len = s.seq_len;
  a.N = s.N; a.H = s.H; a.T = s.T; a.KW = (s.K + 31) / 32; a.causal = s.causal;
  a.f = static_cast<double>(s.scale) * 1.4426950408889634;
  const dim3 grid(static_cast<uint32_t>(s.N) * ((s.T + 15) / 16));
  if (pow2) {
    a.rlog = rlog; a.w = s.T / s.K; a.U = s.K << rlog;
    if (a.w < 1 << 24) hipLaunchKernelGGL(tile_attn_f32_kernel<false>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((tile_attn_f32_kernel<false, true>), grid, dim3(256), 0, st, a);
  } else {
    a.g = column_list(s); a.U = a.g.U;
    hipLaunchKernelGGL(tile_attn_f32_kernel<true>, grid, dim3(256), 0, st, a);
  }
  return hipGetLastError();
}

// Masks without column structure shared by the rows (per-row width geometry): the selection
// arrives as one bit per (row, key), and the same kernel runs with every key its own "column"
// (one key per column, column width 1) -- the walk of the dense kernel with per-key mask bits,
// which every lane reads for its own row one step ahead (no mask words in LDS: four blocks per CU
// as in the other modes).  T <= 8192 is the limit of the kernels that write the bits (beyond it the
// quadratic walk also loses to per-row lists for the budgets in use); the fp32 kernel keeps the mask
// words of its 16 rows in LDS, 128 per row.
bool tile_attn_keybits_supported(const Shape& s, sea_dtype dt) { return s.T <= (dt == SEA_BF16 ? 8192 : 4096); }

// the same for fp32 tensors
hipError_t launch_tile_attn_f32_keybits(const Shape& s, const float* Q, const float* K, const float* V,
                                        const uint32_t* kb, float* O, hipStream_t st) {
  if (s.T > 4096) return hipErrorNotSupported;
  StageScope scope(SEA_STAGE_SPARSE, st);
  TileF32Args a{};
  a.Q = Q; a.K = K; a.V = V; a.mbits = kb; a.O = O; a.seq_len = s.seq_len;
  a.N = s.N; a.H = s.H; a.T = s.T; a.U = s.T; a.KW = (s.T + 31) / 32; a.rlog = 0; a.w = 1; a.causal = s.causal;
  a.f = static_cast<double>(s.scale) * 1.4426950408889634;
  const dim3 grid(static_cast<uint32_t>(s.N) * ((s.T + 15) / 16));
  hipLaunchKernelGGL(tile_attn_f32_kernel<false>, grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_tile_attn_keybits(const Shape& s, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                                    const uint32_t* kb, uint16_t* O, hipStream_t st) {
  if (!tile_attn_keybits_supported(s, SEA_BF16)) return hipErrorNotSupported;
  StageScope scope(SEA_STAGE_SPARSE, st);
  TileArgs a{};
  a.Q = Q; a.K = K; a.V = V; a.mbits = kb; a.O = O; a.seq_len = s.seq_len;
  a.N = s.N; a.H = s.H; a.T = s.T; a.U = s.T; a.KW = (s.T + 31) / 32; a.rlog = 0; a.w = 1; a.causal = s.causal;
  a.group_heads = group_heads_for(s, s.T);
  a.c = s.scale * kLog2e;
  switch (wave_split(s, s.T, true)) {
    case kPairs: launch_tile<0, 3, 2, 4, 1>(s, a, st); break;
    case kHalves: launch_tile<0, 3, 2, 2, 1>(s, a, st); break;
    case kFour: launch_tile<0, 3, 4, 4, 2>(s, a, st); break;
    default: launch_tile<0, 3, 4, 1, 2>(s, a, st); break;
  }
  return hipGetLastError();
}

size_t dense_attn_workspace(const Shape&) { return 0; }

hipError_t launch_dense_attn(const Shape& s, sea_dtype dt, const void* Q, const void* K, const void* V,
                             void* O, void* /*ws*/, hipStream_t st) {
  if (dt != SEA_BF16) return hipErrorNotSupported;
  StageScope scope(SEA_STAGE_DENSE, st);
  // dense: one "column" per key (r = 1, w = 1), so pos(u) = u
  TileArgs a{};
  a.Q = static_cast<const uint16_t*>(Q); a.K = static_cast<const uint16_t*>(K);
  a.V = static_cast<const uint16_t*>(V);
  a.mbits = nullptr; a.O = static_cast<uint16_t*>(O); a.seq_len = s.seq_len;
  a.N = s.N; a.H = s.H; a.T = s.T; a.U = s.T; a.KW = 0; a.rlog = 0; a.w = 1;
  a.causal = s.causal; a.c = s.scale * kLog2e;
  a.group_heads = group_heads_for(s, s.T);
  if (wide_blocks(s)) launch_tile<0, 1, 8, 1, 2>(s, a, st);
  else launch_tile<0, 1, 4, 1, 2>(s, a, st);
  return hipGetLastError();
}

}  // namespace sea
