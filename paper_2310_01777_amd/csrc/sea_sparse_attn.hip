// Sparse attention over per-row key lists (Sec. 3.1.1: rho, sigma, A* V fused).
//
// One wavefront owns one query row and reads its keys one by one (sea_gather.h); nothing of size T x T or
// T x L is ever written.
//
// Lists that hold a good part of the keys they span are better served by tiles: list_tile_kernel turns
// the lists of 128 rows into key bits in LDS and walks the keys once for all of them on the matrix
// cores.  Which form a 128-row block takes is decided on the device from the lists themselves.
#include "sea_gather.h"
#include "sea_internal.h"
#include "sea_tile.h"

#include <type_traits>

namespace sea {
namespace {

constexpr int kWavesPerBlock = 4;

// Where a row's key list lives.  Per-row lists (FLAT = false): idx + row L, cnt[row] entries.  FlatCSR tensor
// (idx = its column array): row (b, h, t) owns the entries of CSR row b T + t whose column h' T + j has
// h' = h -- one contiguous run because columns ascend -- found by two searches; the key is the entry minus h T.
template <bool FLAT>
__device__ __forceinline__ ListKeys key_list(const Shape& s, int64_t row, const int32_t* __restrict__ idx,
                                            const int32_t* __restrict__ cnt, int32_t L,
                                            const int64_t* __restrict__ crow) {
  if (!FLAT) return {idx + row * L, min(cnt[row], L), 0, s.T};
  const int64_t head = row / s.T, t = row - head * s.T;
  const int64_t b = head / s.H, h = head - b * s.H;
  const int64_t beg = crow[b * s.T + t], end = crow[b * s.T + t + 1];
  // First entry >= h T and first entry >= (h + 1) T, both searches in step.  The heads of a time step list
  // about equally many keys, so the first seven probes lie around where that puts the bound (mostly in
  // one or two cache lines) and usually leave a few dozen entries; after that the range is cut in eight.
  int64_t lo[2] = {beg, beg}, hi[2] = {end, end};
  const int64_t key[2] = {h * s.T, (h + 1) * s.T};
  for (bool first = true; lo[0] < hi[0] || lo[1] < hi[1]; first = false) {
    int64_t at[2][7];
    int32_t v[2][7];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int64_t w = hi[e] - lo[e], guess = lo[e] + ((h + e) * w) / s.H;
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        constexpr int32_t kAround[7] = {-65, -17, -5, -1, 3, 15, 63};
        at[e][i] = first ? min(max(guess + kAround[i], lo[e]), hi[e] - 1) : lo[e] + (((i + 1) * w) >> 3);
        v[e][i] = idx[w > 0 ? at[e][i] : beg];
      }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if (lo[e] >= hi[e]) continue;
#pragma unroll
      for (int i = 0; i < 7; ++i) {
        if (v[e][i] < key[e]) lo[e] = max(lo[e], at[e][i] + 1); else hi[e] = min(hi[e], at[e][i]);
      }
    }
  }
  const int64_t bound[2] = {lo[0], lo[1]};
  return {idx + bound[0], static_cast<int32_t>(bound[1] - bound[0]), static_cast<int32_t>(h * s.T), s.T};
}

// The row (or rows) of a wave.  A grid dimension holds fewer than 2^32 threads: from 2^26 rows on, slices of 2^22 blocks.
constexpr uint32_t kSlice = 1u << 22;
dim3 row_grid(int64_t nrows) {
  const int64_t blocks = (nrows + kWavesPerBlock - 1) / kWavesPerBlock;
  return blocks < (int64_t(1) << 24) ? dim3(static_cast<uint32_t>(blocks)) : dim3(kSlice, static_cast<uint32_t>((blocks + kSlice - 1) / kSlice));
}
__device__ __forceinline__ int64_t wave_row() {
  const int64_t block = static_cast<int64_t>(blockIdx.y) * gridDim.x + xcd_contiguous(blockIdx.x, gridDim.x);
  return block * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// key_list for one row, by the whole wave: half the lanes search the run's first entry, half its end.  The heads of a
// time step list about equally many keys, so the first 32 probes lie side by side around where that puts the
// bound (one or two cache lines); after that 32 probes cut the range evenly.
template <bool FLAT>
__device__ __forceinline__ ListKeys wave_key_list(const Shape& s, int64_t row, const int32_t* __restrict__ idx,
                                                 const int32_t* __restrict__ cnt, int32_t L,
                                                 const int64_t* __restrict__ crow) {
  if (!FLAT) return key_list<false>(s, row, idx, cnt, L, crow);
  const int64_t head = row / s.T, t = row - head * s.T;
  const int64_t b = head / s.H, h = head - b * s.H;
  const int64_t beg = crow[b * s.T + t], end = crow[b * s.T + t + 1];
  const int lane = threadIdx.x & 63, probe = lane & 31;
  const int64_t bound = (h + (lane >> 5)) * s.T;
  int32_t lo = 0, hi = static_cast<int32_t>(max(end - beg, static_cast<int64_t>(0)));
  auto passed_by = [&](int32_t at) {  // how many of the half's probes lie below its bound
    const uint64_t mask = __ballot(at < hi && idx[beg + at] < bound);
    return __popc(static_cast<uint32_t>(lane < 32 ? mask : mask >> 32));
  };
  {
    const int32_t guess = static_cast<int32_t>((h + (lane >> 5)) * hi / s.H);
    const int32_t from = max(min(guess - 16, hi - 32), 0), passed = passed_by(from + probe);
    if (passed < 32 && from + passed < hi) hi = from + passed;
    if (passed > 0) lo = from + passed;
  }
  while (__ballot(lo < hi) != 0ull) {
    const int32_t step = (hi - lo + 31) >> 5, passed = passed_by(lo + (probe + 1) * step - 1);
    hi = min(hi, lo + (passed + 1) * step - 1);
    lo += passed * step;
  }
  const int32_t first = __builtin_amdgcn_readlane(lo, 0), past = __builtin_amdgcn_readlane(lo, 32);
  return {idx + beg + first, past - first, static_cast<int32_t>(h * s.T), s.T};
}

// one row of the bf16 lists
__device__ __forceinline__ void gather_list_row(const Shape& s, int64_t head, int64_t row, const ListKeys& kl,
                                                const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                                                const uint16_t* __restrict__ V, uint16_t* __restrict__ O) {
  const int64_t first = head * s.T * kHeadDim, at = row * kHeadDim;
  gather_row_bf16(kl, s.scale * kLog2e, Q + at, K + first, V + first, O + at);
}

// ------------------------------------------------------------------------------------------
// bf16, dense lists: 128 rows of one head per block, tiles of 64 keys on the matrix cores.
//
// The rows' lists are turned into key bits window by window (1024 keys).  A wave takes its 32 rows one
// after the other: a row's entries of the window are at most 1024 consecutive list entries from its
// cursor on.  They come straight to LDS, up to eight pieces of 256 entries ahead, and set the row's bits with one
// atomic OR for four entries of one word.  Then the keys any row of the block uses are ORed together; steps
// without one are skipped, and unused keys of a step are replaced by a used one.  What another row of the block
// lists cannot reach a row either: a value that is not finite gives NaN against a weight of zero, and rows whose
// accumulators are not finite are left to the gather form.
//
// This is right for lists that ascend without repetition.  Whatever else the caller passes is found out
// by counting: the bits set over all windows equal the list lengths exactly when every entry was seen,
// valid and unique.  A block leaves its rows to the gather form at the first window after which a cursor is
// not where it should be.
//
// Bound: unpacking and products take turns.  B = 4, H = 12, T = 2048, 75 M entries from the FlatCSR tensor: 160 us, of
// which the start of a block (its rows' places in the tensor) 28, unpacking alone 78 (3.8 TB/s), products alone 85.
// Before, 210 us: entries loaded through generic pointers, whose loads the compiler lets out one at a time, a byte
// strip per row that was read back and packed, and products on one buffer with two barriers a step.  Windows that
// start staggered over the blocks of a CU, so that their phases alternate, took 171.  See the launcher for when a
// block takes this form and what it gives.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ int32_t wave_sum(int32_t x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, false);   // quad xor 1
  x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, false);   // quad xor 2
  x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, false);  // row_half_mirror
  x += __builtin_amdgcn_update_dpp(0, x, 0x140, 0xf, 0xf, false);  // row_mirror
  const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  const uint32_t y = a[0] + a[1];
  const auto b = __builtin_amdgcn_permlane32_swap(y, y, false, false);
  return static_cast<int32_t>(b[0] + b[1]);
}

constexpr int kTileRows = 128, kWindow = 1024;
constexpr int kChunk = 64, kRow = kHeadDim;  // staged rows as in the power-of-two kernel
constexpr int kRing = 8;                  // pieces of 256 list entries a wave has on their way
constexpr int kBitRow = kWindow / 32 + 4;  // words per row of key bits, padded

// Do the 128 rows from row0 on take tiles?  Both forms cost about a fixed time and one per key.  With the chip
// full: 128 rows read one by one 58 ns + 1.28 ns a listed key per row, the tile walk 96 ns per 1024 keys spanned.
// Inside a launch that has tiles a little less than that counts, since rows left over pay for a second tail,
// and a block takes no less than 115 ns.  The answer comes from eight rows of the block, the lists of all heads
// together and the span of the last one: for a FlatCSR tensor that takes row pointers instead of searches, and
// lists and tensor of the same mask get the same answer.  The whole wave calls.
constexpr float kRowsNs = 58.f, kRowKeyNs = 1.28f, kWindowNs = 96.f, kBlockNs = 115.f;
template <bool FLAT>
__device__ __forceinline__ bool takes_tiles(const Shape& s, int64_t head, int32_t row0, const int32_t* __restrict__ idx,
                                            const int32_t* __restrict__ cnt, int32_t L,
                                            const int64_t* __restrict__ crow) {
  const int lane = threadIdx.x & 63;
  const int32_t t = min(row0 + 16 * (lane & 7) + 15, s.T - 1);
  const int64_t b = head / s.H;
  int32_t n = 0, last = 0;
  if (!FLAT) {
    for (int32_t h = lane >> 3; h < s.H; h += 8) {
      const int64_t at = (b * s.H + h) * s.T + t;
      const int32_t nh = min(max(cnt[at], 0), L);
      n += nh;
      if (h == s.H - 1 && nh > 0) last = idx[at * L + nh - 1];
    }
  } else if (lane < 8) {
    const int64_t beg = crow[b * s.T + t], end = crow[b * s.T + t + 1];
    n = static_cast<int32_t>(max(end - beg, static_cast<int64_t>(0)));
    if (n > 0) last = static_cast<int32_t>(idx[end - 1] - static_cast<int64_t>(s.H - 1) * s.T);
  }
  n = wave_sum(n);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) last = max(last, __shfl_xor(last, off, kWave));
  const float rows = 8.f * static_cast<float>(s.H), windows = static_cast<float>(min(last, s.T - 1) + 1) / static_cast<float>(kWindow);
  return n > 0 && fmaf(kRowKeyNs, static_cast<float>(n), kRowsNs * rows) >= rows * fmaxf(0.9f * kWindowNs * windows, kBlockNs);
}
// block -> (head, first row): heads in groups, the last (longest, if causal) rows first
__device__ __forceinline__ void tile_block(const Shape& s, int32_t group_heads, int64_t* head, int32_t* row0) {
  const uint32_t wgs = (s.T + kTileRows - 1) / kTileRows;
  const uint32_t per_group = static_cast<uint32_t>(group_heads) * wgs;
  const uint32_t place = dealt_in_turn(blockIdx.x, gridDim.x, 3, s.causal);
  const uint32_t grp = place / per_group, rem = place - grp * per_group;
  const uint32_t nh = min(static_cast<uint32_t>(group_heads), static_cast<uint32_t>(s.N) - grp * group_heads);
  *head = static_cast<int64_t>(grp) * group_heads + rem % nh;
  *row0 = static_cast<int32_t>(wgs - 1 - rem / nh) * kTileRows;
}

template <bool FLAT>
__global__ __launch_bounds__(kWavesPerBlock* kWave) void sparse_attn_bf16_kernel(
    Shape s, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ V, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ cnt, int32_t L, const int64_t* __restrict__ crow,
    uint16_t* __restrict__ O) {
  const int64_t row = wave_row();
  const int64_t nrows = static_cast<int64_t>(s.N) * s.T;
  if (row >= nrows) return;
  gather_list_row(s, row / s.T, row, wave_key_list<FLAT>(s, row, idx, cnt, L, crow), Q, K, V, O);
}

// The tile walk leaves rows to the kernel that follows it, four rows a wave, by this pattern in place of their
// result (its first word, where the block took no tiles).  A result may look like that (it is a NaN); the row is
// then computed twice.
constexpr uint32_t kRowLeft = 0xffffffffu;
constexpr int kRestRows = 4;
template <bool FLAT>
__global__ __launch_bounds__(kWavesPerBlock* kWave) void list_rest_kernel(
    Shape s, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt, int32_t L, const int64_t* __restrict__ crow,
    uint16_t* __restrict__ O) {
  const int lane = threadIdx.x & 63;
  const int64_t row0 = wave_row() * kRestRows, nrows = static_cast<int64_t>(s.N) * s.T, mine = row0 + lane;
  const bool left = lane < kRestRows && mine < nrows && *reinterpret_cast<const uint32_t*>(O + mine * kHeadDim) == kRowLeft;
  for (uint64_t rows = __ballot(left); rows != 0ull; rows &= rows - 1ull) {
    const int64_t row = row0 + __ffsll(static_cast<unsigned long long>(rows)) - 1;
    gather_list_row(s, row / s.T, row, wave_key_list<FLAT>(s, row, idx, cnt, L, crow), Q, K, V, O);
  }
}

// ODD: K or V starts between two 4-byte words, so a step's pieces wait in registers.
template <bool FLAT, bool ODD>
__global__ __launch_bounds__(256, 3) void list_tile_kernel(Shape s, const uint16_t* __restrict__ Q,
                                                           const uint16_t* __restrict__ K,
                                                           const uint16_t* __restrict__ V,
                                                           const int32_t* __restrict__ idx,
                                                           const int32_t* __restrict__ cnt, int32_t L,
                                                           const int64_t* __restrict__ crow,
                                                           uint16_t* __restrict__ O, int32_t group_heads) {
  __shared__ __attribute__((aligned(16))) uint16_t KVs[2][2][kChunk * kRow];  // [place][K, V]
  __shared__ __attribute__((aligned(16))) uint32_t bits[kTileRows * kBitRow];
  __shared__ uint32_t used[2][kWindow / 32];  // keys of the window any row of the block lists
  __shared__ int32_t red[4];
  __shared__ uint32_t astray;  // a row whose list is not what the walk takes it for
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ql = lane & 31, g = lane >> 5;
  int64_t head;
  int32_t row0;
  tile_block(s, group_heads, &head, &row0);
  if (!takes_tiles<FLAT>(s, head, row0, idx, cnt, L, crow)) {
    if (tid < kTileRows && row0 + tid < s.T) *reinterpret_cast<uint32_t*>(O + (head * s.T + row0 + tid) * kHeadDim) = kRowLeft;
    return;
  }

  const int32_t t = row0 + 32 * wid + ql;
  // lane r < 32 holds the list of row 32 wid + r
  ListKeys kl = {idx, 0, 0, s.T};
  if (lane < 32 && t < s.T) kl = key_list<FLAT>(s, head * s.T + t, idx, cnt, L, crow);
  kl.n = max(kl.n, 0);
  int32_t span = kl.n > 0 ? min(max(kl.p[kl.n - 1] - kl.base, 0), s.T - 1) + 1 : 0;
  // 256-entry pieces of the row's list that a window of an evenly spread list takes, and a little more
  const int32_t expect = span > 0 ? min(4, static_cast<int32_t>(static_cast<float>(kl.n) * static_cast<float>(kWindow) / static_cast<float>(span) + 64.f) / 256 + 1) : 1;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) span = max(span, __shfl_xor(span, off, kWave));
  if (lane == 0) red[wid] = span;
  if (tid == 0) astray = 0u;
  const uint16_t* Qr = Q + (head * s.T + min(t, s.T - 1)) * kHeadDim + 8 * g;
  bf16x8 bq[4];
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) bq[kc] = *reinterpret_cast<const bf16x8*>(Qr + 16 * kc);
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) asm volatile("" : "+v"(bq[kc]));

  const uint32_t row_bytes = kHeadDim * 2, head_bytes = static_cast<uint32_t>(s.T) * row_bytes;
  const u32x4 Kres = buffer_words(K + head * static_cast<int64_t>(s.T) * kHeadDim, head_bytes);
  const u32x4 Vres = buffer_words(V + head * static_cast<int64_t>(s.T) * kHeadDim, head_bytes);
  const int srow = tid >> 3;
  const uint32_t kpart = 16 * ((tid & 7) ^ ((srow >> 1) & 7)), vpart = 16 * ((tid & 7) ^ (((srow >> 1) & 1) << 2));
  int kat[4];  // this lane's pieces of a K row: slots 2 kc + g of row ql
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) kat[kc] = ql * kRow + 8 * ((2 * kc + g) ^ ((ql >> 1) & 7));

  floatx16 oacc[2];
#pragma unroll
  for (int i = 0; i < 16; ++i) { oacc[0][i] = 0.f; oacc[1][i] = 0.f; }
  float m_ref = 0.f, m_thr = -INFINITY, l_run = 0.f;
  const float c = s.scale * kLog2e;
  const MinusOnes minus = minus_ones();
  const uint32_t inf_bits = 0xff800000u;

  int32_t cursor = 0;    // lane r: list entries of row 32 wid + r taken so far
  if (tid < 2 * (kWindow / 32)) used[tid / (kWindow / 32)][tid % (kWindow / 32)] = 0u;
  __syncthreads();
  span = max(max(red[0], red[1]), max(red[2], red[3]));

  const uint64_t lp = reinterpret_cast<uint64_t>(kl.p);
  for (int32_t w0 = 0, win = 0; w0 < span; w0 += kWindow, ++win) {
    // Four consecutive entries per lane and load; a load that would reach past the list is moved back to
    // end with it (entries unpacked twice set the same bit), so no entry needs a test of its place.
    {
      uint32_t* const rows = &bits[32 * wid * kBitRow];  // the wave's rows
      for (int x = 4 * lane; x < 32 * kBitRow; x += 4 * kWave) *reinterpret_cast<uint4*>(rows + x) = make_uint4(0u, 0u, 0u, 0u);
    }
    const uint32_t nkeys = static_cast<uint32_t>(min(kWindow, s.T - w0));
    // The entries come 256 at a time, straight to LDS in the order of the rows: a ring of eight pieces in the wave's
    // quarter of the place that the products' keys and values take later.
    const int32_t pieces = cursor < kl.n ? min(expect, (kl.n - cursor + 255) >> 8) : 0;
    int32_t issued = 0, taken = 0, next = 0;  // pieces asked for, pieces unpacked, the next row to ask for
    uint16_t* const ring = &KVs[0][0][0] + wid * (kRing * 512);
    auto row_base = [&](int rr) {
      return reinterpret_cast<const int32_t*>(
          static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(lp), rr)) |
          (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(lp >> 32), rr))) << 32));
    };
    auto entry_off = [&](int32_t at, int32_t n) { return static_cast<uint32_t>(4 * min(at, max(n - 4, 0))); };
    auto ask = [&]() {
      while (next < 32) {
        const int32_t c = __builtin_amdgcn_readlane(pieces, next);
        if (issued - taken + c > kRing) break;
        if (c > 0) {
          const int32_t n = __builtin_amdgcn_readlane(kl.n, next), cu = __builtin_amdgcn_readlane(cursor, next);
          const u32x4 list = buffer_words(row_base(next), static_cast<uint32_t>(min(n, 1 << 29)) * 4u);
          for (int32_t q = 0; q < c; ++q, ++issued)
            buffer_load_lds16(list, ring + (issued & (kRing - 1)) * 512, entry_off(cu + 256 * q + 4 * lane, n));
        }
        ++next;
      }
    };
    auto take_row = [&](int rr) {
      const int32_t n = __builtin_amdgcn_readlane(kl.n, rr), cu = __builtin_amdgcn_readlane(cursor, rr);
      const int32_t key0 = __builtin_amdgcn_readlane(kl.base, rr) + w0;
      const int32_t c = __builtin_amdgcn_readlane(pieces, rr);
      if (c == 0) return;  // wave-uniform
      uint32_t* const row = &bits[(32 * wid + rr) * kBitRow];
      // Four entries of one whole word are set at once, which is most of them where lists hold runs of keys.  Entries of
      // other windows (and invalid ones) set nothing, or the spare bit past the window's last key.
      // (not the lanes past the list's end, which all read its last entries)
      auto unpack = [&](const uint4& v, int32_t from) {
        if (from + 4 * lane >= n) return;
        const uint32_t k0 = static_cast<uint32_t>(key0);
        uint32_t e[4] = {v.x - k0, v.y - k0, v.z - k0, v.w - k0};
        if (n < 4) {  // (words past the list are no entries)
#pragma unroll
          for (int i = 1; i < 4; ++i) e[i] = i < n ? e[i] : e[0];
        }
        const uint32_t apart = (e[0] ^ e[1]) | (e[0] ^ e[2]) | (e[0] ^ e[3]);
        if (apart < 32u && e[0] < (nkeys & ~31u)) {
          atomicOr(&row[e[0] >> 5], (1u << (e[0] & 31u)) | (1u << (e[1] & 31u)) | (1u << (e[2] & 31u)) | (1u << (e[3] & 31u)));
        } else if (min(min(e[0], e[1]), min(e[2], e[3])) < nkeys) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t at = min(e[i], nkeys);
            atomicOr(&row[at >> 5], 1u << (at & 31u));
          }
        }
      };
      lds_loads_pending(issued - taken - c);
      int32_t last = 0;
      for (int32_t q = 0; q < c; ++q, ++taken) {
        const uint4 v = *reinterpret_cast<const uint4*>(ring + (taken & (kRing - 1)) * 512 + 8 * lane);
        unpack(v, cu + 256 * q);
        last = __builtin_amdgcn_readlane(static_cast<int>(v.w), 63);
      }
      // more entries than expected: the last one requested still lies in the window
      for (int32_t done = 256 * c; done < kWindow && cu + done < n && static_cast<uint32_t>(last - key0) < nkeys; done += 256) {
        const auto list = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(row_base(rr)), 0, min(n, 1 << 29) * 4, kBufferFlags);
        const uint4 v = buffer_load16(list, entry_off(cu + done + 4 * lane, n));
        unpack(v, cu + done);
        last = __builtin_amdgcn_readlane(static_cast<int>(v.w), 63);
      }
    };
    ask();
#pragma unroll 1
    for (int rr = 0; rr < 32; ++rr) {
      take_row(rr);
      ask();
    }
    __builtin_amdgcn_wave_barrier();
    // (the spare bit lies among the window's words when T ends there)
    if (nkeys < kWindow && lane < 32) bits[(32 * wid + lane) * kBitRow + (nkeys >> 5)] &= ~(1u << (nkeys & 31u));
    __builtin_amdgcn_wave_barrier();
    {
      // entries taken: the bits of row lane / 2, half a row each
      const uint4* const half = reinterpret_cast<const uint4*>(&bits[(32 * wid + (lane >> 1)) * kBitRow + (kWindow / 64) * (lane & 1)]);
      int32_t got = 0;
#pragma unroll
      for (int x = 0; x < kWindow / 256; ++x) {
        const uint4 v = half[x];
        got += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
      }
      got += __shfl_xor(got, 1, kWave);
      got = __shfl(got, 2 * (lane & 31), kWave);
      cursor += lane < 32 ? got : 0;
    }
    // A row's next entry lies past the window, and after the last window there is none.  (The keys found are
    // different entries of the list, so a cursor that ends with the list has met every entry once.)
    const bool lost = w0 + kWindow >= span ? cursor != kl.n : (cursor < kl.n && kl.p[cursor] - kl.base < w0 + kWindow);
    const uint64_t rows_lost = __ballot(lost);
    if (lane == 0 && rows_lost != 0ull) atomicOr(&astray, 1u);
    // keys used by the block, in 32-key words: lanes i and i + 32 go over 16 of the wave's rows each
    static_assert(kWindow == 32 * 32, "a word per lane of half a wave");
    uint32_t wave_used = 0u;
#pragma unroll
    for (int r = 0; r < 16; ++r) wave_used |= bits[(32 * wid + 16 * g + r) * kBitRow + ql];
    atomicOr(&used[win & 1][ql], wave_used);
    __syncthreads();
    if (astray != 0u) break;
    const uint32_t* uw = used[win & 1];
    // 64-key steps with a used key (uniform): lanes 0..15 look at one step each
    uint32_t steps = static_cast<uint32_t>(__ballot(lane < kWindow / 64 && (uw[2 * (lane & 15)] | uw[2 * (lane & 15) + 1]) != 0u));
    u32x4 odd[4];
    auto fetch = [&](int step, int place) __attribute__((always_inline)) {
      // (rows of unused keys repeat the step's first used one)
      const uint32_t u0 = uw[2 * step], u1 = uw[2 * step + 1];
      const uint32_t k0 = static_cast<uint32_t>(w0 + 64 * step);
      const uint32_t first = k0 + (u0 != 0u ? __ffs(u0) - 1 : 31 + __ffs(u1));
      const uint32_t oa = ((u0 >> srow) & 1u ? k0 + srow : first) * row_bytes;
      const uint32_t ob = ((u1 >> srow) & 1u ? k0 + 32 + srow : first) * row_bytes;
      if constexpr (ODD) {
        odd[0] = load16_odd(Kres, oa + kpart);
        odd[1] = load16_odd(Kres, ob + kpart);
        odd[2] = load16_odd(Vres, oa + vpart);
        odd[3] = load16_odd(Vres, ob + vpart);
      } else {
        uint16_t* const at = &KVs[place][0][wid * 8 * kRow];
        buffer_load_lds16(Kres, at, oa + kpart, at + 32 * kRow, ob + kpart);
        buffer_load_lds16(Vres, at + kChunk * kRow, oa + vpart, at + (kChunk + 32) * kRow, ob + vpart);
      }
    };
    auto park = [&](int place) __attribute__((always_inline)) {
      if constexpr (ODD) {
        uint16_t* const at = &KVs[place][0][wid * 8 * kRow];
        park16(at, odd[0]);
        park16(at + 32 * kRow, odd[1]);
        park16(at + kChunk * kRow, odd[2]);
        park16(at + (kChunk + 32) * kRow, odd[3]);
      }
    };
    auto walk = [&](auto place_c) __attribute__((always_inline)) {
      constexpr int place = decltype(place_c)::value;
      const int step = __ffs(steps) - 1;
      steps &= steps - 1u;
      if (steps != 0u) fetch(__ffs(steps) - 1, place ^ 1);
#pragma unroll
      for (int sc = 0; sc < 2; ++sc) {
        const uint32_t word = bits[(32 * wid + ql) * kBitRow + 2 * step + sc];
        if (__ballot(word != 0u) == 0ull) continue;  // no row of the wave uses these keys
        const uint16_t* Kr = &KVs[place][0][32 * sc * kRow];
        floatx16 sv;
#pragma unroll
        for (int i = 0; i < 16; ++i) sv[i] = 0.f;
#pragma unroll
        for (int kc = 0; kc < 4; ++kc)
          sv = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(Kr + kat[kc]), bq[kc], sv, 0, 0, 0);
        // reg i <-> key slot 8 (i / 4) + 4 g + i % 4
        const uint32_t wg = word >> (4 * g);
        float y[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const uint32_t sel = static_cast<uint32_t>(static_cast<int32_t>(wg << (31 - (8 * (i >> 2) + (i & 3)))) >> 31);
          y[i] = __uint_as_float((sel & __float_as_uint(fmaf(sv[i], c, -m_ref))) | (~sel & inf_bits));
        }
        bf16x8 av[2][2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          const uint16_t* Vr = &KVs[place][1][(32 * sc + 4 * g + ((ql & 15) >> 2)) * kRow + 32 * (mt ^ ((ql >> 3) & 1)) + (ql & 16) + 4 * (ql & 3)];
#pragma unroll
          for (int c2 = 0; c2 < 2; ++c2) {
            const bf16x4 lo = lds_transpose4(Vr + (16 * c2) * kRow);
            const bf16x4 hi = lds_transpose4(Vr + (16 * c2 + 8) * kRow);
            av[mt][c2] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          }
        }
        float ymax = max_of(y);
        if (__ballot(ymax > m_thr) != 0ull) {
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
        l_run += add_weighted_rows(y, av, minus, oacc);
      }
      if (steps != 0u) park(place ^ 1);
      lds_loads_done();
      __syncthreads();
    };
    if (steps != 0u) {
      fetch(__ffs(steps) - 1, 0);
      park(0);
      lds_loads_done();
    }
    __syncthreads();
    while (steps != 0u) {
      walk(std::integral_constant<int, 0>{});
      if (steps != 0u) walk(std::integral_constant<int, 1>{});
    }
    if (tid < kWindow / 32) used[(win & 1) ^ 1][tid] = 0u;  // for the next window (nobody reads it now)
    __syncthreads();
  }
  l_run = half_sum(l_run);
  const uint32_t left = astray != 0u ? ~0u : rows_not_finite(l_run, oacc);
  __syncthreads();  // (blocks that stop early leave the loop in front of its last barrier)
  const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
  store_rows(&KVs[0][0][0] + wid * 32 * kRow, oacc, inv, left, [&](int r) -> uint16_t* {
    const int32_t tr = row0 + 32 * wid + r;
    return tr < s.T ? O + (head * s.T + tr) * kHeadDim : nullptr;
  });
}

template <bool FLAT>
__global__ __launch_bounds__(kWavesPerBlock* kWave) void sparse_attn_f32_kernel(
    Shape s, const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const int32_t* __restrict__ idx, const int32_t* __restrict__ cnt, int32_t L,
    const int64_t* __restrict__ crow, float* __restrict__ O) {
  const int64_t row = wave_row();
  const int64_t nrows = static_cast<int64_t>(s.N) * s.T;
  if (row >= nrows) return;
  const int64_t head = row / s.T, first = head * s.T * kHeadDim, at = row * kHeadDim;
  gather_row_f32(wave_key_list<FLAT>(s, row, idx, cnt, L, crow), static_cast<double>(s.scale) * 1.4426950408889634, Q + at, K + first,
                 V + first, O + at);
}

// Tiles from one 128-row block per CU on, where lists of `longest` keys would take them over the whole sequence
// (causal: over three quarters of it, earlier rows span less; a launch of which only a part takes tiles pays for
// both forms' tails), and not where the rows, read one by one, are done before a block could be: alone on its CU a
// block takes 58 us per window.
// us, rows / tiles: 48 heads, T = 2048, bidirectional, 128 keys 150 / 165, 256 keys 285 / 165, causal 128 keys 150 /
// 115; 64 heads, T = 4096, 256 keys 830 / 790, causal 810 / 530; 32 heads, T = 1024, 64 keys 34 / 62, 256 keys 104 /
// 63.
bool tiles_worth_a_launch(const Shape& s, int64_t blocks, int32_t longest) {
  if (blocks < 256 || s.T > (1 << 24) || static_cast<int64_t>(s.H) * s.T > (1 << 28)) return false;
  const float rows = kRowsNs + kRowKeyNs * static_cast<float>(longest), windows = static_cast<float>(s.T) / static_cast<float>(kWindow);
  return rows >= (s.causal ? 0.75f : 1.f) * windows * kWindowNs &&
         rows * static_cast<float>(blocks) >= 58e3f * (windows > 1.f ? windows : 1.f);
}

template <bool FLAT>
void launch_lists(const Shape& s, sea_dtype dt, const void* Q, const void* K, const void* V, const int32_t* idx,
                  const int32_t* cnt, int32_t L, const int64_t* crow, int32_t longest, void* O, hipStream_t st) {
  const int64_t nrows = static_cast<int64_t>(s.N) * s.T, tiles = static_cast<int64_t>(s.N) * ((s.T + kTileRows - 1) / kTileRows);
  const dim3 block(kWavesPerBlock * kWave);
  if (dt == SEA_F32) {
    hipLaunchKernelGGL(sparse_attn_f32_kernel<FLAT>, row_grid(nrows), block, 0, st, s, static_cast<const float*>(Q),
                       static_cast<const float*>(K), static_cast<const float*>(V), idx, cnt, L, crow, static_cast<float*>(O));
    return;
  }
  const uint16_t *q = static_cast<const uint16_t*>(Q), *k = static_cast<const uint16_t*>(K), *v = static_cast<const uint16_t*>(V);
  uint16_t* o = static_cast<uint16_t*>(O);
  // (rows the tiles leave are marked in O and read Q afterwards: not where O lies in the place of Q)
  const uintptr_t at_o = reinterpret_cast<uintptr_t>(o), at_q = reinterpret_cast<uintptr_t>(q), bytes = static_cast<uintptr_t>(nrows) * kHeadDim * 2;
  const bool apart = at_o >= at_q + bytes || at_q >= at_o + bytes;
  if (apart && tiles_worth_a_launch(s, tiles, longest)) {
    const auto kernel = starts_odd(k) || starts_odd(v) ? &list_tile_kernel<FLAT, true> : &list_tile_kernel<FLAT, false>;
    hipLaunchKernelGGL(kernel, dim3(static_cast<uint32_t>(tiles)), dim3(256), 0, st, s, q, k, v, idx, cnt, L, crow, o,
                       group_heads_for(s, s.T));
    hipLaunchKernelGGL(list_rest_kernel<FLAT>, row_grid((nrows + kRestRows - 1) / kRestRows), block, 0, st, s, q, k, v, idx,
                       cnt, L, crow, o);
  } else {
    hipLaunchKernelGGL(sparse_attn_bf16_kernel<FLAT>, row_grid(nrows), block, 0, st, s, q, k, v, idx, cnt, L, crow, o);
  }
}

}  // namespace

hipError_t launch_sparse_attn(const Shape& s, sea_dtype dt, const void* Q, const void* K,
                              const void* V, const int32_t* idx, const int32_t* cnt, int32_t L,
                              const int64_t* crow, int32_t longest, void* O, hipStream_t st) {
  StageScope scope(SEA_STAGE_SPARSE, st);
  if (crow != nullptr) launch_lists<true>(s, dt, Q, K, V, idx, cnt, L, crow, longest, O, st);
  else launch_lists<false>(s, dt, Q, K, V, idx, cnt, L, crow, longest, O, st);
  return hipGetLastError();
}

}  // namespace sea
