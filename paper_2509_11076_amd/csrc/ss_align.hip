// Sequence aligner: longest common subsequence of the reference and the current operator sequence
// and the canonical alignment read off it; the matcher's fourth level (Sec. 5.1 asks for tolerance
// to minor sequence variations with integer-only comparison and gives no algorithm).
//
// The dynamic programme runs in its bit-vector form: bit j of V_i is 0 exactly when
// L[i][j+1] = L[i][j] + 1, V_0 is all ones, and one reference operator advances the row by
//     V' = (V + (V & M)) | (V & ~M),     M = positions of cur holding that operator's key.
// The addition's carry runs through the whole row, so a row is not updated at once: lane l holds word l
// and works on row t - l in step t, taking the carry that lane l - 1 produced for the same row one step
// earlier (all carries of a wavefront are one 64-bit lane mask, so handing them on is one scalar shift).
// A wavefront covers a strip of 2,048 columns; a longer cur takes one workgroup per strip, each reading
// the carries out of the strip before it.  The rows stay where they were written, one step after the
// other, and the alignment is read back from (n, m): equal operators pair, otherwise left if bit j-1 of
// V_i is set (L[i][j-1] = L[i][j]), else up; on the host for short sequences, on the GPU for long ones.
#include <algorithm>
#include <cstring>
#include <unordered_map>

#include "ss_internal.h"

namespace {

typedef unsigned long long u64;

constexpr uint32_t kAlignLenLimit = 1u << 16;          // at most 32 strips
constexpr size_t kAlignRowBytesLimit = 1ull << 30;     // rows kept for the walk back
constexpr uint32_t kBlock = 32;                        // steps between two looks at the neighbouring strip
constexpr uint32_t kGroup = 8;                         // steps whose masks are looked up together
constexpr uint32_t kStripWords = 64;                   // 32-bit words of a row, one per lane
constexpr uint32_t kLdsKeys = 256;                     // mask rows (with the empty one) a strip keeps in LDS at most, 256 bytes each
constexpr size_t kLdsBytes = 160 * 1024;               // for these and the reference's ids
constexpr uint32_t kIdPad = 64;                        // entries before the first id (lanes whose row has not begun)
// Rows up to this many bytes go straight to host memory and are walked there: beside the kernel's pace they cost the
// link nothing up to about 13 GB/s, and the walk on the GPU takes four more launches and two copies.
constexpr size_t kHostRowBytes = 4u << 20;
constexpr uint32_t kCarryPad = 4;                      // carry words a strip may look at beyond its neighbour's last
constexpr uint32_t kPollLimit = 1u << 24;              // looks at a carry word before a strip gives up

// steps a strip takes for n rows, whole blocks of them
static inline uint32_t steps_of(uint32_t n) { return (n + kStripWords - 1 + kBlock - 1) / kBlock * kBlock; }

// entries of a padded id array, a multiple of 16 bytes
static inline __host__ __device__ uint32_t id_length(uint32_t n_steps) { return kIdPad + n_steps + 2 * kBlock; }

// word w of row r: lane w % 64 of strip w / 64 wrote it in step r + w % 64
static inline __host__ __device__ size_t row_word(uint32_t r, uint32_t w, uint32_t steps) {
  const uint32_t l = w % kStripWords;
  return ((size_t)(w / kStripWords) * steps + r + l) * kStripWords + l;
}

// A key id as it is stored: 16 bits, already multiplied by the 256 bytes of an LDS mask row, where the mask rows fit
// LDS; else 32 bits as it is.
static inline __host__ __device__ uint32_t key_of(uint16_t id) { return id >> 8; }
static inline __host__ __device__ uint32_t key_of(uint32_t id) { return id; }
static inline void set_key(uint16_t *id, uint32_t key) { *id = (uint16_t)(key << 8); }
static inline void set_key(uint32_t *id, uint32_t key) { *id = key; }

template <class Id>
__global__ void ss_align_masks_kernel(const Id *__restrict__ cur_id, uint32_t m, uint32_t *__restrict__ masks,
                                      uint32_t W) {
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < m) atomicOr(&masks[(size_t)key_of(cur_id[j]) * W + (j >> 5)], 1u << (j & 31));
}

// One row step of a word, N = ~M: V' = (V + (V & M) + carry in) | (V & ~M); the carries in and out are lane masks.
// Written out because the compiler turns a carry that leaves as a lane mask into a select and a compare.
__device__ __forceinline__ u64 row_step(uint32_t &V, uint32_t N, u64 cin) {
  uint32_t a;
  u64 cout;
  asm("v_bfi_b32 %[a], %[n], 0, %[v]\n\t"
      "v_addc_co_u32_e64 %[a], %[co], %[v], %[a], %[ci]\n\t"
      "v_and_or_b32 %[v], %[v], %[n], %[a]"
      : [v] "+v"(V), [a] "=&v"(a), [co] "=&s"(cout)
      : [n] "v"(N), [ci] "s"(cin));
  return cout;
}

// The same, and hist = 2 * hist + this lane's bit of `before`, the carries out of the previous step (written long
// enough ago: a carry mask may be read again two instructions after it was written at the earliest).
__device__ __forceinline__ u64 row_step_kept(uint32_t &V, uint32_t N, u64 cin, uint32_t &hist, u64 before) {
  uint32_t a;
  u64 cout;
  asm("v_bfi_b32 %[a], %[n], 0, %[v]\n\t"
      "v_addc_co_u32_e64 %[a], %[co], %[v], %[a], %[ci]\n\t"
      "v_addc_co_u32_e64 %[h], vcc, %[h], %[h], %[be]\n\t"
      "v_and_or_b32 %[v], %[v], %[n], %[a]"
      : [v] "+v"(V), [a] "=&v"(a), [co] "=&s"(cout), [h] "+v"(hist)
      : [n] "v"(N), [ci] "s"(cin), [be] "s"(before)
      : "vcc");
  return cout;
}

// The ids of kGroup consecutive steps; 16-bit ids stay packed until they are used, so that reading them is one load
// that nothing waits for.
template <class Id>
struct IdGroup {
  Id v[kGroup];
  __device__ __forceinline__ void load(const Id *p) {
#pragma unroll
    for (uint32_t u = 0; u < kGroup; ++u) v[u] = p[u];
  }
  __device__ __forceinline__ uint32_t operator[](uint32_t u) const { return v[u]; }
};
template <>
struct IdGroup<uint16_t> {
  uint4 v;
  __device__ __forceinline__ void load(const uint16_t *p) { __builtin_memcpy(&v, p, 16); }
  __device__ __forceinline__ uint32_t operator[](uint32_t u) const {
    const uint32_t x = u < 2 ? v.x : u < 4 ? v.y : u < 6 ? v.z : v.w;
    return u & 1 ? x >> 16 : x & 0xFFFFu;
  }
};
static_assert(kGroup == 8, "a group of 16-bit ids is one 16-byte word");

struct RowsArgs {
  const uint32_t *masks;     // wide ids only
  u64 *carry;
  uint32_t *rows, *gave_up;
  uint32_t W, n_steps;
};

// All rows of one strip.  my_ids: entry t is the id of this lane's row in step t; table: this lane's word of an LDS
// mask row of key 0 (inverted).  carry[strip][block]: bit u = carry out of the strip's last lane in step 32 * block + u,
// bit 32 = the word is there (the value and its arrival are one store, so no fence is needed); cleared before the
// launch.  A strip waits only for the strip before it, which waits for no later one, and not for ever (kPollLimit).
template <class Id, bool TAKES, bool GIVES>
__device__ __forceinline__ void strip_rows(const RowsArgs &a, const Id *my_ids, const uint8_t *table) {
  constexpr bool kLds = sizeof(Id) == 2;
  const uint32_t lane = threadIdx.x, strip = blockIdx.x, n_blocks = a.n_steps / kBlock;
  auto mask_of = [&](uint32_t id) -> uint32_t {              // inverted
    if constexpr (kLds) return *reinterpret_cast<const uint32_t *>(table + id);
    return ~a.masks[(size_t)id * a.W + strip * kStripWords + lane];
  };
  const u64 *const cin_words = a.carry + (size_t)(strip - (TAKES ? 1 : 0)) * (n_blocks + kCarryPad);
  u64 *const cout_words = a.carry + (size_t)strip * (n_blocks + kCarryPad);
  auto peek = [&](uint32_t block) { return __hip_atomic_load(cin_words + block, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  // x: what a peek saw earlier; the result is uniform, as it takes part in lane masks
  auto carry_word = [&](uint32_t block, u64 x) -> uint32_t {
    uint32_t word = __builtin_amdgcn_readfirstlane((uint32_t)x);
    if (__builtin_expect(__builtin_amdgcn_readfirstlane((uint32_t)(x >> 32)) != 0, 1)) return word;
#pragma unroll 1
    for (uint32_t tries = 0; tries < kPollLimit; ++tries) {
      __builtin_amdgcn_s_sleep(1);
      const u64 y = peek(block);
      word = __builtin_amdgcn_readfirstlane((uint32_t)y);
      if (__builtin_amdgcn_readfirstlane((uint32_t)(y >> 32))) return word;
    }
    if (lane == 0) __hip_atomic_store(a.gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return 0;
  };

  uint32_t V = ~0u, hist = 0;
  u64 cmask = 0;
  uint32_t N[kBlock];
  IdGroup<Id> ids;
#pragma unroll
  for (uint32_t g = 0; g < kBlock; g += kGroup) {
    ids.load(my_ids + g);
#pragma unroll
    for (uint32_t u = 0; u < kGroup; ++u) N[g + u] = mask_of(ids[u]);
  }
  ids.load(my_ids + kBlock);
  uint32_t prev_word = 0;
  u64 ahead = 0;                      // a carry word, looked at one block before it is needed
  if constexpr (TAKES) {
    prev_word = n_blocks > 1 ? carry_word(1, peek(1)) : 0;
    ahead = peek(2);
    asm volatile("" : "+v"(ahead));   // arrived: inside the loop the wait for it then leaves that block's stores in flight
  }
  uint32_t *out = a.rows + (size_t)strip * a.n_steps * kStripWords;        // uniform: lane l of a step is word l
  for (uint32_t b = 0; b < n_blocks; ++b) {
    // lane 0's row in step t is row t; its carry left the strip before in that strip's step t + 63
    uint32_t in = 0;
    if constexpr (TAKES) {
      const uint32_t next_word = b + 2 < n_blocks ? carry_word(b + 2, ahead) : 0;
      in = __builtin_amdgcn_readfirstlane((prev_word >> 31) | (next_word << 1));
      prev_word = next_word;
      ahead = peek(b + 3);
    }
    const Id *const ids_at = my_ids + (b + 1) * kBlock;
#pragma unroll
    for (uint32_t g = 0; g < kBlock; g += kGroup) {
#pragma unroll
      for (uint32_t u = g; u < g + kGroup; ++u) {
        const u64 cin = TAKES ? (cmask << 1) | ((in >> u) & 1u) : cmask << 1;
        cmask = GIVES ? row_step_kept(V, N[u], cin, hist, cmask) : row_step(V, N[u], cin);
        out[u * kStripWords + lane] = V;
      }
#pragma unroll
      for (uint32_t u = 0; u < kGroup; ++u) N[g + u] = mask_of(ids[u]);  // the same steps of the next block
      ids.load(ids_at + g + kGroup);
      // kept in this order: a refill moved up needs a second register, and the copy back waits for the load
      __builtin_amdgcn_sched_barrier(0);
    }
    out += kBlock * kStripWords;
    if constexpr (GIVES) {            // the last lane's carries, first step lowest; hist is one step behind
      const uint32_t h = __builtin_amdgcn_readlane((int)hist, 63);
      const uint32_t word = __builtin_bitreverse32((h << 1) | (uint32_t)(cmask >> 63));
      if (lane == 0)
        __hip_atomic_store(cout_words + b, (1ull << 32) | word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// One wavefront per workgroup, workgroup = strip.  ref_id: n ids with kIdPad entries of the empty mask row before them
// and id_length() - kIdPad - n after them, so that a lane whose row has not begun or is over adds nothing.  16-bit ids:
// the strip builds its own mask table in LDS from cur_id and keeps all the reference's ids there too; wider ids (more
// keys or operators than fit): masks and ids come from device memory.
//
// Bound by the issue of one wavefront's instructions from one step to the next, seven of them for a single strip
// (words of 32 bits, since a wider word puts a second addition into the chain; the table holds ~M, which saves an
// instruction; masks are looked up one block of steps ahead, a carry word one block before it is needed).  18.9 ns a
// row for one strip, 30 ns for sixteen that hand carries on.  Updating a whole row at once in one wavefront, its
// carries crossing lanes by two ballots and scalar arithmetic, took 128 ns a row at 1,156 columns and 755 ns at
// 32,300: 1,154 x 1,156 operators 149 -> 35 us, 32,312 x 32,297 operators 24.5 -> 1.03 ms.
template <class Id>
__global__ __launch_bounds__(64) void ss_align_rows_kernel(const Id *__restrict__ ref_id,
                                                           const Id *__restrict__ cur_id, uint32_t m, RowsArgs a,
                                                           uint32_t n_mask_rows) {
  constexpr bool kLds = sizeof(Id) == 2;
  extern __shared__ uint32_t lds[];
  const uint32_t lane = threadIdx.x, strip = blockIdx.x;
  const uint32_t w0 = strip * kStripWords;
  const uint32_t lanes = min(kStripWords, a.W - w0);
  Id *const lds_ids = reinterpret_cast<Id *>(lds + n_mask_rows * kStripWords);
  if constexpr (kLds) {
    for (uint32_t i = lane; i < n_mask_rows * kStripWords; i += 64) lds[i] = ~0u;
    const uint4 *src = reinterpret_cast<const uint4 *>(ref_id);
    uint4 *dst = reinterpret_cast<uint4 *>(lds_ids);
    const uint32_t n16 = id_length(a.n_steps) * sizeof(Id) / 16;
    for (uint32_t i0 = lane; i0 < n16; i0 += 8 * 64) {
      uint4 x[8];
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u)
        if (i0 + 64 * u < n16) x[u] = src[i0 + 64 * u];
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u)
        if (i0 + 64 * u < n16) dst[i0 + 64 * u] = x[u];
    }
    __syncthreads();
    // two words' columns a pass, sixteen passes of ids in flight
    for (uint32_t g = 0; g < lanes; g += 32) {
      uint32_t id[16];
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u) {
        const uint32_t j = (w0 + g + 2 * u) * 32 + lane;
        id[u] = j < m ? cur_id[j] : 0xFFFFFFFFu;
      }
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u)
        if (id[u] != 0xFFFFFFFFu)
          atomicAnd(&lds[key_of((uint16_t)id[u]) * kStripWords + g + 2 * u + (lane >> 5)], ~(1u << (lane & 31)));
    }
    __syncthreads();
  }
  if (lane >= lanes) return;                                 // beyond the last word: the rest has no barrier
  const Id *const my_ids = (kLds ? lds_ids : ref_id) + kIdPad - lane;
  const uint8_t *const table = reinterpret_cast<const uint8_t *>(lds + lane);
  const bool takes = strip != 0, gives = strip + 1 < gridDim.x;
  if (takes && gives) strip_rows<Id, true, true>(a, my_ids, table);
  else if (takes) strip_rows<Id, true, false>(a, my_ids, table);
  else if (gives) strip_rows<Id, false, true>(a, my_ids, table);
  else strip_rows<Id, false, false>(a, my_ids, table);
}

// ---- the walk back on the GPU ----------------------------------------------------------------------------------
//
// The walk is one chain of n rows, but what 64 rows do to it is a function of one number: how many columns are left
// when it enters them.  So that function is tabulated for every block of 64 rows at once, one thread per entry
// column of a window around the diagonal (ss_align_tab_kernel); one workgroup then follows the blocks' tables from
// the end (ss_align_chain_kernel), and with every block's entry known the blocks are walked again side by side to
// write the pairs (ss_align_pairs_kernel).  A block whose entry lies outside its window, or whose path leaves the tile
// to the left, is walked in place by a wavefront of the chain.
// 32,312 rows: 63 us for the tables, 145 us for the chain (two dependent LDS reads a block), 24 us for the pairs; single
// steps in one wavefront took 97 ns a row (3.1 ms), the rows over the host link (130 MB) 2.3 ms and a walk there.
constexpr uint32_t kWalkRows = 64;
constexpr uint32_t kWindow = 2048;                     // entry columns tabulated per block of rows
constexpr uint32_t kEntries = 256;                     // of these, per workgroup
constexpr uint32_t kMargin = 256;                      // columns a tile reaches to the left of its first entry
constexpr uint32_t kTileWords = (kEntries + kMargin) / 32;
constexpr uint32_t kTileStride = kTileWords + 1;
constexpr uint16_t kNoEntry = 0xFFFF;

// rows of block k (counted from the end): [lo, hi)
struct RowBlock {
  uint32_t lo, hi;
  __device__ RowBlock(uint32_t k, uint32_t n) : lo(n > (k + 1) * kWalkRows ? n - (k + 1) * kWalkRows : 0), hi(n - k * kWalkRows) {}
};

// first entry (columns left) of the block's window: a multiple of kEntries, the scaled diagonal in the middle
__device__ __forceinline__ uint32_t window_start(uint32_t k, uint32_t n, uint32_t m) {
  const uint32_t mid = (uint32_t)((uint64_t)(n - k * kWalkRows) * m / n);
  return (mid > kWindow / 2 ? mid - kWindow / 2 : 0) / kEntries * kEntries;
}

// M and X = M | ~V of rows [lo, hi) and kTileWords words from word w0 on (w0 may be negative: empty); a step of the
// row buffer holds consecutive words of consecutive rows, so threads run along it
template <class Id>
__device__ __forceinline__ void load_tile(const Id *ref_id, const uint32_t *masks, const uint32_t *rows, uint32_t W,
                                          uint32_t n_steps, RowBlock blk, int w0, uint32_t (*M)[kTileStride],
                                          uint32_t (*X)[kTileStride]) {
  const uint32_t n_rows = blk.hi - blk.lo;
  for (uint32_t i = threadIdx.x; i < (kWalkRows + kTileWords) * kTileWords; i += blockDim.x) {
    const uint32_t l = i % kTileWords, t = i / kTileWords;             // row lo + t - l
    if (t < l || t - l >= n_rows) continue;
    const uint32_t r = blk.lo + t - l, q = blk.hi - 1 - r;             // q: how far from the block's last row
    const int w = w0 + (int)l;
    uint32_t mm = 0, x = 0;
    if (w >= 0 && (uint32_t)w < W) {
      mm = masks[(size_t)key_of(ref_id[kIdPad + r]) * W + w];
      x = mm | ~rows[row_word(r, (uint32_t)w, n_steps)];
    }
    M[q][l] = mm;
    X[q][l] = x;
  }
}

// The walk through a block with j columns left on entry; returns the columns left after it, or -1 if it leaves the
// tile.  Per row: the highest column below j that is equal or steps up.  `pair` is told of every pair.
template <class Pair>
__device__ __forceinline__ int walk_tile(uint32_t n_rows, int w0, int j, const uint32_t (*M)[kTileStride],
                                         const uint32_t (*X)[kTileStride], Pair pair) {
  for (uint32_t q = 0; q < n_rows && j > 0; ++q) {
    int w = ((j - 1) >> 5) - w0;
    if (w < 0) return -1;
    uint32_t bits = X[q][w] & (~0u >> (31 - ((j - 1) & 31)));
    while (!bits && --w >= 0) bits = X[q][w];
    if (!bits) {
      if (w0 > 0) return -1;
      return 0;                                              // nothing left in this row: all the columns are used up
    }
    const int b = 31 - __builtin_clz(bits);
    j = (w + w0) * 32 + b;
    if ((M[q][w] >> b) & 1u) pair(q, j);
    else ++j;
  }
  return j;
}

template <class Id>
__global__ __launch_bounds__(kEntries) void ss_align_tab_kernel(const Id *__restrict__ ref_id, uint32_t n,
                                                                const uint32_t *__restrict__ masks, uint32_t m,
                                                                uint32_t W, uint32_t n_steps,
                                                                const uint32_t *__restrict__ rows,
                                                                uint16_t *__restrict__ table) {
  __shared__ uint32_t M[kWalkRows][kTileStride], X[kWalkRows][kTileStride];
  const uint32_t k = blockIdx.x, e0 = window_start(k, n, m) + blockIdx.y * kEntries;
  if (e0 > m) return;
  const RowBlock blk(k, n);
  const int w0 = (int)(e0 / 32) - (int)(kMargin / 32);
  load_tile(ref_id, masks, rows, W, n_steps, blk, w0, M, X);
  __syncthreads();
  const int j = (int)(e0 + threadIdx.x);
  const int out = j <= (int)m ? walk_tile(blk.hi - blk.lo, w0, j, M, X, [](uint32_t, int) {}) : -1;
  table[(size_t)k * kWindow + blockIdx.y * kEntries + threadIdx.x] = out < 0 ? kNoEntry : (uint16_t)(j - out);
}

// One wavefront walks a block in place and writes its pairs: lane q holds one 64-bit word of row hi - 1 - q.  A run of
// equal operators steps one row and one column at a time, so each lane tests the bit of its own row on the diagonal
// and the run's length is the number of leading ones; then one find-first in the row the run ended in.
template <class Id>
__device__ uint32_t walk_in_place(const Id *ref_id, const uint32_t *masks, const uint32_t *rows, uint32_t W,
                                  uint32_t n_steps, RowBlock blk, uint32_t j, int32_t *ref_to_cur) {
  const int lane = threadIdx.x & 63, n_rows = (int)(blk.hi - blk.lo), r = (int)blk.hi - 1 - lane;
  const bool mine_is_row = lane < n_rows;
  const uint32_t id = mine_is_row ? key_of(ref_id[kIdPad + r]) : 0;
  struct Word { u64 M, V; };
  auto load = [&](int w) -> Word {
    Word x = {0ull, ~0ull};
    if (w >= 0 && mine_is_row) {
      const uint32_t a = 2 * (uint32_t)w, b = min(a + 1, W - 1);       // an odd last word: its upper half is never reached
      x.M = ((u64)masks[(size_t)id * W + b] << 32) | masks[(size_t)id * W + a];
      x.V = ((u64)rows[row_word((uint32_t)r, b, n_steps)] << 32) | rows[row_word((uint32_t)r, a, n_steps)];
    }
    return x;
  };
  int w = (int)(j - 1) >> 6, p = (int)(j - 1) & 63, q = 0;
  Word here = load(w), left = load(w - 1);
  int32_t mine = -1;
  while (w >= 0 && q < n_rows) {
    const int sh = p - (lane - q);
    const bool hit = lane >= q && sh >= 0 && ((here.M >> (sh & 63)) & 1ull);
    const u64 diag = __builtin_amdgcn_ballot_w64(hit) >> q;
    const int run = ~diag ? __builtin_ctzll(~diag) : 64;     // the shift brings in zeros: at most 64 - q
    if (lane >= q && lane < q + run) mine = w * 64 + sh;
    q += run;
    p -= run;
    if (q < n_rows && p >= 0) {
      const u64 x = here.M | ~here.V;
      const u64 xq = ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), q) << 32) |
                     (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, q);
      const u64 cand = xq & (~0ull >> (63 - p));
      if (cand) {
        p = 63 - __builtin_clzll(cand);
        const u64 mq = ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(here.M >> 32), q) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)here.M, q);
        if (!((mq >> p) & 1ull)) ++q;                        // not equal there: up
      } else {
        p = -1;
      }
    }
    if (p < 0) {                                             // on to the word to the left
      p = 63;
      --w;
      here = left;
      left = load(w - 1);
    }
  }
  if (mine_is_row) ref_to_cur[r] = mine;
  return w < 0 ? 0 : (uint32_t)(64 * w + p + 1);
}

constexpr uint32_t kChainBlocks = 16;                  // tables in LDS at a time
constexpr uint32_t kChainThreads = 256;

// entry[k]: columns left when the walk enters block k, or -1 if the block has been walked here
template <class Id>
__global__ __launch_bounds__(kChainThreads) void ss_align_chain_kernel(const Id *__restrict__ ref_id, uint32_t n,
                                                                       const uint32_t *__restrict__ masks, uint32_t m,
                                                                       uint32_t W, uint32_t n_steps,
                                                                       const uint32_t *__restrict__ rows,
                                                                       const uint16_t *__restrict__ table,
                                                                       int32_t *__restrict__ entry,
                                                                       int32_t *__restrict__ ref_to_cur) {
  __shared__ uint4 tabs[kChainBlocks * kWindow / 8];
  __shared__ uint32_t start[kChainBlocks];
  constexpr uint32_t kPer = kChainBlocks * kWindow / 8 / kChainThreads;
  const uint32_t K = (n + kWalkRows - 1) / kWalkRows;
  const uint4 *src = reinterpret_cast<const uint4 *>(table);
  const size_t total = (size_t)K * kWindow / 8;
  uint4 next[kPer];
  auto fetch = [&](uint32_t k0) {
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      const size_t at = (size_t)k0 * kWindow / 8 + i * kChainThreads + threadIdx.x;
      next[i] = at < total ? src[at] : uint4{0, 0, 0, 0};
    }
  };
  fetch(0);
  uint32_t j = m;                                            // wavefront 0's own
  for (uint32_t k0 = 0; k0 < K; k0 += kChainBlocks) {
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) tabs[i * kChainThreads + threadIdx.x] = next[i];
    if (threadIdx.x < kChainBlocks && k0 + threadIdx.x < K) start[threadIdx.x] = window_start(k0 + threadIdx.x, n, m);
    __syncthreads();
    fetch(k0 + kChainBlocks);
    if (threadIdx.x < 64) {
      const uint16_t *t = reinterpret_cast<const uint16_t *>(tabs);
      const uint32_t k1 = min(K, k0 + kChainBlocks);
      for (uint32_t k = k0; k < k1; ++k) {
        const uint32_t at = j - start[k - k0];               // before the window: wraps to a large number
        uint32_t d = at < kWindow ? t[(k - k0) * kWindow + at] : kNoEntry;
        d = __builtin_amdgcn_readfirstlane(d);
        if (d != kNoEntry) {
          if (threadIdx.x == 0) entry[k] = (int32_t)j;
          j -= d;
        } else {
          if (threadIdx.x == 0) entry[k] = -1;
          j = __builtin_amdgcn_readfirstlane(
              walk_in_place(ref_id, masks, rows, W, n_steps, RowBlock(k, n), j, ref_to_cur));
        }
      }
    }
    __syncthreads();
  }
}

template <class Id>
__global__ __launch_bounds__(64) void ss_align_pairs_kernel(const Id *__restrict__ ref_id, uint32_t n,
                                                            const uint32_t *__restrict__ masks, uint32_t W,
                                                            uint32_t n_steps, const uint32_t *__restrict__ rows,
                                                            const int32_t *__restrict__ entry,
                                                            int32_t *__restrict__ ref_to_cur) {
  __shared__ uint32_t M[kWalkRows][kTileStride], X[kWalkRows][kTileStride];
  __shared__ int32_t paired[kWalkRows];
  const uint32_t k = blockIdx.x;
  const int j = entry[k];
  if (j < 0) return;
  const RowBlock blk(k, n);
  const int w0 = j / (int)kEntries * (int)(kEntries / 32) - (int)(kMargin / 32);     // the tile the table came from
  paired[threadIdx.x] = -1;
  load_tile(ref_id, masks, rows, W, n_steps, blk, w0, M, X);
  __syncthreads();
  if (threadIdx.x == 0) walk_tile(blk.hi - blk.lo, w0, j, M, X, [&](uint32_t q, int c) { paired[q] = c; });
  __syncthreads();
  if (threadIdx.x < blk.hi - blk.lo) ref_to_cur[blk.hi - 1 - threadIdx.x] = paired[threadIdx.x];
}

struct KeyHash {
  size_t operator()(const std::pair<uint64_t, uint32_t> &k) const {
    uint64_t x = k.first * 0x9E3779B97F4A7C15ull ^ ((uint64_t)k.second * 0xC2B2AE3D27D4EB4Full);
    x ^= x >> 29;
    return (size_t)x;
  }
};

// LDS of the rows kernel with 16-bit ids: mask rows and all ids of the reference
size_t lds_need(uint32_t n_keys, uint32_t n) {
  return (size_t)(n_keys + 1) * kStripWords * 4 + (size_t)id_length(steps_of(n)) * 2;
}

// ref_to_cur (host, all -1 on entry) from the ids of both sequences
template <class Id>
int align_ids(ss_ctx *ctx, const std::vector<uint32_t> &ref_id, const std::vector<uint32_t> &cur_id, uint32_t n_keys,
              int32_t *ref_to_cur, uint32_t *lcs) {
  const uint32_t n = (uint32_t)ref_id.size(), m = (uint32_t)cur_id.size();
  constexpr bool kLds = sizeof(Id) == 2;
  const uint32_t W = (m + 31) / 32;                      // 32-bit words of a row
  const uint32_t strips = (W + kStripWords - 1) / kStripWords;
  const uint32_t n_steps = steps_of(n), n_blocks = n_steps / kBlock;
  const size_t row_bytes = (size_t)strips * n_steps * kStripWords * 4;
  const size_t id_len = id_length(n_steps);
  // short: the kernel writes the rows to pinned host memory and the host walks them; else they stay in device memory
  // and are walked there
  const bool short_rows = row_bytes <= kHostRowBytes;
  const bool ids_mapped = kLds && short_rows;            // each id is read once: straight from host memory
  const bool masks_needed = !kLds || !short_rows;
  size_t off = 0, hoff = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += ss_align_up(bytes, 256); return o; };
  auto htake = [&](size_t bytes) { size_t o = hoff; hoff += ss_align_up(bytes, 256); return o; };
  const size_t ho_ref = htake(id_len * sizeof(Id)), ho_cur = htake((size_t)m * sizeof(Id)), ids_end = hoff;
  const size_t ho_flag = htake(4), ho_out = htake(short_rows ? row_bytes : (size_t)n * 4);
  const size_t o_ids = take(ids_mapped ? 0 : ids_end);
  const size_t o_mask = take(masks_needed ? (size_t)(n_keys + 1) * W * 4 : 0);   // mask table, then the carry words:
  const size_t o_carry = take((size_t)(strips - 1) * (n_blocks + kCarryPad) * 8), o_end = off; // cleared in one go
  const size_t o_rows = take(short_rows ? 0 : row_bytes), o_pair = take(short_rows ? 0 : (size_t)n * 4);
  const uint32_t walk_blocks = (n + kWalkRows - 1) / kWalkRows;
  const size_t o_table = take(short_rows ? 0 : (size_t)walk_blocks * kWindow * 2);
  const size_t o_entry = take(short_rows ? 0 : (size_t)walk_blocks * 4);
  const int rc = ss_scratch_reserve(ctx, off, hoff);
  if (rc != SS_OK) return rc;
  uint8_t *d = (uint8_t *)ctx->d_scratch, *h = (uint8_t *)ctx->h_scratch, *hd = nullptr;
  SS_HIP(hipHostGetDevicePointer((void **)&hd, h, 0));
  hipStream_t s = ctx->s_aux;
  Id *h_ref = (Id *)(h + ho_ref), *h_cur = (Id *)(h + ho_cur);
  for (uint32_t i = 0; i < kIdPad; ++i) set_key(h_ref + i, n_keys);
  for (uint32_t i = 0; i < n; ++i) set_key(h_ref + kIdPad + i, ref_id[i]);
  for (size_t i = kIdPad + n; i < id_len; ++i) set_key(h_ref + i, n_keys);
  for (uint32_t j = 0; j < m; ++j) set_key(h_cur + j, cur_id[j]);
  volatile uint32_t *h_flag = (volatile uint32_t *)(h + ho_flag);
  *h_flag = 0;
  uint8_t *const ids_at = ids_mapped ? hd : d + o_ids;
  const Id *dref = (const Id *)(ids_at + ho_ref), *dcur = (const Id *)(ids_at + ho_cur);
  if (!ids_mapped) SS_HIP(hipMemcpyAsync(ids_at, h, ids_end, hipMemcpyHostToDevice, s));
  uint32_t *masks = (uint32_t *)(d + o_mask), *rows = (uint32_t *)(short_rows ? hd + ho_out : d + o_rows);
  if (o_end > o_mask) ss_launch_fill(s, d + o_mask, o_end - o_mask, 0);
  if (masks_needed)
    hipLaunchKernelGGL(ss_align_masks_kernel<Id>, dim3((m + 255) / 256), dim3(256), 0, s, dcur, m, masks, W);
  const RowsArgs args = {masks, (u64 *)(d + o_carry), rows, (uint32_t *)(hd + ho_flag), W, n_steps};
  hipLaunchKernelGGL(ss_align_rows_kernel<Id>, dim3(strips), dim3(64), kLds ? lds_need(n_keys, n) : 0, s, dref, dcur, m, args,
                     n_keys + 1);
  SS_HIP(hipGetLastError());
  uint32_t pairs = 0;
  if (!short_rows) {
    int32_t *dpair = (int32_t *)(d + o_pair);
    uint16_t *table = (uint16_t *)(d + o_table);
    int32_t *entry = (int32_t *)(d + o_entry);
    const uint32_t *cmasks = masks, *crows = rows;
    hipLaunchKernelGGL(ss_align_tab_kernel<Id>, dim3(walk_blocks, kWindow / kEntries), dim3(kEntries), 0, s, dref, n, cmasks,
                       m, W, n_steps, crows, table);
    hipLaunchKernelGGL(ss_align_chain_kernel<Id>, dim3(1), dim3(kChainThreads), 0, s, dref, n, cmasks, m, W, n_steps, crows,
                       (const uint16_t *)table, entry, dpair);
    hipLaunchKernelGGL(ss_align_pairs_kernel<Id>, dim3(walk_blocks), dim3(64), 0, s, dref, n, cmasks, W, n_steps, crows,
                       (const int32_t *)entry, dpair);
    SS_HIP(hipGetLastError());
    SS_HIP(hipMemcpyAsync(h + ho_out, dpair, (size_t)n * 4, hipMemcpyDeviceToHost, s));
    SS_HIP(hipStreamSynchronize(s));
    if (*h_flag) return SS_E_TIMEOUT;
    std::memcpy(ref_to_cur, h + ho_out, (size_t)n * 4);
    for (uint32_t i = 0; i < n; ++i) pairs += ref_to_cur[i] >= 0;
    *lcs = pairs;
    return SS_OK;
  }
  SS_HIP(hipStreamSynchronize(s));
  if (*h_flag) return SS_E_TIMEOUT;

  // walk back from (n, m)
  const uint32_t *hr = (const uint32_t *)(h + ho_out);
  uint32_t i = n, j = m;
  while (i > 0 && j > 0) {
    if (ref_id[i - 1] == cur_id[j - 1]) {
      ref_to_cur[i - 1] = (int32_t)(j - 1);
      ++pairs;
      --i;
      --j;
    } else if ((hr[row_word(i - 1, (j - 1) >> 5, n_steps)] >> ((j - 1) & 31)) & 1u) {
      --j;
    } else {
      --i;
    }
  }
  *lcs = pairs;
  return SS_OK;
}

}  // namespace

// ref_to_cur: n entries (host), filled; *lcs out.  Shared by ss_align_sequence and the SS_MATCH_ALIGN
// branch of ss_match_sequence.
int ss_align_core(ss_ctx *ctx, const ss_op_t *ref, uint32_t n, const ss_op_t *cur, uint32_t m,
                  int32_t *ref_to_cur, uint32_t *lcs, uint32_t *n_keys_out) {
  if (n > kAlignLenLimit || m > kAlignLenLimit) return SS_E_CAPACITY;
  for (uint32_t i = 0; i < n; ++i) ref_to_cur[i] = -1;
  *lcs = 0;
  if (n_keys_out) *n_keys_out = 0;
  if (n == 0 || m == 0) return SS_OK;

  // dense key ids: the keys of cur in first-seen order; reference operators whose key cur does not
  // hold share the id n_keys, whose mask row stays zero
  std::unordered_map<std::pair<uint64_t, uint32_t>, uint32_t, KeyHash> ids;
  ids.reserve(256);
  std::vector<uint32_t> cur_id(m), ref_id(n);
  for (uint32_t j = 0; j < m; ++j) {
    const std::pair<uint64_t, uint32_t> key{((uint64_t)cur[j].op_token << 32) | cur[j].stack_hash, cur[j].sig};
    auto it = ids.find(key);
    if (it == ids.end()) it = ids.emplace(key, (uint32_t)ids.size()).first;
    cur_id[j] = it->second;
  }
  const uint32_t n_keys = (uint32_t)ids.size();
  for (uint32_t i = 0; i < n; ++i) {
    const std::pair<uint64_t, uint32_t> key{((uint64_t)ref[i].op_token << 32) | ref[i].stack_hash, ref[i].sig};
    auto it = ids.find(key);
    ref_id[i] = it == ids.end() ? n_keys : it->second;
  }
  if (n_keys_out) *n_keys_out = n_keys;
  const uint64_t W64 = (m + 63) / 64;
  if (n * W64 * 8 > kAlignRowBytesLimit || (n_keys + 1) * W64 * 8 > kAlignRowBytesLimit) return SS_E_CAPACITY;
  return n_keys + 1 <= kLdsKeys && lds_need(n_keys, n) <= kLdsBytes
             ? align_ids<uint16_t>(ctx, ref_id, cur_id, n_keys, ref_to_cur, lcs)
             : align_ids<uint32_t>(ctx, ref_id, cur_id, n_keys, ref_to_cur, lcs);
}

void ss_align_anchors(const ss_op_t *ref, uint32_t n, const ss_op_t *cur, const int32_t *ref_to_cur,
                      const ss_anchor_t *anchors, uint32_t k, int32_t *new_idx, uint8_t *level,
                      uint32_t *n_unmatched) {
  (void)ref;
  uint32_t unm = 0;
  for (uint32_t a = 0; a < k; ++a) {
    const uint32_t i = anchors[a].ref_op;
    int32_t j = -1;
    if (i < n && ref_to_cur[i] >= 0 && anchors[a].out_slot < cur[ref_to_cur[i]].n_out) j = ref_to_cur[i];
    new_idx[a] = j;
    level[a] = j >= 0 ? (uint8_t)SS_LEVEL_ALIGN : (uint8_t)255;
    unm += j < 0;
  }
  *n_unmatched = unm;
}

extern "C" int ss_align_sequence(ss_ctx *ctx, const ss_op_t *ref, uint32_t n_ref, const ss_op_t *cur,
                                 uint32_t n_cur, const ss_anchor_t *anchors, uint32_t n_anchors,
                                 int32_t *ref_to_cur, int32_t *new_idx, uint8_t *level, ss_align_result_t *res) {
  return ss_guard([&]() -> int {
    if (!ctx || !res || (n_ref && !ref) || (n_cur && !cur)) return SS_E_INVAL;
    if (n_anchors && (!anchors || !new_idx || !level)) return SS_E_INVAL;
    std::vector<int32_t> local;
    if (!ref_to_cur) {
      local.resize(n_ref);
      ref_to_cur = local.data();
    }
    std::memset(res, 0, sizeof(*res));
    uint32_t lcs = 0, n_keys = 0;
    int rc = ss_align_core(ctx, ref, n_ref, cur, n_cur, ref_to_cur, &lcs, &n_keys);
    if (rc != SS_OK) return rc;
    res->lcs = lcs;
    res->distance = n_ref + n_cur - 2 * lcs;
    res->n_keys = n_keys;
    ss_align_anchors(ref, n_ref, cur, ref_to_cur, anchors, n_anchors, new_idx, level, &res->n_unmatched);
    for (uint32_t a = 0; a < n_anchors; ++a) ctx->stats.match_levels[level[a] <= SS_LEVEL_ALIGN ? level[a] : 4]++;
    return SS_OK;
  });
}
