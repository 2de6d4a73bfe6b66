// Sequence aligner: longest common subsequence of the reference and the current operator sequence
// and the canonical alignment read off it; the matcher's fourth level (Sec. 5.1 asks for tolerance
// to minor sequence variations with integer-only comparison and gives no algorithm).
//
// The dynamic programme runs in its bit-vector form: bit j of V_i is 0 exactly when
// L[i][j+1] = L[i][j] + 1, V_0 is all ones, and one reference operator advances the row by
//     V' = (V + (V & M)) | (V & ~M),     M = positions of cur holding that operator's key.
// The addition's carry runs through the whole row, so a row is not updated at once: lane l holds word l
// and works on row t - 2 l in step t, taking the carry that lane l - 1 produced for the same row two steps
// earlier (all carries of a wavefront are one 64-bit lane mask, so handing them on is one scalar shift;
// with one step in between, the way through the scalar unit and back was the longest chain).
// A wavefront covers a strip of 2,048 columns; a longer cur takes one workgroup per strip of 1,984, each
// reading the carries out of the strip before it.  The rows stay where they were written, four steps of a
// lane together, and the alignment is read back from (n, m): equal operators pair, otherwise left if bit
// j-1 of V_i is set (L[i][j-1] = L[i][j]), else up; on the host for short sequences, on the GPU for long
// ones.
#include <algorithm>
#include <cstring>

#include "ss_internal.h"

namespace {

typedef unsigned long long u64;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kAlignLenLimit = SS_ALIGN_LEN_LIMIT;       // at most 34 strips
constexpr uint32_t kBlock = 32;                        // steps between two looks at the neighbouring strip
constexpr uint32_t kStripWords = 64;                   // 32-bit words of a row, one per lane, in a single strip
constexpr uint32_t kInnerWords = 62;                   // the same where there are several strips: lanes 1 to 62
constexpr uint32_t kLdsKeys = 256;                     // mask rows (with the empty one) a strip keeps in LDS at most, 256 bytes each
constexpr uint32_t kFeeds = 4;                         // blocks of steps whose masks lie in LDS, and carries
constexpr uint32_t kFeedWords = kBlock * kStripWords;
constexpr uint32_t kRowsThreads = 320;
constexpr uint32_t kSkew = 2;                          // steps that a lane is behind the one before it
constexpr uint32_t kIdPad = 64 * kSkew;                // entries before the first id (lanes whose row has not begun)
// Rows up to this many bytes go straight to host memory and are walked there: beside the kernel's pace they cost the
// link nothing up to about 13 GB/s, and the walk on the GPU takes four more launches.  us a call, walked on the host and on the
// GPU: 2,694 x 2,704 operators (1.4 MiB) 93 and 101, 3,100 x 3,100 (1.6) 109 and 108, 3,300 x 3,300 (1.7) 124 and 111, 3,882 x 3,880
// 143 and 123, 5,192 x 5,196 195 and 140, 16,000 x 1,000 332 and 280; paths beside the diagonal: kAllTables.  Where cur is more than
// twice as long, a block's path leaves the tile of columns that is looked at for it: 2,200 x 6,000 (2.3), all of ref at the front of
// cur, 124 and 186, spread over cur 112 and 113; 1,800 x 9,000 126 and 228, 500 x 30,000 192 and 384.
constexpr size_t kHostRowBytes = 1700u << 10, kHostRowBytesSteep = 4u << 20;
constexpr uint32_t kCarryPad = 8;                      // carry words beyond a strip's last (the first of them is looked at)

// steps a strip takes for n rows, whole blocks of them: the last lane with a word is that far behind the first
static constexpr uint32_t steps_of(uint32_t n, uint32_t lanes = kStripWords) {
  return (n + kSkew * (lanes - 1) + kBlock - 1) / kBlock * kBlock;
}

// entries of a padded id array, a multiple of 16 bytes
static inline __host__ __device__ uint32_t id_length(uint32_t n_steps) { return kIdPad + n_steps + 6 * kBlock; }

static constexpr __host__ __device__ uint32_t strips_of(uint32_t W) {
  return W <= kStripWords ? 1 : (W + kInnerWords - 1) / kInnerWords;
}

// Word w (of W) of row r: lane l of its strip wrote it in step r + 2 l, four steps of a lane to a 16-byte store.
static inline __host__ __device__ size_t row_word(uint32_t r, uint32_t w, uint32_t W, uint32_t steps) {
  const bool one = W <= kStripWords;
  const uint32_t strip = one ? 0 : w / kInnerWords, l = one ? w : w % kInnerWords + 1, t = r + kSkew * l;
  return (size_t)strip * steps * kStripWords + ((size_t)(t / 4) * kStripWords + l) * 4 + t % 4;
}

// A key id as it is stored: 16 bits, already multiplied by the 256 bytes of an LDS mask row, where the mask rows fit
// LDS; else 32 bits as it is.
static __device__ __forceinline__ uint32_t key_of(uint16_t id) { return id >> 8; }
static __device__ __forceinline__ uint32_t key_of(uint32_t id) { return id; }

// ---- key ids ---------------------------------------------------------------------------------------------------
//
// The distinct (op_token, stack_hash, sig) of cur get dense ids through an open-addressing table whose slots hold
// 1 + the operator that stands for a key; which key gets which id does not matter.  Operators of ref whose key cur does
// not hold share the id n_keys, whose mask row is empty.  Ids are written in the form the rows kernel reads (key_of):
// 16 bits if there are few enough keys, 32 bits otherwise.  2,310 operators: one workgroup, 6.4 us; 64,609: three
// launches, 36 us, of which 24 bring the operators over the link and clear what the rows need clear; the third one makes the masks
// as well.  An unordered map on the host took about 23 and 260 us.

struct KeyArgs {
  const ss_op_t *ref, *cur;
  uint32_t n, m, n_steps;
  uint32_t few;                // up to this many keys the ids take 16 bits
  void *ref_id, *cur_id;       // id_length(n_steps) entries, padded; m entries
  uint32_t *n_keys;            // device: distinct keys so far
  uint32_t *n_keys_out;        // pinned: how many there are
  ss_done done;                // long sequences: the host waits for them
  // long sequences
  uint32_t *rep, *id;          // per slot
  uint32_t *slot;              // per operator of cur
  uint32_t mask, shift;
  uint32_t *masks, W;          // if given, cleared: mask rows of W words, made with the ids where there are few keys
  ss_cosine_part *part;        // pinned, if wanted: of each workgroup that reads the operators
};

__device__ __forceinline__ void put_id(void *ids, size_t at, uint32_t key, bool few) {
  if (few) static_cast<uint16_t *>(ids)[at] = (uint16_t)(key << 8);
  else static_cast<uint32_t *>(ids)[at] = key;
}

// Both sequences in one workgroup, keys and table in LDS, ops read from pinned host memory.
constexpr uint32_t kWgOps = 4096, kWgSlots = 8192, kWgThreads = 1024, kWgPer = kWgOps / kWgThreads;

constexpr size_t kWgLds = (2 * kWgSlots + 3 * kWgOps) * 4;

// mine[u]: the id of operator u * kWgThreads + tid of cur.  Returns how many keys there are.  (Whether the sums are wanted is asked
// by the host: code of theirs in a kernel that leaves it out cost 1,154 x 1,156 operators 0.6 us of 43.3.)
template <bool kSums>
__device__ __forceinline__ uint32_t keys_of_wg(const KeyArgs &a, uint32_t *lds, uint32_t (&mine)[kWgPer]) {
  uint32_t *const rep = lds, *const id = rep + kWgSlots, *const tok = id + kWgSlots, *const stk = tok + kWgOps, *const sig = stk + kWgOps;
  __shared__ uint32_t n_keys;
  constexpr uint32_t kShift = 64 - 13;
  static_assert(kWgSlots == 1u << 13, "hash bits");
  const uint32_t tid = threadIdx.x, total = a.m + a.n;       // cur first
  ss_op_t o[kWgPer];
#pragma unroll
  for (uint32_t u = 0; u < kWgPer; ++u) {
    const uint32_t i = u * kWgThreads + tid;
    if (i < total) o[u] = i < a.m ? a.cur[i] : a.ref[i - a.m];
  }
  for (uint32_t i = tid; i < kWgSlots; i += kWgThreads) rep[i] = 0;
  if (tid == 0) n_keys = 0;
  uint32_t slot[kWgPer];
#pragma unroll
  for (uint32_t u = 0; u < kWgPer; ++u) {
    const uint32_t i = u * kWgThreads + tid;
    if (i < total) { tok[i] = o[u].op_token; stk[i] = o[u].stack_hash; sig[i] = o[u].sig; }
  }
  __syncthreads();
  if constexpr (kSums) {
    uint64_t dot = 0, na = 0, nb = 0;
    uint32_t bad = 0;
    for (uint32_t i = tid; i < max(a.n, a.m); i += kWgThreads) {               // the shorter sequence is padded with token 0
      const uint32_t x = i < a.m ? tok[i] : 0, y = i < a.n ? tok[a.m + i] : 0;
      bad |= x >= SS_TOKEN_LIMIT || y >= SS_TOKEN_LIMIT;
      dot += (uint64_t)x * y; na += (uint64_t)x * x; nb += (uint64_t)y * y;
    }
    ss_put_part<kWgThreads>(a.part, dot, na, nb, bad);
  }
  // at most m <= kWgSlots / 2 keys: a free or matching slot is met
  auto find = [&](uint32_t u, bool insert) -> uint32_t {
    const uint32_t i = u * kWgThreads + tid;
    uint32_t h = ss_key_hash(o[u].op_token, o[u].stack_hash, o[u].sig, kShift);
    for (uint32_t probe = 0; probe < kWgSlots; ++probe) {
      uint32_t seen = *(volatile uint32_t *)(rep + h);
      if (!seen) {
        if (!insert) return kWgSlots;
        seen = atomicCAS(rep + h, 0u, i + 1);
        if (!seen) {
          id[h] = atomicAdd(&n_keys, 1u);
          return h;
        }
      }
      const uint32_t r = seen - 1;
      if (tok[r] == o[u].op_token && stk[r] == o[u].stack_hash && sig[r] == o[u].sig) return h;
      h = (h + 1) % kWgSlots;
    }
    return kWgSlots;
  };
#pragma unroll
  for (uint32_t u = 0; u < kWgPer; ++u)
    if (u * kWgThreads + tid < a.m) slot[u] = find(u, true);
  __syncthreads();
  const uint32_t keys = n_keys;
  const bool few = keys <= a.few;
  if (tid == 0) { *a.n_keys = keys; *a.n_keys_out = keys; }
#pragma unroll
  for (uint32_t u = 0; u < kWgPer; ++u) {
    const uint32_t i = u * kWgThreads + tid;
    mine[u] = 0;
    if (i < a.m) {
      mine[u] = id[slot[u]];
      put_id(a.cur_id, i, mine[u], few);
    } else if (i < total) {
      const uint32_t h = find(u, false);
      put_id(a.ref_id, kIdPad + i - a.m, h < kWgSlots ? id[h] : keys, few);
    }
  }
  for (uint32_t i = tid; i < id_length(a.n_steps); i += kWgThreads)
    if (i < kIdPad || i >= kIdPad + a.n) put_id(a.ref_id, i, keys, few);
  return keys;
}

template <bool kSums>
__global__ __launch_bounds__(kWgThreads) void ss_align_keys_kernel(KeyArgs a) {
  extern __shared__ uint32_t lds[];
  uint32_t mine[kWgPer];
  keys_of_wg<kSums>(a, lds, mine);
}

constexpr uint32_t kFetchWgs = 256;

// Long sequences: ops copied from pinned host memory, the table cleared and what the rows need clear; keys of cur inserted; ids of
// both, and the masks (the clearing and the masks in launches of their own: 32,312 operators 663 us a call, so 654).
__global__ __launch_bounds__(256) void ss_align_fetch_kernel(const ss_op_t *__restrict__ ref, ss_op_t *__restrict__ dref,
                                                             uint32_t n, const ss_op_t *__restrict__ cur,
                                                             ss_op_t *__restrict__ dcur, uint32_t m, uint32_t *rep,
                                                             uint32_t slots, uint32_t *n_keys, uint4 *zeros, uint32_t n_zeros,
                                                             ss_cosine_part *part) {
  const uint32_t first = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
  if (part) {
    uint64_t dot = 0, na = 0, nb = 0;
    uint32_t bad = 0;
    for (uint32_t i = first; i < max(n, m); i += stride) {
      ss_op_t c = {0, 0, 0, 0}, r = {0, 0, 0, 0};              // the shorter sequence is padded with token 0
      if (i < m) c = cur[i];
      if (i < n) r = ref[i];
      if (i < m) dcur[i] = c;
      if (i < n) dref[i] = r;
      bad |= c.op_token >= SS_TOKEN_LIMIT || r.op_token >= SS_TOKEN_LIMIT;
      dot += (uint64_t)c.op_token * r.op_token; na += (uint64_t)c.op_token * c.op_token; nb += (uint64_t)r.op_token * r.op_token;
    }
    ss_put_part<256>(part, dot, na, nb, bad);
  } else {
    for (uint32_t i = first; i < n; i += stride) dref[i] = ref[i];
    for (uint32_t i = first; i < m; i += stride) dcur[i] = cur[i];
  }
  for (uint32_t i = first; i < slots; i += stride) rep[i] = 0;
  for (uint32_t i = first; i < n_zeros; i += stride) zeros[i] = uint4{0, 0, 0, 0};
  if (first == 0) *n_keys = 0;
}

__device__ __forceinline__ bool same_key(const ss_op_t &x, const ss_op_t &y) {
  return x.op_token == y.op_token && x.stack_hash == y.stack_hash && x.sig == y.sig;
}

// A workgroup's operators share few keys, and every one of them would go for the same few slots: the first of each key
// within the workgroup (found through a table in LDS) goes, the others take over its slot.
__global__ __launch_bounds__(256) void ss_align_insert_kernel(KeyArgs a) {
  constexpr uint32_t kSlots = 512, kShift = 64 - 9;
  __shared__ uint32_t first[kSlots], slot_of[kSlots];
  __shared__ ss_op_t ops[256];
  const uint32_t j = blockIdx.x * 256 + threadIdx.x;
  const bool live = j < a.m;
  ss_op_t o = {0, 0, 0, 0};
  if (live) o = a.cur[j];
  ops[threadIdx.x] = o;
  for (uint32_t i = threadIdx.x; i < kSlots; i += 256) first[i] = 0;
  __syncthreads();
  uint32_t l = ss_key_hash(o.op_token, o.stack_hash, o.sig, kShift);
  bool goes = false;
  for (uint32_t probe = 0; live && probe < kSlots; ++probe) {  // at most 256 keys in 512 slots
    uint32_t seen = *(volatile uint32_t *)(first + l);
    if (!seen) {
      seen = atomicCAS(first + l, 0u, threadIdx.x + 1);
      if (!seen) { goes = true; break; }
    }
    if (same_key(ops[seen - 1], o)) break;
    l = (l + 1) % kSlots;
  }
  if (goes) {
    uint32_t h = ss_key_hash(o.op_token, o.stack_hash, o.sig, a.shift);
    for (uint32_t probe = 0; probe <= a.mask; ++probe) {       // at most m keys in at least 2m slots
      uint32_t seen = __hip_atomic_load(a.rep + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (!seen) {
        seen = atomicCAS(a.rep + h, 0u, j + 1);
        if (!seen) {
          a.id[h] = atomicAdd(a.n_keys, 1u);
          break;
        }
      }
      if (same_key(a.cur[seen - 1], o)) break;
      h = (h + 1) & a.mask;
    }
    slot_of[l] = h;
  }
  __syncthreads();
  if (live) a.slot[j] = slot_of[l];
}

__device__ __forceinline__ void operator_ids(const KeyArgs &a) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x, keys = *a.n_keys;
  const bool few = keys <= a.few;
  if (i == 0) *a.n_keys_out = keys;
  if (i < a.m) {
    const uint32_t key = a.id[a.slot[i]];
    put_id(a.cur_id, i, key, few);
    if (few && a.masks) atomicOr(&a.masks[(size_t)key * a.W + (i >> 5)], 1u << (i & 31));
  }
  if (i >= id_length(a.n_steps)) return;
  uint32_t key = keys;
  if (i >= kIdPad && i < kIdPad + a.n) {
    const ss_op_t o = a.ref[i - kIdPad];
    uint32_t h = ss_key_hash(o.op_token, o.stack_hash, o.sig, a.shift);
    for (uint32_t probe = 0; probe <= a.mask; ++probe) {
      const uint32_t seen = a.rep[h];
      if (!seen) break;
      if (same_key(a.cur[seen - 1], o)) { key = a.id[h]; break; }
      h = (h + 1) & a.mask;
    }
  }
  put_id(a.ref_id, i, key, few);
}

__global__ __launch_bounds__(256) void ss_align_ids_kernel(KeyArgs a) {
  operator_ids(a);
  ss_tell_host(a.done);
}

template <class Id>
__global__ void ss_align_masks_kernel(const Id *__restrict__ cur_id, uint32_t m, uint32_t *__restrict__ masks,
                                      uint32_t W) {
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < m) atomicOr(&masks[(size_t)key_of(cur_id[j]) * W + (j >> 5)], 1u << (j & 31));
}

// Four row steps of a word: V' = (V + (V & M) + carry in) | (V & ~M); the carries in and out are lane masks, `even` and
// `odd` those out of the two steps before.
// Written out because the compiler turns a carry that leaves as a lane mask into a select and a compare, and for the order.
// (bitop3's number is its truth table, S0 = 0xF0, S1 = 0xCC, S2 = 0xAA: (S0 & ~S1) | S2.)
__device__ __forceinline__ void row_steps(uint32_t V, const u32x4 &M, u64 &even, u64 &odd, u32x4 &rows) {
  uint32_t a, v0, v1, v2, v3;
  asm("v_and_b32_e32 %[a], %[m0], %[v]\n\t"
      "s_lshl_b64 %[c0], %[c0], 1\n\t"
      "s_lshl_b64 %[c1], %[c1], 1\n\t"
      "v_addc_co_u32_e64 %[a], %[c0], %[v], %[a], %[c0]\n\t"
      "v_bitop3_b32 %[v0], %[v], %[m0], %[a] bitop3:0xba\n\t"
      "v_and_b32_e32 %[a], %[m1], %[v0]\n\t"
      "v_addc_co_u32_e64 %[a], %[c1], %[v0], %[a], %[c1]\n\t"
      "v_bitop3_b32 %[v1], %[v0], %[m1], %[a] bitop3:0xba\n\t"
      "v_and_b32_e32 %[a], %[m2], %[v1]\n\t"
      "s_lshl_b64 %[c0], %[c0], 1\n\t"
      "s_lshl_b64 %[c1], %[c1], 1\n\t"
      "v_addc_co_u32_e64 %[a], %[c0], %[v1], %[a], %[c0]\n\t"
      "v_bitop3_b32 %[v2], %[v1], %[m2], %[a] bitop3:0xba\n\t"
      "v_and_b32_e32 %[a], %[m3], %[v2]\n\t"
      "v_addc_co_u32_e64 %[a], %[c1], %[v2], %[a], %[c1]\n\t"
      "v_bitop3_b32 %[v3], %[v2], %[m3], %[a] bitop3:0xba"
      : [v0] "=&v"(v0), [v1] "=&v"(v1), [v2] "=&v"(v2), [v3] "=v"(v3), [a] "=&v"(a), [c0] "+s"(even), [c1] "+s"(odd)
      : [v] "v"(V), [m0] "v"(M.x), [m1] "v"(M.y), [m2] "v"(M.z), [m3] "v"(M.w)
      : "scc");
  rows = u32x4{v0, v1, v2, v3};
}

struct RowsArgs {
  const uint32_t *masks;     // wide ids only
  u64 *carry;
  uint32_t *rows;
  uint32_t *gave_up;         // device, cleared before the launch (several strips only): a strip has given up
  uint32_t *gave_up_host;    // pinned: the same
  uint32_t W, n_steps, strips, strip0;       // strips of a row; the one of workgroup 0
  uint32_t wait_looks;       // looks at a carry word before a strip gives up
  ss_done done;              // where the host walks the rows
};

static __device__ const uint32_t all_ones = ~0u;

// Mask words of a block of steps of this lane.  The ids are read from device memory as 16 bytes (a row's distance between
// lanes keeps them aligned to 4), long before they are used.
typedef uint32_t ids16 __attribute__((ext_vector_type(4), aligned(4)));

// Wide ids: masks from device memory; a lane that holds no word of the row has W = 0 and `word` = &all_ones.
template <class Id>
struct Masks {
  const __attribute__((address_space(1))) uint32_t *word;      // this lane's word of the mask row of key 0
  const uint32_t *ids;       // entry t is the id of this lane's row in step t
  uint32_t W;
  ids16 id[kBlock / 4];
  __device__ __forceinline__ void load(uint32_t b) {
#pragma unroll
    for (uint32_t u = 0; u < kBlock / 4; ++u) id[u] = *reinterpret_cast<const ids16 *>(ids + b * kBlock + 4 * u);
  }
  __device__ __forceinline__ uint32_t look_up(uint32_t step) const { return word[(size_t)id[step / 4][step % 4] * W]; }
};

// 16-bit ids: masks in LDS.
template <>
struct Masks<uint16_t> {
  const uint8_t *table;      // this lane's word of the LDS mask row of key 0
  const uint16_t *ids;
  ids16 id[kBlock / 8];
  __device__ __forceinline__ void load(uint32_t b) {
#pragma unroll
    for (uint32_t u = 0; u < kBlock / 8; ++u) id[u] = *reinterpret_cast<const ids16 *>(ids + b * kBlock + 8 * u);
  }
  __device__ __forceinline__ uint32_t look_up(uint32_t step) const {
    const uint32_t x = id[step / 8][step / 2 % 4];
    return *reinterpret_cast<const uint32_t *>(table + (step & 1 ? x >> 16 : x & 0xFFFFu));
  }
};

struct alignas(16) RowsShared {             // read and written 16 bytes at a time
  uint32_t feed[kFeeds][kFeedWords];     // masks of a block of steps, four steps of a lane together
  uint32_t in[kFeeds];                   // what lane 0 hands on during a block
  uint32_t out[kFeeds][kStripWords];     // V after a block; lane 63's is what the strip hands on
};

// The wavefronts of a strip meet after every block of steps.  Those that write LDS have done so by then; what the first one
// reads is not written again before it has used it (kFeeds), and it waits for none of its reads here.  In several strips it
// also leaves its words, one store a block; the store of the block before has been done by then: the eight reads for the next
// block were issued after it, and LDS operations of a wavefront end in order.  (They were issued a block of steps ago: the
// wait takes no time.)
__device__ __forceinline__ void meet() { asm volatile("s_barrier" ::: "memory"); }
static_assert(kBlock / 4 == 8, "reads of a block of steps");
__device__ __forceinline__ void meet_written_before() { asm volatile("s_waitcnt lgkmcnt(8)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void meet_written() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Masks for the first wavefront: two feeders take the blocks in turn.  Block c lies in LDS when the first one enters block
// c - 1 (it reads ahead by a block); its masks are looked up one block of steps before they are written there.
template <class Id>
__device__ __forceinline__ void feed_masks(RowsShared &sh, Masks<Id> masks, uint32_t feeder, uint32_t n_blocks) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t M[kBlock];
  auto look = [&]() {
#pragma unroll
    for (uint32_t u = 0; u < kBlock; ++u) M[u] = masks.look_up(u);
  };
  auto put = [&](uint32_t block) {
    u32x4 *const out = reinterpret_cast<u32x4 *>(sh.feed[block % kFeeds]) + lane;
#pragma unroll
    for (uint32_t u = 0; u < kBlock; u += 4) out[u / 4 * kStripWords] = u32x4{M[u], M[u + 1], M[u + 2], M[u + 3]};
  };
  masks.load(feeder);
  look();
  put(feeder);
  masks.load(feeder + 2);
  if (!feeder) {
    look();                            // block 2
    masks.load(4);
  }
  meet_written();
#pragma unroll 1
  for (uint32_t b = 0; b < n_blocks; ++b) {
    if ((b ^ feeder) & 1) {
      look();                          // block b + 3
      masks.load(b + 5);
    } else {
      put(b + 2);
    }
    meet_written();
  }
  meet_written();
}

// What strips tell each other.  carry[strip][block]: lane 63's word after step 32 * block + 31 of that strip, bit 32 = the
// word is there (the value and its arrival are one store, so no fence is needed); cleared before the launch.  Lane 0 hands
// row t on in step t, and lane 63 of the strip before received that carry in step t + 126: block b needs words b + 3 and
// b + 4.  A word takes about a us from one strip to the other, three blocks of steps, so several looks are on their way at a
// time, one begun in every block, each at the 64 words from the one needed on; the oldest that shows the word will do.  (One
// look at each word, begun four blocks before it is needed, finds it only if the strip before is that much further ahead:
// 32,312 x 32,297 operators 523 us against 515.)
// A strip waits only for the strip before it, which waits for no later one.  That one may not be running, though (compute
// units held by others), so a wait ends after a.wait_looks; whoever gives up says so and goes on with zeros, and so does
// every strip that waits or comes to wait, after one look: a word that never comes costs one limit, not one per block and
// strip.  The host then starts the strips one by one.
__device__ __forceinline__ void take_carries(RowsShared &sh, const RowsArgs &a, bool takes) {
  constexpr uint32_t kLooks = 4;
  const uint32_t lane = threadIdx.x & 63, strip = a.strip0 + blockIdx.x, n_blocks = a.n_steps / kBlock;
  const u64 *const words = a.carry + (size_t)(strip - (takes ? 1 : 0)) * (n_blocks + kCarryPad);
  auto look = [&](uint32_t from) {                             // lane l: word from + l
    return __hip_atomic_load(words + min(from + lane, n_blocks), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  // the word that `seen` shows in lane l; false: it was not there
  auto found = [&](u64 seen, uint32_t l, uint32_t &word) {
    word = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)seen, l);
    return __builtin_amdgcn_readlane((int)(uint32_t)(seen >> 32), l) != 0;
  };
  auto wait_for = [&](uint32_t block) -> uint32_t {
    uint32_t word;
#pragma unroll 1
    for (uint32_t looks = 0; looks <= a.wait_looks; ++looks) {
      const u64 y = look(block);
      const uint32_t over = __hip_atomic_load(a.gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (found(y, 0, word)) return word;
      if (__builtin_amdgcn_readfirstlane(over)) break;
    }
    if (lane == 0) {
      __hip_atomic_store(a.gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(a.gave_up_host, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return 0;
  };
  uint32_t prev = 0;
  u64 x[kLooks];
  auto give = [&](uint32_t block, uint32_t word) {             // the input of `block`, with word block + 4
    if (lane == 0) sh.in[block % kFeeds] = (prev << 30) | (word >> 2);
    prev = word;
  };
  if (takes) {
    prev = 3 < n_blocks ? wait_for(3) : 0;
    give(0, 4 < n_blocks ? wait_for(4) : 0);
    give(1, 5 < n_blocks ? wait_for(5) : 0);
#pragma unroll
    for (uint32_t u = 0; u < kLooks; ++u) x[u] = look(u + 2);
  } else if (lane < kFeeds) {
    sh.in[lane] = 0;
  }
  meet_written();
  // kLooks blocks a turn, so that what is on its way stays in its register
#pragma unroll 1
  for (uint32_t b = 0; b < n_blocks; b += kLooks) {
#pragma unroll
    for (uint32_t u = 0; u < kLooks; ++u) {
      if (b + u >= n_blocks) break;
      if (takes) {
        const uint32_t need = b + u + 6;                       // the looks were begun at need - 4, ... need - 1
        uint32_t word = 0;
        if (need < n_blocks && !found(x[u], 4, word) && !found(x[(u + 1) % kLooks], 3, word) &&
            !found(x[(u + 2) % kLooks], 2, word) && !found(x[(u + 3) % kLooks], 1, word))
          word = wait_for(need);
        give(need - 4, word);
        x[u] = look(need);
      }
      meet_written();
    }
  }
  meet_written();
}

// The first wavefront leaves its words in LDS (a store of its own, by one lane, took it 70 cycles a block) and doesn't wait
// for that: they are there a block later (meet_written_before).  Taking and giving are two wavefronts' work: behind its own stores the one that
// looks at the other strip's words waits for them too (32,312 x 32,297 operators 623 us against 500).
__device__ __forceinline__ void give_carries(const RowsShared &sh, const RowsArgs &a, bool gives) {
  const uint32_t lane = threadIdx.x & 63, strip = a.strip0 + blockIdx.x, n_blocks = a.n_steps / kBlock;
  u64 *const own = a.carry + (size_t)strip * (n_blocks + kCarryPad);
  auto hand_on = [&](uint32_t block) {
    const uint32_t word = sh.out[block % kFeeds][kStripWords - 1];
    if (lane == 0) __hip_atomic_store(own + block, (1ull << 32) | word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  meet_written();
#pragma unroll 1
  for (uint32_t b = 0; b < n_blocks; ++b) {
    if (gives && b >= 2) hand_on(b - 2);
    meet_written();
  }
  meet_written();
  if (gives)
    for (uint32_t b = max(n_blocks, 2u) - 2; b < n_blocks; ++b) hand_on(b);
}

// All rows of one strip.  Where there are several (kMany), lanes 0 and 63 hold no word: their M is all ones, which
// makes a step V' = 2 V + carry in with V's top bit as the carry out.  So lane 63 collects what lane 62 hands on, one bit
// a step, first step highest, and lane 0 hands on what it was given as a word, likewise: strips exchange carries without
// an instruction in any step (a history kept beside the row and bits put into the lane mask took 3.7 of 11.1 instructions).
template <bool kMany>
__device__ __forceinline__ void strip_rows(RowsShared &sh, const RowsArgs &a, bool stored) {
  const uint32_t lane = threadIdx.x & 63, strip = a.strip0 + blockIdx.x, n_blocks = a.n_steps / kBlock;
  uint32_t V = ~0u;
  u64 even = 0, odd = 0;
  u32x4 M[kBlock / 4];
  // A lane whose word nobody reads stores beyond the end of the buffer, which drops it: all lanes stay in step, and
  // no store needs a lane mask of its own.
  const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(
      a.rows + (size_t)strip * a.n_steps * kStripWords, 0, (int)(a.n_steps * kStripWords * 4), 0x00027000);
  uint32_t at = stored ? lane * 16 : 0x80000000u;
  meet();
  auto feed = [&](uint32_t block) { return reinterpret_cast<const u32x4 *>(sh.feed[block % kFeeds]) + lane; };
  uint32_t in = sh.in[0];              // read in the same order as in the loop, whose waits then count the reads that are later
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (uint32_t q = 0; q < kBlock / 4; ++q) {
    M[q] = feed(0)[q * kStripWords];
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll 1
  for (uint32_t b = 0; b < n_blocks; ++b) {
    const u32x4 *const ahead = feed(b + 1);
    if constexpr (kMany) {
      V = lane ? V : in;
      in = sh.in[(b + 1) % kFeeds];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (uint32_t q = 0; q < kBlock / 4; ++q) {
      u32x4 v;
      row_steps(V, M[q], even, odd, v);
      V = v.w;
      __builtin_amdgcn_raw_buffer_store_b128(v, out, at, q * kStripWords * 16, 0);
      M[q] = ahead[q * kStripWords];
      __builtin_amdgcn_sched_barrier(0);
    }
    at += kBlock * kStripWords * 4;
    if constexpr (kMany) {
      sh.out[b % kFeeds][lane] = V;
      meet_written_before();
    } else {
      meet();
    }
  }
  meet_written();
}

// A workgroup per strip (all of them, or one to a launch): the first wavefront does the rows, two look its masks up for it,
// and two take and give carries where there are several strips.  ref_id: n ids with kIdPad entries of the empty mask row before them
// and id_length() - kIdPad - n after them, so that a lane whose row has not begun or is over adds nothing.  16-bit ids: the
// strip builds its own mask table in LDS from cur_id; wider ids (more keys than fit): masks come from device memory.
//
// Bound by the issue of the first wavefront's instructions from one step to the next: three vector instructions in a chain
// and a shift of the carries, with a half of one for the masks' coming and the row's going (words of 32 bits, since a wider
// word puts a second addition into the chain).  A scalar instruction that comes soon after a vector instruction that wrote a
// lane mask waits for it, whichever mask it reads: so lanes are two steps apart and the shifts of two steps' carries stand
// together, as far from the additions as they can.  A loop of nothing but these steps, reads and stores takes 24.8 cycles a
// step, without the shifts 18.8; with a shift in every step 28.8, with the parts of V that the next row needs worked out
// beside V, one operation less in the chain and one more to issue, 28.3, with the carries in vector registers 34.8.
// One wavefront that also looked up its masks and exchanged carries took seven instructions a step and 15.5 ns (20.1 in
// several strips): 1,154 x 1,156 operators 27.0 us, now 23.0; 32,312 x 32,297 in 17 strips 650 us, now 500, of which some 80
// are the strips' start one after the other.  Updating a whole row at once in one wavefront, its carries crossing lanes by
// two ballots and scalar arithmetic, took 149 us and 24.5 ms.
template <class Id>
__global__ __launch_bounds__(kRowsThreads) void ss_align_rows_kernel(const Id *__restrict__ ref_id,
                                                                     const Id *__restrict__ cur_id, uint32_t m, RowsArgs a,
                                                                     const uint32_t *__restrict__ n_keys) {
  constexpr bool kLds = sizeof(Id) == 2;
  __shared__ RowsShared sh;
  extern __shared__ uint4 lds4[];                            // written 16 bytes at a time
  uint32_t *const lds = reinterpret_cast<uint32_t *>(lds4);
  const uint32_t tid = threadIdx.x, lane = tid & 63, role = __builtin_amdgcn_readfirstlane(tid >> 6), strip = a.strip0 + blockIdx.x;
  const bool many = a.strips > 1;
  const uint32_t first = many ? 1 : 0;                       // lane of the strip's first word
  const uint32_t w0 = strip * kInnerWords;
  const uint32_t words = min(many ? kInnerWords : kStripWords, a.W - w0);
  const bool stored = lane >= first && lane < first + words;
  const uint32_t n_mask_rows = *n_keys + 1, n_blocks = a.n_steps / kBlock;
  if (kLds && n_mask_rows > kLdsKeys) {                      // launched before the number was known, and the ids are wide
    ss_tell_host(a.done);
    return;
  }
  Masks<Id> masks;
  if constexpr (kLds) {
    for (uint32_t i = tid; i < n_mask_rows * (kStripWords / 4); i += kRowsThreads) {
      const uint32_t part = i % (kStripWords / 4);
      lds4[i] = uint4{many && part == 0 ? ~0u : 0, 0, 0, many && part == kStripWords / 4 - 1 ? ~0u : 0};
    }
    // ten words' columns at a time, all of them in flight
    constexpr uint32_t kPer = (kStripWords * 32 + kRowsThreads - 1) / kRowsThreads;
    uint32_t id[kPer];
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u) {
      const uint32_t w = u * (kRowsThreads / 32) + (tid >> 5), j = (w0 + w) * 32 + (tid & 31);
      id[u] = w < words && j < m ? cur_id[j] : 0xFFFFFFFFu;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < kPer; ++u)
      if (id[u] != 0xFFFFFFFFu)
        atomicOr(&lds[key_of((uint16_t)id[u]) * kStripWords + first + u * (kRowsThreads / 32) + (tid >> 5)], 1u << (tid & 31));
    __syncthreads();
    masks.table = reinterpret_cast<const uint8_t *>(lds + lane);
  } else {
    using Global = const __attribute__((address_space(1))) uint32_t *;
    masks.word = stored ? (Global)(a.masks + w0 + lane - first) : (Global)&all_ones;
    masks.W = stored ? a.W : 0;
  }
  masks.ids = ref_id + kIdPad - kSkew * lane;
  if (role == 0) {
    if (many) strip_rows<true>(sh, a, stored);
    else strip_rows<false>(sh, a, stored);
  } else if (role < 3) {
    feed_masks(sh, masks, role - 1, n_blocks);
  } else if (role == 3) {
    take_carries(sh, a, many && strip != 0);
  } else {
    give_carries(sh, a, many && strip + 1 < a.strips);
  }
  ss_tell_host(a.done);
}

// Ids and rows of short sequences in one launch, where one strip holds them: the workgroup that makes the ids goes on with
// the rows, in the same LDS, the masks made from the ids in its registers; the wavefronts that have no part in them end.  If
// there turn out to be too many keys nothing more is done.  1,154 x 1,156 operators: 27.1 us, by two launches 6.3 and 23.0 and
// about 2.5 between them.  (With LDS aligned to 4 bytes, 16-byte reads lose that again and more: 35.2.)
constexpr uint32_t kFewRows = kLdsKeys * kStripWords * 4;
constexpr size_t kShortLds = kWgLds > kFewRows + sizeof(RowsShared) ? kWgLds : kFewRows + sizeof(RowsShared);

template <bool kSums>
__global__ __launch_bounds__(kWgThreads) void ss_align_short_kernel(KeyArgs k, RowsArgs a) {
  extern __shared__ uint4 lds4[];                            // behind n_keys: 16-byte reads want it aligned
  uint32_t *const lds = reinterpret_cast<uint32_t *>(lds4);
  const uint32_t tid = threadIdx.x, lane = tid & 63, role = __builtin_amdgcn_readfirstlane(tid >> 6), n_blocks = a.n_steps / kBlock;
  uint32_t mine[kWgPer];
  const uint32_t keys = keys_of_wg<kSums>(k, lds, mine);
  if (keys > k.few) {                                        // the ids are wide
    ss_tell_host(a.done);
    return;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // the ids that other wavefronts read
  __syncthreads();
  for (uint32_t i = tid; i < (keys + 1) * (kStripWords / 4); i += kWgThreads) lds4[i] = uint4{0, 0, 0, 0};
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kWgPer; ++u) {
    const uint32_t j = u * kWgThreads + tid;
    if (j < k.m) atomicOr(&lds[mine[u] * kStripWords + (j >> 5)], 1u << (j & 31));
  }
  __syncthreads();
  if (role >= kRowsThreads / 64) return;
  RowsShared &sh = *reinterpret_cast<RowsShared *>(lds + kFewRows / 4);
  Masks<uint16_t> masks;
  masks.table = reinterpret_cast<const uint8_t *>(lds + lane);
  masks.ids = static_cast<const uint16_t *>(k.ref_id) + kIdPad - kSkew * lane;
  if (role == 0) strip_rows<false>(sh, a, lane < a.W);
  else if (role < 3) feed_masks(sh, masks, role - 1, n_blocks);
  else if (role == 3) take_carries(sh, a, false);
  else give_carries(sh, a, false);
  ss_tell_host(a.done);
}

// ---- the walk back on the GPU ----------------------------------------------------------------------------------
//
// The walk is one chain of n rows, but what 64 rows do to it is a function of one number: how many columns are left
// when it enters them.  So that function is tabulated for every block of 64 rows at once, one thread per entry
// column of a window around the diagonal (ss_align_tab_kernel), and eight blocks' tables are put together to one
// (ss_align_compose_kernel); one workgroup then follows these from the end (ss_align_chain_kernel), and with every
// group's entry known the blocks are walked again side by side to write the pairs (ss_align_pairs_kernel).  Where a group's
// table has no entry the chain follows its blocks' own, and a block whose entry lies outside its window, or whose path
// leaves the tile to the left, is walked in place by a wavefront of the chain.
// 32,312 rows: 28 us for the tables, 5 us for the groups' and 12 us for the chain (an LDS read and a few vector operations
// per group; 17 where each group's went through the scalar unit, 90 block by block), 15 us for the pairs; single steps in one
// wavefront took 97 ns a row (3.1 ms), the rows over the host link (130 MB) 2.3 ms and a walk there.
constexpr uint32_t kWalkRows = 64;
// Entry columns tabulated per block of rows (windows).  Where lengths differ by more than half of kWindow and that takes no more than
// kAllTables workgroups, all columns: no path leaves them.  Otherwise kWindow; or, where the lengths differ by at most kNearlyEqual, kNarrowWindow first, since a path of operators that
// come and go all along the sequences strays from the diagonal by some hundred columns (32,312 rows: tables 48 us, half as many 28).
// If it leaves them after all, the walk goes on from there with kWindow columns around the diagonal of what is left, which finds a
// path that has come to lie beside the first one.
// us a call, sequences of 9,000 with 700 foreign operators in a quarter of one and as many missing in the last of it: 244, by a second
// walk of all blocks 275, with kWindow alone and the kernels of that time 254; with 1,500 foreign ones 251, 392 and 351; without any
// 209, 207 and 243.
// All columns, kWindow or kNarrowWindow first: lengths that are nearly equal, the path near the diagonal, 3,300 operators 110 us and
// 107, 3,600 117 and 112, 4,000 126 and 120; 700 or 1,500 beside it 119 to 148 and 126 to 165 (the host 124 to 169, a second walk of all
// blocks 136 to 188), but sequences that are that far apart are the rarer.  Operators missing all along one of them, 4,000 and 3,400 of
// them 125 and 120, 6,000 and 5,100 171 and 157; 5,000 and 4,100 of them from one end on 145 and 136.  Lengths that differ by more are
// seldom those of a path near the diagonal: 8,000 operators and the first 3,000 of them 192 us, with kWindow 704, on the host 235;
// 5,000 and the first 3,500 149 and 158, with operators missing all along 142 and 139.
constexpr uint32_t kWindow = 2048, kNarrowWindow = 1024, kNearlyEqual = 512, kMostColumns = 8192;
constexpr uint32_t kAllTables = 2600;
constexpr uint32_t kEntries = 256;                     // of these, per workgroup
constexpr uint32_t kMargin = 256;                      // columns a tile reaches to the left of its first entry
constexpr uint32_t kTileWords = (kEntries + kMargin) / 32;
// A word of a tile: columns that are equal, and those where the walk stops (equal, or it steps up).  In front of a row's first is
// one without a stop.
struct TileWord { uint32_t stops, equal; };
typedef TileWord Tile[kWalkRows][kTileWords + 1];
constexpr uint16_t kNoEntry = 0xFFFF;

// rows of block k (counted from the end): [lo, hi)
struct RowBlock {
  uint32_t lo, hi;
  __device__ RowBlock(uint32_t k, uint32_t n) : lo(n > (k + 1) * kWalkRows ? n - (k + 1) * kWalkRows : 0), hi(n - k * kWalkRows) {}
};

// The windows' size, and where a block's starts (columns left): a multiple of kEntries, the scaled diagonal in the middle, or, of
// windows of all columns, 0.
struct Windows {
  uint64_t slope;                      // columns to a row, 32 bits of them behind the point
  uint32_t n, m, size;
  // of a walk that begins with `rows` rows and `columns` columns left
  Windows(uint32_t n_, uint32_t m_, uint32_t size_, uint32_t rows, uint32_t columns)
      : slope(size_ > m_ ? 0 : ((uint64_t)columns << 32) / rows), n(n_), m(m_), size(size_) {}
  __device__ __forceinline__ uint32_t start(uint32_t k) const {
    const uint32_t mid = (uint32_t)((n - k * kWalkRows) * slope >> 32);
    return (mid > size / 2 ? mid - size / 2 + kEntries / 2 : 0) / kEntries * kEntries;
  }
  // columns that block k takes off j, or kNoEntry
  __device__ __forceinline__ uint32_t taken(const uint16_t *table, uint32_t k, uint32_t j) const {
    const uint32_t at = j - start(k);                        // before the window: wraps to a large number
    return at < size ? table[(size_t)k * size + at] : kNoEntry;
  }
};

// 0 to 31, or all ones for 0
__device__ __forceinline__ uint32_t leading_zeros(uint32_t x) {
  uint32_t n;
  asm("v_ffbh_u32_e32 %0, %1" : "=v"(n) : "v"(x));
  return n;
}

// Rows [lo, hi) and kTileWords words from word w0 on (w0 may be negative: empty); stops = M | ~V.  A step of the row buffer holds
// consecutive words of consecutive rows, so threads run along it there, and along a mask row for the masks; each thread's loads are
// all on their way before the first is waited for.  n_keys, if given: false, and nothing read but ids, where there are too many for
// ids of this form (looked at while the ids are on their way; in front of them it takes 0.4 us).
constexpr uint32_t kTileThreads = 256;

template <class Id>
__device__ __forceinline__ bool load_tile(const Id *ref_id, const uint32_t *masks, const uint32_t *rows, uint32_t W,
                                          uint32_t n_steps, RowBlock blk, int w0, Tile &tile, const uint32_t *n_keys = nullptr) {
  constexpr uint32_t kMasks = kWalkRows * kTileWords / kTileThreads, kRows = (kWalkRows + kSkew * kTileWords) * kTileWords / kTileThreads;
  static_assert(kMasks * kTileThreads == kWalkRows * kTileWords && kRows * kTileThreads == (kWalkRows + kSkew * kTileWords) * kTileWords, "");
  const uint32_t n_rows = blk.hi - blk.lo, l = threadIdx.x % kTileWords;
  const int w = w0 + (int)l;
  const bool there = w >= 0 && (uint32_t)w < W;
  Id id[kMasks];
#pragma unroll
  for (uint32_t u = 0; u < kMasks; ++u) {                    // q: how far from the block's last row
    const uint32_t q = (u * kTileThreads + threadIdx.x) / kTileWords;
    id[u] = q < n_rows ? ref_id[kIdPad + blk.hi - 1 - q] : Id(0);
  }
  if (sizeof(Id) == 2 && n_keys && *n_keys >= kLdsKeys) return false;
  uint32_t V[kRows], M[kMasks];
#pragma unroll
  for (uint32_t u = 0; u < kRows; ++u) {                     // row lo + t - back
    const uint32_t t = (u * kTileThreads + threadIdx.x) / kTileWords, back = kSkew * l;
    V[u] = there && t >= back && t - back < n_rows ? rows[row_word(blk.lo + t - back, (uint32_t)w, W, n_steps)] : ~0u;
  }
#pragma unroll
  for (uint32_t u = 0; u < kMasks; ++u) M[u] = there ? masks[(size_t)key_of(id[u]) * W + w] : 0;
  if (threadIdx.x < kWalkRows) tile[threadIdx.x][0] = TileWord{0, 1};
#pragma unroll
  for (uint32_t u = 0; u < kMasks; ++u) tile[(u * kTileThreads + threadIdx.x) / kTileWords][l + 1].equal = M[u];
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kRows; ++u) {
    const uint32_t t = (u * kTileThreads + threadIdx.x) / kTileWords, back = kSkew * l;
    if (t < back || t - back >= n_rows) continue;
    TileWord &x = tile[n_rows - 1 - (t - back)][l + 1];
    x.stops = x.equal | ~V[u];
  }
  return true;
}

// Lane q: which words of the block's row q hold a stop (bit l + 1: word l).
__device__ __forceinline__ uint32_t words_that_stop(uint32_t n_rows, const Tile &tile) {
  const uint32_t q = threadIdx.x & 63;
  uint32_t some = 0;
  if (q < n_rows)
#pragma unroll
    for (uint32_t l = 0; l < kTileWords; ++l) some |= tile[q][l + 1].stops ? 2u << l : 0;
  return some;
}

// The walk through a block with j columns left on entry; returns the columns left after it, or -1 if it leaves the
// tile.  Per row: the highest column below j where it stops, in the word of column j - 1 or else in the highest one below with a
// stop (beside the path hundreds of columns in a row may hold none).  Both words are read at once and there is no branch: bound
// by the instructions of a row, some 25 for a wavefront's 64 entries; with a search from word to word and early ends 65.
// at: the column, counted from 32 before the tile's first; 31 (nothing left in the tile) leads to the empty word in front of the
// row, which leads back to 31.
struct TileStep { uint32_t stops, equal; };                  // whether there is a stop; whether the row's operator is equal there

__device__ __forceinline__ TileStep step_row(const Tile &tile, uint32_t q, uint32_t some, uint32_t &at) {
  const uint32_t word = at >> 5;
  const uint32_t other = ~(uint32_t)leading_zeros(__builtin_amdgcn_ubfe(some, 0, word)) & 31u;
  const TileWord here = tile[q][word], below = tile[q][other];
  const uint32_t upto = here.stops & (~0u >> (~at & 31u));
  const uint32_t stops = upto ? upto : below.stops, equal = upto ? here.equal : below.equal;
  const uint32_t lead = leading_zeros(stops), there = equal >> (~lead & 31u) & 1u;
  at = ((upto ? word : other) << 5) + (31 - lead) - there;
  return TileStep{stops, there};
}

__device__ __forceinline__ int walk_tile(uint32_t n_rows, int w0, int j, const Tile &tile) {
  const uint32_t rows_some = words_that_stop(n_rows, tile);
  uint32_t at = (uint32_t)(j - 1 - w0 * 32 + 32);
  for (uint32_t q = 0; q < n_rows; ++q) step_row(tile, q, (uint32_t)__builtin_amdgcn_readlane((int)rows_some, q), at);
  return at == 31 && w0 > 0 ? -1 : max(0, (int)at - 31 + w0 * 32);
}

template <class Id>
__global__ __launch_bounds__(kEntries) void ss_align_tab_kernel(const Id *__restrict__ ref_id, Windows win,
                                                                const uint32_t *__restrict__ masks,
                                                                uint32_t W, uint32_t n_steps,
                                                                const uint32_t *__restrict__ rows,
                                                                uint16_t *__restrict__ table, const uint32_t *__restrict__ n_keys, uint32_t k_first) {
  __shared__ Tile tile;
  const uint32_t k = k_first + blockIdx.x, e0 = win.start(k) + blockIdx.y * kEntries;
  if (e0 > win.m) return;
  const RowBlock blk(k, win.n);
  const int w0 = (int)(e0 / 32) - (int)(kMargin / 32);
  if (!load_tile(ref_id, masks, rows, W, n_steps, blk, w0, tile, n_keys)) return;        // launched before the number was known: no rows
  __syncthreads();
  const int j = (int)(e0 + threadIdx.x);
  const int out = walk_tile(blk.hi - blk.lo, w0, min(j, (int)win.m), tile);
  table[(size_t)k * win.size + blockIdx.y * kEntries + threadIdx.x] = out < 0 || j > (int)win.m ? kNoEntry : (uint16_t)(j - out);
}

// One wavefront walks a block in place and writes its pairs: lane q holds 64-bit words of row hi - 1 - q, id is the row's key.  A run
// of equal operators steps one row and one column at a time, so each lane tests the bit of its own row on the diagonal
// and the run's length is the number of leading ones; then one find-first in the row the run ended in.
// Bound by the latency of the words' loads: four words to the left are loaded at a time, by every lane, also beside the rows and
// the words, whose bits nobody looks at (one word ahead at a time, handed on from word to word, is copied behind its load, which is
// waited for: 15,000 operators and the first 5,000 of them, most of whose path lies outside the windows, 2,050 us a call, so up to
// 2,500).  Through columns without a stop it goes 4,096 at a time (word by word 16,000 operators with nothing in common 587 us
// a call, so 378).
__device__ uint32_t walk_in_place(uint32_t id, const uint32_t *masks, const uint32_t *rows, uint32_t W, uint32_t n_steps, RowBlock blk,
                                  uint32_t j, int32_t *ref_to_cur) {
  const int lane = threadIdx.x & 63, n_rows = (int)(blk.hi - blk.lo), r = max((int)blk.hi - 1 - lane, (int)blk.lo);
  const int row = lane < n_rows ? lane : -1;
  struct Word { u64 M, V; };
  // Every lane loads, also beside the rows and the words, whose bits nobody looks at: no value is put together behind a load, which
  // would be waited for.
  auto load = [&](int w) -> Word {
    const uint32_t a = 2 * (uint32_t)max(w, 0), b = min(a + 1, W - 1);     // an odd last word: its upper half is never reached
    return Word{((u64)masks[(size_t)id * W + b] << 32) | masks[(size_t)id * W + a],
                ((u64)rows[row_word((uint32_t)r, b, W, n_steps)] << 32) | rows[row_word((uint32_t)r, a, W, n_steps)]};
  };
  // the highest word below w with a stop in the block's row q, 64 words at a time; -1: there is none
  auto jump = [&](int w, int q) -> int {
    const uint32_t row = blk.hi - 1 - (uint32_t)q, mask_row = (uint32_t)__builtin_amdgcn_readlane((int)id, q);
    for (int at = w - 1; at >= 0; at -= 64) {
      u64 stops = 0;
      if (at >= lane) {
        const uint32_t a = 2 * (uint32_t)(at - lane);
        stops = ((u64)masks[(size_t)mask_row * W + a + 1] << 32) | masks[(size_t)mask_row * W + a];
        stops |= ~(((u64)rows[row_word(row, a + 1, W, n_steps)] << 32) | rows[row_word(row, a, W, n_steps)]);
      }
      const u64 there = __builtin_amdgcn_ballot_w64(stops != 0);
      if (there) return at - __builtin_ctzll(there);
    }
    return -1;
  };
  int w = (int)(j - 1) >> 6, p = (int)(j - 1) & 63, q = 0, empty = 0, empty_row = -1;
  int32_t mine = -1;
  while (w >= 0 && q < n_rows) {
    constexpr int kAhead = 4, kStepped = 2;                  // words loaded at a time; without a stop gone through one by one
    Word words[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) words[i] = load(w - i);
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const Word here = words[i];
      if (w < 0) break;
      while (p >= 0 && q < n_rows) {
        const int sh = p - (lane - q);
        const bool hit = row >= q && sh >= 0 && ((here.M >> (sh & 63)) & 1ull);
        const u64 diag = __builtin_amdgcn_ballot_w64(hit) >> q;
        const int run = ~diag ? __builtin_ctzll(~diag) : 64; // the shift brings in zeros: at most 64 - q
        if (lane >= q && lane < q + run) mine = w * 64 + sh;
        q += run;
        p -= run;
        if (q >= n_rows || p < 0) break;
        const u64 x = here.M | ~here.V;
        const u64 xq = ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), q) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, q);
        const u64 cand = xq & (~0ull >> (63 - p));
        if (!cand) {
          p = -1;
          empty = q == empty_row ? empty + 1 : 1;
          empty_row = q;
          break;
        }
        p = 63 - __builtin_clzll(cand);
        const u64 mq = ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(here.M >> 32), q) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)here.M, q);
        if (!((mq >> p) & 1ull)) ++q;                        // not equal there: up
      }
      if (p < 0) {                                           // on to the word to the left
        p = 63;
        --w;
      }
      if (q >= n_rows) break;
    }
    if (empty > kStepped && q == empty_row) {                // or to the next that holds a stop
      w = jump(w + 1, q);
      empty = 0;
    }
  }
  if (row >= 0) ref_to_cur[r] = mine;
  return w < 0 ? 0 : (uint32_t)(64 * w + p + 1);
}

constexpr uint32_t kGroupBlocks = 8;                   // blocks whose tables are put together
constexpr uint32_t kChainGroups = 16;                  // tables in LDS at a time
constexpr uint32_t kChainThreads = 256;

// The table of a group of blocks, for the window of its first: at most 8 * (kEntries + kMargin) columns.  upto: what the group's
// blocks take up to each of them, so that a block finds its entry from its group's with one read (block by block 4 us).
template <class Id>
__global__ __launch_bounds__(256) void ss_align_compose_kernel(const uint16_t *__restrict__ table, Windows win, uint32_t K,
                                                               uint16_t *__restrict__ upto, uint32_t upto_stride, uint16_t *__restrict__ groups,
                                                               const uint32_t *__restrict__ n_keys, uint32_t g_first) {
  if (sizeof(Id) == 2 && *n_keys >= kLdsKeys) return;        // nor tables
  const uint32_t g = g_first + blockIdx.x, k0 = g * kGroupBlocks, i = blockIdx.y * 256 + threadIdx.x, entry = win.start(k0) + i;
  uint32_t j = entry;
  bool known = j <= win.m;
  const uint32_t end = min(k0 + kGroupBlocks, K);
  for (uint32_t k = k0; k < end; ++k) {
    const uint32_t d = known ? win.taken(table, k, j) : kNoEntry;
    known = d != kNoEntry;
    if (known) j -= d;
    upto[(size_t)k * upto_stride + i] = known ? (uint16_t)(entry - j) : kNoEntry;
  }
  groups[(size_t)g * win.size + i] = known ? (uint16_t)(entry - j) : kNoEntry;
}

// Where a walk with narrow windows ends because the path has left them: the block's number and 1, and the columns left there.  The
// host is told at once; the pairs are left to the walk that goes on from there.
struct Strayed { uint32_t *device, *host_block, *host_columns; ss_done done; };

// group_entry[g]: columns left when the walk enters group g, or -1 if its blocks have been followed one by one here;
// then entry[k] is that of block k, or -1 if the block has been walked here.  The walk begins at block k_first with j_first columns
// left and ends with the last block, or at the one it strays at: what lies before that is as it would have been.
template <class Id>
__global__ __launch_bounds__(kChainThreads) void ss_align_chain_kernel(const Id *__restrict__ ref_id, Windows win,
                                                                       const uint32_t *__restrict__ masks,
                                                                       uint32_t W, uint32_t n_steps,
                                                                       const uint32_t *__restrict__ rows,
                                                                       const uint16_t *__restrict__ table,
                                                                       const uint16_t *__restrict__ upto, uint32_t upto_stride,
                                                                       const uint16_t *__restrict__ groups,
                                                                       int32_t *__restrict__ entry,
                                                                       int32_t *__restrict__ group_entry,
                                                                       int32_t *__restrict__ ref_to_cur, Strayed strayed,
                                                                       const uint32_t *__restrict__ n_keys, uint32_t k_first, uint32_t j_first) {
  constexpr uint32_t kTabs = kChainGroups * kWindow / 8, kPer = kTabs / kChainThreads;
  __shared__ uint4 tabs[kTabs];
  __shared__ uint32_t left;
  const uint32_t n = win.n, size = win.size;
  if (sizeof(Id) == 2 && *n_keys >= kLdsKeys) return;
  if (threadIdx.x == 0) left = 0;
  const uint32_t K = (n + kWalkRows - 1) / kWalkRows, G = (K + kGroupBlocks - 1) / kGroupBlocks;
  const uint4 *src = reinterpret_cast<const uint4 *>(groups);
  const uint32_t of_turn = min(kChainGroups, kTabs * 8 / size);
  const uint32_t total = G * (size / 8), turn = of_turn * (size / 8);      // at most 2^10 tables of 2^13 entries
  uint4 next[kPer];
  auto fetch = [&](uint32_t g0) {
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      const uint32_t x = i * kChainThreads + threadIdx.x, at = g0 * (size / 8) + x;
      next[i] = x < turn && at < total ? src[at] : uint4{0, 0, 0, 0};
    }
  };
  uint32_t j = j_first;                                      // wavefront 0's own
  // block by block, up to block `end`; false: the path has left the windows
  auto row_id = [&](uint32_t k) {
    const RowBlock blk(k, n);
    const uint32_t q = threadIdx.x & 63;
    return q < blk.hi - blk.lo ? ref_id[kIdPad + blk.hi - 1 - q] : Id(0);
  };
  auto follow = [&](uint32_t k, uint32_t end) {
    Id ahead = row_id(k);
    for (; k < end; ++k) {
      const Id id = ahead;
      if (k + 1 < end) ahead = row_id(k + 1);
      if (strayed.device && j - win.start(k) >= size) {
        if (threadIdx.x == 0) {
          left = 1;
          *strayed.device = k + 1;
          __hip_atomic_store(strayed.host_block, k + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          __hip_atomic_store(strayed.host_columns, j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          if (strayed.done.flag) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
            __hip_atomic_store(strayed.done.flag, strayed.done.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          }
        }
        return false;
      }
      const uint32_t e = __builtin_amdgcn_readfirstlane(win.taken(table, k, j));
      if (threadIdx.x == 0) entry[k] = e != kNoEntry ? (int32_t)j : -1;
      if (e != kNoEntry)
        j -= e;
      else
        j = __builtin_amdgcn_readfirstlane(walk_in_place(key_of(id), masks, rows, W, n_steps, RowBlock(k, n), j, ref_to_cur));
    }
    return true;
  };
  const uint32_t g_first = (k_first + kGroupBlocks - 1) / kGroupBlocks;    // the walk may begin within the group before
  fetch(g_first);
  if (k_first % kGroupBlocks && threadIdx.x < 64) follow(k_first, min(g_first * kGroupBlocks, K));
  for (uint32_t g0 = g_first; g0 < G; g0 += of_turn) {
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) tabs[i * kChainThreads + threadIdx.x] = next[i];
    __syncthreads();
    fetch(g0 + of_turn);
    if (threadIdx.x < 64) {
      const uint16_t *t = reinterpret_cast<const uint16_t *>(tabs);
      const uint32_t here = min(of_turn, G - g0), mine = min(g0 + (threadIdx.x & (kChainGroups - 1)), G - 1);
      const uint32_t starts = win.start(mine * kGroupBlocks);               // lane u: group g0 + u's
      int32_t entries = 0;                                   // likewise
      // where every table has its entry: nothing goes through the scalar unit between two of them
      uint32_t v = j;
      bool known = true;
#pragma unroll
      for (uint32_t u = 0; u < kChainGroups; ++u) {
        const uint32_t at = v - (uint32_t)__builtin_amdgcn_readlane((int)starts, u);       // before the window: wraps to a large number
        const uint32_t d = u < here ? at < size ? t[u * size + min(at, size - 1)] : kNoEntry : 0;
        entries = threadIdx.x == u ? (int32_t)v : entries;
        known &= d != kNoEntry;
        v -= d;
      }
      const bool all = __builtin_amdgcn_ballot_w64(known) == ~0ull;
      if (all) j = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
#pragma unroll 1
      for (uint32_t u = 0; !all && u < here; ++u) {
        const uint32_t at = j - (uint32_t)__builtin_amdgcn_readlane((int)starts, u);       // before the window: wraps to a large number
        const uint32_t d = at < size ? __builtin_amdgcn_readfirstlane((uint32_t)t[u * size + at]) : kNoEntry;
        if (threadIdx.x == u) entries = d != kNoEntry ? (int32_t)j : -1;
        if (__builtin_expect(d != kNoEntry, 1)) {
          j -= d;
          continue;
        }
        const uint32_t k0 = (g0 + u) * kGroupBlocks;
        uint32_t known_blocks = 0;                           // whose way through the group's first blocks is tabulated
        if (at < size) {
          const uint32_t b = threadIdx.x & 63;
          const uint32_t c = b < kGroupBlocks && k0 + b < K ? upto[(size_t)(k0 + b) * upto_stride + at] : kNoEntry;
          known_blocks = (uint32_t)__builtin_ctzll(__builtin_amdgcn_ballot_w64(c == kNoEntry));
          const uint32_t before = dpp_u32<0x111, 0xF>(c, 0);               // of the block before
          if (b < known_blocks) entry[k0 + b] = (int32_t)(j - before);
          if (known_blocks) j -= (uint32_t)__builtin_amdgcn_readlane((int)c, known_blocks - 1);
        }
        if (!follow(k0 + known_blocks, min(k0 + kGroupBlocks, K))) break;
      }
      if (threadIdx.x < here) group_entry[g0 + threadIdx.x] = entries;
    }
    __syncthreads();
    if (left) return;
  }
}

// The walk through a block from j columns left by one wavefront, lane q the block's row q; returns the column that the row pairs
// with, or -1.  Equal operators run along the diagonal: each lane tests its own row's bit there and a ballot tells how long the
// run is; in the row that it ends in, sixteen lanes look for the highest column below that is equal or steps up.  A block whose
// first kManyRuns runs were of no more than kTheirRows rows is then gone through row by row as by walk_tile: 0.1 us a row, a run's end
// takes 0.2.  The pairs of 6,000 unrelated operators of 40 keys 17.6 us, by runs alone 24.3, of 9,270 of a training trace 12.3 and 12.3;
// after sixteen runs of any length 17.3 and 13.2.
constexpr uint32_t kManyRuns = 16, kTheirRows = 36;

__device__ __forceinline__ int32_t walk_runs(uint32_t n_rows, int w0, int j, const Tile &tile) {
  const int lane = threadIdx.x & 63, l = lane % (int)kTileWords;
  int32_t mine = -1;
  uint32_t q = 0;
  for (uint32_t runs = 0; runs != kManyRuns || q > kTheirRows; ++runs) {
    if (q >= n_rows || j <= 0) return mine;
    const int c = j - 1 - (lane - (int)q), w = (c >> 5) - w0;
    const bool hit = lane >= (int)q && lane < (int)n_rows && c >= 0 && w >= 0 && (tile[lane][w + 1].equal >> (c & 31) & 1u);
    const u64 missed = ~(__builtin_amdgcn_ballot_w64(hit) >> q);       // the shift brings in zeros
    const uint32_t run = missed ? (uint32_t)__builtin_ctzll(missed) : 64;
    if (lane >= (int)q && lane < (int)(q + run)) mine = c;
    q += run;
    j -= (int)run;
    if (q >= n_rows || j <= 0) return mine;
    const int at = ((j - 1) >> 5) - w0;
    if (at < 0) return mine;                                 // left of the tile: the table had no entry
    const TileWord x = tile[q][l + 1];
    const uint32_t bits = l <= at ? x.stops & (l == at ? ~0u >> (31 - ((j - 1) & 31)) : ~0u) : 0;
    const uint32_t there = (uint32_t)__builtin_amdgcn_ballot_w64(bits != 0) & ((1u << kTileWords) - 1);
    if (!there) return mine;                                 // all the columns are used up
    const int word = 31 - __builtin_clz(there);
    const int b = 31 - __builtin_clz((uint32_t)__builtin_amdgcn_readlane((int)bits, word));
    j = (word + w0) * 32 + b + 1;
    if (!((uint32_t)__builtin_amdgcn_readlane((int)x.equal, word) >> b & 1u)) ++q;            // up; else the next run begins there
  }
  const uint32_t rows_some = words_that_stop(n_rows, tile);
  uint32_t at = (uint32_t)(j - 1 - w0 * 32 + 32);
  for (; q < n_rows; ++q) {
    const TileStep x = step_row(tile, q, (uint32_t)__builtin_amdgcn_readlane((int)rows_some, q), at);
    if (x.stops && x.equal && lane == (int)q) mine = (int32_t)(at - 32) + w0 * 32 + 1;
  }
  return mine;
}

// Blocks from k_win on were walked by the chain with windows `win`, those before with `first`.
// One wavefront walks, all of them load its tile.  Bound by the latency of loads that need each other (the group's entry, the
// block's, the tile's ids and masks) and of the walk's LDS reads: 32,312 rows 15.3 us; with one thread that walks row by row, the
// block's entry by up to seven reads one after the other and the tile's loads one after the other 20.1.
constexpr uint32_t kPairThreads = kTileThreads;
static_assert(kEntries == kTileThreads, "a table's workgroup loads its tile");

template <class Id>
__global__ __launch_bounds__(kPairThreads) void ss_align_pairs_kernel(const Id *__restrict__ ref_id, Windows first, Windows win, uint32_t k_win,
                                                            const uint32_t *__restrict__ masks, uint32_t W,
                                                            uint32_t n_steps, const uint32_t *__restrict__ rows,
                                                            const uint16_t *__restrict__ upto, uint32_t upto_stride,
                                                            const int32_t *__restrict__ entry,
                                                            const int32_t *__restrict__ group_entry,
                                                            int32_t *__restrict__ ref_to_cur, const uint32_t *strayed, const uint32_t *n_keys,
                                                            ss_done done) {
  __shared__ Tile tile;
  const uint32_t k = blockIdx.x, k0 = k / kGroupBlocks * kGroupBlocks;
  if (strayed && *strayed) return;                           // the chain has ended early, and has told the host
  if (sizeof(Id) == 2 && *n_keys >= kLdsKeys) {
    ss_tell_host(done);
    return;
  }
  int j = group_entry[k / kGroupBlocks];
  if (j >= 0) {                                              // known: the group's table is
    if (k > k0) j -= (int)upto[(size_t)(k - 1) * upto_stride + (uint32_t)j - (k < k_win ? first.start(k0) : win.start(k0))];
  } else {
    j = entry[k];
  }
  if (j < 0) {                                               // the chain has walked it
    ss_tell_host(done);
    return;
  }
  const RowBlock blk(k, win.n);
  const int w0 = j / (int)kEntries * (int)(kEntries / 32) - (int)(kMargin / 32);     // the tile the table came from
  load_tile(ref_id, masks, rows, W, n_steps, blk, w0, tile);
  __syncthreads();
  if (threadIdx.x < 64) {
    const int32_t mine = walk_runs(blk.hi - blk.lo, w0, __builtin_amdgcn_readfirstlane(j), tile);
    if (threadIdx.x < blk.hi - blk.lo) ref_to_cur[blk.hi - 1 - threadIdx.x] = mine;
  }
  ss_tell_host(done);
}

// LDS of the rows kernel with 16-bit ids, beside what it always has: its mask rows
size_t lds_need(uint32_t n_keys) { return (size_t)(n_keys + 1) * kStripWords * 4; }

// Where everything lies.  `d` device scratch, `h` pinned scratch.
struct Layout {
  size_t h_ref, h_cur, h_flag, h_n_keys, h_part, h_out, h_end;
  size_t ref, cur, ref_id, cur_id, n_keys, rep, id, slot, carry, gave_up, rows, table, entry, upto, groups, group_entry, masks, end;
  uint32_t n, m, W, strips, n_steps, n_blocks, walk_blocks, walk_groups, window, upto_stride, slots, bits;
  bool one_wg, short_rows;

  Layout(uint32_t n_, uint32_t m_) : n(n_), m(m_) {
    W = (m + 31) / 32;                                     // 32-bit words of a row
    strips = strips_of(W);
    n_steps = strips == 1 ? steps_of(n, W) : steps_of(n);
    n_blocks = n_steps / kBlock;
    walk_blocks = (n + kWalkRows - 1) / kWalkRows;
    walk_groups = (walk_blocks + kGroupBlocks - 1) / kGroupBlocks;
    const size_t row_bytes = (size_t)strips * n_steps * kStripWords * 4;
    one_wg = n + m <= kWgOps;
    // the kernel writes the rows to pinned host memory and the host walks them; else they stay in device memory and
    // are walked there
    short_rows = row_bytes <= (m > 2 * (uint64_t)n ? kHostRowBytesSteep : kHostRowBytes);
    // The windows that the walk begins with (kWindow)
    const uint32_t all = (uint32_t)ss_align_up(m + 1, kEntries);
    const uint32_t differ = std::max(n, m) - std::min(n, m);
    const bool few_tables = all <= kMostColumns && walk_blocks * (all / kEntries) <= kAllTables;
    window = all <= kWindow || (few_tables && differ > kWindow / 2) ? all : differ <= kNearlyEqual ? kNarrowWindow : kWindow;
    upto_stride = std::max(window, kWindow);               // the same for a second walk, of whose blocks it leaves the others'
    const size_t entries = upto_stride;
    bits = 13;
    while ((1u << bits) < 2 * m) ++bits;
    slots = 1u << bits;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += ss_align_up(bytes, 256); return at; };
    h_ref = take((size_t)n * sizeof(ss_op_t));
    h_cur = take((size_t)m * sizeof(ss_op_t));
    h_flag = take(16);                                     // the same; the number of keys; columns left where the walk strays
    h_n_keys = h_flag + 8;
    h_part = take(kFetchWgs * sizeof(ss_cosine_part));
    h_out = take(short_rows ? row_bytes : (size_t)n * 4);
    h_end = o;
    o = 0;
    ref = take(one_wg ? 0 : (size_t)n * sizeof(ss_op_t));
    cur = take(one_wg ? 0 : (size_t)m * sizeof(ss_op_t));
    ref_id = take((size_t)id_length(n_steps) * 4);
    cur_id = take((size_t)m * 4);
    n_keys = take(4);
    rep = take(one_wg ? 0 : (size_t)slots * 4);
    id = take(one_wg ? 0 : (size_t)slots * 4);
    slot = take(one_wg ? 0 : (size_t)m * 4);
    rows = take(short_rows ? 0 : row_bytes);
    table = take(short_rows ? 0 : walk_blocks * entries * 2);
    entry = take(short_rows ? 0 : (size_t)walk_blocks * 4);
    upto = take(short_rows ? 0 : walk_blocks * entries * 2);
    groups = take(short_rows ? 0 : walk_groups * entries * 2);
    group_entry = take(short_rows ? 0 : (size_t)walk_groups * 4);
    carry = take((size_t)(strips - 1) * (n_blocks + kCarryPad) * 8);
    gave_up = take(8);                                     // by a strip; by the walk (strayed)
    masks = o;                                             // last: its size needs the number of keys
    end = o;
  }
  size_t with_masks(uint32_t keys) const { return end + (size_t)(keys + 1) * W * 4; }
  size_t to_clear(bool with, uint32_t keys) const { return (with ? with_masks(keys) : end) - carry; }          // carry words, then masks
};
// With both lengths at their limit the rows take 545 MiB, a strip 16 MiB (the kernel's buffer offsets have 31 bits), and the
// masks, with every key distinct, 512 MiB.
static_assert((uint64_t)steps_of(kAlignLenLimit) * kStripWords * 4 * strips_of(kAlignLenLimit / 32) <= 1ull << 30, "rows");
static_assert((uint64_t)steps_of(kAlignLenLimit) * kStripWords * 4 < 1ull << 31, "a strip's rows");
static_assert(((uint64_t)kAlignLenLimit + 1) * (kAlignLenLimit / 32) * 4 <= 1ull << 30, "masks");

// The walk over rows in device memory, with windows of that size, from block k on with j columns left.
template <class Id>
int launch_walk(ss_ctx *ctx, const Layout &y, uint8_t *d, uint8_t *hd, uint32_t size, uint32_t k, uint32_t j, ss_done &done) {
  hipStream_t s = ctx->s_aux;
  const Id *ref_id = (const Id *)(d + y.ref_id);
  const uint32_t *masks = (const uint32_t *)(d + y.masks), *rows = (const uint32_t *)(d + y.rows);
  uint16_t *table = (uint16_t *)(d + y.table), *upto = (uint16_t *)(d + y.upto), *groups = (uint16_t *)(d + y.groups);
  int32_t *entry = (int32_t *)(d + y.entry), *group_entry = (int32_t *)(d + y.group_entry), *pair = (int32_t *)(hd + y.h_out);
  const uint32_t *n_keys = (const uint32_t *)(d + y.n_keys);
  uint32_t *const h_flag = (uint32_t *)(hd + y.h_flag);
  const Windows win(y.n, y.m, size, y.n - k * kWalkRows, j), first(y.n, y.m, y.window, y.n, y.m);
  const uint32_t g = k / kGroupBlocks, k0 = g * kGroupBlocks;              // the tables' first group and block
  done = ss_next_done(ctx);
  ss_told_by(done, y.walk_blocks);
  const Strayed strayed = size == kNarrowWindow && size <= y.m ? Strayed{(uint32_t *)(d + y.gave_up) + 1, h_flag + 1, h_flag + 3, done} : Strayed{};
  hipLaunchKernelGGL(ss_align_tab_kernel<Id>, dim3(y.walk_blocks - k0, size / kEntries), dim3(kEntries), 0, s, ref_id, win, masks,
                     y.W, y.n_steps, rows, table, n_keys, k0);
  hipLaunchKernelGGL(ss_align_compose_kernel<Id>, dim3(y.walk_groups - g, size / 256), dim3(256), 0, s, table, win, y.walk_blocks, upto,
                     y.upto_stride, groups, n_keys, g);
  hipLaunchKernelGGL(ss_align_chain_kernel<Id>, dim3(1), dim3(kChainThreads), 0, s, ref_id, win, masks, y.W, y.n_steps, rows, table,
                     upto, y.upto_stride, groups, entry, group_entry, pair, strayed, n_keys, k, j);
  hipLaunchKernelGGL(ss_align_pairs_kernel<Id>, dim3(y.walk_blocks), dim3(kPairThreads), 0, s, ref_id, first, win, k, masks, y.W,
                     y.n_steps, rows, upto, y.upto_stride, entry, group_entry, pair, strayed.device, n_keys, done);
  SS_HIP(hipGetLastError());
  return SS_OK;
}

// cleared: with what the rows need clear, and the masks made, by the kernels of the ids.
// Rows (and, long ones, the walk) for ids of the given form.  The masks are needed where the rows kernel does not keep its
// own in LDS, and by the walk.
template <class Id>
int launch_rows(ss_ctx *ctx, const Layout &y, uint8_t *d, uint8_t *hd, uint32_t keys, ss_done &done, bool one_by_one = false,
                bool cleared = false) {
  constexpr bool kLds = sizeof(Id) == 2;
  hipStream_t s = ctx->s_aux;
  const Id *ref_id = (const Id *)(d + y.ref_id), *cur_id = (const Id *)(d + y.cur_id);
  uint32_t *masks = (uint32_t *)(d + y.masks), *rows = (uint32_t *)(y.short_rows ? hd + y.h_out : d + y.rows);
  const bool masks_needed = !kLds || !y.short_rows;
  if (!cleared) ss_launch_fill(s, d + y.carry, y.to_clear(masks_needed, keys), 0);
  if (!cleared && masks_needed)
    hipLaunchKernelGGL(ss_align_masks_kernel<Id>, dim3((y.m + 255) / 256), dim3(256), 0, s, cur_id, y.m, masks, y.W);
  RowsArgs args = {masks, (u64 *)(d + y.carry), rows, (uint32_t *)(d + y.gave_up), (uint32_t *)(hd + y.h_flag),
                   y.W, y.n_steps, y.strips, 0, ctx->align_wait_looks, {}};
  const uint32_t *n_keys = (const uint32_t *)(d + y.n_keys);
  const uint32_t per_launch = one_by_one ? 1 : y.strips;
  if (y.short_rows) {
    done = ss_next_done(ctx);
    ss_told_by(done, y.strips);
    args.done = done;
  }
  for (; args.strip0 < y.strips; args.strip0 += per_launch)
    hipLaunchKernelGGL(ss_align_rows_kernel<Id>, dim3(per_launch), dim3(kRowsThreads), kLds ? lds_need(keys) : 0, s, ref_id,
                       cur_id, y.m, args, n_keys);
  SS_HIP(hipGetLastError());
  return y.short_rows ? SS_OK : launch_walk<Id>(ctx, y, d, hd, y.window, 0, y.m, done);
}

}  // namespace

// ref_to_cur: n entries (host), filled; *lcs out.  Shared by ss_align_sequence and the SS_MATCH_ALIGN
// branch of ss_match_sequence.
int ss_align_core(ss_ctx *ctx, const ss_op_t *ref, uint32_t n, const ss_op_t *cur, uint32_t m,
                  int32_t *ref_to_cur, uint32_t *lcs, uint32_t *n_keys_out, ss_cosine_part *sums) {
  if (n > kAlignLenLimit || m > kAlignLenLimit) return SS_E_CAPACITY;
  for (uint32_t i = 0; i < n; ++i) ref_to_cur[i] = -1;
  *lcs = 0;
  if (n_keys_out) *n_keys_out = 0;
  if (n == 0 || m == 0) return SS_OK;
  const Layout y(n, m);
  const uint32_t few = kLdsKeys - 1;
  hipStream_t s = ctx->s_aux;
  uint8_t *d = nullptr, *h = nullptr, *hd = nullptr;
  volatile uint32_t *h_flag = nullptr, *h_n_keys = nullptr;
  ss_done keys_known = {}, done = {};
  uint32_t parts = 1;
  // key ids; again if the mask table then turns out not to fit (the first call with that many keys)
  auto make_ids = [&](size_t dev_bytes, bool again) -> int {
    const int rc = ss_scratch_reserve(ctx, dev_bytes, y.h_end);
    if (rc != SS_OK) return rc;
    d = (uint8_t *)ctx->d_scratch;
    h = (uint8_t *)ctx->h_scratch;
    SS_HIP(hipHostGetDevicePointer((void **)&hd, h, 0));
    std::memcpy(h + y.h_ref, ref, (size_t)n * sizeof(ss_op_t));
    std::memcpy(h + y.h_cur, cur, (size_t)m * sizeof(ss_op_t));
    h_flag = (volatile uint32_t *)(h + y.h_flag);
    h_n_keys = (volatile uint32_t *)(h + y.h_n_keys);
    h_flag[0] = h_flag[1] = 0;
    KeyArgs a = {};
    a.n = n; a.m = m; a.n_steps = y.n_steps;
    a.few = few;
    a.ref_id = d + y.ref_id;
    a.cur_id = d + y.cur_id;
    a.n_keys = (uint32_t *)(d + y.n_keys);
    a.n_keys_out = (uint32_t *)(hd + y.h_n_keys);
    if (sums) a.part = (ss_cosine_part *)(hd + y.h_part);
    const ss_op_t *mref = (const ss_op_t *)(hd + y.h_ref), *mcur = (const ss_op_t *)(hd + y.h_cur);
    if (y.one_wg) {
      a.ref = mref;
      a.cur = mcur;
      if (y.strips == 1 && !again) {
        RowsArgs r = {nullptr, nullptr, (uint32_t *)(hd + y.h_out), nullptr, nullptr, y.W, y.n_steps, 1, 0, 0, ss_next_done(ctx)};
        done = r.done;
        hipLaunchKernelGGL(a.part ? ss_align_short_kernel<true> : ss_align_short_kernel<false>, dim3(1), dim3(kWgThreads), kShortLds, s, a, r);
      } else {
        hipLaunchKernelGGL(a.part ? ss_align_keys_kernel<true> : ss_align_keys_kernel<false>, dim3(1), dim3(kWgThreads), kWgLds, s, a);
      }
    } else {
      ss_op_t *dref = (ss_op_t *)(d + y.ref), *dcur = (ss_op_t *)(d + y.cur);
      a.ref = dref;
      a.cur = dcur;
      a.rep = (uint32_t *)(d + y.rep);
      a.id = (uint32_t *)(d + y.id);
      a.slot = (uint32_t *)(d + y.slot);
      a.mask = y.slots - 1;
      a.shift = 64 - y.bits;
      const uint32_t wgs = parts = std::min(kFetchWgs, (std::max(n, m) + 255) / 256), len = std::max(m, id_length(y.n_steps));
      const bool for_rows = !ctx->align_many_keys;
      if (for_rows && !y.short_rows) {
        a.masks = (uint32_t *)(d + y.masks);
        a.W = y.W;
      }
      hipLaunchKernelGGL(ss_align_fetch_kernel, dim3(wgs), dim3(256), 0, s, mref, dref, n, mcur, dcur, m, a.rep, y.slots, a.n_keys,
                         (uint4 *)(d + y.carry), for_rows ? (uint32_t)((y.to_clear(a.masks, few) + 15) / 16) : 0, a.part);
      hipLaunchKernelGGL(ss_align_insert_kernel, dim3((m + 255) / 256), dim3(256), 0, s, a);
      if (ctx->align_many_keys) {
        a.done = ss_next_done(ctx);
        ss_told_by(a.done, (len + 255) / 256);
        keys_known = a.done;
      }
      hipLaunchKernelGGL(ss_align_ids_kernel, dim3((len + 255) / 256), dim3(256), 0, s, a);
    }
    SS_HIP(hipGetLastError());
    return SS_OK;
  };
  int rc = make_ids(y.with_masks(kLdsKeys), false);
  if (rc != SS_OK) return rc;
  uint32_t keys = kLdsKeys - 1;
  bool done_rows = false;
  auto rows = [&](bool one_by_one) -> int {
    int r = keys <= few ? launch_rows<uint16_t>(ctx, y, d, hd, keys, done, one_by_one)
                        : launch_rows<uint32_t>(ctx, y, d, hd, keys, done, one_by_one);
    return r != SS_OK ? r : ss_wait_done(ctx, done);
  };
  // Rows and walk at once, as if there were few keys (every kernel looks again): one wait less, some 8 us.  If there are more the
  // launches are for nothing, so a context whose last call had more waits for their number before.
  if (y.one_wg || !ctx->align_many_keys) {
    if (!(y.one_wg && y.strips == 1) && (rc = launch_rows<uint16_t>(ctx, y, d, hd, keys, done, false, !y.one_wg)) != SS_OK) return rc;
    if ((rc = ss_wait_done(ctx, done)) != SS_OK) return rc;
    keys = *h_n_keys;
    done_rows = keys <= few;
  } else {
    if ((rc = ss_wait_done(ctx, keys_known)) != SS_OK) return rc;
    keys = *h_n_keys;
  }
  ctx->align_many_keys = keys > few;
  if (!done_rows) {
    h_flag[0] = h_flag[1] = 0;
    if (y.with_masks(keys) > ctx->d_scratch_bytes) {
      if ((rc = make_ids(y.with_masks(keys), true)) != SS_OK) return rc;
    }
    if ((rc = rows(false)) != SS_OK) return rc;
  }
  if (*h_flag) {                        // a strip gave up: each after the one before it, then every word is there and none waits
    ctx->align_one_by_one += 1;
    h_flag[1] = 0;                      // what the walk made of these rows
    if ((rc = rows(true)) != SS_OK) return rc;
  }
  if (h_flag[1]) {                      // the path has left the narrow windows: on from there with wide ones
    const uint32_t k = h_flag[1] - 1, j = h_flag[3];
    rc = keys <= few ? launch_walk<uint16_t>(ctx, y, d, hd, kWindow, k, j, done) : launch_walk<uint32_t>(ctx, y, d, hd, kWindow, k, j, done);
    if (rc != SS_OK || (rc = ss_wait_done(ctx, done)) != SS_OK) return rc;
  }
  if (n_keys_out) *n_keys_out = keys;
  if (sums) {
    const ss_cosine_part *const part = (const ss_cosine_part *)(h + y.h_part);
    *sums = ss_cosine_part{0, 0, 0, 0};
    for (uint32_t w = 0; w < parts; ++w) {
      sums->dot += part[w].dot; sums->na += part[w].na; sums->nb += part[w].nb; sums->bad |= part[w].bad;
    }
  }
  uint32_t pairs = 0;
  if (!y.short_rows) {
    std::memcpy(ref_to_cur, h + y.h_out, (size_t)n * 4);
    for (uint32_t i = 0; i < n; ++i) pairs += ref_to_cur[i] >= 0;
    *lcs = pairs;
    return SS_OK;
  }
  // walk back from (n, m)
  const uint32_t *hr = (const uint32_t *)(h + y.h_out);
  constexpr uint32_t kAhead = 24;
  uint32_t i = n, j = m;
  while (i > 0 && j > 0) {
    // the rows came over the link: none is in a cache, and the path's next rows lie near the diagonal
    if (i > kAhead && j > kAhead) __builtin_prefetch(hr + row_word(i - 1 - kAhead, (j - 1 - kAhead) >> 5, y.W, y.n_steps));
    const ss_op_t &a = ref[i - 1], &b = cur[j - 1];
    if (a.op_token == b.op_token && a.stack_hash == b.stack_hash && a.sig == b.sig) {
      ref_to_cur[i - 1] = (int32_t)(j - 1);
      ++pairs;
      --i;
      --j;
    } else if ((hr[row_word(i - 1, (j - 1) >> 5, y.W, y.n_steps)] >> ((j - 1) & 31)) & 1u) {
      --j;
    } else {
      --i;
    }
  }
  *lcs = pairs;
  return SS_OK;
}

// For tests: the context's limit of a strip's wait, in looks at the word; returns how many of its calls have started the
// strips one by one so far.
extern "C" uint32_t ss_align_wait_limit(ss_ctx *ctx, uint32_t looks) {
  if (!ctx) return 0;
  ctx->align_wait_looks = looks;
  return ctx->align_one_by_one;
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
