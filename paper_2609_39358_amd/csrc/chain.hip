// Device-side key chains and a device index (gfx950).
//
// The key of block k of a chain is SHA-256(key of block k-1 | the block's
// token ids as u32 little-endian), rooted at the namespace digest or at a
// caller-supplied parent key (Sec. 2.2: state is stored under a fingerprint
// of the exact input bytes, the model and the tenant; Sec. 5: reuse is of
// whole blocks at exact positions). A chain is inherently sequential; the
// chip's parallelism is across chains. Few chains get a workgroup of four
// wavefronts each (k_chain_waves), which divides the work of one chain; many
// share wavefronts, up to 64 of them (k_chain; chain_waves draws the line).
//
// The walk probes the device index while it computes, so the lookup of key k
// hides behind the hash of key k+1. Key k+1 is kept only once key k is known
// to be a hit.
//
// Device index: linear probing over 64-byte slots
//   word 0  tag = first 8 key bytes | 1 (0 = empty)
//   word 1  writer (0 outside a put; the winning duplicate's index + 1 inside)
//   word 2  handle
//   word 3  0
//   words 4..7  the key
// after a 256-byte header (word 0 occupied slots, word 1 longest probe). A
// put has three phases (kernels; few keys: one kernel with barriers), so that
// no lane ever waits on another: claim (find the key's slot by tag, or take a
// free one with a compare-and-swap and write the key), vote (each lane checks the full key in its slot, now
// complete, and takes the maximum of its index into the writer word), and
// publish (the winner writes the handle and clears the writer word).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"

namespace {

constexpr uint32_t kMaxProbe = 1024;  // slots a key may sit past its home slot
constexpr uint32_t kNoSlot = 0xffffffffu;
constexpr uint64_t kMiss = ~0ull;
constexpr uint32_t kHeaderWords = 32;  // 256-byte header
constexpr uint32_t kSlotWords = 8;

// ---- SHA-256 compression (FIPS 180-4, 6.2.2) --------------------------------
__device__ __forceinline__ uint32_t rotr(uint32_t x, uint32_t n) {
  return __builtin_amdgcn_alignbit(x, x, n);
}
// gfx950 has any function of three words in one instruction (v_bitop3_b32;
// the immediate is the function of 0xf0, 0xcc and 0xaa); the compiler forms
// it from only some of these expressions.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96);
}
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t a, uint32_t b) {  // bits of a where mask is set
  return (uint32_t)__builtin_amdgcn_bitop3_b32((int)mask, (int)a, (int)b, 0xca);
}
__device__ __forceinline__ uint32_t bsig0(uint32_t a) { return xor3(rotr(a, 2), rotr(a, 13), rotr(a, 22)); }
__device__ __forceinline__ uint32_t bsig1(uint32_t e) { return xor3(rotr(e, 6), rotr(e, 11), rotr(e, 25)); }
__device__ __forceinline__ uint32_t ssig0(uint32_t x) { return xor3(rotr(x, 7), rotr(x, 18), x >> 3); }
__device__ __forceinline__ uint32_t ssig1(uint32_t x) { return xor3(rotr(x, 17), rotr(x, 19), x >> 10); }
__device__ __forceinline__ uint32_t ch(uint32_t e, uint32_t f, uint32_t g) { return pick(e, f, g); }
__device__ __forceinline__ uint32_t maj(uint32_t a, uint32_t b, uint32_t c) {
  return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0xe8);
}

// Rounds R..63 with the working variables passed by value, so that the
// unrolled rounds rename registers instead of moving them; K[R] is a
// constant expression, hence an immediate.
template <int R>
__device__ __forceinline__ void rounds(uint32_t (&out)[8], uint32_t a, uint32_t b, uint32_t c,
                                       uint32_t d, uint32_t e, uint32_t f, uint32_t g, uint32_t h,
                                       uint32_t (&w)[16]) {
  if constexpr (R == 64) {
    out[0] = a; out[1] = b; out[2] = c; out[3] = d;
    out[4] = e; out[5] = f; out[6] = g; out[7] = h;
  } else {
    constexpr uint32_t k = tl::kSha256K[R];
    if constexpr (R >= 16)
      w[R & 15] += ssig1(w[(R + 14) & 15]) + w[(R + 9) & 15] + ssig0(w[(R + 1) & 15]);
    const uint32_t t1 = h + bsig1(e) + ch(e, f, g) + k + w[R & 15];
    const uint32_t t2 = bsig0(a) + maj(a, b, c);
    rounds<R + 1>(out, t1 + t2, a, b, c, d + t1, e, f, g, w);
  }
}

__device__ __forceinline__ void compress(uint32_t (&st)[8], uint32_t (&w)[16]) {
  uint32_t o[8];
  rounds<0>(o, st[0], st[1], st[2], st[3], st[4], st[5], st[6], st[7], w);
#pragma unroll
  for (int i = 0; i < 8; ++i) st[i] += o[i];
}

// SHA-256 of PW big-endian prefix words followed by bt u32 token ids (as
// little-endian bytes): the message is 4*PW + 4*bt bytes, then 0x80, zeros
// and the 64-bit bit length, in nb 64-byte blocks (the same for every lane).
// PW = 8 gives a chain key (the previous key, then the block's tokens);
// PW = 10 a block fingerprint (namespace digest and position, then tokens).
template <int PW>
__device__ __forceinline__ void sha_tokens(uint32_t (&out)[8], const uint32_t (&pre)[PW],
                                           const uint32_t* tok, uint32_t bt, uint32_t nb,
                                           uint32_t len_hi, uint32_t len_lo) {
  uint32_t st[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) st[i] = tl::kSha256IV[i];
  const uint32_t last = 16 * nb - 1;
  for (uint32_t c = 0; c < nb; ++c) {
    // all sixteen loads go out before the first is needed (an index past the
    // tokens reads the last one), so a compression waits for memory once
    uint32_t w[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) w[t] = tok[min(16 * c + t - PW, bt - 1)];
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const uint32_t g = 16 * c + t;  // word index in the message
      const uint32_t j = g - PW;      // token index (wraps for g < PW)
      uint32_t v = j < bt ? __builtin_bswap32(w[t]) : j == bt ? 0x80000000u : 0;
      if (t < PW && g < PW) v = pre[t < PW ? t : 0];
      if (t == 14 && g == last - 1) v = len_hi;
      if (t == 15 && g == last) v = len_lo;
      w[t] = v;
    }
    compress(st, w);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) out[i] = st[i];
}

// Message geometry of sha_tokens for PW prefix words and bt tokens.
struct MsgLen {
  uint32_t nb, hi, lo;
};
__host__ __device__ inline MsgLen msg_len(uint32_t pw, uint32_t bt) {
  const uint64_t bytes = 4ull * pw + 4ull * bt;
  return MsgLen{(uint32_t)((bytes + 8) / 64 + 1), (uint32_t)((bytes * 8) >> 32), (uint32_t)(bytes * 8)};
}

// ---- device index ---------------------------------------------------------
struct Dx {
  uint64_t* mem;  // header, then slots
  uint64_t mask;  // capacity - 1
};

__device__ __forceinline__ uint64_t* slot_ptr(const Dx& x, uint64_t s) {
  return x.mem + kHeaderWords + s * kSlotWords;
}

// Key words as little-endian u64 from a byte array of 32 bytes.
__device__ __forceinline__ void load_key(uint64_t (&k)[4], const uint8_t* p) {
  const uint64_t* q = (const uint64_t*)p;
#pragma unroll
  for (int i = 0; i < 4; ++i) k[i] = q[i];
}

// The same words from a chain key held as big-endian SHA-256 state words.
__device__ __forceinline__ void key_words(uint64_t (&k)[4], const uint32_t (&h)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    k[i] = (uint64_t)__builtin_bswap32(h[2 * i]) | (uint64_t)__builtin_bswap32(h[2 * i + 1]) << 32;
}

__device__ __forceinline__ uint64_t tag_of(const uint64_t (&k)[4]) { return k[0] | 1; }

__device__ __forceinline__ uint64_t atomic_read(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(256) void k_dindex_clear(uint64_t* mem, uint64_t n_words) {
  const uint64_t step = (uint64_t)gridDim.x * 256;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n_words; i += step) mem[i] = 0;
}

struct PutArgs {
  Dx x;
  const uint8_t* keys;
  const uint64_t* handles;
  uint8_t* status;
  uint32_t* target;  // workspace [n]
  uint32_t n;
};

__device__ __forceinline__ void put_claim(const PutArgs& a, uint32_t i) {
  uint64_t k[4];
  load_key(k, a.keys + 32ull * i);
  const uint64_t tag = tag_of(k);
  const uint64_t home = k[1] & a.x.mask;
  const uint32_t reach = a.x.mask < kMaxProbe ? (uint32_t)a.x.mask + 1 : kMaxProbe;
  uint32_t target = kNoSlot;
  for (uint32_t d = 0; d < reach; ++d) {
    const uint64_t s = (home + d) & a.x.mask;
    uint64_t* slot = slot_ptr(a.x, s);
    uint64_t t = atomic_read(slot);
    if (t == 0) {
      t = atomicCAS((unsigned long long*)slot, 0ull, (unsigned long long)tag);
      if (t == 0) {  // this lane owns the slot: it alone writes the key
#pragma unroll
        for (int q = 0; q < 4; ++q) slot[4 + q] = k[q];
        atomicAdd((unsigned long long*)&a.x.mem[0], 1ull);
        atomicMax((unsigned long long*)&a.x.mem[1], (unsigned long long)d);
        target = (uint32_t)s;
        break;
      }
    }
    if (t == tag) {  // the key's slot (or a tag clash, found by the vote)
      target = (uint32_t)s;
      break;
    }
  }
  a.target[i] = target;
}

__device__ __forceinline__ void put_vote(const PutArgs& a, uint32_t i) {
  const uint32_t s = a.target[i];
  uint8_t st = TL_INDEX_FULL;
  if (s != kNoSlot) {
    uint64_t k[4];
    load_key(k, a.keys + 32ull * i);
    uint64_t* slot = slot_ptr(a.x, s);
    const bool same = slot[4] == k[0] && slot[5] == k[1] && slot[6] == k[2] && slot[7] == k[3];
    if (same) {
      atomicMax((unsigned long long*)&slot[1], (unsigned long long)i + 1);
      st = TL_INDEX_STORED;
    } else {
      st = TL_INDEX_TAG_CLASH;
      a.target[i] = kNoSlot;
    }
  }
  if (a.status) a.status[i] = st;
}

__device__ __forceinline__ void put_publish(const PutArgs& a, uint32_t i) {
  const uint32_t s = a.target[i];
  if (s == kNoSlot) return;
  uint64_t* slot = slot_ptr(a.x, s);
  if (atomic_read(&slot[1]) == (uint64_t)i + 1) {
    slot[2] = a.handles[i];
    slot[1] = 0;
  }
}

__global__ __launch_bounds__(256) void k_dindex_claim(PutArgs a) {
  const uint32_t step = gridDim.x * 256;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < a.n; i += step) put_claim(a, i);
}

__global__ __launch_bounds__(256) void k_dindex_vote(PutArgs a) {
  const uint32_t step = gridDim.x * 256;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < a.n; i += step) put_vote(a, i);
}

__global__ __launch_bounds__(256) void k_dindex_publish(PutArgs a) {
  const uint32_t step = gridDim.x * 256;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < a.n; i += step) put_publish(a, i);
}

// A put of at most kPutThreads keys in one launch: barriers stand where the
// others have the ends of kernels. One compute unit has to do it, which shows
// with inserts, above all where keys sit far from their home slots. Keys new to
// an index that is 45 % full (three kernels, one): 62 13.5 and 11.7 us, 256 16.7
// and 16.1, 320 18.4 and 18.8, 512 17.8 and 21.9; to an empty one 256 9.3 and
// 9.1, 320 9.5 and 10.3, 512 10.5 and 15.0; hence the bound. (Puts of keys that
// are there already: 256 10.6 and 6.7, 512 10.9 and 10.1.)
constexpr uint32_t kPutThreads = 256;

__global__ __launch_bounds__(kPutThreads) void k_dindex_put(PutArgs a) {
  const uint32_t i = threadIdx.x;
  if (i < a.n) put_claim(a, i);
  __threadfence();
  __syncthreads();
  if (i < a.n) put_vote(a, i);
  __threadfence();
  __syncthreads();
  if (i < a.n) put_publish(a, i);
}

// Handle of key k, or kMiss; probes at most maxp + 1 slots.
__device__ __forceinline__ uint64_t probe_from(const Dx& x, const uint64_t (&k)[4], uint64_t maxp,
                                               uint64_t d0) {
  const uint64_t tag = tag_of(k);
  const uint64_t home = k[1] & x.mask;
  for (uint64_t d = d0; d <= maxp; ++d) {
    // the slot's words in one request (it is one 64-byte line)
    const uint64_t* slot = slot_ptr(x, (home + d) & x.mask);
    const uint64_t t = slot[0], hv = slot[2], k0 = slot[4], k1 = slot[5], k2 = slot[6], k3 = slot[7];
    if (t == 0) return kMiss;
    if (t == tag && k0 == k[0] && k1 == k[1] && k2 == k[2] && k3 == k[3]) return hv;
  }
  return kMiss;
}

struct GetArgs {
  Dx x;
  const uint8_t* keys;
  uint64_t* out;
  uint32_t n;
};

__global__ __launch_bounds__(256) void k_dindex_get(GetArgs a) {
  const uint64_t maxp = a.x.mem[1];
  const uint32_t step = gridDim.x * 256;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < a.n; i += step) {
    uint64_t k[4];
    load_key(k, a.keys + 32ull * i);
    a.out[i] = probe_from(a.x, k, maxp, 0);
  }
}

__global__ void k_dindex_stats(const uint64_t* mem, uint64_t* out) {
  if (threadIdx.x < 2) out[threadIdx.x] = mem[threadIdx.x];
}

// ---- chain walk -------------------------------------------------------------
// Inputs shared by the walks.
struct ChainIn {
  const uint32_t* tokens;
  uint64_t n_tokens;
  const uint64_t* tok_off;
  const uint64_t* slot_off;
  uint64_t n_slots;
  const uint8_t* parents;
  const uint64_t* first_block;
  uint32_t n_chains;
  uint32_t bt;     // tokens per block
  uint32_t tail;   // 1: a chain's partial last block is keyed too
  MsgLen key;      // chain key message of a full block
  MsgLen fp;       // fingerprint message of a full block
  uint32_t ns[8];  // namespace digest as big-endian words
};

struct Range {
  uint64_t t0, s0, n;  // first token, first slot, blocks (full ones, then the tail if keyed)
  uint64_t slots;      // slots in the chain's range
  uint64_t full;       // full blocks among the n
  uint32_t tail_tok;   // tokens of the keyed partial last block, 0 if none
};

__device__ __forceinline__ Range chain_range(const uint64_t* tok_off, const uint64_t* slot_off,
                                             uint64_t n_tokens, uint64_t n_slots, uint32_t bt,
                                             uint32_t tail, uint32_t c) {
  Range r;
  const uint64_t a = tok_off[c], b = tok_off[c + 1];
  r.t0 = a < n_tokens ? a : n_tokens;
  const uint64_t t1 = b < r.t0 ? r.t0 : (b < n_tokens ? b : n_tokens);
  const uint64_t p = slot_off[c], q = slot_off[c + 1];
  r.s0 = p < n_slots ? p : n_slots;
  const uint64_t s1 = q < r.s0 ? r.s0 : (q < n_slots ? q : n_slots);
  r.slots = s1 - r.s0;
  const uint64_t nf = (t1 - r.t0) / bt;
  const uint32_t rem = (uint32_t)(t1 - r.t0 - nf * bt);
  r.full = nf < r.slots ? nf : r.slots;
  r.tail_tok = tail && rem && nf < r.slots ? rem : 0;
  r.n = r.full + (r.tail_tok ? 1 : 0);
  return r;
}

__device__ __forceinline__ Range chain_range(const ChainIn& in, uint32_t c) {
  return chain_range(in.tok_off, in.slot_off, in.n_tokens, in.n_slots, in.bt, in.tail, c);
}

// Tokens of block k of a chain.
__device__ __forceinline__ uint32_t block_len(const Range& r, uint64_t k, uint32_t bt) {
  return k < r.full ? bt : r.tail_tok;
}

__device__ __forceinline__ void parent_words(uint32_t (&h)[8], const ChainIn& in, uint32_t c) {
  if (in.parents) {
    const uint32_t* p = (const uint32_t*)(in.parents + 32ull * c);
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = __builtin_bswap32(p[i]);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = in.ns[i];
  }
}

__device__ __forceinline__ void chain_key(uint32_t (&out)[8], const ChainIn& in, const uint32_t (&prev)[8],
                                          const uint32_t* tok, uint32_t len) {
  const MsgLen m = len == in.bt ? in.key : msg_len(8, len);
  sha_tokens<8>(out, prev, tok, len, m.nb, m.hi, m.lo);
}

__device__ __forceinline__ void store_key(uint8_t* keys, uint64_t slot, const uint32_t (&h)[8]) {
  uint32_t* p = (uint32_t*)(keys + 32 * slot);
#pragma unroll
  for (int i = 0; i < 8; ++i) p[i] = __builtin_bswap32(h[i]);
}

// Resolves a lookup from the home slot's words (already loaded) and, past a
// mismatch in a full slot, by probing on.
__device__ __forceinline__ uint64_t resolve(const Dx& x, const uint64_t (&kw)[4],
                                            const uint64_t (&sv)[8], uint64_t maxp) {
  if (sv[0] == 0) return kMiss;
  if (sv[0] == tag_of(kw) && sv[4] == kw[0] && sv[5] == kw[1] && sv[6] == kw[2] && sv[7] == kw[3])
    return sv[2];
  return probe_from(x, kw, maxp, 1);
}

// Sequential walk over blocks [k0, r.n) of one chain, `cur` holding the key
// of block k0 - 1. Stores every key it keeps and, with an index (x.mem set),
// the handle of every hit; stops after the first miss unless all_keys.
// Iteration k computes key k while the lookup of key k-1, issued at the end
// of iteration k-1, is in flight; key k is kept only if k-1 was a hit (or
// all_keys). Returns the number of hits from k0 on.
__device__ uint64_t seq_walk(const ChainIn& in, const Dx& x, bool all_keys, const Range& r,
                             uint64_t k0, uint32_t (&cur)[8], uint8_t* keys, uint64_t* handles) {
  const bool lookup = x.mem != nullptr;
  const uint64_t maxp = lookup ? x.mem[1] : 0;
  uint64_t n_hit = 0;
  bool pending = false, missed = false;
  uint64_t kw[4] = {0, 0, 0, 0}, sv[8];
  for (uint64_t k = k0; k <= r.n; ++k) {
    uint32_t nk[8];
    const bool compute = k < r.n && (!missed || all_keys);
    if (compute) chain_key(nk, in, cur, in.tokens + r.t0 + k * in.bt, block_len(r, k, in.bt));
    if (pending) {
      const uint64_t hv = resolve(x, kw, sv, maxp);
      if (hv == kMiss) {
        missed = true;
      } else {
        handles[r.s0 + k - 1] = hv;
        ++n_hit;
      }
      pending = false;
    }
    if (!compute || (missed && !all_keys)) break;
#pragma unroll
    for (int i = 0; i < 8; ++i) cur[i] = nk[i];
    store_key(keys, r.s0 + k, cur);
    if (lookup && !missed) {
      key_words(kw, cur);
      const uint64_t* slot = slot_ptr(x, kw[1] & x.mask);
#pragma unroll
      for (int i = 0; i < 8; ++i) sv[i] = slot[i];
      pending = true;
    }
  }
  return lookup ? n_hit : r.n - k0;
}

struct ChainArgs {
  ChainIn in;
  uint32_t lanes;  // chains per wavefront
  uint32_t all_keys;
  Dx x;            // x.mem == nullptr: keys only
  uint8_t* keys;
  uint64_t* handles;
  uint32_t* hits;
};

// ---- one chain on a workgroup of four wavefronts -------------------------------
// What bounds a chain is its serial path: a lone wavefront issues one vector
// instruction every 4.4 cycles (1.86 ns, the same for every instruction the
// walk uses), so a block costs its instruction count. k_chain below issues
// about 4,700 per 16-token block (8.7 us), most of them message schedule,
// padding selection and waits for token loads. Here the serial path holds
// nothing but the 64 rounds of each compression, and the other wavefronts of
// the workgroup, each on its own SIMD, feed it through LDS. Measured: one to
// 256 chains 3.4 us per 16-token block against 8.2 (k_chain), 1,024 chains 4.1
// against 20.8; each further compression of a block 1.4 us (64-token blocks
// 7.5 against 21.6):
//   wave 0  the rounds, ten instructions each (TL_ROUND below)
//   wave 1  the message schedule of a block's first compression, the only one
//           that depends on the previous key, published eight words at a time
//   wave 2  stores the keys and looks them up; a miss stops the others
//   wave 3  tiles of 64 compressions, one per lane: the schedule plus round
//           constants of every later compression (they hold tokens and padding
//           only), and words 8..15 of first compressions
// Every wait is for a wavefront of the same workgroup (all four are resident)
// and also ends when wave 2 stops the walk. LDS accesses of one wavefront are
// performed in order, so a reader that loads a counter and then the data it
// covers, in one go, may use the data when the counter says so.
constexpr uint32_t kTileComps = 64;
constexpr uint32_t kRowWords = 68;  // a tile row: 64 words, padded against bank conflicts
constexpr uint32_t kRing = 16;      // keys between wave 0 and their readers

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Control words: read together, written one by one.
enum : uint32_t { kSchedSeq, kKeySeq, kKeyUsed, kStop, kTileReady, kTileDone, kCtlWords = 8 };

struct SeqShared {
  uint32_t tile[2][kTileComps * kRowWords];
  uint32_t sched[48];  // K + W for rounds 16..63 of a block's first compression (get_sched)
  uint32_t ring[kRing][8];
  uint32_t ctl[kCtlWords];
};

// LDS accesses that other wavefronts' accesses meet: kept in program order.
typedef __attribute__((address_space(3))) volatile uint32_t lds_u32;
typedef __attribute__((address_space(3))) volatile u32x4 lds_u32x4;
__device__ __forceinline__ uint32_t lds_get(const uint32_t* p) { return *(const lds_u32*)p; }
__device__ __forceinline__ u32x4 lds_get4(const uint32_t* p) { return *(const lds_u32x4*)p; }
__device__ __forceinline__ void lds_put(uint32_t* p, uint32_t v) { *(lds_u32*)p = v; }
__device__ __forceinline__ void lds_put4(uint32_t* p, u32x4 v) { *(lds_u32x4*)p = v; }
__device__ __forceinline__ uint32_t scalar(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Waits until control word i reaches `want` (modulo 2^32); false when the walk
// was stopped.
template <bool kSleep>
__device__ __forceinline__ bool wait_for(const SeqShared& s, uint32_t i, uint32_t want) {
  uint32_t v = scalar(lds_get(&s.ctl[i])), stop = scalar(lds_get(&s.ctl[kStop]));
  while (((int32_t)(v - want) < 0) & !stop) {
    if constexpr (kSleep) __builtin_amdgcn_s_sleep(1);
    v = scalar(lds_get(&s.ctl[i]));
    stop = scalar(lds_get(&s.ctl[kStop]));
  }
  return !stop;
}

// One round with the working variables split over lanes: lanes 0-3 and 8-11
// of a row of 16 hold (e, f, g, h), the other eight (a, b, c, d), so that one
// instruction does a step of Sigma1 and of Sigma0 (shift amounts per lane), or
// of Ch and of Maj: with u = m ? ~(x ^ y) : x, u ? y : z is Ch(x, y, z) where
// m = 0 and Maj(x, y, z) where m = ~0. X = Sigma + Ch|Maj + hk with
// hk = h + K + W in the e-lanes and 0 in the a-lanes; the new e is X + d and
// the new a is X + the e-lanes' X, the other half's value read with a rotation
// of the row by 4. w (h and d) becomes the new variable. hk is set for the
// next round from its h (now z) and its kw. A DPP operand may be read only two
// wait states after a vector instruction wrote it: the two instructions
// between X and its rotated use are those, and z and w are older than that.
#define TL_ROUND(x, y, z, w, kw_next)                                              \
  "v_alignbit_b32 %[t0], %[" x "], %[" x "], %[s0]\n\t"                             \
  "v_alignbit_b32 %[t1], %[" x "], %[" x "], %[s1]\n\t"                             \
  "v_alignbit_b32 %[t2], %[" x "], %[" x "], %[s2]\n\t"                             \
  "v_bitop3_b32 %[u], %[" x "], %[" y "], %[m] bitop3:0xd2\n\t"                     \
  "v_bitop3_b32 %[t0], %[t0], %[t1], %[t2] bitop3:0x96\n\t"                         \
  "v_bitop3_b32 %[u], %[u], %[" y "], %[" z "] bitop3:0xca\n\t"                     \
  "v_add3_u32 %[t1], %[t0], %[u], %[hk]\n\t"                                        \
  "v_add_u32_dpp %[" w "], %[" w "], %[t1] row_ror:4 row_mask:0xf bank_mask:0xf\n\t" \
  "v_add_u32_dpp %[hk], %[" z "], %[" kw_next "] quad_perm:[0,1,2,3] row_mask:0xf bank_mask:0x5\n\t" \
  "v_add_u32_dpp %[" w "], %[t1], %[t1] row_ror:4 row_mask:0xf bank_mask:0xa\n\t"
#define TL_ROUND_OPERANDS(...)                                                               \
  : [a] "+v"(v[0]), [b] "+v"(v[1]), [c] "+v"(v[2]), [d] "+v"(v[3]), [hk] "+v"(hk), [t0] "=&v"(t0), \
    [t1] "=&v"(t1), [t2] "=&v"(t2), [u] "=&v"(u)                                            \
  : [s0] "v"(s0), [s1] "v"(s1), [s2] "v"(s2), [m] "v"(m), __VA_ARGS__

// Lane constants and working variables of wave 0.
struct Rounds {
  uint32_t s0, s1, s2, m;
  uint32_t v[4];  // e-lanes: e, f, g, h; a-lanes: a, b, c, d
  uint32_t hk;    // stays 0 in the a-lanes

  __device__ __forceinline__ void init(uint32_t lane) {
    const bool a = lane >> 2 & 1;
    s0 = a ? 2 : 6;
    s1 = a ? 13 : 11;
    s2 = a ? 22 : 25;
    m = a ? 0xffffffffu : 0;
    hk = 0;
  }
  // hk of a compression's first round
  __device__ __forceinline__ void start(uint32_t kw0) {
    asm("s_nop 1\n\tv_add_u32_dpp %0, %1, %2 quad_perm:[0,1,2,3] row_mask:0xf bank_mask:0x5"
        : "+v"(hk) : "v"(v[3]), "v"(kw0));
  }
  // Four rounds; k1, k2, k3 and next are the words of the rounds after the
  // first. After four rounds v is in its first order again.
  __device__ __forceinline__ void four(uint32_t k1, uint32_t k2, uint32_t k3, uint32_t next) {
    uint32_t t0, t1, t2, u;
    asm(TL_ROUND("a", "b", "c", "d", "k1") TL_ROUND("d", "a", "b", "c", "k2") TL_ROUND("c", "d", "a", "b", "k3")
            TL_ROUND("b", "c", "d", "a", "k4")
        TL_ROUND_OPERANDS([k1] "v"(k1), [k2] "v"(k2), [k3] "v"(k3), [k4] "v"(next)));
  }
  // The first three and the last of four rounds, for a `next` that comes late.
  __device__ __forceinline__ void three(uint32_t k1, uint32_t k2, uint32_t k3) {
    uint32_t t0, t1, t2, u;
    asm(TL_ROUND("a", "b", "c", "d", "k1") TL_ROUND("d", "a", "b", "c", "k2") TL_ROUND("c", "d", "a", "b", "k3")
        TL_ROUND_OPERANDS([k1] "v"(k1), [k2] "v"(k2), [k3] "v"(k3)));
  }
  __device__ __forceinline__ void fourth(uint32_t next) {
    uint32_t t0, t1, t2, u;
    asm(TL_ROUND("b", "c", "d", "a", "k4") TL_ROUND_OPERANDS([k4] "v"(next)));
  }
};

__device__ __forceinline__ void get8(uint32_t (&out)[8], const uint32_t* p) {
  const u32x4 a = lds_get4(p), b = lds_get4(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[i] = a[i];
    out[4 + i] = b[i];
  }
}

// Eight words of wave 1's schedule: the even ones come first.
__device__ __forceinline__ void get_sched(uint32_t (&out)[8], const uint32_t* p) {
  const u32x4 a = lds_get4(p), b = lds_get4(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[2 * i] = a[i];
    out[2 * i + 1] = b[i];
  }
}

// Wave 0: the rounds of every compression of the chain, in order.
__device__ __forceinline__ void seq_rounds(SeqShared& s, const ChainIn& in, const Range& r, const uint32_t (&parent)[8],
                                           uint32_t lane) {
  Rounds R;
  R.init(lane);
  const bool a_lane = lane >> 2 & 1;
  uint32_t key[4], iv[4];  // e-lanes: words 4..7, a-lanes: words 0..3
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    key[i] = pick(R.m, parent[i], parent[4 + i]);
    iv[i] = pick(R.m, tl::kSha256IV[i], tl::kSha256IV[4 + i]);
  }
  uint32_t at = 0, tiles = 0;  // place in the current tile, tiles begun
  uint32_t used = 0;           // keys that wave 2 has taken, as last seen
  if (!wait_for<false>(s, kTileReady, 1)) return;
  for (uint64_t k = 0; k < r.n; ++k) {
    const uint32_t nb = k < r.full ? in.key.nb : msg_len(8, r.tail_tok).nb;
    uint32_t h[4], stop = 0;
    for (uint32_t c = 0; c < nb; ++c) {
      if (at == kTileComps) {
        at = 0;
        ++tiles;
        if (lane == 0) lds_put(&s.ctl[kTileDone], tiles);
        if (!wait_for<false>(s, kTileReady, tiles + 1)) return;
      }
      const uint32_t* row = &s.tile[tiles & 1][at * kRowWords];
      ++at;
      uint32_t p[8], q[8];
      if (c == 0) {
        get8(q, row + 8);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          h[i] = R.v[i] = iv[i];
          p[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key[i], 0x124, 0xf, 0xf, false) + tl::kSha256K[i];
          p[4 + i] = key[i] + tl::kSha256K[4 + i];
        }
        R.start(p[0]);
        R.four(p[1], p[2], p[3], p[4]);
        R.four(p[5], p[6], p[7], q[0]);
        // rounds 8..63, eight at a time, while the next eight words are on their way
#pragma unroll
        for (int g = 1; g < 8; ++g) {
          uint32_t(&cur)[8] = g & 1 ? q : p;
          uint32_t(&nxt)[8] = g & 1 ? p : q;
          const uint32_t* words = &s.sched[8 * (g - 1)];
          const uint32_t want = 6 * (uint32_t)k + g;
          u32x4 ctl;
          if (g > 2 && g < 7) {  // wave 1 is that far ahead by now
            ctl = lds_get4(s.ctl);
            get_sched(nxt, words);
          }
          R.four(cur[1], cur[2], cur[3], cur[4]);
          if (g == 7) {
            R.four(cur[5], cur[6], cur[7], 0);
            break;
          }
          if (g <= 2) {
            ctl = lds_get4(s.ctl);
            get_sched(nxt, words);
          }
          R.three(cur[5], cur[6], cur[7]);
          if (__builtin_expect((int32_t)(scalar(ctl[kSchedSeq]) - want) < 0, 0)) {
            do {
              ctl = lds_get4(s.ctl);
              get_sched(nxt, words);
              stop = scalar(ctl[kStop]);
            } while (((int32_t)(scalar(ctl[kSchedSeq]) - want) < 0) & !stop);
          }
          if (g == 6) used = scalar(ctl[kKeyUsed]);
          R.fourth(nxt[0]);
        }
        if (stop) return;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) R.v[i] = h[i];
        get8(p, row);
        get8(q, row + 8);
        R.start(p[0]);
#pragma unroll
        for (int g = 0; g < 8; ++g) {
          uint32_t(&cur)[8] = g & 1 ? q : p;
          uint32_t(&nxt)[8] = g & 1 ? p : q;
          R.four(cur[1], cur[2], cur[3], cur[4]);
          R.four(cur[5], cur[6], cur[7], g < 7 ? nxt[0] : 0);
          if (g < 6) get8(cur, row + 8 * (g + 2));
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) h[i] += R.v[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) key[i] = h[i];
    if ((uint32_t)k - used >= kRing && !wait_for<false>(s, kKeyUsed, (uint32_t)k + 1 - kRing)) return;
    if ((lane & ~4u) == 0) lds_put4(&s.ring[k % kRing][a_lane ? 0 : 4], u32x4{key[0], key[1], key[2], key[3]});
    if (lane == 0) lds_put(&s.ctl[kKeySeq], (uint32_t)k + 1);
  }
}

// Row of 16 lanes rotated by 4: swaps the two kinds of lanes.
__device__ __forceinline__ uint32_t other_lanes(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, true);
}

// Wave 1: words 16..63 of every block's first compression, plus the round
// constants. Words 0..7 are the previous key; the tile row holds words 8..15.
// It has to stay ahead of wave 0's rounds, so it makes two words at a time:
// P[i] is word 2i in the e-lanes (lanes 0-3 and 8-11 of a row) and word 2i + 1
// in the others, Q[i] words 2i - 1 and 2i, and
//   P[i] = ssig1(P[i-1]) + Q[i-3] + ssig0(Q[i-7]) + P[i-8].
// That is 13 instructions for two words against 22 one by one.
__device__ __forceinline__ void seq_schedule(SeqShared& s, const ChainIn& in, const Range& r,
                                             uint32_t lane) {
  const uint64_t nb = in.key.nb;
  const bool odd = lane >> 2 & 1;  // the lanes of the odd words
  const uint32_t m = odd ? 0xffffffffu : 0;
  uint32_t K[32];
#pragma unroll
  for (int i = 8; i < 32; ++i) K[i] = tl::kSha256K[2 * i] ^ (m & (tl::kSha256K[2 * i] ^ tl::kSha256K[2 * i + 1]));
  uint64_t q = 0;  // the block's first compression
  for (uint64_t k = 0; k < r.n; ++k, q += nb) {
    if (!wait_for<false>(s, kTileReady, (uint32_t)(q / kTileComps) + 1)) return;
    uint32_t lo[8], hi[8], P[8], Q[8];
    get8(hi, &s.tile[q / kTileComps & 1][(uint32_t)(q % kTileComps) * kRowWords]);
#pragma unroll
    for (int i = 4; i < 8; ++i) P[i] = pick(m, hi[2 * i - 7], hi[2 * i - 8]);
#pragma unroll
    for (int i = 5; i < 8; ++i) Q[i] = pick(m, hi[2 * i - 8], hi[2 * i - 9]);
    uint32_t seq, stop;
    do {
      const u32x4 ctl = lds_get4(s.ctl);
      get8(lo, s.ring[(k - 1) % kRing]);
      seq = scalar(ctl[kKeySeq]);
      stop = scalar(ctl[kStop]);
    } while (((int32_t)(seq - (uint32_t)k) < 0) & !stop);
    if (stop) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) P[i] = pick(m, lo[2 * i + 1], lo[2 * i]);
#pragma unroll
    for (int i = 1; i < 4; ++i) Q[i] = pick(m, lo[2 * i], lo[2 * i - 1]);
    Q[4] = pick(m, hi[0], lo[7]);
#pragma unroll
    for (int t = 8; t < 32; t += 4) {
      u32x4 kw;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = t + j;
        const uint32_t x = ssig1(P[(i + 7) & 7]) + (P[i & 7] + ssig0(Q[(i + 1) & 7]) + Q[(i + 5) & 7]);
        // Q[i]: word 2i - 1 from the odd lanes' P[i-1], word 2i from the even lanes' P[i]
        const uint32_t before = other_lanes(P[(i + 7) & 7]), now = other_lanes(x);
        P[i & 7] = x;
        Q[i & 7] = pick(m, now, before);
        kw[j] = x + K[i];
      }
      // eight words: the even ones, then the odd ones
      if ((lane & ~4u) == 0) lds_put4(&s.sched[2 * (t - 8) + (odd ? 4 : 0)], kw);
      if (lane == 0) lds_put(&s.ctl[kSchedSeq], 6 * (uint32_t)k + (t - 8) / 4 + 1);
    }
  }
}

// Wave 2: keys to memory, lookups, hits. Keys are stored in order and only
// while every block before them was found (or all_keys), as in seq_walk.
__device__ __forceinline__ void seq_lookup(SeqShared& s, const Dx& x, bool all_keys, const Range& r, uint8_t* keys,
                                           uint64_t* handles, uint32_t* hits, uint32_t lane) {
  const bool lookup = x.mem != nullptr;
  const uint64_t maxp = lookup ? x.mem[1] : 0;
  uint64_t n_hit = 0;
  bool missed = false;
  for (uint64_t k = 0; k < r.n; ++k) {
    wait_for<true>(s, kKeySeq, (uint32_t)k + 1);
    uint32_t h[8];
    get8(h, s.ring[k % kRing]);
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) mine = lane == (uint32_t)i ? h[i] : mine;
    if (lane < 8) ((uint32_t*)(keys + 32 * (r.s0 + k)))[lane] = __builtin_bswap32(mine);
    if (lane == 0) lds_put(&s.ctl[kKeyUsed], (uint32_t)k + 1);  // after the reads of the ring
    if (lookup && !missed) {
      uint64_t kw[4];
      key_words(kw, h);
      const uint64_t hv = probe_from(x, kw, maxp, 0);
      if (hv == kMiss) {
        missed = true;
        if (!all_keys) break;
      } else {
        if (lane == 0) handles[r.s0 + k] = hv;
        ++n_hit;
      }
    }
  }
  if (lane == 0) lds_put(&s.ctl[kStop], 1);
  if (lookup) {
    for (uint64_t j = n_hit + lane; j < r.n; j += 64) handles[r.s0 + j] = kMiss;
  }
  if (lane == 0) *hits = (uint32_t)(lookup ? n_hit : r.n);
}

// Wave 3: tiles of 64 compressions ahead of wave 0, one per lane.
__device__ __forceinline__ void seq_tiles(SeqShared& s, const ChainIn& in, const Range& r, uint32_t lane) {
  const uint64_t nb = in.key.nb;
  const uint64_t total = r.full * nb + (r.tail_tok ? msg_len(8, r.tail_tok).nb : 0);
  for (uint64_t t = 0; t * kTileComps < total; ++t) {
    if (t >= 2 && !wait_for<true>(s, kTileDone, (uint32_t)t - 1)) return;
    const uint64_t q = t * kTileComps + lane;
    if (q < total) {
      const uint64_t k = q / nb;
      const uint32_t c = (uint32_t)(q - k * nb), len = block_len(r, k, in.bt);
      const MsgLen m = len == in.bt ? in.key : msg_len(8, len);
      const uint32_t* tok = in.tokens + r.t0 + k * in.bt;
      const uint32_t last = 16 * m.nb - 1;
      uint32_t w[16], hi[8];
#pragma unroll
      for (int i = 0; i < 16; ++i) w[i] = tok[min(16 * c + i - 8, len - 1)];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t g = 16 * c + i, j = g - 8;
        w[i] = j < len ? __builtin_bswap32(w[i])
                       : j == len ? 0x80000000u : g == last ? m.lo : g == last - 1 ? m.hi : 0;
      }
      if (c == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = 0;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) hi[i] = w[8 + i];
      uint32_t* row = &s.tile[t & 1][lane * kRowWords];
#pragma unroll
      for (int i = 0; i < 64; i += 4) {
        u32x4 kw;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int g = i + j;
          if (g >= 16) w[g & 15] += ssig1(w[(g + 14) & 15]) + w[(g + 9) & 15] + ssig0(w[(g + 1) & 15]);
          kw[j] = w[g & 15] + tl::kSha256K[g];
        }
        *(u32x4*)(row + i) = kw;
      }
      if (c == 0) {  // words 8..15 as they are, for wave 1
        *(u32x4*)(row) = u32x4{hi[0], hi[1], hi[2], hi[3]};
        *(u32x4*)(row + 4) = u32x4{hi[4], hi[5], hi[6], hi[7]};
      }
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);  // the tile is written before it is announced
    if (lane == 0) lds_put(&s.ctl[kTileReady], (uint32_t)t + 1);
  }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_chain_waves(ChainArgs a) {
  __shared__ __align__(16) SeqShared s;
  const uint32_t lane = threadIdx.x & 63, wave = scalar(threadIdx.x >> 6), c = blockIdx.x;
  const Range r = chain_range(a.in, c);
  uint32_t parent[8];
  parent_words(parent, a.in, c);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) s.ring[kRing - 1][i] = parent[i];  // the key before block 0's
  }
  if (threadIdx.x < kCtlWords) s.ctl[threadIdx.x] = 0;
  __syncthreads();
  if (wave == 2) {
    seq_lookup(s, a.x, a.all_keys != 0, r, a.keys, a.handles, &a.hits[c], lane);
  } else if (wave == 3) {
    seq_tiles(s, a.in, r, lane);
  } else if (r.n && wave == 0) {
    __builtin_amdgcn_s_setprio(3);
    seq_rounds(s, a.in, r, parent, lane);
  } else if (r.n) {
    __builtin_amdgcn_s_setprio(2);
    seq_schedule(s, a.in, r, lane);
  }
}

__global__ __launch_bounds__(64) void k_chain(ChainArgs a) {
  const uint32_t lane = threadIdx.x;
  if (lane >= a.lanes) return;
  const uint32_t c = blockIdx.x * a.lanes + lane;
  if (c >= a.in.n_chains) return;
  const Range r = chain_range(a.in, c);
  uint32_t cur[8];
  parent_words(cur, a.in, c);
  const uint64_t n_hit = seq_walk(a.in, a.x, a.all_keys != 0, r, 0, cur, a.keys, a.handles);
  if (a.x.mem) {
    for (uint64_t j = n_hit; j < r.n; ++j) a.handles[r.s0 + j] = kMiss;
  }
  a.hits[c] = (uint32_t)n_hit;
}

// ---- block fingerprints and the verified parallel walk -----------------------
// Fingerprint of a block: SHA-256(namespace digest | u64 LE position | token
// ids), the key of the token index that proposes, for a block of a request,
// the chain key of a stored block with the same tokens at the same position.
__device__ __forceinline__ void fingerprint(uint32_t (&out)[8], const ChainIn& in, uint64_t pos,
                                            const uint32_t* tok, uint32_t len) {
  uint32_t pre[10];
#pragma unroll
  for (int i = 0; i < 8; ++i) pre[i] = in.ns[i];
  pre[8] = __builtin_bswap32((uint32_t)pos);
  pre[9] = __builtin_bswap32((uint32_t)(pos >> 32));
  const MsgLen m = len == in.bt ? in.fp : msg_len(10, len);
  sha_tokens<10>(out, pre, tok, len, m.nb, m.hi, m.lo);
}

struct FpArgs {
  ChainIn in;
  const uint32_t* tokens;    // [n][bt]
  const uint64_t* pos;       // [n]
  const uint32_t* n_tokens;  // [n] or null (all full); a count outside [1, bt] counts as bt
  uint8_t* out;              // [n][32]
  uint32_t n;
};

__global__ __launch_bounds__(256) void k_fingerprint(FpArgs a) {
  const uint32_t step = gridDim.x * 256;
  for (uint32_t b = blockIdx.x * 256 + threadIdx.x; b < a.n; b += step) {
    uint32_t f[8];
    uint32_t len = a.n_tokens ? a.n_tokens[b] : a.in.bt;
    if (len < 1 || len > a.in.bt) len = a.in.bt;
    fingerprint(f, a.in, a.pos[b], a.tokens + (uint64_t)b * a.in.bt, len);
    store_key(a.out, b, f);
  }
}

struct ParArgs {
  ChainIn in;
  Dx x;                  // key index
  Dx t;                  // token index: fingerprint -> handle
  const uint8_t* hkeys;  // [n_handles][32] chain key of each handle's record
  uint64_t n_handles;
  uint8_t* keys;
  uint64_t* handles;
  uint32_t* hits;
};

// The parallel walk. For block k the token index proposes cand_k, the key a
// stored block with the same tokens at the same position has; every block then
// computes c_k = SHA-256(cand_{k-1} | tokens_k) (cand_{-1} = the chain's
// parent) and looks c_k up in the key index, all independently. If cand_j =
// c_j for every j < k, induction from c_0 (computed from the true parent)
// makes c_0..c_k the true chain keys, so the walk is exact up to the first
// block m where c_m is not in the index (flag 1: reuse ends at m) or cand_m !=
// c_m (flag 2: c_m is true and a hit, but c_{m+1} is not known: the chain goes
// on sequentially from m+1). Results equal the sequential walk's; candidates
// only decide how much of it runs in parallel.
//
// A tile is kTileBlocks blocks of one chain on one wavefront: lane 0 makes the
// candidate of the block before the tile (in step with the others' own), lanes
// 1.. are the tile's blocks. What bounds a tile is the instruction count of
// its four SHA-256 compressions on one lane (about 1,400 each, 1.86 ns per
// instruction for a wavefront that has its SIMD to itself), so a call's tiles
// go to as many SIMDs as there are: the corpus's one chain of 6,062 blocks is
// 97 tiles and takes 25 us (87 us as six tiles of 1,024 blocks, each on one
// compute unit). A compression's token loads go out together, a slot of an
// index is one request (28.7 us with loads and compares one after another).
constexpr uint32_t kTileBlocks = 63;

struct TileShared {
  uint32_t cand[64][8];  // candidate of the block before the tile, then the tile's blocks'
  uint32_t has[64];
};

// LDS written by a wavefront is seen by its own later reads.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Walks blocks [t0, t0 + kTileBlocks) of chain c; returns the tile's first
// flagged block as (block << 2 | flag), or all ones. One wavefront, whose s is.
__device__ uint64_t walk_tile(TileShared& s, const ParArgs& a, const Range& r, uint32_t c, uint64_t t0, uint64_t maxp,
                              uint64_t tmaxp) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t k = t0 + lane - 1;  // lane 0 of the first tile: the parent
  const bool live = k < r.n;
  const uint32_t* tok = a.in.tokens + r.t0 + k * a.in.bt;
  const uint32_t len = block_len(r, k, a.in.bt);
  uint32_t cand[8], hc = 0;
  if (live) {
    uint32_t f[8];
    fingerprint(f, a.in, (a.in.first_block ? a.in.first_block[c] : 0) + k, tok, len);
    uint64_t fw[4];
    key_words(fw, f);
    const uint64_t h = probe_from(a.t, fw, tmaxp, 0);
    if (h < a.n_handles) {
      const uint32_t* hk = (const uint32_t*)(a.hkeys + 32 * h);
#pragma unroll
      for (int i = 0; i < 8; ++i) cand[i] = __builtin_bswap32(hk[i]);
      hc = 1;
    }
  }
  if (t0 == 0 && lane == 0) {
    parent_words(cand, a.in, c);
    hc = 1;
  }
  wave_sync();  // the last tile's reads come first
  if (hc) {
#pragma unroll
    for (int i = 0; i < 8; ++i) s.cand[lane][i] = cand[i];
  }
  s.has[lane] = hc;
  wave_sync();
  uint32_t flag = 0;
  if (live && lane && s.has[lane - 1]) {
    uint32_t prev[8], ck[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) prev[i] = s.cand[lane - 1][i];
    chain_key(ck, a.in, prev, tok, len);
    store_key(a.keys, r.s0 + k, ck);
    uint64_t kw[4];
    key_words(kw, ck);
    const uint64_t hv = probe_from(a.x, kw, maxp, 0);
    a.handles[r.s0 + k] = hv;
    bool same = hc != 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) same = same && cand[i] == ck[i];
    flag = hv == kMiss ? 1u : (same ? 0u : 2u);
  }
  // (a block without a candidate for its predecessor is never the first
  // flagged one: that predecessor is flagged, in this tile or before)
  const uint64_t any = __ballot(flag != 0);
  if (!any) return ~0ull;
  const int at = __builtin_ctzll(any);
  return (t0 + at - 1) << 2 | (uint32_t)__builtin_amdgcn_readlane((int)flag, at);
}

// Hits of a chain whose first flagged block is known; for a disagreement at
// block m the chain goes on sequentially from m + 1, after the key that the
// walk stored for m. Handles past the last hit become misses.
template <uint32_t kThreads>
__device__ void finish_chain(const ParArgs& a, const Range& r, uint32_t c, uint64_t first, uint64_t* seq_hits) {
  const uint32_t tid = threadIdx.x;
  const uint64_t stop = first >> 2;
  uint64_t n_hit = first == ~0ull ? r.n : stop;
  if (first != ~0ull && (first & 3) == 2) {
    if (tid == 0) {
      const uint32_t* sk = (const uint32_t*)(a.keys + 32 * (r.s0 + stop));
      uint32_t cur[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) cur[i] = __builtin_bswap32(sk[i]);
      *seq_hits = stop + 1 + seq_walk(a.in, a.x, false, r, stop + 1, cur, a.keys, a.handles);
    }
    __syncthreads();
    n_hit = *seq_hits;
  }
  for (uint64_t j = n_hit + tid; j < r.n; j += kThreads) a.handles[r.s0 + j] = kMiss;
  __syncthreads();  // every thread has read what it needs of hits[c] and *seq_hits
  if (tid == 0) a.hits[c] = (uint32_t)n_hit;
}

// A workgroup walks whole chains, a tile per wavefront at a time.
constexpr uint32_t kParWaves = 4;

__global__ __launch_bounds__(64 * kParWaves) void k_chain_par(ParArgs a) {
  __shared__ TileShared s[kParWaves];
  __shared__ uint64_t flagged[kParWaves];
  __shared__ uint64_t seq_hits;
  const uint32_t wave = scalar(threadIdx.x >> 6);
  const uint64_t maxp = a.x.mem[1], tmaxp = a.t.mem[1];
  for (uint32_t c = blockIdx.x; c < a.in.n_chains; c += gridDim.x) {
    const Range r = chain_range(a.in, c);
    uint64_t first = ~0ull;
    for (uint64_t base = 0; base < r.n && first == ~0ull; base += kParWaves * kTileBlocks) {
      const uint64_t t0 = base + wave * kTileBlocks;
      const uint64_t f = t0 < r.n ? walk_tile(s[wave], a, r, c, t0, maxp, tmaxp) : ~0ull;
      if ((threadIdx.x & 63) == 0) flagged[wave] = f;
      __threadfence_block();  // thread 0 may read a key that another thread stored
      __syncthreads();
#pragma unroll
      for (uint32_t w = 0; w < kParWaves; ++w) first = min(first, flagged[w]);
      __syncthreads();
    }
    finish_chain<64 * kParWaves>(a, r, c, first, &seq_hits);
  }
}

// The same with a chain's tiles on `spread` wavefronts of their own. Pass 1
// runs the tiles; a tile's first flagged block k goes to hits[c] as
// min(k << 2 | flag) (k_par_init sets every hits[c] to all ones first). Tiles
// after a block already flagged are skipped: only the first flag counts. Pass
// 2 (k_chain_par_finish, one workgroup per chain) turns hits[c] into the hit
// count. Results equal k_chain_par's.
__global__ __launch_bounds__(256) void k_par_init(uint32_t* hits, uint32_t n) {
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) hits[i] = 0xffffffffu;
}

__global__ __launch_bounds__(64) void k_chain_par_tiles(ParArgs a, uint32_t spread) {
  __shared__ TileShared s;
  const uint64_t maxp = a.x.mem[1], tmaxp = a.t.mem[1];
  const uint32_t c = blockIdx.x % a.in.n_chains;
  const Range r = chain_range(a.in, c);
  const uint64_t t_first = (uint64_t)(blockIdx.x / a.in.n_chains) * kTileBlocks;
  for (uint64_t t0 = t_first; t0 < r.n; t0 += (uint64_t)spread * kTileBlocks) {
    if (t0 != t_first) {  // (the first tiles all start at the same time)
      const uint32_t seen = scalar(__hip_atomic_load(&a.hits[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      if (seen != 0xffffffffu && (seen >> 2) < t0) return;
    }
    const uint64_t first = walk_tile(s, a, r, c, t0, maxp, tmaxp);
    if (first != ~0ull) {
      if (threadIdx.x == 0) atomicMin(&a.hits[c], (uint32_t)first);
      return;
    }
  }
}

__global__ __launch_bounds__(256) void k_chain_par_finish(ParArgs a) {
  __shared__ uint64_t seq_hits;
  for (uint32_t c = blockIdx.x; c < a.in.n_chains; c += gridDim.x) {
    const uint32_t f = a.hits[c];  // final: pass 1 has completed
    finish_chain<256>(a, chain_range(a.in, c), c, f == 0xffffffffu ? ~0ull : f, &seq_hits);
    __syncthreads();
  }
}

// ---- staging of tl_load's inputs --------------------------------------------
struct StageArgs {
  const uint32_t* tokens;
  uint64_t n_tokens;
  const uint64_t* tok_off;
  const uint64_t* slot_off;
  uint64_t n_slots;
  const uint64_t* first_block;
  uint32_t n_chains;
  uint32_t bt;
  uint32_t ppb;
  uint32_t page_tokens;
  uint32_t n_groups;
  uint32_t tail;               // chains key their partial last block
  uint32_t* n_tokens_out;      // [n_slots] tokens per slot, or null
  const uint32_t* hits;
  const uint64_t* handles;
  const uint64_t* hptr;
  const uint64_t* hlen;
  uint64_t n_handles;
  uint64_t* rec_ptrs;
  uint64_t* rec_lens;
  uint64_t* bidx;
  uint32_t* tokens_out;
  const int32_t* tables_in;  // null: page j of slot q is q * ppb + j
  int32_t* tables_out;
};

__device__ __forceinline__ bool stage_hit(const StageArgs& a, uint64_t slot, uint64_t k,
                                          uint64_t hits, uint64_t* h) {
  if (k >= hits) return false;
  *h = a.handles[slot];
  return *h < a.n_handles;
}

// Workgroups of kStageThreads: blockIdx.x strides over chains, and the
// gridDim.y workgroups of a chain take equal contiguous parts of its slots
// (with their token ids and table entries), so that a few long chains still
// spread over many compute units.
constexpr uint32_t kStageThreads = 256;

__global__ __launch_bounds__(kStageThreads) void k_chain_stage(StageArgs a) {
  const uint32_t tid = threadIdx.x;
  for (uint32_t c = blockIdx.x; c < a.n_chains; c += gridDim.x) {
    const Range r = chain_range(a.tok_off, a.slot_off, a.n_tokens, a.n_slots, a.bt, a.tail, c);
    const uint64_t hits_raw = a.hits[c];
    const uint64_t hits = hits_raw < r.n ? hits_raw : r.n;
    const uint64_t first = a.first_block ? a.first_block[c] : 0;
    // this workgroup's slots [k0, k1) of the chain's r.slots
    const uint64_t k0 = r.slots * blockIdx.y / gridDim.y, k1 = r.slots * (blockIdx.y + 1) / gridDim.y;
    for (uint64_t k = k0 + tid; k < k1; k += kStageThreads) {
      const uint64_t q = r.s0 + k;
      uint64_t h = 0;
      const bool hit = stage_hit(a, q, k, hits, &h);
      a.rec_ptrs[q] = hit ? a.hptr[h] : 0;
      a.rec_lens[q] = hit ? a.hlen[h] : 0;
      a.bidx[q] = first + k;
      if (a.n_tokens_out) a.n_tokens_out[q] = k == r.full && r.tail_tok ? r.tail_tok : a.bt;
    }
    if (a.tokens_out) {
      const uint64_t have = r.full * a.bt + r.tail_tok;
      uint32_t* dst = a.tokens_out + r.s0 * a.bt;
      const uint32_t* src = a.tokens + r.t0;
      for (uint64_t e = k0 * a.bt + tid; e < k1 * a.bt; e += kStageThreads) dst[e] = e < have ? src[e] : 0;
    }
    if (a.tables_out) {
      const uint64_t row = a.n_slots * a.ppb;
      // a restored partial block restores only the pages holding its tokens
      const uint64_t tail_pages = (r.tail_tok + a.page_tokens - 1) / a.page_tokens;
      for (uint64_t e = k0 * a.ppb + tid; e < k1 * a.ppb; e += kStageThreads) {
        const uint64_t k = e / a.ppb, j = e - k * a.ppb, at = r.s0 * a.ppb + e;
        uint64_t h = 0;
        const bool hit = stage_hit(a, r.s0 + k, k, hits, &h) && !(r.tail_tok && k == r.full && j >= tail_pages);
        for (uint32_t g = 0; g < a.n_groups; ++g) {
          const uint64_t i = (uint64_t)g * row + at;
          a.tables_out[i] = !hit ? -1 : (a.tables_in ? a.tables_in[i] : (int32_t)at);
        }
      }
    }
  }
}

int launched() { return hipGetLastError() == hipSuccess ? TL_OK : TL_EDEVICE; }

uint32_t grid_for(uint64_t n, uint32_t per, uint32_t cap) {
  const uint64_t g = (n + per - 1) / per;
  return (uint32_t)(g < cap ? (g ? g : 1) : cap);
}

int sm_count() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    return 256;
  return cus;
}

}  // namespace

namespace tl {

int launch_dindex_clear(void* mem, uint64_t capacity, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const uint64_t words = kHeaderWords + capacity * kSlotWords;
  (void)hipGetLastError();
  {
    TimedLaunch t(TL_KERNEL_INDEX, stream);
    hipLaunchKernelGGL(k_dindex_clear, dim3(grid_for(words, 256, 8192)), dim3(256), 0, s,
                       (uint64_t*)mem, words);
  }
  return launched();
}

int launch_dindex_put(void* mem, uint64_t capacity, void* stream, size_t n, const uint8_t* d_keys,
                      const uint64_t* d_handles, uint8_t* d_status, uint32_t* d_ws) {
  hipStream_t s = (hipStream_t)stream;
  PutArgs a;
  a.x.mem = (uint64_t*)mem;
  a.x.mask = capacity - 1;
  a.keys = d_keys;
  a.handles = d_handles;
  a.status = d_status;
  a.target = d_ws;
  a.n = (uint32_t)n;
  const uint32_t g = grid_for(n, 256, 1u << 16);
  (void)hipGetLastError();
  if (n <= kPutThreads) {
    TimedLaunch t(TL_KERNEL_INDEX, stream);
    hipLaunchKernelGGL(k_dindex_put, dim3(1), dim3((uint32_t)(n + 63) / 64 * 64), 0, s, a);
    return launched();
  }
  {
    TimedLaunch t(TL_KERNEL_INDEX, stream);
    hipLaunchKernelGGL(k_dindex_claim, dim3(g), dim3(256), 0, s, a);
  }
  {
    TimedLaunch t(TL_KERNEL_INDEX, stream);
    hipLaunchKernelGGL(k_dindex_vote, dim3(g), dim3(256), 0, s, a);
  }
  {
    TimedLaunch t(TL_KERNEL_INDEX, stream);
    hipLaunchKernelGGL(k_dindex_publish, dim3(g), dim3(256), 0, s, a);
  }
  return launched();
}

int launch_dindex_get(const void* mem, uint64_t capacity, void* stream, size_t n,
                      const uint8_t* d_keys, uint64_t* d_out) {
  hipStream_t s = (hipStream_t)stream;
  GetArgs a;
  a.x.mem = (uint64_t*)mem;
  a.x.mask = capacity - 1;
  a.keys = d_keys;
  a.out = d_out;
  a.n = (uint32_t)n;
  (void)hipGetLastError();
  {
    TimedLaunch t(TL_KERNEL_INDEX, stream);
    hipLaunchKernelGGL(k_dindex_get, dim3(grid_for(n, 256, 1u << 16)), dim3(256), 0, s, a);
  }
  return launched();
}

int launch_dindex_stats(const void* mem, void* stream, uint64_t* d_out) {
  hipStream_t s = (hipStream_t)stream;
  (void)hipGetLastError();
  {
    TimedLaunch t(TL_KERNEL_INDEX, stream);
    hipLaunchKernelGGL(k_dindex_stats, dim3(1), dim3(64), 0, s, (const uint64_t*)mem, d_out);
  }
  return launched();
}

namespace {
ChainIn chain_in(const tl_ctx* ctx, size_t n_chains, const tl_chains* ch, uint32_t flags) {
  ChainIn in;
  in.tokens = ch ? ch->d_tokens : nullptr;
  in.n_tokens = ch ? ch->n_tokens : 0;
  in.tok_off = ch ? ch->d_tok_off : nullptr;
  in.slot_off = ch ? ch->d_slot_off : nullptr;
  in.n_slots = ch ? ch->n_slots : 0;
  in.parents = ch ? ch->d_parents : nullptr;
  in.first_block = ch ? ch->d_first_block : nullptr;
  in.n_chains = (uint32_t)n_chains;
  in.bt = ctx->geo.block_tokens;
  in.tail = (flags & TL_CHAIN_TAIL) ? 1 : 0;
  in.key = msg_len(8, in.bt);
  in.fp = msg_len(10, in.bt);
  for (int i = 0; i < 8; ++i)
    in.ns[i] = (uint32_t)ctx->ns[4 * i] << 24 | (uint32_t)ctx->ns[4 * i + 1] << 16 |
               (uint32_t)ctx->ns[4 * i + 2] << 8 | ctx->ns[4 * i + 3];
  return in;
}
}  // namespace

// Whether each chain gets a workgroup (k_chain_waves) rather than a lane
// (k_chain). A compute unit holds four such workgroups, and each of them begins
// with a tile of schedules, so with many chains it takes work to be worth it.
// Up to 8 chains per compute unit it always is: 2,048 chains of one key 16.7 us
// and 16.4, of 2 28.4 and 42.7, of 65 0.70 ms and 1.66. Up to 16 with 8
// compressions per chain that are sure to be made (a lookup may end at its second
// key): 4,096 chains of 4 keys of 16 tokens (8 compressions) 92 us and 95, of 17
// 354 and 433, of 2 of 64 tokens (looked up, none stored) 106 and 132; but of one
// key 31.2 and 16.4 us, of 2 53.0 and 42.5, of 5 keys of 5 tokens 77.9 and 70.0,
// 17 of 16 tokens looked up and none stored 65.3 and 56.1. Beyond that lanes are
// faster: 8,192 chains of 64 blocks 2.47 ms and 1.46.
bool chain_waves(const ChainIn& in, bool ends_early) {
  const uint64_t cus = (uint64_t)sm_count();
  if (in.n_chains <= 8 * cus) return true;
  uint64_t keys = in.n_slots / in.n_chains;
  if (ends_early) keys = std::min<uint64_t>(keys, 2);
  // (slots may be more than there are tokens for: 16 of them to a compression, and one for the key)
  const uint64_t work = std::min(keys * in.key.nb, in.n_tokens / in.n_chains / 16 + keys);
  return in.n_chains <= 16 * cus && work >= 8;
}

int launch_chain(const tl_ctx* ctx, void* stream, size_t n_chains, const tl_chains* ch,
                 const void* index_mem, uint64_t capacity, uint32_t flags, uint8_t* d_keys,
                 uint64_t* d_handles, uint32_t* d_hits) {
  hipStream_t s = (hipStream_t)stream;
  ChainArgs a;
  a.in = chain_in(ctx, n_chains, ch, flags);
  a.all_keys = (flags & TL_CHAIN_ALL_KEYS) ? 1 : 0;
  a.x.mem = (uint64_t*)index_mem;
  a.x.mask = index_mem ? capacity - 1 : 0;
  a.keys = d_keys;
  a.handles = d_handles;
  a.hits = d_hits;
  a.lanes = 0;
  (void)hipGetLastError();
  if (chain_waves(a.in, index_mem && !a.all_keys)) {
    TimedLaunch t(TL_KERNEL_CHAIN, stream);
    hipLaunchKernelGGL(k_chain_waves, dim3((uint32_t)n_chains), dim3(256), 0, s, a);
  } else {
    // chains spread over the SIMDs, up to 64 on a wavefront's lanes
    const uint64_t simds = 4ull * (uint64_t)sm_count();
    a.lanes = (uint32_t)std::min<uint64_t>((n_chains + simds - 1) / simds, 64);
    TimedLaunch t(TL_KERNEL_CHAIN, stream);
    hipLaunchKernelGGL(k_chain, dim3((uint32_t)((n_chains + a.lanes - 1) / a.lanes)), dim3(64), 0, s, a);
  }
  return launched();
}

int launch_chain_par(const tl_ctx* ctx, void* stream, size_t n_chains, const tl_chains* ch,
                     const void* index_mem, uint64_t capacity, const void* tok_mem,
                     uint64_t tok_capacity, const uint8_t* d_handle_keys, uint64_t n_handles,
                     uint32_t flags, uint8_t* d_keys, uint64_t* d_handles, uint32_t* d_hits) {
  hipStream_t s = (hipStream_t)stream;
  ParArgs a;
  a.in = chain_in(ctx, n_chains, ch, flags);
  a.x.mem = (uint64_t*)index_mem;
  a.x.mask = capacity - 1;
  a.t.mem = (uint64_t*)tok_mem;
  a.t.mask = tok_capacity - 1;
  a.hkeys = d_handle_keys;
  a.n_handles = d_handle_keys ? n_handles : 0;
  a.keys = d_keys;
  a.handles = d_handles;
  a.hits = d_hits;
  (void)hipGetLastError();
  // A chain's blocks never exceed the call's slots. Its tiles go to wavefronts
  // of their own while that keeps the call at 16 wavefronts per compute unit
  // (measured: 25 us for one chain of 6,062 blocks, 42 us for 256 of 400);
  // past that, and where the workgroup of one chain holds all its tiles (one
  // launch instead of three), a workgroup walks a whole chain. hits[c] holds
  // a flagged block in 30 bits.
  const uint64_t tiles = (ch->n_slots + kTileBlocks - 1) / kTileBlocks;
  const uint64_t spread = std::min<uint64_t>(tiles, 16 * (uint64_t)sm_count() / n_chains);
  {
    TimedLaunch t(TL_KERNEL_CHAIN, stream);
    if (tiles > kParWaves && spread >= 2 && ch->n_slots < (1ull << 29)) {
      hipLaunchKernelGGL(k_par_init, dim3(grid_for(n_chains, 256, 4096)), dim3(256), 0, s, d_hits,
                         (uint32_t)n_chains);
      hipLaunchKernelGGL(k_chain_par_tiles, dim3((uint32_t)(n_chains * spread)), dim3(64), 0, s, a, (uint32_t)spread);
      hipLaunchKernelGGL(k_chain_par_finish, dim3(grid_for(n_chains, 1, 1u << 16)), dim3(256), 0, s, a);
    } else {
      hipLaunchKernelGGL(k_chain_par, dim3(grid_for(n_chains, 1, 1u << 16)), dim3(64 * kParWaves), 0, s, a);
    }
  }
  return launched();
}

int launch_fingerprints(const tl_ctx* ctx, void* stream, size_t n, const uint32_t* d_tokens,
                        const uint64_t* d_pos, const uint32_t* d_n_tokens, uint8_t* d_out) {
  hipStream_t s = (hipStream_t)stream;
  FpArgs a;
  a.in = chain_in(ctx, 0, nullptr, 0);
  a.tokens = d_tokens;
  a.pos = d_pos;
  a.n_tokens = d_n_tokens;
  a.out = d_out;
  a.n = (uint32_t)n;
  (void)hipGetLastError();
  {
    TimedLaunch t(TL_KERNEL_INDEX, stream);
    hipLaunchKernelGGL(k_fingerprint, dim3(grid_for(n, 256, 1u << 16)), dim3(256), 0, s, a);
  }
  return launched();
}

int launch_stage(const tl_ctx* ctx, void* stream, size_t n_chains, const tl_chains* ch, uint32_t flags,
                 const uint32_t* d_hits, const uint64_t* d_handles, const uint64_t* d_hptr,
                 const uint64_t* d_hlen, uint64_t n_handles, uint64_t* d_ptrs, uint64_t* d_lens,
                 uint64_t* d_bidx, uint32_t* d_tokens_out, uint32_t* d_n_tokens_out,
                 const int32_t* d_tables_in, int32_t* d_tables_out) {
  hipStream_t s = (hipStream_t)stream;
  StageArgs a;
  a.tokens = ch->d_tokens;
  a.n_tokens = ch->n_tokens;
  a.tok_off = ch->d_tok_off;
  a.slot_off = ch->d_slot_off;
  a.n_slots = ch->n_slots;
  a.first_block = ch->d_first_block;
  a.n_chains = (uint32_t)n_chains;
  a.bt = ctx->geo.block_tokens;
  a.ppb = ctx->geo.ppb;
  a.page_tokens = ctx->geo.page_tokens;
  a.n_groups = ctx->geo.n_groups;
  a.tail = (flags & TL_CHAIN_TAIL) ? 1 : 0;
  a.n_tokens_out = d_n_tokens_out;
  a.hits = d_hits;
  a.handles = d_handles;
  a.hptr = d_hptr;
  a.hlen = d_hlen;
  a.n_handles = n_handles;
  a.rec_ptrs = d_ptrs;
  a.rec_lens = d_lens;
  a.bidx = d_bidx;
  a.tokens_out = d_tokens_out;
  a.tables_in = d_tables_in;
  a.tables_out = d_tables_out;
  (void)hipGetLastError();
  // Few chains for the device: split each chain's slots over up to 64
  // workgroups of about 512 slots (one chain of 6,062 slots: 11 workgroups).
  uint32_t parts = 1;
  if (n_chains && n_chains < 256) {
    const uint64_t per_chain = (ch->n_slots + n_chains - 1) / n_chains;
    parts = (uint32_t)std::min<uint64_t>(std::max<uint64_t>(per_chain / 512, 1), 64);
  }
  {
    TimedLaunch t(TL_KERNEL_STAGE, stream);
    hipLaunchKernelGGL(k_chain_stage, dim3(grid_for(n_chains, 1, 1u << 16), parts), dim3(kStageThreads), 0, s, a);
  }
  return launched();
}

}  // namespace tl
