// C0 averaging over shared GLL nodes, global edge keys and welded output.
//
// Elements store their own copy of every node; a global id per stored node
// says which copies coincide.  The direct-stiffness average (the
// gather-scatter sum of spectral-element codes, Deville, Fischer & Mund
// 2002, ch. 4, divided by the multiplicity) replaces each copy by the mean
// over all copies of its node, which makes per-element derived fields
// continuous and their isosurfaces closed across element faces.
//
// sem_gs_setup lists the copies of every shared node in increasing storage
// order, so every average is summed in one fixed order and the result does
// not depend on scheduling.  The structure follows the storage: 64 stored
// nodes have one word of flags that says which of them are the first copy of
// their node and which of those have other copies; only the other copies are
// listed by index, in 32 bits (a launch covers fewer than 2^32 work-items, so
// there are never more nodes).
// Welding numbers the distinct global edge keys of a triangle soup in order
// of first occurrence: a hash table records each key's first corner, flags
// mark those corners, and their exclusive prefix gives the vertex index.
#include <hip/hip_runtime.h>

#include "sem_internal.h"

namespace sem {
namespace {

constexpr int kThreads = 256;
constexpr uint64_t kEmpty = ~0ull;
constexpr int kGsExt = 2048;             // listed copies a workgroup holds in LDS
constexpr int kWeldT = 512;              // threads of weld_insert
constexpr int64_t kWeldMany = 1 << 22;   // corners from which a thread takes four

inline unsigned blocks_for(int64_t n) {
  return (unsigned)((n + kThreads - 1) / kThreads > 0 ? (n + kThreads - 1) / kThreads : 1);
}

__host__ __device__ constexpr size_t al256(size_t b) { return (b + 255) & ~size_t(255); }

// the listed copies follow the flag words
__device__ __forceinline__ const uint32_t* gs_col(const GsWord* words, int64_t n_words) {
  return reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(words) +
                                           al256((size_t)(n_words + 1) * sizeof(GsWord)));
}

// Workgroups go to the eight XCDs in turn; this gives each XCD runs of 64
// neighbouring ones, so that most copies of a node meet in one L2 while the
// XCDs stay close enough in the mesh to meet in the shared cache (32,768
// elements of order 7 in FP64: 100 us without, 98 with an eighth of the mesh
// per XCD, 92 with runs of 64).
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned n) {
  constexpr unsigned kRun = 64, kRound = 8 * kRun;
  if (b >= n / kRound * kRound) return b;
  const unsigned z = b % kRound;
  return b - z + (z % 8) * kRun + z / 8;
}

// all ones in n pairs of words
__global__ void fill_ones(uint64_t* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < n) p[2 * i] = p[2 * i + 1] = ~0ull;
}

__device__ __forceinline__ int below(uint64_t mask, int lane) {
  return __popcll(mask & ((1ull << lane) - 1));
}

__global__ void gs_clear(int64_t n_global, uint32_t* __restrict__ first, int64_t n_others,
                         uint32_t* __restrict__ others, GsHead* __restrict__ head,
                         int64_t n_words) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i == 0) head->n_words = n_words;
  if (i < n_global) first[i] = ~0u;
  if (i < n_others) others[i] = 0;
}

// first copy of each global node
__global__ void gs_first(int64_t n_nodes, const int64_t* __restrict__ gid, int64_t n_global,
                         uint32_t* __restrict__ first, int32_t* __restrict__ status) {
  const int64_t n = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (n >= n_nodes) return;
  const int64_t g = gid[n];
  if (g < 0 || g >= n_global) {
    if (status) atomicOr(status, SEM_FLAG_BAD_ID);
    return;
  }
  atomicMin(&first[g], (uint32_t)n);
}

// The later copies of a node are counted, and its row filled, at others[] of its
// id (DENSE) or of its first copy: by first copies the counts lie in storage
// order and are read without a look at the ids, by ids they are closer together
// for the atomics, which wins where nodes have many copies.
// Set-up, bound by the atomics on scattered nodes: 32,768 order-7 elements 417 us
// (435 by ids), 262,144 order-2 elements 349 by ids (399 by first copies), where
// one pass that counted all copies and took the first by two atomics a node gave
// 570 and 375.
template <bool DENSE>
__device__ __forceinline__ int64_t gs_at(int64_t g, uint32_t f) {
  return DENSE ? g : (int64_t)f;
}

// which stored nodes are first copies, and how many others each node has
template <bool DENSE>
__global__ void gs_others(int64_t n_nodes, const int64_t* __restrict__ gid, int64_t n_global,
                          const uint32_t* __restrict__ first, GsWord* __restrict__ words,
                          uint32_t* __restrict__ others) {
  const int64_t n = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t g = n < n_nodes ? gid[n] : -1;
  const bool good = g >= 0 && g < n_global;
  const uint32_t f = good ? first[g] : 0;
  const uint64_t own = __ballot(good && f == (uint32_t)n);
  if (good && f != (uint32_t)n) atomicAdd(&others[gs_at<DENSE>(g, f)], 1u);
  if ((threadIdx.x & 63) == 0 && n < n_nodes) words[n >> 6].own = own;
}

// later copies of the node whose first copy n is (0 where it is none)
template <bool DENSE>
__device__ __forceinline__ uint32_t gs_later(int64_t n, int64_t n_nodes,
                                             const int64_t* __restrict__ gid, uint64_t own,
                                             const uint32_t* others) {
  if constexpr (DENSE) return (own >> (n & 63)) & 1 ? others[gid[n]] : 0;
  else return n < n_nodes ? others[n] : 0;
}

// which first copies have others, and how many rows (upper half) and listed
// copies (lower half) each word starts
template <bool DENSE>
__global__ void gs_words(int64_t n_nodes, const int64_t* __restrict__ gid,
                         const uint32_t* __restrict__ others, GsWord* __restrict__ words,
                         int64_t* __restrict__ starts) {
  const int64_t n = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const uint64_t own = n < n_nodes ? words[n >> 6].own : 0;
  uint32_t sum = gs_later<DENSE>(n, n_nodes, gid, own, others);
  const uint64_t ms = __ballot(sum > 0);
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
  if ((threadIdx.x & 63) == 0 && n < n_nodes) {
    words[n >> 6].shared = ms;
    starts[n >> 6] = ((int64_t)__popcll(ms) << 32) | sum;
  }
}

// where the row of each shared node starts, in others[] too, from which gs_fill
// counts on
template <bool DENSE>
__global__ void gs_rows(int64_t n_nodes, const int64_t* __restrict__ gid, int64_t n_words,
                        const int64_t* __restrict__ begin, GsWord* __restrict__ words,
                        uint32_t* __restrict__ others, uint32_t* __restrict__ rowptr) {
  const int64_t n = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t w = n >> 6;
  const int lane = threadIdx.x & 63;
  if (n == 0) {
    const int64_t end = begin[n_words];
    rowptr[end >> 32] = (uint32_t)end;
    words[n_words].copy = (uint32_t)end;
  }
  if (w >= n_words) return;
  const int64_t at = begin[w];
  const uint32_t mine = gs_later<DENSE>(n, n_nodes, gid, words[w].own, others);
  const uint64_t ms = __ballot(mine > 0);
  uint32_t pre = mine;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(pre, d);
    if (lane >= d) pre += up;
  }
  if (lane == 0) {
    words[w].rank = (uint32_t)(at >> 32);
    words[w].copy = (uint32_t)at;
  }
  if (mine == 0) return;
  const uint32_t start = (uint32_t)at + pre - mine;
  rowptr[(at >> 32) + below(ms, lane)] = start;
  others[DENSE ? gid[n] : n] = start;
}

// place every later copy in its node's row (arbitrary order within the row)
template <bool DENSE>
__global__ void gs_fill(int64_t n_nodes, const int64_t* __restrict__ gid, int64_t n_global,
                        const uint32_t* __restrict__ first, uint32_t* __restrict__ cursor,
                        uint32_t* __restrict__ col) {
  const int64_t n = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (n >= n_nodes) return;
  const int64_t g = gid[n];
  if (g < 0 || g >= n_global) return;
  const uint32_t f = first[g];
  if (f != (uint32_t)n) col[atomicAdd(&cursor[gs_at<DENSE>(g, f)], 1u)] = (uint32_t)n;
}

// order each row by storage index (rows are short: the copies of one node)
__global__ void gs_sort(const int64_t* __restrict__ end, const uint32_t* __restrict__ rowptr,
                        uint32_t* __restrict__ col) {
  const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (r >= (*end >> 32)) return;
  const int64_t a = rowptr[r], b = rowptr[r + 1];
  for (int64_t i = a + 1; i < b; ++i) {
    const uint32_t v = col[i];
    int64_t j = i - 1;
    while (j >= a && col[j] > v) {
      col[j + 1] = col[j];
      --j;
    }
    col[j + 1] = v;
  }
}

// Mean over the copies of each global node, summed in storage order, then
// written back to every copy (in may equal out: a node's copies are read and
// written by one workgroup, that of its first copy).  The listed copies of a
// workgroup's rows are contiguous, so they are read and written as one flat
// list through LDS: a lane that walks its own row instead waits for up to
// seven loads one after the other, and the wave for its longest row.  Only a
// list that does not fit is walked by row.  Bound by the field once in and
// once out plus 2.6 bytes a node of structure (62 us at copy rate for 32,768
// elements of order 7 in FP64).  Measured there: 162 us with 64-bit rows for
// all global nodes, 195 with words and per-lane walks, 92 so; the rest is
// the chain flags -> list -> copies -> average -> copies of each workgroup
// (8 words a wave: 121 us, too few waves; 2 words: 107).  Where nodes have more
// than eight copies on average (no mesh of hexahedra does) the first words own
// nearly all of them, and a wave takes one word (4.2 million nodes at random, 64
// copies each: 235 us, 509 with four; a thread for each node took 124).
template <typename T, int kGsWords>
__global__ void __launch_bounds__(kThreads)
    dsavg_k(const GsHead* __restrict__ head, const uint32_t* __restrict__ rowptr,
            const GsWord* __restrict__ words, const T* in, T* out) {
  __shared__ T ext[kGsExt];
  const int64_t n_words = head->n_words;
  const uint32_t* __restrict__ col = gs_col(words, n_words);
  const int t = threadIdx.x, lane = t & 63;
  constexpr int kBlockWords = kGsWords * (kThreads / 64);
  for (int64_t b0 = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlockWords; b0 < n_words;
       b0 += (int64_t)gridDim.x * kBlockWords) {
    const int64_t w0 = b0 + __builtin_amdgcn_readfirstlane(t >> 6) * kGsWords;
    const uint32_t c0 = words[b0].copy;
    const uint32_t n_ext = words[b0 + kBlockWords <= n_words ? b0 + kBlockWords : n_words].copy - c0;
    const bool flat = n_ext <= kGsExt;
    GsWord g[kGsWords];
    T v[kGsWords];
    uint32_t a[kGsWords], b[kGsWords];
#pragma unroll
    for (int k = 0; k < kGsWords; ++k) {
      g[k].own = g[k].shared = 0;
      g[k].rank = 0;
      if (w0 + k < n_words) g[k] = words[w0 + k];
      if ((g[k].own >> lane) & 1) v[k] = in[(w0 + k) * 64 + lane];
      if ((g[k].shared >> lane) & 1) {
        const uint32_t r = g[k].rank + below(g[k].shared, lane);
        a[k] = rowptr[r] - c0;
        b[k] = rowptr[r + 1] - c0;
      }
    }
    uint32_t c[kGsExt / kThreads];
    if (flat) {
#pragma unroll
      for (int j = 0; j < kGsExt / kThreads; ++j)
        if (t + j * kThreads < n_ext) c[j] = col[c0 + t + j * kThreads];
#pragma unroll
      for (int j = 0; j < kGsExt / kThreads; ++j)
        if (t + j * kThreads < n_ext) ext[t + j * kThreads] = in[c[j]];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kGsWords; ++k) {
      if (!((g[k].own >> lane) & 1)) continue;
      T s = T(0) + v[k];
      if ((g[k].shared >> lane) & 1) {
        if (flat) {
          for (uint32_t i = a[k]; i < b[k]; ++i) s += ext[i];
          s = s / (T)(b[k] - a[k] + 1);
          for (uint32_t i = a[k]; i < b[k]; ++i) ext[i] = s;
        } else {
          for (uint32_t i = a[k]; i < b[k]; ++i) s += in[col[c0 + i]];
          s = s / (T)(b[k] - a[k] + 1);
          for (uint32_t i = a[k]; i < b[k]; ++i) out[col[c0 + i]] = s;
        }
      }
      out[(w0 + k) * 64 + lane] = s;
    }
    __syncthreads();
    if (flat) {
#pragma unroll
      for (int j = 0; j < kGsExt / kThreads; ++j)
        if (t + j * kThreads < n_ext) out[c[j]] = ext[t + j * kThreads];
    }
    __syncthreads();
  }
}

// element-local key (e P^3 + n_lo) * 3 + axis  ->  (min gid << 32) | max gid
__global__ void global_keys_k(int64_t n_ref, int p, int64_t n_elem,
                              const uint64_t* __restrict__ local,
                              const int64_t* __restrict__ gid, uint64_t* __restrict__ global,
                              int32_t* __restrict__ status) {
  const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (r >= n_ref) return;
  const uint64_t k = local[r];
  const int axis = (int)(k % 3u);
  const uint64_t flat = k / 3u;
  const uint64_t p3 = (uint64_t)p * p * p;
  const uint64_t e = flat / p3, lo = flat % p3;
  const uint64_t step = axis == 0 ? 1u : (axis == 1 ? (uint64_t)p : (uint64_t)p * p);
  const uint64_t hi = lo + step;
  if (e >= (uint64_t)n_elem || hi >= p3) {
    if (status) atomicOr(status, SEM_FLAG_BAD_ID);
    global[r] = kEmpty;
    return;
  }
  const int64_t a = gid[e * p3 + lo], b = gid[e * p3 + hi];
  if (a < 0 || b < 0 || a >= (int64_t)0xffffffffll || b >= (int64_t)0xffffffffll) {
    if (status) atomicOr(status, SEM_FLAG_BAD_ID);
    global[r] = kEmpty;
    return;
  }
  const uint64_t mn = (uint64_t)(a < b ? a : b), mx = (uint64_t)(a < b ? b : a);
  global[r] = (mn << 32) | mx;
}

// 64-bit finaliser of SplitMix64 (Steele, Lea & Flood 2014) as the hash
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// Table slot of every corner's key (linear probing; the table is at least
// twice the number of corners, so a free slot is always reached).  A slot
// holds the smallest corner of its key, and the key is looked up there: one
// atomic claims a slot and records the corner, and an entry is 4 bytes.  A
// workgroup finds the distinct keys of its consecutive corners in LDS first,
// in the same way (also at most half full), and only the first corner of each
// goes to the table in memory; local[] marks these corners, 64 to a word.
// 535,000 triangles of two isovalues: 165 us with an atomic each for key and
// corner of every corner, 48 with the distinct keys of a workgroup only, 26
// with the key looked up at the corner.  Corners a thread (PER): one up to
// kWeldMany, where a probe's round trip is hidden by other waves only; four
// beyond, where the table is far larger than the caches and a workgroup of
// four times the corners sends fewer of them there.  All passes of the weld,
// one corner and four: 1,000 triangles that share no key 22 and 39 us; the
// first 100,000 triangles of a channel snapshot's soup 29 and 32, 1,000,000
// 115 and 117, 2,000,000 218 and 214, 7,900,000 873 and 834.
template <int PER>
__global__ void __launch_bounds__(kWeldT)
    weld_insert(int64_t n_ref, const uint64_t* __restrict__ keys, uint32_t* __restrict__ table,
                int32_t* __restrict__ slot, uint64_t* __restrict__ local, int64_t cap,
                int32_t* __restrict__ status) {
  constexpr int kRefs = kWeldT * PER;
  __shared__ uint64_t lkey[kRefs];
  __shared__ uint32_t lpos[2 * kRefs];
  const int64_t base = (int64_t)blockIdx.x * kRefs;
  uint64_t k[PER], hash[PER];
  uint32_t l[PER];
  bool own[PER], bad = false;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const uint32_t me = j * kWeldT + threadIdx.x;
    k[j] = base + me < n_ref ? keys[base + me] : kEmpty;
    bad |= base + me < n_ref && k[j] == kEmpty;
    hash[j] = mix64(k[j]);
    lkey[me] = k[j];
    lpos[me] = lpos[kRefs + me] = ~0u;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (k[j] == kEmpty) continue;
    const uint32_t me = j * kWeldT + threadIdx.x;
    l[j] = (uint32_t)(hash[j] >> 40) & (2 * kRefs - 1);
    for (;;) {   // ends: at most kRefs of the 2 kRefs entries are taken
      const uint32_t prev = atomicCAS(&lpos[l[j]], ~0u, me);
      if (prev == ~0u) break;
      if (lkey[prev] == k[j]) {
        if (me < prev) atomicMin(&lpos[l[j]], me);
        break;
      }
      l[j] = (l[j] + 1) & (2 * kRefs - 1);
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const uint32_t me = j * kWeldT + threadIdx.x;
    own[j] = k[j] != kEmpty && lpos[l[j]] == me;
    const uint64_t marks = __ballot(own[j]);
    if ((me & 63) == 0 && base + me < n_ref) local[(base + me) >> 6] = marks;
  }
  __syncthreads();
  const uint64_t mask = (uint64_t)cap - 1;
  uint32_t prev[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (own[j])
      prev[j] = atomicCAS(&table[hash[j] & mask], ~0u, (uint32_t)(base + j * kWeldT + threadIdx.x));
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (!own[j]) continue;
    const uint32_t r = (uint32_t)(base + j * kWeldT + threadIdx.x);
    uint64_t h = hash[j] & mask;
    for (int64_t probe = 1; prev[j] != ~0u; ++probe) {
      if (keys[prev[j]] == k[j]) {
        if (r < prev[j]) atomicMin(&table[h], r);
        break;
      }
      if (probe == cap) break;   // not reached in a half-empty table
      h = (h + 1) & mask;
      prev[j] = atomicCAS(&table[h], ~0u, r);
    }
    lpos[l[j]] = (uint32_t)h;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int64_t r = base + j * kWeldT + threadIdx.x;
    if (r < n_ref) slot[r] = k[j] != kEmpty ? (int32_t)lpos[l[j]] : -1;
  }
  if (bad && status) atomicOr(status, SEM_FLAG_BAD_ID);
}

// first corners of the keys, 64 corners a wave
__global__ void weld_flag(int64_t n_words, const int32_t* __restrict__ slot,
                          const uint32_t* __restrict__ table, uint64_t* __restrict__ marks,
                          int32_t* __restrict__ count) {
  const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t w = r >> 6;
  if (w >= n_words) return;
  bool first = false;
  if ((marks[w] >> (r & 63)) & 1) first = table[slot[r]] == (uint32_t)r;
  const uint64_t m = __ballot(first);
  if ((r & 63) == 0) {
    marks[w] = m;
    count[w] = __popcll(m);
  }
}

// number the vertices (in the table, in place of their corners) and write their coordinates
template <typename T>
__global__ void weld_emit(int64_t n_words, const int32_t* __restrict__ slot,
                          const uint64_t* __restrict__ marks, const int64_t* __restrict__ offs,
                          const T* __restrict__ tri_xyz, uint32_t* __restrict__ table,
                          T* __restrict__ vert_xyz, int64_t vert_cap,
                          int64_t* __restrict__ n_vert, int32_t* __restrict__ status) {
  const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (r == 0) {
    const int64_t total = offs[n_words];
    *n_vert = total;
    if (status && total > vert_cap) atomicOr(status, SEM_FLAG_VERT_OVERFLOW);
  }
  const int64_t w = r >> 6;
  if (w >= n_words) return;
  const uint64_t m = marks[w];
  if (!((m >> (r & 63)) & 1)) return;
  const int64_t v = offs[w] + below(m, (int)(r & 63));
  table[slot[r]] = (uint32_t)v;
  if (v < vert_cap) {
    vert_xyz[3 * v] = tri_xyz[3 * r];
    vert_xyz[3 * v + 1] = tri_xyz[3 * r + 1];
    vert_xyz[3 * v + 2] = tri_xyz[3 * r + 2];
  }
}

__global__ void weld_index(int64_t n_ref, const int32_t* __restrict__ slot,
                           const uint32_t* __restrict__ table, int64_t* __restrict__ tri_index) {
  const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (r >= n_ref) return;
  const int32_t h = slot[r];
  tri_index[r] = h < 0 ? -1 : (int64_t)table[h];
}

}  // namespace

GsLayout gs_layout(void* base, int64_t n_nodes, int64_t n_global) {
  GsLayout l;
  char* p = static_cast<char*>(base);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char* q = p ? p + o : nullptr;
    o += al256(bytes);
    return q;
  };
  const int64_t nw = (n_nodes + 63) / 64;
  l.n_words = nw;
  // what sem_dsavg reads comes first, at offsets that depend on n_global only
  l.head = reinterpret_cast<GsHead*>(take(sizeof(GsHead)));
  l.first = reinterpret_cast<uint32_t*>(take((size_t)n_global * 4));
  l.rowptr = reinterpret_cast<uint32_t*>(take((size_t)(n_global + 1) * 4));
  l.words = reinterpret_cast<GsWord*>(take((size_t)(nw + 1) * sizeof(GsWord)));
  l.col = reinterpret_cast<uint32_t*>(take((size_t)n_nodes * 4));
  l.starts = reinterpret_cast<int64_t*>(take((size_t)nw * 8));
  l.begin = reinterpret_cast<int64_t*>(take((size_t)(nw + 1) * 8));
  l.dense = n_global < n_nodes / 2;
  l.many = n_global < n_nodes / 8;
  l.others = reinterpret_cast<uint32_t*>(take((size_t)(l.dense ? n_global : n_nodes) * 4));
  l.partial = reinterpret_cast<int64_t*>(take((size_t)(scan_partials_capacity(nw) + 1) * 8));
  l.bytes = o;
  return l;
}

namespace {
template <bool DENSE>
hipError_t gs_build(int64_t n_nodes, const int64_t* gid, int64_t n_global, const GsLayout& gs,
                    hipStream_t s) {
  const unsigned nb = blocks_for(n_nodes);
  hipLaunchKernelGGL(gs_others<DENSE>, dim3(nb), dim3(kThreads), 0, s, n_nodes, gid, n_global,
                     (const uint32_t*)gs.first, gs.words, gs.others);
  hipLaunchKernelGGL(gs_words<DENSE>, dim3(nb), dim3(kThreads), 0, s, n_nodes, gid,
                     (const uint32_t*)gs.others, gs.words, gs.starts);
  const hipError_t e = launch_exclusive_scan(gs.starts, gs.n_words, gs.partial, gs.begin, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gs_rows<DENSE>, dim3(nb), dim3(kThreads), 0, s, n_nodes, gid, gs.n_words,
                     (const int64_t*)gs.begin, gs.words, gs.others, gs.rowptr);
  hipLaunchKernelGGL(gs_fill<DENSE>, dim3(nb), dim3(kThreads), 0, s, n_nodes, gid, n_global,
                     (const uint32_t*)gs.first, gs.others, gs.col);
  const int64_t rows = n_nodes / 2 < n_global ? n_nodes / 2 : n_global;   // at most
  hipLaunchKernelGGL(gs_sort, dim3(blocks_for(rows)), dim3(kThreads), 0, s,
                     (const int64_t*)gs.begin + gs.n_words, (const uint32_t*)gs.rowptr, gs.col);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_gs_setup(int64_t n_nodes, const int64_t* gid, int64_t n_global,
                           const GsLayout& gs, int32_t* status, hipStream_t s) {
  if (n_nodes > (int64_t)0xffffff00) return hipErrorInvalidConfiguration;
  const int64_t n_others = gs.dense ? n_global : n_nodes;
  hipLaunchKernelGGL(gs_clear, dim3(blocks_for(n_global > n_others ? n_global : n_others)),
                     dim3(kThreads), 0, s, n_global, gs.first, n_others, gs.others, gs.head,
                     gs.n_words);
  if (n_nodes == 0) return hipGetLastError();
  hipLaunchKernelGGL(gs_first, dim3(blocks_for(n_nodes)), dim3(kThreads), 0, s, n_nodes, gid,
                     n_global, gs.first, status);
  return gs.dense ? gs_build<true>(n_nodes, gid, n_global, gs, s)
                  : gs_build<false>(n_nodes, gid, n_global, gs, s);
}

hipError_t launch_dsavg(sem_dtype dt, const GsLayout& gs, const void* in, void* out,
                        hipStream_t s) {
  auto go = [&](auto kern, int words, auto zero) {
    using T = decltype(zero);
    hipLaunchKernelGGL(kern, dim3(blocks_for((gs.n_words * 64 + words - 1) / words)),
                       dim3(kThreads), 0, s, (const GsHead*)gs.head, (const uint32_t*)gs.rowptr,
                       (const GsWord*)gs.words, (const T*)in, (T*)out);
  };
  if (dt == SEM_F64)
    gs.many ? go(dsavg_k<double, 1>, 1, 0.0) : go(dsavg_k<double, 4>, 4, 0.0);
  else
    gs.many ? go(dsavg_k<float, 1>, 1, 0.f) : go(dsavg_k<float, 4>, 4, 0.f);
  return hipGetLastError();
}

hipError_t launch_global_keys(int64_t n_ref, int order, int64_t n_elem, const uint64_t* local,
                              const int64_t* gid, uint64_t* global, int32_t* status,
                              hipStream_t s) {
  hipLaunchKernelGGL(global_keys_k, dim3(blocks_for(n_ref)), dim3(kThreads), 0, s, n_ref,
                     order + 1, n_elem, local, gid, global, status);
  return hipGetLastError();
}

WeldLayout weld_layout(void* base, int64_t n_ref) {
  WeldLayout w;
  int64_t cap = 64;
  while (cap < 2 * n_ref) cap <<= 1;
  w.cap = cap;
  w.n_words = (n_ref + 63) / 64;
  char* p = static_cast<char*>(base);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    char* q = p ? p + o : nullptr;
    o += al256(bytes);
    return q;
  };
  w.table = reinterpret_cast<uint32_t*>(take((size_t)cap * 4));
  w.slot = reinterpret_cast<int32_t*>(take((size_t)n_ref * 4));
  w.marks = reinterpret_cast<uint64_t*>(take((size_t)w.n_words * 8));
  w.count = reinterpret_cast<int32_t*>(take((size_t)w.n_words * 4));
  w.offs = reinterpret_cast<int64_t*>(take((size_t)(w.n_words + 1) * 8));
  w.partial =
      reinterpret_cast<int64_t*>(take((size_t)(scan_partials_capacity(w.n_words) + 1) * 8));
  // one size for all small soups: a workspace kept between them fits
  constexpr size_t kLeast = 16 << 10;
  w.bytes = o > kLeast ? o : kLeast;
  return w;
}

namespace {
template <typename T>
hipError_t weld_t(int64_t n_ref, const T* tri_xyz, const uint64_t* keys, int64_t* tri_index,
                  T* vert_xyz, int64_t vert_cap, int64_t* n_vert, const WeldLayout& w,
                  int32_t* status, hipStream_t s) {
  if (n_ref > 0) {
    hipLaunchKernelGGL(fill_ones, dim3(blocks_for(w.cap / 4)), dim3(kThreads), 0, s,
                       reinterpret_cast<uint64_t*>(w.table), w.cap / 4);
    auto insert = [&](auto kern, int per) {
      const int64_t refs = (int64_t)kWeldT * per;
      hipLaunchKernelGGL(kern, dim3((unsigned)((n_ref + refs - 1) / refs)), dim3(kWeldT), 0, s,
                         n_ref, keys, w.table, w.slot, w.marks, w.cap, status);
    };
    if (n_ref > kWeldMany) insert(weld_insert<4>, 4);
    else insert(weld_insert<1>, 1);
    hipLaunchKernelGGL(weld_flag, dim3(blocks_for(w.n_words * 64)), dim3(kThreads), 0, s,
                       w.n_words, (const int32_t*)w.slot, (const uint32_t*)w.table, w.marks,
                       w.count);
  }
  const hipError_t e = launch_exclusive_scan(w.count, w.n_words, w.partial, w.offs, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(weld_emit<T>, dim3(blocks_for(w.n_words * 64)), dim3(kThreads), 0, s,
                     w.n_words, (const int32_t*)w.slot, (const uint64_t*)w.marks,
                     (const int64_t*)w.offs, tri_xyz, w.table, vert_xyz, vert_cap, n_vert,
                     status);
  if (n_ref > 0)
    hipLaunchKernelGGL(weld_index, dim3(blocks_for(n_ref)), dim3(kThreads), 0, s, n_ref,
                       (const int32_t*)w.slot, (const uint32_t*)w.table, tri_index);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_weld(int64_t n_ref, sem_dtype dt, const void* tri_xyz, const uint64_t* keys,
                       int64_t* tri_index, void* vert_xyz, int64_t vert_cap, int64_t* n_vert,
                       const WeldLayout& w, int32_t* status, hipStream_t s) {
  if (dt == SEM_F64)
    return weld_t(n_ref, (const double*)tri_xyz, keys, tri_index, (double*)vert_xyz, vert_cap,
                  n_vert, w, status, s);
  return weld_t(n_ref, (const float*)tri_xyz, keys, tri_index, (float*)vert_xyz, vert_cap,
                n_vert, w, status, s);
}

}  // namespace sem
