// Exact selection engine and step 3a (top-k).  Per row, a 3-pass radix select (11 + 11 + 10
// bits of an order-preserving key) finds the threshold key T and how many slots equal to T
// are needed; a counting pass plus a chunk prefix then lets an ordered pass emit the
// selected slots in ascending order with ties resolved towards the lower slot:
//   selected(j) = key_j > T  or  (key_j == T and #{i < j : key_i == T} < r_eq)
//   position(j) = #{i < j : key_i > T} + min(#{i < j : key_i == T}, r_eq)
// This is the sorted prefix Pi_k of Sec. 3.2 without sorting.  The engine serves the eviction's keep-set, whose
// values are accumulated softmax weights: a first counting pass against 0 settles T for every row whose
// wanted-th largest value is 0 (sel_try_zero), and the radix passes skip those rows.
#include "hca_internal.h"

namespace hca {

constexpr int kBins = 2048;

__device__ __forceinline__ int pass_shift(int p) { return p == 0 ? 21 : (p == 1 ? 10 : 0); }

size_t select_workspace_bytes(int rows, int64_t nmax) {
  (void)nmax;
  size_t b = 0;
  b += align_up((int64_t)rows * 3 * kBins * 4, 256);
  b += align_up((int64_t)rows * 4 * 4, 256);
  b += align_up((int64_t)rows * 1024 * 2 * 4, 256);
  return b;
}

void select_plan(SelectPlan* p, void* ws, int rows, int64_t nmax) {
  int64_t chunk = align_up((nmax + 1023) / 1024, 1024);
  if (chunk < 4096) chunk = 4096;
  p->chunk = chunk;
  p->nchunks = (int32_t)((nmax + chunk - 1) / chunk);
  if (p->nchunks < 1) p->nchunks = 1;
  uint8_t* w = (uint8_t*)ws;
  p->hist = (uint32_t*)w;   w += align_up((int64_t)rows * 3 * kBins * 4, 256);
  p->state = (uint32_t*)w;  w += align_up((int64_t)rows * 4 * 4, 256);
  p->ccount = (uint32_t*)w;
}

// Sixteen loads of a 4096-slot tile in flight per thread (256 threads); slots at or past `end` are not live.
template <typename F>
__device__ __forceinline__ void sel_each(const float* __restrict__ v, int64_t c0, int64_t c1, F&& f) {
  for (int64_t s0 = c0; s0 < c1; s0 += 4096) {
    float x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int64_t j = s0 + i * 256 + threadIdx.x;
      x[i] = v[j < c1 ? j : c1 - 1];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) f(order_key(x[i]), s0 + i * 256 + threadIdx.x < c1);
  }
}

// The bin of a 2048-bin histogram that holds the rem-th largest key, and how many of it are left to take: the same for
// every thread of the workgroup (256).  Every workgroup of the pass that needs a bin finds it from the finished
// histogram by itself - 8 KB from L2 - instead of waiting for a launch of its own that would.
__device__ __forceinline__ void sel_find_bin(const uint32_t* __restrict__ gh, uint32_t* bin, uint32_t* rem) {
  __shared__ uint32_t wsum[4], s_bin, s_rem;
  const int t = threadIdx.x;
  uint32_t h[8];
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) { h[i] = gh[kBins - 1 - (8 * t + i)]; sum += h[i]; }     // bins from the top
  __syncthreads();
  uint32_t running = block_scan_excl<4>(sum, wsum);
  const uint32_t want = *rem;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (running < want && want <= running + h[i]) { s_bin = (uint32_t)(kBins - 1 - (8 * t + i)); s_rem = want - running; }
    running += h[i];
  }
  __syncthreads();
  *bin = s_bin;
  *rem = s_rem;
}

// Leading digits of the threshold key known after PASSES histograms, and how many are left to take among the keys that
// share them.
template <int PASSES>
__device__ __forceinline__ void sel_prefix(const uint32_t* __restrict__ hist, int row, uint32_t want, uint32_t* prefix,
                                           uint32_t* rem) {
  *prefix = 0;
  *rem = want;
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    uint32_t bin;
    sel_find_bin(hist + ((int64_t)row * 3 + p) * kBins, &bin, rem);
    *prefix |= bin << pass_shift(p);
  }
}

// Per-chunk counts of keys above and equal to T; clears the row's histograms on the way (AT_ZERO).
// AT_ZERO: against the key of +0.0f, before any radix pass (the shortcut below); otherwise against the row's threshold -
// found here from the three histograms -, and rows that the shortcut resolved keep the counts they already have.
template <bool AT_ZERO>
__global__ __launch_bounds__(256) void sel_count(const float* __restrict__ vals, int64_t stride, int64_t chunk,
                                                 int n_kv_heads, SelRows sr, uint32_t* __restrict__ state,
                                                 uint32_t* __restrict__ hist, uint32_t* __restrict__ ccount) {
  __shared__ uint32_t red[2][4];
  const int row = blockIdx.y;
  const int64_t want = sr.want[row / n_kv_heads];
  if (want < 0) return;
  if (!AT_ZERO && state[4 * row + 3] != 0) return;
  uint32_t T = order_key(0.0f);
  if constexpr (AT_ZERO) {
    uint32_t* gh = hist + (int64_t)row * 3 * kBins;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < 3 * kBins; i += gridDim.x * 256) gh[i] = 0;
  } else if (want == 0) {
    T = 0xffffffffu;
  } else {
    uint32_t rem;
    sel_prefix<3>(hist, row, (uint32_t)want, &T, &rem);
    if (blockIdx.x == 0 && threadIdx.x == 0) { state[4 * row] = T; state[4 * row + 1] = rem; }
  }
  const int64_t nsel = sr.nsel[row / n_kv_heads];
  const int64_t c0 = (int64_t)blockIdx.x * chunk;
  int64_t c1 = c0 + chunk;
  if (c1 > nsel) c1 = nsel;
  uint32_t gt = 0, eq = 0;
  sel_each(vals + (int64_t)row * stride, c0, c1, [&](uint32_t key, bool live) {
    gt += live && key > T;
    eq += live && key == T;
  });
  gt = wave_sum(gt);
  eq = wave_sum(eq);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[0][w] = gt; red[1][w] = eq; }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t* o = ccount + ((int64_t)row * gridDim.x + blockIdx.x) * 2;
    o[0] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    o[1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
  }
}

// The zero-threshold shortcut, decided by every workgroup of the first histogram pass from the chunk counts (at most
// 1024 pairs).  Accumulated scores are sums of softmax weights: never negative, and exactly 0 for every token that was
// never selected - most of a long context.  When fewer than `want` slots lie above 0 and the zeros make up the rest,
// the want-th largest key is the key of +0.0f and the number of zeros to take is want - #(above 0): exactly what the
// three radix passes would find, from one pass whose per-chunk counts are also the ones the ordered pass needs.
__device__ __forceinline__ bool sel_try_zero(const uint32_t* __restrict__ ccount, int nchunks, int row, int64_t want,
                                             uint32_t* __restrict__ state, bool writer) {
  __shared__ uint32_t red[2][4];
  const int t = threadIdx.x;
  uint32_t g = 0, e = 0;
  for (int c = t; c < nchunks; c += 256) {
    g += ccount[((int64_t)row * nchunks + c) * 2];
    e += ccount[((int64_t)row * nchunks + c) * 2 + 1];
  }
  g = wave_sum(g);
  e = wave_sum(e);
  if ((t & 63) == 0) { red[0][t >> 6] = g; red[1][t >> 6] = e; }
  __syncthreads();
  const uint64_t above = (uint64_t)red[0][0] + red[0][1] + red[0][2] + red[0][3];
  const uint64_t zeros = (uint64_t)red[1][0] + red[1][1] + red[1][2] + red[1][3];
  const bool zero = want > 0 && above < (uint64_t)want && (uint64_t)want <= above + zeros;
  if (writer && t == 0) {
    state[4 * row + 0] = zero ? order_key(0.0f) : 0xffffffffu;
    state[4 * row + 1] = zero ? (uint32_t)((uint64_t)want - above) : 0u;
    state[4 * row + 2] = 0xffffffffu;        // lowest slot that is not selected (filled in by the eviction's ordered pass)
    state[4 * row + 3] = zero ? 1u : 0u;     // 1: threshold found here, the radix passes skip the row
  }
  return zero;
}

template <int PASS>
__global__ __launch_bounds__(256) void sel_hist(const float* __restrict__ vals, int64_t stride, int64_t chunk,
                                                int n_kv_heads, SelRows sr, uint32_t* __restrict__ hist,
                                                uint32_t* __restrict__ state, const uint32_t* __restrict__ ccount) {
  __shared__ uint32_t lh[kBins];
  const int row = blockIdx.y;
  const int64_t nsel = sr.nsel[row / n_kv_heads], want = sr.want[row / n_kv_heads];
  if constexpr (PASS == 0) {
    if (want < 0) return;
    if (sel_try_zero(ccount, (int)gridDim.x, row, want, state, blockIdx.x == 0)) return;
  } else if (want > 0 && state[4 * row + 3] != 0) {
    return;
  }
  if (want <= 0) return;
  const int64_t c0 = (int64_t)blockIdx.x * chunk;
  if (c0 >= nsel) return;
  int64_t c1 = c0 + chunk;
  if (c1 > nsel) c1 = nsel;
  uint32_t prefix, rem;
  sel_prefix<PASS>(hist, row, (uint32_t)want, &prefix, &rem);
  for (int i = threadIdx.x; i < kBins; i += 256) lh[i] = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  sel_each(vals + (int64_t)row * stride, c0, c1, [&](uint32_t key, bool live) {
    bool hit = live;
    uint32_t bin;
    if (PASS == 0) {
      bin = key >> 21;
    } else if (PASS == 1) {
      hit = hit && (key >> 21) == (prefix >> 21);
      bin = (key >> 10) & 2047u;
    } else {
      hit = hit && (key >> 10) == (prefix >> 10);
      bin = key & 1023u;
    }
    // accumulated scores are mostly equal (0), so a whole wave usually lands in one bin: one
    // atomic for the wave instead of 64 on the same LDS word
    const uint64_t m = __ballot(hit);
    if (m != 0) {
      const int leader = __ffsll((unsigned long long)m) - 1;
      const uint32_t b0 = __shfl(bin, leader);
      if (__ballot(hit && bin != b0) == 0) {
        if (lane == leader) atomicAdd(&lh[b0], (uint32_t)__popcll(m));
      } else if (hit) {
        atomicAdd(&lh[bin], 1u);
      }
    }
  });
  __syncthreads();
  uint32_t* gh = hist + ((int64_t)row * 3 + PASS) * kBins;
  for (int i = threadIdx.x; i < kBins; i += 256) {
    const uint32_t c = lh[i];
    if (c) atomicAdd(&gh[i], c);
  }
}

// Five launches: counts against 0; first histogram (and the shortcut); second; third; counts against the threshold.
// The last three find nothing to do for rows that the shortcut resolved.  With a launch each for clearing, for the
// shortcut, for every bin search and for the chunk prefixes it was eleven: 8 rows of 512 Ki slots 52 us, 25 now.
int32_t select_run(const SelectPlan& p, const float* vals, int64_t stride, int rows, int n_kv_heads,
                   const SelRows& sr, hipStream_t st) {
  dim3 g((unsigned)p.nchunks, (unsigned)rows);
  sel_count<true><<<g, 256, 0, st>>>(vals, stride, p.chunk, n_kv_heads, sr, p.state, p.hist, p.ccount);
  sel_hist<0><<<g, 256, 0, st>>>(vals, stride, p.chunk, n_kv_heads, sr, p.hist, p.state, p.ccount);
  sel_hist<1><<<g, 256, 0, st>>>(vals, stride, p.chunk, n_kv_heads, sr, p.hist, p.state, p.ccount);
  sel_hist<2><<<g, 256, 0, st>>>(vals, stride, p.chunk, n_kv_heads, sr, p.hist, p.state, p.ccount);
  sel_count<false><<<g, 256, 0, st>>>(vals, stride, p.chunk, n_kv_heads, sr, p.state, p.hist, p.ccount);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// ---------------------------------------------------------------------------------------
// Top-k fast path: one 12-bit histogram pass finds the bin b* that holds the k-th largest key;
// a second pass counts, per chunk, the slots above that bin and collects the (few) slots inside
// it as (key, slot) candidates; one workgroup per row then finishes the radix select on the
// candidates only and turns the counts into chunk offsets for the ordered emit.
constexpr int kBins12 = 4096;
constexpr int kMaxChunks = 1024;

struct TopkWs {
  uint32_t* hist;      // [rows][4096]
  uint32_t* ncand;     // [rows][1024] entries in each chunk's list
  uint32_t* state;     // [rows][4]: T (after resolve), r_eq / still-to-take, b*, unused; the cumulative walk has the smallest
                       // and the largest key of its bin in the last two
  uint32_t* above;     // [rows][1024] slots strictly above bin b* per chunk; before that, the cumulative walk's row maxima
                       // per group of chunks
  uint32_t* coff;      // [rows][1024][2]; before the chunk prefixes, the cumulative walk's wave extremes
  uint2* cand;         // [rows][row_entries]: chunk c owns entries [c*chunk, (c+1)*chunk)
  int64_t row_entries;
  // cumulative-weight selection only
  uint32_t* pcount;    // [rows][4096] slots per bin, the first kTpBins in use
  uint64_t* pmass;     // [rows][4096] integer weight per bin, likewise
  uint64_t* pstate;    // [rows][4]: weight still to reach inside the bin; window of the fine bins (two floats)
  uint32_t* prow;      // [rows][4]: key of the row maximum, slots still allowed, selected count, (unused)
  // scan + top-k in one call only
  uint32_t* samples;   // [rows][kSampleMax] keys of the sampled slots; after a second scan by tk_finish, the pair counts of
                       // the rows that it scanned, [rows][kSelectMaxChunks]
  uint32_t* spec;      // [rows][4]: see SelectOut
  uint32_t* mon;       // [rows][4] since the last reset: fused selections, fewest and most pairs a first scan let
                       // through, selections that needed the second scan
};

// chunk geometry for a row of n slots: at most 1024 chunks, each a multiple of 1024 slots, >= 4096
static void chunk_geometry(int64_t n, int64_t* chunk, int32_t* nchunks) {
  if (n < 1) n = 1;
  int64_t c = align_up((n + 1023) / 1024, 1024);
  if (c < 4096) c = 4096;
  *chunk = c;
  *nchunks = (int32_t)((n + c - 1) / c);
}

static int64_t list_entries_per_row(int64_t cap) {
  int64_t chunk;
  int32_t nchunks;
  chunk_geometry(cap, &chunk, &nchunks);
  return align_up(cap, 1024) + 2 * chunk;     // nchunks(n) * chunk(n) < n + chunk(n) <= this, for any n <= cap
}

size_t topk_workspace_bytes(int rows, int64_t cap) {
  size_t b = 0;
  b += align_up((int64_t)rows * kBins12 * 4, 256);
  b += align_up((int64_t)rows * kMaxChunks * 4, 256);
  b += align_up((int64_t)rows * 4 * 4, 256);
  b += align_up((int64_t)rows * 1024 * 4, 256);
  b += align_up((int64_t)rows * 1024 * 2 * 4, 256);
  b += align_up((int64_t)rows * list_entries_per_row(cap) * 8, 256);
  b += align_up((int64_t)rows * kBins12 * 4, 256);
  b += align_up((int64_t)rows * kBins12 * 8, 256);
  b += align_up((int64_t)rows * 4 * 8, 256);
  b += align_up((int64_t)rows * 4 * 4, 256);
  b += align_up((int64_t)rows * kSampleMax * 4, 256);
  b += align_up((int64_t)rows * 4 * 4, 256);
  b += align_up((int64_t)rows * 4 * 4, 256);
  return b;
}

static void topk_carve(TopkWs* t, void* ws, int rows, int64_t cap) {
  uint8_t* w = (uint8_t*)ws;
  t->hist = (uint32_t*)w;  w += align_up((int64_t)rows * kBins12 * 4, 256);
  t->ncand = (uint32_t*)w; w += align_up((int64_t)rows * kMaxChunks * 4, 256);
  t->state = (uint32_t*)w; w += align_up((int64_t)rows * 4 * 4, 256);
  t->above = (uint32_t*)w; w += align_up((int64_t)rows * 1024 * 4, 256);
  t->coff = (uint32_t*)w;  w += align_up((int64_t)rows * 1024 * 2 * 4, 256);
  t->cand = (uint2*)w;
  t->row_entries = list_entries_per_row(cap);
  w += align_up((int64_t)rows * t->row_entries * 8, 256);
  t->pcount = (uint32_t*)w; w += align_up((int64_t)rows * kBins12 * 4, 256);
  t->pmass = (uint64_t*)w;  w += align_up((int64_t)rows * kBins12 * 8, 256);
  t->pstate = (uint64_t*)w; w += align_up((int64_t)rows * 4 * 8, 256);
  t->prow = (uint32_t*)w;   w += align_up((int64_t)rows * 4 * 4, 256);
  t->samples = (uint32_t*)w; w += align_up((int64_t)rows * kSampleMax * 4, 256);
  t->spec = (uint32_t*)w;    w += align_up((int64_t)rows * 4 * 4, 256);
  t->mon = (uint32_t*)w;
}

__global__ void tk_zero(uint32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// LDS counter updates, to be called by all lanes of a wave together.  When every participating lane
// targets the same counter (ties, clustered scores) the wave issues one atomic instead of up to 64
// serialised ones on the same word.
__device__ __forceinline__ void lds_count(uint32_t* h, uint32_t bin, bool hit, bool aggregate) {
  if (!aggregate) {                       // wave-uniform choice: short candidate sets do not pay for the ballots
    if (hit) atomicAdd(&h[bin], 1u);
    return;
  }
  const uint64_t m = __ballot(hit);
  if (m == 0) return;
  const int leader = __ffsll((unsigned long long)m) - 1;
  const uint32_t b0 = __shfl(bin, leader);
  if (__ballot(hit && bin != b0) == 0) {
    if ((int)(threadIdx.x & 63) == leader) atomicAdd(&h[b0], (uint32_t)__popcll(m));
  } else if (hit) {
    atomicAdd(&h[bin], 1u);
  }
}

// The same for a counter and an integer weight; one pair of atomics when all participating lanes hold the
// same key (and therefore the same weight).
__device__ __forceinline__ void lds_count_mass(uint32_t* h, unsigned long long* hm, uint32_t bin, uint32_t key,
                                               uint64_t w, bool hit, bool aggregate) {
  if (!aggregate) {
    if (hit) {
      atomicAdd(&h[bin], 1u);
      if (w) atomicAdd(&hm[bin], (unsigned long long)w);
    }
    return;
  }
  const uint64_t m = __ballot(hit);
  if (m == 0) return;
  const int leader = __ffsll((unsigned long long)m) - 1;
  const uint32_t k0 = __shfl(key, leader);
  if (__ballot(hit && key != k0) == 0) {
    if ((int)(threadIdx.x & 63) == leader) {
      const uint32_t c = (uint32_t)__popcll(m);
      atomicAdd(&h[bin], c);
      if (w) atomicAdd(&hm[bin], (unsigned long long)w * c);
    }
  } else if (hit) {
    atomicAdd(&h[bin], 1u);
    if (w) atomicAdd(&hm[bin], (unsigned long long)w);
  }
}

// Appends the participating lanes' (key, slot) pairs to an LDS list with one counter update per wave.
__device__ __forceinline__ void lds_append(uint32_t* counter, uint2* list, uint32_t room, uint32_t key, uint32_t slot,
                                           bool hit) {
  const uint64_t m = __ballot(hit);
  if (m == 0) return;
  const int lane = threadIdx.x & 63;
  const int leader = __ffsll((unsigned long long)m) - 1;
  uint32_t base = 0;
  if (lane == leader) base = atomicAdd(counter, (uint32_t)__popcll(m));
  base = __shfl(base, leader);
  if (hit) {
    const uint32_t at = base + (uint32_t)__popcll(m & ((1ull << lane) - 1));
    if (at < room) list[at] = uint2{key, slot};
  }
}

// Keys of the 16 slots s0 + x*256 + tid (x = 0..15) of a 4096-slot tile, all loads issued before
// any use; slots at or past `end` yield valid[x] = false.
__device__ __forceinline__ void load_tile_keys(const float* __restrict__ v, int64_t s0, int64_t end,
                                               uint32_t (&key)[16], bool (&valid)[16]) {
  float f[16];
#pragma unroll
  for (int x = 0; x < 16; ++x) {
    const int64_t j = s0 + x * 256 + threadIdx.x;
    valid[x] = j < end;
    f[x] = v[valid[x] ? j : end - 1];
  }
#pragma unroll
  for (int x = 0; x < 16; ++x) key[x] = order_key(f[x]);
}

// 12-bit histogram of a row's keys.
__global__ __launch_bounds__(256) void tk_hist(const float* __restrict__ vals, int64_t stride, int64_t chunk,
                                               int n_kv_heads, SelRows sr, TopkWs t) {
  __shared__ uint32_t lh[kBins12];
  const int row = blockIdx.y;
  const int64_t want = sr.want[row / n_kv_heads];
  if (want <= 0) return;
  const int64_t nsel = sr.nsel[row / n_kv_heads];
  const int64_t c0 = (int64_t)blockIdx.x * chunk;
  if (c0 >= nsel) return;
  int64_t c1 = c0 + chunk;
  if (c1 > nsel) c1 = nsel;
  for (int i = threadIdx.x; i < kBins12; i += 256) lh[i] = 0;
  __syncthreads();
  const float* v = vals + (int64_t)row * stride;
  for (int64_t s0 = c0; s0 < c1; s0 += 4096) {
    uint32_t key[16];
    bool valid[16];
    load_tile_keys(v, s0, c1, key, valid);
#pragma unroll
    for (int x = 0; x < 16; ++x)
      if (valid[x]) atomicAdd(&lh[key[x] >> 20], 1u);
  }
  __syncthreads();
  uint32_t* gh = t.hist + (int64_t)row * kBins12;
  for (int i = threadIdx.x; i < kBins12; i += 256) {
    const uint32_t c = lh[i];
    if (c) atomicAdd(&gh[i], c);
  }
}

// One workgroup per row: locates the bin b* of the `want`-th largest key (bins scanned from the
// top) and leaves (still-to-take, b*, too-many-candidates flag) in state.
__global__ __launch_bounds__(256) void tk_findbin(int n_kv_heads, SelRows sr, TopkWs t) {
  __shared__ uint32_t wsum[4];
  const int row = blockIdx.x;
  const int64_t want = sr.want[row / n_kv_heads];
  if (want <= 0) return;
  uint32_t* gh = t.hist + (int64_t)row * kBins12;
  uint32_t h[16], sum = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int b = kBins12 - 1 - (16 * threadIdx.x + i);
    h[i] = gh[b];
    gh[b] = 0;                 // leave the histogram clean for the next selection on this workspace
    sum += h[i];
  }
  uint32_t running = block_scan_excl<4>(sum, wsum);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (running < (uint32_t)want && (uint32_t)want <= running + h[i]) {
      t.state[4 * row + 1] = (uint32_t)want - running;                 // still to take inside the bin
      t.state[4 * row + 2] = kBins12 - 1 - (16 * threadIdx.x + i);     // b*
    }
    running += h[i];
  }
}

// Second pass over the row.  Every chunk writes, in slot order, the (key, slot) pairs of its slots
// in bin b* or above into its own list (room for the whole chunk, so it cannot overflow), and
// counts the ones strictly above the bin.  Lists are per chunk so that no two workgroups ever
// contend for an append position.
// range(&first, &last): the smallest and the largest key of the bin, asked for while the first tile is on its way.
// ABOVE: the keys above `first` are listed, in `room`, and those equal to it counted.
struct ListRoom {          // lists of a selection by a sampled key
  uint2* pairs;            // [rows][pair_row]: (key, slot), pair_chunk per chunk, the rest of a longer list left out
  uint32_t* slots;         // [rows][slot_row]: the whole list's slots, a chunk's slots per chunk (null: pair_chunk suffices)
  int64_t pair_row, pair_chunk, slot_row;
};
template <bool ABOVE, typename F>
__device__ __forceinline__ void collect_chunk(const float* __restrict__ vals, int64_t stride, int64_t chunk, int64_t nsel,
                                              int row, const TopkWs& t, F&& range, const ListRoom& room = ListRoom{}) {
  __shared__ uint32_t wsum[4];
  __shared__ uint32_t pc[64], po[64];
  __shared__ uint32_t s_total;
  const int64_t c0 = (int64_t)blockIdx.x * chunk;
  uint32_t* ncand = t.ncand + (int64_t)row * kMaxChunks + blockIdx.x;
  if (c0 >= nsel) {
    if (threadIdx.x == 0) { t.above[(int64_t)row * 1024 + blockIdx.x] = 0; *ncand = 0; }
    return;
  }
  int64_t c1 = c0 + chunk;
  if (c1 > nsel) c1 = nsel;
  const float* v = vals + (int64_t)row * stride;
  uint2* dst = t.cand + (int64_t)row * t.row_entries + (int64_t)blockIdx.x * chunk;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t cnt = 0, base = 0;
  uint32_t key[16];
  bool valid[16];
  load_tile_keys(v, c0, c1, key, valid);
  uint32_t first, last;
  range(&first, &last);
  for (int64_t s0 = c0; s0 < c1; s0 += 4096) {
    if (s0 != c0) load_tile_keys(v, s0, c1, key, valid);
    // slot order inside the tile is (x, wave, lane): one ballot per (x, wave), prefix over the 64 of them
    uint64_t mask[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      cnt += valid[x] && (ABOVE ? key[x] == first : key[x] > last);
      mask[x] = __ballot(valid[x] && (ABOVE ? key[x] > first : key[x] >= first));
      if (lane == 0) pc[x * 4 + w] = (uint32_t)__popcll(mask[x]);
    }
    __syncthreads();
    if (w == 0) {
      const uint32_t mine = pc[lane];
      const uint32_t inc = wave_scan_incl(mine);
      po[lane] = inc - mine;
      if (lane == 63) s_total = inc;
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      if ((mask[x] >> lane) & 1) {
        const uint32_t at = base + po[x * 4 + w] + (uint32_t)__popcll(mask[x] & ((1ull << lane) - 1));
        const uint32_t slot = (uint32_t)(s0 + x * 256 + threadIdx.x);
        if constexpr (ABOVE) {
          if (at < room.pair_chunk) room.pairs[row * room.pair_row + blockIdx.x * room.pair_chunk + at] = uint2{key[x], slot};
          if (room.slots != nullptr) room.slots[row * room.slot_row + blockIdx.x * chunk + at] = slot;
        } else {
          dst[at] = uint2{key[x], slot};
        }
      }
    }
    base += s_total;
    __syncthreads();
  }
  cnt = wave_sum(cnt);
  if (lane == 0) wsum[w] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    t.above[(int64_t)row * 1024 + blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    *ncand = base;
  }
}

__global__ __launch_bounds__(256) void tk_collect(const float* __restrict__ vals, int64_t stride, int64_t chunk,
                                                  int n_kv_heads, SelRows sr, TopkWs t) {
  const int row = blockIdx.y;
  if (sr.want[row / n_kv_heads] <= 0) return;
  collect_chunk<false>(vals, stride, chunk, sr.nsel[row / n_kv_heads], row, t, [&](uint32_t* first, uint32_t* last) {
    *first = t.state[4 * row + 2] << 20;
    *last = *first | 0xfffffu;
  });
}

// The same with a sampled key in place of a bin: the keys above it.
__global__ __launch_bounds__(256) void tk_collect_sampled(const float* __restrict__ vals, int64_t stride, int64_t chunk,
                                                          int n_kv_heads, SelRows sr, TopkWs t,
                                                          ListRoom room) {
  const int row = blockIdx.y;
  if (sr.want[row / n_kv_heads] <= 0) return;
  collect_chunk<true>(vals, stride, chunk, sr.nsel[row / n_kv_heads], row, t, [&](uint32_t* first, uint32_t* last) {
    *first = t.state[4 * row];
    *last = 0;
  }, room);
}

// One workgroup per row: finishes the select inside bin b* (two 10-bit passes over the
// candidates, or over the whole row when there were too many to keep) and builds the chunk
// offsets of (#key > T, #key == T) for the ordered emit.
constexpr int kResolveLds = 5120;   // candidates staged in LDS by tk_resolve (40 KiB)

// One workgroup per row: finishes the select inside bin b* (two 10-bit passes over the list
// entries that lie in that bin) and builds the chunk offsets of (#key > T, #key == T) for the
// ordered emit.
__global__ __launch_bounds__(1024) void tk_resolve(int64_t chunk, int nchunks, int n_kv_heads, SelRows sr, TopkWs t) {
  __shared__ uint32_t h[1024], e[1024], cnt[1024], wsum[16];
  __shared__ uint32_t s_prefix, s_rem, s_n;
  __shared__ uint2 lc[kResolveLds];
  const int row = blockIdx.x;
  if (sr.want[row / n_kv_heads] <= 0) return;
  const uint32_t bin = t.state[4 * row + 2];
  const uint2* cand = t.cand + (int64_t)row * t.row_entries;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t prefix = bin << 20, rem = t.state[4 * row + 1];
  cnt[tid] = tid < nchunks ? t.ncand[(int64_t)row * kMaxChunks + tid] : 0;
  if (tid == 0) s_n = 0;
  __syncthreads();
  // sweep(f): f(key, slot, hit) over every list entry of the row, hit = the entry exists and lies in bin
  // b*; f is called by all lanes of a wave together.  Each wave takes 16 chunks per step and fetches the
  // first 64 entries of all of them in one batch of loads (most lists are shorter than that), so a step
  // costs one memory round trip; longer lists follow, 8 loads in flight.
  auto sweep = [&](auto&& f) {
    for (int c0 = 0; c0 < nchunks; c0 += 256) {
      uint2 ent[16];
      uint32_t m[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int c = c0 + wv * 16 + u;
        m[u] = c < nchunks ? cnt[c] : 0;
        ent[u] = uint2{0, 0};
        if ((uint32_t)lane < m[u]) ent[u] = cand[(int64_t)c * chunk + lane];
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) f(ent[u].x, ent[u].y, (uint32_t)lane < m[u] && (ent[u].x >> 20) == bin);
#pragma unroll 1
      for (int u = 0; u < 16; ++u) {      // long lists (clustered heavy hitters, mass ties)
        const int c = c0 + wv * 16 + u;
        for (uint32_t i0 = 64 + lane; i0 < m[u] + lane; i0 += 512) {
          uint2 x[8];
#pragma unroll
          for (int v = 0; v < 8; ++v) {
            x[v] = uint2{0, 0};
            if (i0 + 64 * v < m[u]) x[v] = cand[(int64_t)c * chunk + i0 + 64 * v];
          }
#pragma unroll
          for (int v = 0; v < 8; ++v) f(x[v].x, x[v].y, i0 + 64 * v < m[u] && (x[v].x >> 20) == bin);
        }
      }
    }
  };
  // staging: the in-bin entries go to the LDS list; one counter update per wave and batch of loads
  {
    const uint64_t lt = (1ull << lane) - 1;
    auto stage = [&](const uint2* x, const bool* hit, int cntx) {
      uint64_t mk[16];
      uint32_t off[16], tot = 0;
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (u < cntx) { mk[u] = __ballot(hit[u]); off[u] = tot; tot += (uint32_t)__popcll(mk[u]); }
      if (tot == 0) return;
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(&s_n, tot);
      base = __shfl(base, 0);
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (u < cntx && hit[u]) {
          const uint32_t at = base + off[u] + (uint32_t)__popcll(mk[u] & lt);
          if (at < (uint32_t)kResolveLds) lc[at] = x[u];
        }
    };
    for (int c0 = 0; c0 < nchunks; c0 += 256) {
      uint2 ent[16];
      bool hit[16];
      uint32_t m[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int c = c0 + wv * 16 + u;
        m[u] = c < nchunks ? cnt[c] : 0;
        ent[u] = uint2{0, 0};
        if ((uint32_t)lane < m[u]) ent[u] = cand[(int64_t)c * chunk + lane];
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) hit[u] = (uint32_t)lane < m[u] && (ent[u].x >> 20) == bin;
      stage(ent, hit, 16);
#pragma unroll 1
      for (int u = 0; u < 16; ++u) {
        const int c = c0 + wv * 16 + u;
        for (uint32_t i0 = 64 + lane; i0 < m[u] + lane; i0 += 512) {
          uint2 x[8];
          bool hx[8];
#pragma unroll
          for (int v = 0; v < 8; ++v) {
            x[v] = uint2{0, 0};
            if (i0 + 64 * v < m[u]) x[v] = cand[(int64_t)c * chunk + i0 + 64 * v];
          }
#pragma unroll
          for (int v = 0; v < 8; ++v) hx[v] = i0 + 64 * v < m[u] && (x[v].x >> 20) == bin;
          stage(x, hx, 8);
        }
      }
    }
  }
  __syncthreads();
  const uint32_t nst = s_n;
  const bool staged = nst <= (uint32_t)kResolveLds;
  auto visit = [&](auto&& f) {
    if (staged) {
      for (uint32_t i0 = 0; i0 < nst; i0 += 1024) {
        const bool hit = i0 + tid < nst;
        const uint2 x = lc[hit ? i0 + tid : 0];
        f(x.x, x.y, hit);
      }
    } else {
      sweep(f);
    }
  };
  for (int pass = 0; pass < 2; ++pass) {
    const int shift = pass == 0 ? 10 : 0;
    h[tid] = 0;
    __syncthreads();
    visit([&](uint32_t key, uint32_t, bool hit) {
      lds_count(h, (key >> shift) & 1023u, hit && (key >> (shift + 10)) == (prefix >> (shift + 10)), !staged);
    });
    __syncthreads();
    const uint32_t mine = h[1023 - tid];                    // thread tid owns bin 1023 - tid
    const uint32_t running = block_scan_excl<16>(mine, wsum);
    if (running < rem && rem <= running + mine) {
      s_prefix = prefix | ((uint32_t)(1023 - tid) << shift);
      s_rem = rem - running;
    }
    __syncthreads();
    prefix = s_prefix;
    rem = s_rem;
    __syncthreads();
  }
  const uint32_t T = prefix;
  h[tid] = 0;
  e[tid] = 0;
  __syncthreads();
  visit([&](uint32_t key, uint32_t slot, bool hit) {
    lds_count(h, (uint32_t)(slot / chunk), hit && key > T, !staged);
    lds_count(e, (uint32_t)(slot / chunk), hit && key == T, !staged);
  });
  __syncthreads();
  const uint32_t g = (tid < nchunks) ? t.above[(int64_t)row * 1024 + tid] + h[tid] : 0;
  const uint32_t q = (tid < nchunks) ? e[tid] : 0;
  const uint32_t og = block_scan_excl<16>(g, wsum);
  const uint32_t oe = block_scan_excl<16>(q, wsum);
  if (tid < nchunks) {
    t.coff[((int64_t)row * nchunks + tid) * 2] = og;
    t.coff[((int64_t)row * nchunks + tid) * 2 + 1] = oe;
  }
  if (tid == 0) { t.state[4 * row] = T; t.state[4 * row + 1] = rem; }
}

// Ordered emit from the per-chunk lists (already in slot order): no further pass over the row.
//   selected(j) = key_j > T  or  (key_j == T and #{i < j : key_i == T} < r_eq)
//   position(j) = #{i < j : key_i > T} + min(#{i < j : key_i == T}, r_eq)
__global__ __launch_bounds__(256) void tk_emit_lists(int64_t chunk, int nchunks, int n_kv_heads, SelRows sr, TopkWs t,
                                                     int32_t k, int32_t* __restrict__ idx, int32_t* __restrict__ count,
                                                     bool count_from_state) {
  __shared__ uint32_t wsum[2][4];
  const int row = blockIdx.y;
  const int64_t want = sr.want[row / n_kv_heads];
  if (blockIdx.x == 0 && threadIdx.x == 0)
    count[row] = want > 0 ? (count_from_state ? (int32_t)t.prow[4 * row + 2] : (int32_t)want) : 0;
  if (want <= 0) return;
  const uint32_t m = t.ncand[(int64_t)row * kMaxChunks + blockIdx.x];
  if (m == 0) return;
  const uint32_t T = t.state[4 * row], req = t.state[4 * row + 1];
  uint32_t base_g = t.coff[((int64_t)row * nchunks + blockIdx.x) * 2];
  uint32_t base_e = t.coff[((int64_t)row * nchunks + blockIdx.x) * 2 + 1];
  const uint2* src = t.cand + (int64_t)row * t.row_entries + (int64_t)blockIdx.x * chunk;
  int32_t* out = idx + (int64_t)row * k;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (uint32_t p0 = 0; p0 < m; p0 += 512) {
    uint2 en[2];
    bool fg[2], fe[2];
    uint32_t ng = 0, ne = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t p = p0 + 2 * threadIdx.x + i;
      en[i] = src[p < m ? p : m - 1];
      fg[i] = p < m && en[i].x > T;
      fe[i] = p < m && en[i].x == T;
      ng += fg[i]; ne += fe[i];
    }
    const uint32_t ig = wave_scan_incl(ng), ie = wave_scan_incl(ne);
    if (lane == 63) { wsum[0][w] = ig; wsum[1][w] = ie; }
    __syncthreads();
    uint32_t pg = base_g + ig - ng, pe = base_e + ie - ne;
    for (int x = 0; x < w; ++x) { pg += wsum[0][x]; pe += wsum[1][x]; }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (fg[i] || (fe[i] && pe < req)) out[pg + (pe < req ? pe : req)] = (int32_t)en[i].y;
      pg += fg[i]; pe += fe[i];
    }
    base_g += wsum[0][0] + wsum[0][1] + wsum[0][2] + wsum[0][3];
    base_e += wsum[1][0] + wsum[1][1] + wsum[1][2] + wsum[1][3];
    __syncthreads();
  }
}


// the float of an order key (the +0 of the two zeros)
__device__ __forceinline__ float key_to_float(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// ---------------------------------------------------------------------------------------
// Top-k of short rows in one launch: a 1024-thread workgroup holds a whole row of scores in registers, KPT values per
// thread, wave w owning the KPT * 64 consecutive slots from w * KPT * 64 on (a wave's x-th load is 64 of them, so slot
// order is (wave, x, lane)).  hca_topk, 8 rows of 4 Ki / 16 Ki / 32 Ki / 40 Ki slots, 1024 to select: 8 / 10.3 / 13.5 / 14.9
// us (8 / 11.2 / 18.1 / 21.6 without step 0), against 31 / 35 / - / 39 us for the six launches over the whole chip; with
// the scan in front (hca_score_topk), 4 Ki / 16 Ki / 32 Ki: 13 / 18 / 23 (13 / 19 / 28 without step 0) against 39 / 39 / 41 us
// for sample, threshold, selecting scan, selection and its fall-back pair.
//   0. Rows of 8 Ki slots and more, in a call whose longest has more than 12 Ki, of which few are wanted: a bound below which the want-th largest lies almost never, from
//      1024 samples (their rank-th largest, rank = the expected one + 3.5 standard deviations + 6; binned as in step 1).  The
//      values at or above it and the NaNs - 2000 of 32 Ki for 1024 to select - go to a list in LDS in slot order, and only
//      those, P per thread, are binned, ranked and placed.  A list longer than that, or more than kRankMax of it in the bin of
//      the last one (ties): all steps, their window over the values at or above the bound; too short a list: all steps.  The
//      lists are expected to fill three quarters of the room at most (six entries per thread for rows beyond 16 Ki; of four
//      one row in fifty was too long at the rule's end, 18.5 -> 22 us), so it takes ties or a row that follows the samples' places.
//      What those cost, 8 rows of 32 Ki, 1024 to select, without step 0 / with it: all samples among the smallest 18.6 / 24,
//      among the largest 18 / 24, all slots equal 12.2 / 16; steps of 0.5 between the values 43.6 / 31, a NaN in every
//      row 36.6 / 13.5.  Of 11.4 us in the kernel loads and window take 3.5, the bound 1, the list 4, the rest 3, for 16.5.
//   1. smallest and largest value per wave; 4096 bins spread evenly over a window in which most of the row lies, so that
//      neither the counters are fought over nor most of them stay empty (the keys of one row share their exponent bits).
//      The window reaches a quarter of its width beyond the fourth smallest and the fourth largest of the waves' extremes:
//      a few values far outside - a sink, a few masked slots - fall into the end bins and do not move it (a window from
//      the smallest to the largest value took 89 us for 8 rows of 40 Ki slots with one such value, 39 over the whole
//      chip).  Where masked slots are everywhere the smallest values are taken again without them.  Binning by value is
//      monotone in the key - a difference, a product, a clamp and a truncation - which is all the selection needs.  Rows
//      with +inf or NaNs, or too wide for a finite scale, are binned by the key's leading 12 bits.  The lowest bin
//      is not counted, it holds the row's others.
//   2. the bin that holds the want-th largest key; its keys are ranked against each other when there are at most 512,
//      else by radix levels over the distance from the bin's smallest key (ties, one far outlier).
//   3. the ordered emit, positions by ballot:  selected(j) = key_j > T  or  (key_j == T and fewer than r_eq equals
//      before it), position(j) = #{i < j : key_i > T} + min(#{i < j : key_i == T}, r_eq).
// Steps 1 to 3 are bound by the issue of one compute unit's vector ALUs, about 40 instructions per slot, with step 0 about 13;
// then the chain of its dozen barriers counts as much.  The row in LDS with rolled
// loops instead of registers: 35.6 us per 32 Ki slots.
constexpr int kRankMax = 512;
// entries of the list per thread, and how many are expected at most: rows of up to 16 Ki slots, longer ones
__host__ __device__ constexpr int sift_per(int kpt) { return kpt <= 16 ? 4 : 6; }
__host__ __device__ constexpr uint32_t sift_expected(int kpt) { return kpt <= 16 ? 3072 : 3584; }
constexpr uint32_t kSiftMin = 8192;           // slots of a row; of the longest one of a call:
constexpr int64_t kSiftCall = 12288;
// rank among 1024 samples, expected number of those among the wanted and a margin, whose value bounds the list of step 0
__host__ __device__ __forceinline__ uint32_t sift_rank(uint32_t want, uint32_t n) {
  const float mean = (float)want * 1024.0f / (float)n;
  return (uint32_t)(mean + 3.5f * sqrtf(mean) + 6.0f);
}

struct RowSelectFused {      // what hca_score_topk keeps beside the result (null spec: a plain top-k)
  uint32_t* spec;
  uint32_t* ncand;
  uint32_t* mon;
  int32_t nchunks;
};

// f(turn) for the fifteen other lanes of a row of sixteen, turn(v) = that lane's v; and what the row's lanes hold at most
// and at least, on every lane.
template <int N>
struct Row16 {
  __device__ __forceinline__ float operator()(float v) const {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, false));
  }
};
template <int N = 1, typename F>
__device__ __forceinline__ void row16_each(F&& f) {
  f(Row16<N>());
  if constexpr (N < 15) row16_each<N + 1>(f);
}
__device__ __forceinline__ float row16_min(float v) {
  v = fminf(v, Row16<8>()(v));
  v = fminf(v, Row16<4>()(v));
  v = fminf(v, Row16<2>()(v));
  return fminf(v, Row16<1>()(v));
}
__device__ __forceinline__ float row16_max(float v) { return -row16_min(-v); }

template <int KPT, bool kSift>
__global__ __launch_bounds__(1024) void tk_row_select(const float* __restrict__ vals, int64_t stride, int n_kv_heads,
                                                      SelRows sr, int32_t k, int32_t* __restrict__ idx,
                                                      int32_t* __restrict__ count, RowSelectFused fu) {
  __shared__ uint32_t h[kBins12], list[kRankMax], wsum[16], wlo[16], whi[16], wplain[16];
  __shared__ uint32_t s_bin, s_rem, s_cb, s_n, s_T, s_req, s_flags;
  __shared__ __align__(16) float s_win[8];
  constexpr int P = sift_per(KPT), kSiftMax = 1024 * P;
  __shared__ __align__(16) float s_kept[kSift ? kSiftMax : 4];
  __shared__ __align__(16) uint16_t s_slot[kSift ? kSiftMax : 4];         // (rows have at most kRowSelectMax slots)
  const int row = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t want64 = sr.want[row / n_kv_heads];
  const uint32_t n = want64 > 0 ? (uint32_t)sr.nsel[row / n_kv_heads] : 0u;
  if (fu.spec != nullptr) {
    // every resident slot is a candidate, none of them came through a threshold
    for (int c = tid; c < fu.nchunks; c += 1024) fu.ncand[(int64_t)row * kSelectMaxChunks + c] = c == 0 ? n : 0u;
    if (tid == 0) {
      fu.spec[4 * row + 1] = 0;
      if (want64 > 0 && fu.mon != nullptr) {
        uint32_t* m = fu.mon + 4 * row;
        m[0] += 1;
        m[1] = n < m[1] ? n : m[1];
        m[2] = n > m[2] ? n : m[2];
      }
    }
  }
  if (want64 <= 0) {
    if (tid == 0) count[row] = 0;
    return;
  }
  const uint32_t want = (uint32_t)want64;
  const float* v = vals + (int64_t)row * stride;
  uint32_t s0 = (uint32_t)wv * (KPT * 64) + (uint32_t)lane;
  // the sample of step 0, one place in each of 1024 equal parts of the row
  float sample = 0.0f;
  const uint32_t rank = kSift ? sift_rank(want, n) : 0u;
  const bool sift = kSift && n >= kSiftMin && rank * n <= sift_expected(KPT) * 1024u;
  if (sift) {
    const uint32_t from = ((uint32_t)tid * n) >> 10, part = n >> 10;
    sample = v[from + ((((uint32_t)tid * 40503u) & 0xffffu) * part >> 16)];
  }
  float f[KPT];                                             // (lanes past the row's end hold its last slot for now)
#pragma unroll
  for (int x = 0; x < KPT; ++x) f[x] = v[s0 + x * 64 < n ? s0 + x * 64 : n - 1];
  // between the phases: what a phase derived from the values (bins, lane masks, KPT of each) is not carried along in
  // registers to the next one, which would spill
  auto forget = [&]() {
    asm volatile("" : "+v"(s0));
#pragma unroll
    for (int x = 0; x < KPT; ++x) asm volatile("" : "+v"(f[x]));
  };
  for (int i = tid; i < kBins12; i += 1024) h[i] = 0;
  if (tid == 0) { s_n = 0; s_T = 0xffffffffu; s_req = 0; }
  float vlo = INFINITY, vhi = -INFINITY, from = 0.0f, scale = 0.0f;
  bool plain = true;                                        // no NaN and no +infinity
  // the window of the bins, from the extremes and the plainness of each lane's values; `waves`: those with values;
  // lowest(cut): the smallest of the lane's values that are not below cut
  auto find_window = [&](uint32_t waves, auto&& lowest) {
    vlo = wave_min(vlo);
    vhi = wave_max(vhi);
    plain = __builtin_amdgcn_ballot_w64(!plain) == 0;
    if (lane == 0) { wlo[wv] = __float_as_uint(vlo); whi[wv] = __float_as_uint(vhi); wplain[wv] = plain; }
    __syncthreads();
    // lo4, hi4: the fourth smallest and the fourth largest extreme of the waves with slots
    auto window = [&](float lo4, float hi4) {
      const float edge = lo4 < hi4 ? 0.25f * (hi4 - lo4) : INFINITY;
      const float first = fmaxf(vlo, lo4 - edge);
      return float2{first, 4095.0f / (fminf(vhi, hi4 + edge) - first)};
    };
    if (wv == 0) {
      const uint32_t i = (uint32_t)(lane & 15);
      const uint32_t fourth = waves > 3 ? 3 : waves - 1;
      vlo = i < waves ? __uint_as_float(wlo[i]) : INFINITY;
      vhi = i < waves ? __uint_as_float(whi[i]) : -INFINITY;
      plain = i >= waves || wplain[i] != 0;
      uint32_t below = 0, over = 0;
      row16_each([&](auto turn) {
        below += turn(vlo) < vlo;
        over += turn(vhi) > vhi;
      });
      float lo4 = i < waves && below <= fourth ? vlo : -INFINITY;      // the largest of those with at most three before them
      float hi4 = i < waves && over <= fourth ? vhi : INFINITY;
      lo4 = row16_max(lo4);
      hi4 = row16_min(hi4);
      vlo = row16_min(vlo);
      // how much the waves' largest values differ, those left out that hold nothing but the row's smallest value
      const float apart = hi4 - row16_min(vhi > vlo ? vhi : INFINITY);
      vhi = row16_max(vhi);
      plain = __builtin_amdgcn_ballot_w64(!plain) == 0;
      const float2 w = window(lo4, hi4);
      if (lane == 0) {
        // far more below the top than that: masked slots in most waves, say
        const bool masked = plain && apart > 0.0f && hi4 - lo4 > 512.0f * apart;
        s_win[0] = vlo; s_win[1] = vhi; s_win[2] = w.x; s_win[3] = w.y;
        s_win[4] = hi4; s_win[5] = hi4 - 256.0f * apart;
        s_flags = (plain ? 1u : 0u) | (masked ? 2u : 0u);
      }
    }
    __syncthreads();
    vlo = s_win[0];
    vhi = s_win[1];
    plain = (s_flags & 1u) != 0;
    from = s_win[2];
    scale = s_win[3];
    forget();
    if (s_flags & 2u) {                                     // the smallest value again, without those
      float m = lowest(s_win[5]);
      m = wave_min(m);
      if (lane == 0) wlo[wv] = __float_as_uint(m);
      __syncthreads();
      for (int x = 0; x < 16; ++x) m = fminf(m, __uint_as_float(wlo[x]));
      const float2 w = window(m, s_win[4]);
      from = w.x;
      scale = w.y;
      forget();
    }
  };
  // the bin that holds the rem-th largest entry of the counters in h: published to s_bin / s_rem / s_cb.  all: the
  // number of entries, of which the lowest bin's are not counted (0: it is counted)
  auto find_bin = [&](uint32_t rem, uint32_t all) {
    uint32_t hb[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) { hb[i] = h[kBins12 - 1 - (4 * tid + i)]; sum += hb[i]; }
    uint32_t running = block_scan_excl<16>(sum, wsum);
    if (tid == 1023 && all != 0) hb[3] = all - (running + sum);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (running < rem && rem <= running + hb[i]) {
        s_bin = (uint32_t)(kBins12 - 1 - (4 * tid + i));
        s_rem = rem - running;
        s_cb = hb[i];
      }
      running += hb[i];
    }
    __syncthreads();
  };
  // the rem-th largest of the cb keys in `list`, published to s_T, and how many of its equals are taken to s_req
  auto rank_list = [&](uint32_t cb, uint32_t rem) {
    __syncthreads();
    if ((uint32_t)tid < cb) {
      const uint32_t ki = list[tid];
      uint32_t gt = 0, eq = 0;
      for (uint32_t j = 0; j < cb; ++j) {
        const uint32_t kj = list[j];
        gt += kj > ki;
        eq += kj == ki;
      }
      if (gt < rem && rem <= gt + eq) { s_T = ki; s_req = rem - gt; }         // equal keys write equal values
    }
    __syncthreads();
  };
  float bound = -INFINITY;                                  // at least `want` values are not below it
  if constexpr (kSift) {
    // 0. (uniform over the workgroup)
    if (sift) {
      vlo = vhi = sample;
      plain = sample < INFINITY;
      find_window(16u, [&](float cut) { return sample >= cut ? sample : INFINITY; });
      // up to the largest sample, where that is not far outside: the largest may all be one wave's
      if (vhi - from < 16.0f * 4095.0f / scale) scale = 4095.0f / (vhi - from);
      if (plain && scale > 0.0f && scale < INFINITY) {
        atomicAdd(&h[(uint32_t)__builtin_amdgcn_fmed3f((sample - from) * scale, 0.0f, 4095.0f)], 1u);
        __syncthreads();
        find_bin(rank, 0u);
        const float cut = from + ((float)s_bin - 0.25f) / scale, top = from + 4095.0f / scale;     // (ties on a bin's edge)
        const float fine = 4093.0f / (top - cut);
        for (int i = tid; i < kBins12; i += 1024) h[i] = 0;
        // those at or above it and the NaNs, in slot order: (wave, x, lane)
        uint32_t mine = 0;
        const bool whole = (uint32_t)(wv + 1) * (KPT * 64) <= n;
        if (whole) {
#pragma unroll
          for (int x = 0; x < KPT; ++x) mine += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(!(f[x] < cut)));
        } else {
#pragma unroll
          for (int x = 0; x < KPT; ++x) mine += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(!(f[x] < cut) && s0 + x * 64 < n));
        }
        forget();
        if (lane == 0) wlo[wv] = mine;
        __syncthreads();
        uint32_t at = 0, all = 0;
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          at += x < wv ? wlo[x] : 0u;
          all += wlo[x];
        }
        if (all >= want) bound = cut;
        if (all >= want && all <= (uint32_t)kSiftMax && fine > 0.0f && fine < INFINITY) {
          auto keep = [&](auto&& hit) {
#pragma unroll
            for (int x = 0; x < KPT; ++x) {
              const uint64_t m = __builtin_amdgcn_ballot_w64(hit(x));
              const uint32_t p = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, at));
              if (hit(x)) {
                s_kept[p] = f[x];
                s_slot[p] = (uint16_t)(s0 + x * 64);
              }
              at += (uint32_t)__popcll(m);
            }
          };
          if (whole) keep([&](int x) { return !(f[x] < cut); });
          else keep([&](int x) { return !(f[x] < cut) && s0 + x * 64 < n; });
          __syncthreads();
          forget();
          // P of them per thread, one behind the other; bin 0 is for the negative NaNs alone, the smallest keys of all
          float c[P];
          uint32_t bin[P];
#pragma unroll
          for (int i = 0; i < P; ++i) {
            c[i] = s_kept[P * tid + i];
            const bool in = (uint32_t)(P * tid + i) < all, nan = c[i] != c[i];
            const float at_bin = __builtin_amdgcn_fmed3f((c[i] - cut) * fine + 2.0f, 1.0f, 4095.0f);
            bin[i] = !in ? 0xffffffffu : nan ? ((__float_as_uint(c[i]) >> 31) != 0 ? 0u : 4095u) : (uint32_t)at_bin;
            if (in) atomicAdd(&h[bin[i]], 1u);
          }
          __syncthreads();
          find_bin(want, 0u);
          const uint32_t cb = s_cb, rem = s_rem, b0 = s_bin;
          if (cb <= (uint32_t)kRankMax && b0 != 0) {        // (bin 0: values below the bound come before these)
#pragma unroll
            for (int i = 0; i < P; ++i)
              if (bin[i] == b0) list[atomicAdd(&s_n, 1u)] = order_key(c[i]);
            rank_list(cb, rem);
            const uint32_t T = s_T, req = s_req;
            uint32_t ng = 0, ne = 0;
#pragma unroll
            for (int i = 0; i < P; ++i) {
              const bool in = bin[i] != 0xffffffffu;
              ng += in && order_key(c[i]) > T;
              ne += in && order_key(c[i]) == T;
            }
            const uint32_t before = block_scan_excl<16>(ng | ne << 16, wsum);
            uint32_t g = before & 0xffffu, e = before >> 16;
            int32_t* out = idx + (int64_t)row * k;
            if (tid == 0) count[row] = (int32_t)want;
#pragma unroll
            for (int i = 0; i < P; ++i) {
              const bool in = bin[i] != 0xffffffffu, is_g = in && order_key(c[i]) > T, is_e = in && order_key(c[i]) == T;
              if (is_g || (is_e && e < req)) out[g + (e < req ? e : req)] = (int32_t)s_slot[P * tid + i];
              g += is_g;
              e += is_e;
            }
            return;
          }
        }
        __syncthreads();                                    // everybody has read what the steps below write again
        for (int i = tid; i < kBins12; i += 1024) h[i] = 0;
      }
      vlo = INFINITY;
      vhi = -INFINITY;
      plain = true;
      __syncthreads();
    }
  }
  // the window of the values that are not below the bound (without one: of all), which at least `want` are
#pragma unroll
  for (int x = 0; x < KPT; ++x) {
    const bool counts = !kSift || f[x] >= bound;
    vlo = counts ? fminf(vlo, f[x]) : vlo;
    vhi = counts ? fmaxf(vhi, f[x]) : vhi;
    plain = plain && f[x] < INFINITY;
  }
  find_window((n + KPT * 64 - 1) / (KPT * 64), [&](float cut) {
    float m = INFINITY;
    if (kSift) cut = fmaxf(cut, bound);
#pragma unroll
    for (int x = 0; x < KPT; ++x) m = f[x] >= cut ? fminf(m, f[x]) : m;
    return m;
  });
  if (kSift && bound > -INFINITY) from -= 1.5f / scale;     // (the lowest bin is the others')
  const bool by_value = plain && scale > 0.0f && scale < INFINITY;
  if (plain) {                                              // past the row's end: the lowest bin, below every threshold
#pragma unroll
    for (int x = 0; x < KPT; ++x) f[x] = s0 + x * 64 < n ? f[x] : -INFINITY;
  }
  uint32_t T, req;
  if (plain && vlo == vhi) {                               // all equal: the want lowest slots
    T = order_key(vlo);
    req = want;
  } else {
    auto live = [&](int x) { return s0 + x * 64 < n; };
    auto bin_of = [&](int x) {
      return by_value ? (uint32_t)__builtin_amdgcn_fmed3f((f[x] - from) * scale, 0.0f, 4095.0f) : order_key(f[x]) >> 20;
    };
    if (by_value) {
#pragma unroll
      for (int x = 0; x < KPT; ++x) {
        const uint32_t b = bin_of(x);
        if (b != 0) atomicAdd(&h[b], 1u);
      }
    } else {
#pragma unroll
      for (int x = 0; x < KPT; ++x)
        if (live(x)) atomicAdd(&h[bin_of(x)], 1u);
    }
    __syncthreads();
    find_bin(want, by_value ? n : 0u);
    forget();
    const uint32_t b0 = s_bin;
    uint32_t rem = s_rem, cb = s_cb;
    // the keys still in question: those of bin b0, and among them those whose distance from `base` starts with pd
    uint32_t base = 0, pd = 0;
    int sbits = 32;                                         // unknown bits of the distance; 32: every key of the bin
    if (cb > (uint32_t)kRankMax) {
      uint32_t lo = 0xffffffffu, hi = 0;
#pragma unroll
      for (int x = 0; x < KPT; ++x)
        if (live(x) && bin_of(x) == b0) {
          const uint32_t kk = order_key(f[x]);
          lo = kk < lo ? kk : lo;
          hi = kk > hi ? kk : hi;
        }
      lo = wave_min(lo);
      hi = wave_max(hi);
      __syncthreads();                                      // everybody has read the row's extremes
      if (lane == 0) { wlo[wv] = lo; whi[wv] = hi; }
      __syncthreads();
      for (int x = 0; x < 16; ++x) { lo = wlo[x] < lo ? wlo[x] : lo; hi = whi[x] > hi ? whi[x] : hi; }
      base = lo;
      int left = lo == hi ? 0 : 32 - __clz((int)(hi - lo));           // 0: all equal
      bool first = true;
      while (left > 0 && cb > (uint32_t)kRankMax) {         // uniform over the workgroup
        forget();
        const int width = left > 12 ? 12 : left, ns = left - width;
        __syncthreads();
        for (int i = tid; i < kBins12; i += 1024) h[i] = 0;
        __syncthreads();
#pragma unroll
        for (int x = 0; x < KPT; ++x) {
          const uint32_t d = order_key(f[x]) - base;
          lds_count(h, (d >> ns) & ((1u << width) - 1u), live(x) && bin_of(x) == b0 && (first || (d >> left) == pd), true);
        }
        __syncthreads();
        find_bin(rem, 0);
        pd = first ? s_bin : ((pd << width) | s_bin);
        rem = s_rem;
        cb = s_cb;
        left = ns;
        first = false;
      }
      sbits = left;
    }
    forget();
    if (sbits == 0) {                                       // the distance is fully known
      T = base + pd;
      req = rem;
    } else {
#pragma unroll
      for (int x = 0; x < KPT; ++x) {
        bool hit = live(x) && bin_of(x) == b0;
        if (__builtin_amdgcn_ballot_w64(hit) == 0) continue;
        const uint32_t kk = order_key(f[x]);
        hit = hit && (sbits == 32 || ((kk - base) >> sbits) == pd);
        const uint64_t m = __builtin_amdgcn_ballot_w64(hit);
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s_n, (uint32_t)__popcll(m));
        at = __builtin_amdgcn_readfirstlane(at);
        if (hit) list[at + (uint32_t)__popcll(m & ((1ull << lane) - 1))] = kk;
      }
      rank_list(cb, rem);
      T = s_T;
      req = s_req;
    }
  }
  // ordered emit
  int32_t* out = idx + (int64_t)row * k;
  if (tid == 0) count[row] = (int32_t)want;
  auto emit = [&](auto&& above, auto&& equal) {
    forget();
    uint32_t ng = 0, ne = 0;
#pragma unroll
    for (int x = 0; x < KPT; ++x) {
      ng += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(above(x)));
      ne += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(equal(x)));
    }
    forget();
    __syncthreads();                                        // (wlo and whi have been read)
    if (lane == 0) { wlo[wv] = ng; whi[wv] = ne; }
    __syncthreads();
    uint32_t pg = 0, pe = 0;
#pragma unroll
    for (int x = 0; x < 16; ++x) { pg += x < wv ? wlo[x] : 0; pe += x < wv ? whi[x] : 0; }
#pragma unroll
    for (int x = 0; x < KPT; ++x) {
      const bool is_g = above(x), is_e = equal(x);
      const uint64_t mg = __builtin_amdgcn_ballot_w64(is_g), me = __builtin_amdgcn_ballot_w64(is_e);
      if ((mg | me) == 0) continue;
      const uint32_t g = pg + __builtin_amdgcn_mbcnt_hi((uint32_t)(mg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mg, 0u));
      if (me == 0) {
        if (is_g) out[g + (pe < req ? pe : req)] = (int32_t)(s0 + x * 64);
      } else {
        const uint32_t e = pe + __builtin_amdgcn_mbcnt_hi((uint32_t)(me >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)me, 0u));
        if (is_g || (is_e && e < req)) out[g + (e < req ? e : req)] = (int32_t)(s0 + x * 64);
        pe += (uint32_t)__popcll(me);
      }
      pg += (uint32_t)__popcll(mg);
    }
  };
  const float tf = key_to_float(T);
  if (plain && tf > -INFINITY) {
    // values compare like their keys (the two zeros are equal both ways); past the row's end: -inf
    emit([&](int x) { return f[x] > tf; }, [&](int x) { return f[x] == tf; });
  } else {
    emit([&](int x) { return s0 + x * 64 < n && order_key(f[x]) > T; },
         [&](int x) { return s0 + x * 64 < n && order_key(f[x]) == T; });
  }
}

// Longest row of the one-launch form: 40 Ki slots are what fits the 128 registers of a 1024-thread workgroup, and keep a
// 32 Ki context on this side while it grows by the tokens it decodes.  The line lies where the registers end and not where
// the forms are level.  hca_topk / hca_score_topk on the GPU, us, 40 960 slots here and 40 961 over the chip: 8 rows, 1024 to
// select 13.9 / 20.8 and 27.4 / 33.7, 4096 to select (no step 0) 22.3 / 28.6 and 28.7 / 34.7; 32 rows, 4096: 22.9 / 45.4 and
// 29.2 / 45.8; one row, 4096: 21.9 / 25.7 and 25.3 / 30.8.
constexpr int64_t kRowSelectMax = 40960;

static int32_t launch_row_select(const float* vals, int64_t stride, int rows, int n_kv_heads, const SelRows& sr,
                                 int64_t nmax, int32_t k, int32_t* idx, int32_t* count, const RowSelectFused& fu,
                                 hipStream_t st) {
  // step 0 where the longest row's list is expected to fit (a shorter row's is no longer); its code beside the other's costs
  // a row that does without 1 us of 23.  Up to 12 Ki slots it saves nothing: 8 rows of 9000, 256 / 1024 / 2250 to select, without
  // and with it 10.1 / 10.4 / 10.5 and 10.4 / 10.5 / 10.6 us; of 14 336 10.6 / 11.1 / 11.2 and 10.4 / 10.6 / 10.8
  const bool sift = nmax > kSiftCall && k < nmax &&
                    sift_rank((uint32_t)k, (uint32_t)nmax) * (uint64_t)nmax <= (uint64_t)sift_expected(nmax <= 16 * 1024 ? 16 : 32) * 1024u;
#define HCA_ROW_SELECT(KPT, SIFT) tk_row_select<KPT, SIFT><<<rows, 1024, 0, st>>>(vals, stride, n_kv_heads, sr, k, idx, count, fu)
  if (nmax <= 4 * 1024) HCA_ROW_SELECT(4, false);
  else if (nmax <= 8 * 1024) HCA_ROW_SELECT(8, false);
  else if (nmax <= 16 * 1024 && sift) HCA_ROW_SELECT(16, true);
  else if (nmax <= 16 * 1024) HCA_ROW_SELECT(16, false);
  else if (nmax <= 32 * 1024 && sift) HCA_ROW_SELECT(32, true);
  else if (nmax <= 32 * 1024) HCA_ROW_SELECT(32, false);
  else if (sift) HCA_ROW_SELECT(40, true);
  else HCA_ROW_SELECT(40, false);
#undef HCA_ROW_SELECT
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// ---------------------------------------------------------------------------------------
// Top-k straight from the scan (Sec. 3.2): the selecting scan has left, per chunk and in slot order, the
// (key, slot) pairs at or above the row's sampled threshold.  One workgroup per row takes the chunks' lists one behind
// the other - the row's candidates in ascending slot order, their keys in registers when they fit -, runs the whole
// radix select (12 + 10 + 10 bits) over them and writes the selected slots in ascending order:
//   selected(j) = key_j > T  or  (key_j == T and #{i < j : key_i == T} < r_eq)
//   position(j) = #{i < j : key_i > T} + min(#{i < j : key_i == T}, r_eq)
// A row with fewer pairs than it has to select is marked for a second scan without threshold; `only_failed`
// launches handle exactly those rows.
constexpr uint32_t kDirectRank = 128;   // keys ranked against each other: 1.5 us; a round of digits takes 2
constexpr int kHeldPairs = 16384;   // pairs per row held in registers
constexpr int kSearchMax = 65536;   // pairs still addressed by position when they are not held

// counter updates when the lanes of a wave share a handful of bins (the leading bits of keys that all lie
// just above one threshold): one atomic per distinct bin for the first few, single updates for the rest
__device__ __forceinline__ void lds_count_few(uint32_t* h, uint32_t bin, bool hit) {
  uint64_t todo = __ballot(hit);
  const int lane = threadIdx.x & 63;
#pragma unroll 1
  for (int it = 0; it < 4 && todo != 0; ++it) {
    const int leader = __ffsll((unsigned long long)todo) - 1;
    const uint32_t b0 = __shfl(bin, leader);
    const uint64_t same = __ballot(hit && bin == b0) & todo;
    if (lane == leader) atomicAdd(&h[b0], (uint32_t)__popcll(same));
    todo &= ~same;
  }
  if ((todo >> lane) & 1) atomicAdd(&h[bin], 1u);
}

template <int NT>
struct ResolveShared {
  uint32_t h[kBins12], off[1025], wsum[16];
  uint16_t cmap[1024];                     // chunk of position 16 i
  uint32_t s_prefix, s_rem, s_cb;
};

// A row's lists: (key, slot) pairs, or slots alone beside the row's scores.
struct PairList {
  const uint2* p;
  __device__ __forceinline__ uint2 operator[](int64_t at) const { return p[at]; }
  __device__ __forceinline__ uint32_t key(int64_t at) const { return p[at].x; }
  __device__ __forceinline__ uint32_t slot(int64_t at) const { return p[at].y; }
};
struct SlotList {
  const uint32_t* p;
  const float* scores;
  __device__ __forceinline__ uint2 operator[](int64_t at) const { return uint2{order_key(scores[p[at]]), p[at]}; }
  __device__ __forceinline__ uint32_t key(int64_t at) const { return order_key(scores[p[at]]); }
  __device__ __forceinline__ uint32_t slot(int64_t at) const { return p[at]; }
};

// The selection proper, once the chunks' offsets are in sh.off.  HELD: every pair's key in a register.
template <int NT, bool HELD, typename List>
__device__ __forceinline__ void tk_resolve_pairs(ResolveShared<NT>& sh, const int64_t chunk, const int nchunks,
                                                 const int64_t want, const List& gl, const uint32_t base_key,
                                                 const int32_t k, int32_t* __restrict__ idx, int32_t* __restrict__ count,
                                                 const int row, const uint32_t total) {
  constexpr int NW = NT / 64;              // waves
  constexpr int PER = 1024 / NT;           // chunks (and 10-bit bins) per thread
  auto& h = sh.h;
  auto& off = sh.off;
  auto& wsum = sh.wsum;
  auto& cmap = sh.cmap;
  uint32_t &s_prefix = sh.s_prefix, &s_rem = sh.s_rem, &s_cb = sh.s_cb;
  const int tid = threadIdx.x;
  // beyond kHeldPairs: up to kSearchMax pairs are still addressed by their position in slot order (short lists:
  // walking them chunk by chunk would cost a memory round trip per chunk), more than that are walked chunk by chunk
  const bool by_position = total <= (uint32_t)kSearchMax;
  // pair p of the row in slot order: the chunk c with off[c] <= p < off[c + 1], entry p - off[c] of its list
  auto fetch = [&](uint32_t p) {
    uint32_t c = 0;
#pragma unroll
    for (int s = 512; s >= 1; s >>= 1)
      if (off[c + s] <= p) c += s;
    return gl[(int64_t)c * chunk + (p - off[c])];
  };
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t kmax = 0;                                        // largest key this thread has seen
  constexpr int kPer = kHeldPairs / NT, kStep = NT == 512 ? 4 : 8;
  const uint32_t per = (total + NT - 1) / NT;               // HELD: pairs per thread ...
  const uint32_t pos0 = (uint32_t)wv * 64 * per + lane;     // ... the first one's position, 64 apart
  constexpr bool kKeep = HELD && NT == 1024;                // room for the slots too: 147 -> 142 us for a codebook step at 1 Mi
  uint32_t held_slot[kKeep ? kPer : 1];
  uint32_t held[HELD ? kPer : 1];                           // their keys (0: no pair; no finite score has it)
  // this thread's pairs u0 .. u0 + kStep - 1: their places in the lists (or -1).  `reach`: the first step of the search
  // from the chunk of a position's group of 16, from the widest such group of the wave.  Spread pairs need 0 to 2 steps;
  // where they lie in a few chunks far apart, the empty chunks between are halved, not walked: 8 rows of 1 Mi tokens whose
  // keys come in runs of up to 4096, k = 4096: 109 -> 22 us for this kernel, 242 -> 153 for the call (independent keys 17)
  uint32_t reach = 0;
  auto locate = [&](int u0, uint32_t (&at)[kStep]) {
    uint32_t c[kStep], first = pos0 + 64 * u0;
    asm volatile("" : "+v"(first));        // (or every call's comparisons are kept for the next one: registers)
#pragma unroll
    for (int u = 0; u < kStep; ++u) {
      const uint32_t p = first + 64 * u;
      c[u] = cmap[p < total ? p >> 4 : 0];
    }
    for (uint32_t s = reach; s != 0; s >>= 1) {
#pragma unroll
      for (int u = 0; u < kStep; ++u) {
        const uint32_t p = first + 64 * u, next = c[u] + s < 1024 ? c[u] + s : 1024;
        if (p < total && off[next] <= p) c[u] = next;
      }
    }
#pragma unroll
    for (int u = 0; u < kStep; ++u) {
      const uint32_t p = first + 64 * u;
      at[u] = (uint32_t)(u0 + u) < per && p < total ? c[u] * (uint32_t)chunk + (p - off[c[u]]) : 0xffffffffu;
    }
  };
  if constexpr (HELD) {
    // chunk of every 16th position, from there on to the chunk of each position
    for (int c = tid; c < 1024; c += NT) {
      const uint32_t end = off[c + 1];
      for (uint32_t i = (off[c] + 15) >> 4; i * 16 < end; ++i) cmap[i] = (uint16_t)c;
    }
    __syncthreads();
    uint32_t gap = 0;
    for (uint32_t g = lane; g < 4 * per; g += 64) {
      const uint32_t i = 4 * (uint32_t)wv * per + g;
      if (16 * i < total) {
        const uint32_t d = (16 * (i + 1) < total ? (uint32_t)cmap[i + 1] : (uint32_t)nchunks - 1) - cmap[i];
        gap = d > gap ? d : gap;
      }
    }
    gap = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max(gap));
    reach = gap != 0 ? 1u << (31 - __clz((int)gap)) : 0u;
#pragma unroll
    for (int u0 = 0; u0 < kPer; u0 += kStep) {
      uint32_t at[kStep];
      if ((uint32_t)u0 < per) {
        locate(u0, at);
#pragma unroll
        for (int u = 0; u < kStep; ++u) {
          if constexpr (kKeep) {
            const uint2 x = at[u] != 0xffffffffu ? gl[at[u]] : uint2{0, 0};
            held[u0 + u] = x.x;
            held_slot[u0 + u] = x.y;
          } else {
            held[u0 + u] = at[u] != 0xffffffffu ? gl.key(at[u]) : 0;
          }
        }
      } else {
#pragma unroll
        for (int u = 0; u < kStep; ++u) held[u0 + u] = 0;
      }
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) kmax = held[u] > kmax ? held[u] : kmax;
  }
  __syncthreads();
  // visit(f): f(key, slot, exists) over every pair of the row, in any order, called by all lanes of a wave
  // together.  HELD: from the registers.  By position: through fetch, four pairs in flight per thread.  Otherwise the lists where they are: wave w takes chunks w, w + NW, ... and reads each list 1024
  // pairs at a time (sixteen loads in flight per lane).
  auto visit = [&](auto&& f) {
    if constexpr (HELD) {
#pragma unroll
      for (int u0 = 0; u0 < kPer; u0 += kStep) {
        if ((uint32_t)u0 >= per) break;
        uint32_t none = 0;
        asm volatile("" : "+s"(none));                      // (no pass's comparisons are kept for the next: registers)
#pragma unroll
        for (int u = 0; u < kStep; ++u) f(held[u0 + u], 0u, held[u0 + u] != none);
      }
    } else if (by_position) {
      for (uint32_t i0 = 0; i0 < total; i0 += 4 * NT) {
        uint2 x[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = fetch(i0 + v * NT + tid < total ? i0 + v * NT + tid : 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) f(x[v].x, x[v].y, i0 + v * NT + tid < total);
      }
    } else {
      for (int c = wv; c < nchunks; c += NW) {
        const uint32_t m = off[c + 1] - off[c];
        const int64_t src = (int64_t)c * chunk;
        for (uint32_t i0 = 0; i0 < m; i0 += 1024) {
          uint2 x[16];
#pragma unroll
          for (int v = 0; v < 16; ++v) x[v] = i0 + v * 64 + lane < m ? gl[src + i0 + v * 64 + lane] : uint2{0, 0};
#pragma unroll
          for (int v = 0; v < 16; ++v) f(x[v].x, x[v].y, i0 + v * 64 + lane < m);
        }
      }
    }
  };
  if (!HELD) visit([&](uint32_t key, uint32_t, bool hit) { if (hit && key > kmax) kmax = key; });
  kmax = wave_max(kmax);
  if (lane == 0) wsum[wv] = kmax;
  __syncthreads();
#pragma unroll
  for (int x = 0; x < NW; ++x) kmax = wsum[x] > kmax ? wsum[x] : kmax;
  __syncthreads();
  // Radix select on d = key - base (every key of the list is >= base, the scan's threshold): pd = the leading
  // digits of d found so far, s = the number of bits of d below them; rem = how many are still to take among the
  // pairs whose d starts with pd, cb = how many such pairs there are.  The first level spreads the occupied
  // range of d over 4096 bins, so the counters are not fought over although the keys share their leading bits.
  const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base_key);
  const uint32_t maxd = kmax - base;
  int sbits = 32 - __clz((int)(maxd | 1)) - 12;             // bits of maxd beyond the 12 of the first level
  if (sbits < 0) sbits = 0;
  uint32_t pd = 0, rem = (uint32_t)want, cb = total;
  {
    for (int i = tid; i < kBins12; i += NT) h[i] = 0;
    __syncthreads();
    visit([&](uint32_t key, uint32_t, bool hit) { lds_count(h, (key - base) >> sbits, hit, !HELD); });
    __syncthreads();
    constexpr int BPT = kBins12 / NT;                       // bins per thread, from the top
    uint32_t hb[BPT], sum = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) { hb[i] = h[kBins12 - 1 - (BPT * tid + i)]; sum += hb[i]; }
    uint32_t running = block_scan_excl<NT / 64>(sum, wsum);
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      if (running < rem && rem <= running + hb[i]) {
        s_prefix = (uint32_t)(kBins12 - 1 - (BPT * tid + i));
        s_rem = rem - running;
        s_cb = hb[i];
      }
      running += hb[i];
    }
    __syncthreads();
    pd = s_prefix;
    rem = s_rem;
    cb = s_cb;
    __syncthreads();
  }
  uint32_t T = 0, req = 0;
  while (true) {                                            // every condition below is uniform over the workgroup
    if (sbits == 0) {                                       // d is fully known: the pairs left all hold one key
      T = base + pd;
      req = rem;
      break;
    }
    if (cb <= (HELD ? kDirectRank : 1024)) {                // (unheld, a round is one more walk through the lists)
      // few pairs left: rank them against each other.  sl = their keys; T is the key with fewer than rem keys
      // above it that, together with its equals, reaches rem.
      uint32_t* sl = h;
      if (tid == 0) s_cb = 0;
      __syncthreads();
      uint32_t base1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
      asm volatile("" : "+s"(base1));                       // (nor the differences)
      visit([&](uint32_t key, uint32_t, bool hit) {
        if (hit && ((key - base1) >> sbits) == pd) sl[atomicAdd(&s_cb, 1u)] = key;
      });
      __syncthreads();
      for (uint32_t me = (uint32_t)tid; me < cb; me += NT) {
        const uint32_t ki = sl[me];
        uint32_t gt = 0, eq = 0;
#pragma unroll 4
        for (uint32_t j = 0; j < cb; ++j) {
          const uint32_t kj = sl[j];
          gt += kj > ki;
          eq += kj == ki;
        }
        if (gt < rem && rem <= gt + eq) { s_prefix = ki; s_rem = rem - gt; }   // equal keys write equal values
      }
      __syncthreads();
      T = s_prefix;
      req = s_rem;
      break;
    }
    const int ns = sbits > 10 ? sbits - 10 : 0, width = sbits - ns;
    for (int i = tid; i < 1024; i += NT) h[i] = 0;
    __syncthreads();
    uint32_t base1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    asm volatile("" : "+s"(base1));
    visit([&](uint32_t key, uint32_t, bool hit) {
      const uint32_t d = key - base1;
      lds_count(h, (d >> ns) & ((1u << width) - 1), hit && (d >> sbits) == pd, !HELD);
    });
    __syncthreads();
    uint32_t mine[PER], msum = 0;                           // thread tid owns bins 1023 - (PER tid + x)
#pragma unroll
    for (int x = 0; x < PER; ++x) { mine[x] = h[1023 - (PER * tid + x)]; msum += mine[x]; }
    uint32_t running = block_scan_excl<NT / 64>(msum, wsum);
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      if (running < rem && rem <= running + mine[x]) {
        s_prefix = (pd << width) | (uint32_t)(1023 - (PER * tid + x));
        s_rem = rem - running;
        s_cb = mine[x];
      }
      running += mine[x];
    }
    __syncthreads();
    pd = s_prefix;
    rem = s_rem;
    cb = s_cb;
    sbits = ns;
    __syncthreads();
  }
  int32_t* out = idx + (int64_t)row * k;
  if (tid == 0) count[row] = (int32_t)want;
  if constexpr (HELD) {
    // the wave's pairs above and equal to T, those of the waves before, then every pair's place
    const uint64_t lt = (1ull << lane) - 1;
    uint32_t ng = 0, ne = 0;
#pragma unroll
    for (int u0 = 0; u0 < kPer; u0 += kStep) {
      if ((uint32_t)u0 >= per) break;
#pragma unroll
      for (int u = 0; u < kStep; ++u) {
        ng += (uint32_t)__popcll(__ballot(held[u0 + u] > T));
        ne += (uint32_t)__popcll(__ballot(held[u0 + u] == T));
      }
    }
    if (lane == 0) { wsum[wv] = ng; h[wv] = ne; }
    __syncthreads();
    uint32_t pg = 0, pe = 0;
#pragma unroll
    for (int x = 0; x < NW; ++x) { pg += x < wv ? wsum[x] : 0; pe += x < wv ? h[x] : 0; }
#pragma unroll
    for (int u0 = 0; u0 < kPer; u0 += kStep) {
      if ((uint32_t)u0 >= per) break;
      uint32_t slot[kStep];
      if constexpr (kKeep) {
#pragma unroll
        for (int u = 0; u < kStep; ++u) slot[u] = held_slot[u0 + u];
      } else {
        uint32_t at[kStep];
        locate(u0, at);
#pragma unroll
        for (int u = 0; u < kStep; ++u) slot[u] = held[u0 + u] >= T ? gl.slot(at[u]) : 0;    // (T > 0: a pair)
      }
#pragma unroll
      for (int u = 0; u < kStep; ++u) {
        const bool fg = held[u0 + u] > T, fe = held[u0 + u] == T;
        const uint64_t mg = __ballot(fg), me = __ballot(fe);
        const uint32_t gb = pg + (uint32_t)__popcll(mg & lt), eb = pe + (uint32_t)__popcll(me & lt);
        if (fg) out[gb + (eb < req ? eb : req)] = (int32_t)slot[u];
        else if (fe && eb < req) out[gb + eb] = (int32_t)slot[u];
        pg += (uint32_t)__popcll(mg);
        pe += (uint32_t)__popcll(me);
      }
    }
    return;
  }
  if (by_position) {
    // ordered part by position (slot order): thread tid owns the run [tid * E, tid * E + E)
    const uint32_t E = (total + NT - 1) / NT;
    const uint32_t p0 = (uint32_t)tid * E;
    const uint32_t p1 = p0 + E < total ? p0 + E : total;
    uint32_t ng = 0, ne = 0;
    if (p0 < p1) {
      // the run lies in consecutive entries of consecutive chunks' lists: one search for its start, then a walk
      uint32_t c = 0;
#pragma unroll
      for (int s = 512; s >= 1; s >>= 1)
        if (off[c + s] <= p0) c += s;
      uint32_t e = p0 - off[c];
      for (uint32_t p = p0; p < p1; ++p) {
        while (e >= off[c + 1] - off[c]) { ++c; e = 0; }
        const uint32_t key = gl.key((int64_t)c * chunk + e);
        ng += key > T;
        ne += key == T;
        ++e;
      }
    }
    uint32_t rg = block_scan_excl<NT / 64>(ng, wsum);            // pairs above T on lower slots
    uint32_t re = block_scan_excl<NT / 64>(ne, wsum);            // pairs equal to T on lower slots
    if (p0 < p1) {
      uint32_t c = 0;
#pragma unroll
      for (int s = 512; s >= 1; s >>= 1)
        if (off[c + s] <= p0) c += s;
      uint32_t e = p0 - off[c];
      for (uint32_t p = p0; p < p1; ++p) {
        while (e >= off[c + 1] - off[c]) { ++c; e = 0; }
        const uint2 x = gl[(int64_t)c * chunk + e];
        if (x.x > T) { out[rg + (re < req ? re : req)] = (int32_t)x.y; ++rg; }
        else if (x.x == T) { if (re < req) out[rg + re] = (int32_t)x.y; ++re; }
        ++e;
      }
    }
    return;
  }
  // ordered part on the lists where they are: per chunk the pairs above / equal to T, a prefix over the chunks,
  // then every wave walks its chunks again, 64 pairs at a time, positions by ballot
  uint32_t* cg = h;            // [1024] pairs above T per chunk -> pairs above T in the chunks before
  uint32_t* ce = h + 1024;     // the same for pairs equal to T
  __syncthreads();
  for (int c = wv; c < 1024; c += NW) {
    uint32_t g = 0, e = 0;
    if (c < nchunks) {
      const uint32_t m = off[c + 1] - off[c];
      const int64_t src = (int64_t)c * chunk;
      for (uint32_t i0 = 0; i0 < m; i0 += 1024) {
        uint32_t key[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) key[v] = i0 + v * 64 + lane < m ? gl.key(src + i0 + v * 64 + lane) : 0u;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const bool live = i0 + v * 64 + lane < m;
          g += (uint32_t)__popcll(__ballot(live && key[v] > T));
          e += (uint32_t)__popcll(__ballot(live && key[v] == T));
        }
      }
    }
    if (lane == 0) { cg[c] = g; ce[c] = e; }
  }
  __syncthreads();
  {
    uint32_t g[PER], e[PER], gs = 0, es = 0;
#pragma unroll
    for (int x = 0; x < PER; ++x) { g[x] = cg[PER * tid + x]; e[x] = ce[PER * tid + x]; gs += g[x]; es += e[x]; }
    uint32_t og = block_scan_excl<NT / 64>(gs, wsum);
    uint32_t oe = block_scan_excl<NT / 64>(es, wsum);
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      cg[PER * tid + x] = og;
      ce[PER * tid + x] = oe;
      og += g[x];
      oe += e[x];
    }
  }
  __syncthreads();
  const uint64_t lt = (1ull << lane) - 1;
  for (int c = wv; c < nchunks; c += NW) {
    const uint32_t m = off[c + 1] - off[c];
    const int64_t src = (int64_t)c * chunk;
    uint32_t pg = cg[c], pe = ce[c];
    for (uint32_t i0 = 0; i0 < m; i0 += 512) {
      uint2 xs[8];
#pragma unroll
      for (int v = 0; v < 8; ++v) xs[v] = i0 + v * 64 + lane < m ? gl[src + i0 + v * 64 + lane] : uint2{0, 0};
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const bool live = i0 + v * 64 + lane < m;
        const uint2 x = xs[v];
        const bool fg = live && x.x > T, fe = live && x.x == T;
        const uint64_t mg = __ballot(fg), me = __ballot(fe);
        const uint32_t gb = pg + (uint32_t)__popcll(mg & lt), eb = pe + (uint32_t)__popcll(me & lt);
        if (fg) out[gb + (eb < req ? eb : req)] = (int32_t)x.y;
        else if (fe && eb < req) out[gb + eb] = (int32_t)x.y;
        pg += (uint32_t)__popcll(mg);
        pe += (uint32_t)__popcll(me);
      }
    }
  }
}

// One workgroup per row; the keys of the row's pairs (up to 16384 of them) are held in registers, wave w those of the
// positions [64 w E, 64 (w + 1) E), lane l its positions l, l + 64, ...: the loads are whole lines, no pass over the pairs
// touches memory, and the order of the slots is that of (wave, u, lane), so ranks are popcounts of ballots.  What bounds it
// is the chain of passes and barriers.  8 rows of 14 Ki pairs, alone: 28 us with the pairs in 128 KiB of LDS, 21 so.
// NT = 1024 is the quickest where the chip is free (2 Mi slots x 8, k = 8192: 172 -> 165 us for the call).  Beside a
// running scan what counts is the room it needs: a scan workgroup has 128 registers and 33 KiB, four of them fill a compute
// unit, and another launch's workgroup only gets in where one of them ends.  NT = 512 has 64 registers, three spilled (two waves per SIMD)
// and 23 KiB: 62 us from launch to end beside a scan where the 1024-thread form waited for the scan's end, 200 us; four
// layers of 1 Mi tokens in a step driver 810 -> 720 us, eight 1315 -> 1087.  NT = 256 (48 us alone) is for launches that
// nearly always find nothing to do.  All give the same result.
// Returns true for a row whose lists hold too little (mark: its spec then asks for a second scan).
template <int NT>
__device__ __forceinline__ bool tk_resolve_emit_body(const int64_t chunk, const int nchunks, const int64_t want,
                                                     const SelectOut& so, const int32_t k, int32_t* __restrict__ idx,
                                                     int32_t* __restrict__ count, const bool only_failed, const int row,
                                                     const bool mark = true) {
  constexpr int PER = 1024 / NT;           // chunks per thread
  __shared__ ResolveShared<NT> sh;
  auto& off = sh.off;
  auto& wsum = sh.wsum;
  const int tid = threadIdx.x;
  uint32_t* spec = so.spec + 4 * row;
  if (want <= 0) {
    if (tid == 0 && !only_failed) count[row] = 0;
    return false;
  }
  if (only_failed && spec[1] == 0) return false;
  // off[c] = pairs in the chunks before c; off[1024] = all of them.  Thread tid owns chunks [PER tid, PER tid + PER)
  {
    uint32_t mine[PER], sum = 0;
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      const int c = tid * PER + x;
      mine[x] = c < nchunks ? so.ncand[(int64_t)row * kSelectMaxChunks + c] : 0;
      sum += mine[x];
    }
    uint32_t before = block_scan_excl<NT / 64>(sum, wsum);
#pragma unroll
    for (int x = 0; x < PER; ++x) { off[tid * PER + x] = before; before += mine[x]; }
    if (tid == NT - 1) off[1024] = before;
  }
  __syncthreads();
  const uint32_t total = off[1024];
  if (!only_failed && tid == 0 && so.mon != nullptr) {      // one workgroup per row and launches in stream order: no atomics
    uint32_t* m = so.mon + 4 * row;
    m[0] += 1;
    m[1] = total < m[1] ? total : m[1];
    m[2] = total > m[2] ? total : m[2];
    if (total < (uint32_t)want) m[3] += 1;
  }
  if (total < (uint32_t)want && !mark) return true;         // (the launch itself scans the row again)
  if (total < (uint32_t)want) {
    // the sampled threshold was too high: scan the row again, with the second threshold if the first scan counted
    // enough slots at or above it, else without one
    uint32_t sum1 = 0;
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      const int c = tid * PER + x;
      sum1 += c < nchunks ? so.n1[(int64_t)row * kSelectMaxChunks + c] : 0;
    }
    const uint32_t before1 = block_scan_excl<NT / 64>(sum1, wsum);
    if (tid == NT - 1) {
      const uint32_t enough = before1 + sum1 >= (uint32_t)want;
      spec[0] = enough && spec[1] == 0 ? spec[2] : 0;       // (a second failure cannot happen: the count is exact)
      spec[1] = 1;
    }
    return true;
  }
  const uint32_t base = spec[0];
  const PairList lists{so.lists + (int64_t)row * so.row_entries};
  if (total <= (uint32_t)kHeldPairs) tk_resolve_pairs<NT, true>(sh, chunk, nchunks, want, lists, base, k, idx, count, row, total);
  else tk_resolve_pairs<NT, false>(sh, chunk, nchunks, want, lists, base, k, idx, count, row, total);
  return false;
}

template <int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 512 ? 8 : 4))) void tk_resolve_emit(int64_t chunk, int nchunks, int n_kv_heads, SelRows sr,
                                                      SelectOut so, int32_t k, int32_t* __restrict__ idx,
                                                      int32_t* __restrict__ count, bool only_failed) {
  tk_resolve_emit_body<NT>(chunk, nchunks, sr.want[blockIdx.x / n_kv_heads], so, k, idx, count, only_failed,
                           (int)blockIdx.x);
}

// The last launch of hca_score_topk's selecting scan, one 1024-thread workgroup per row and behind them some for rows that have
// to be scanned again.  A row whose lists hold enough is selected by its own workgroup.  The others add up every row's
// counts and return, nearly always, as none falls short; those that do are dealt out among them and their own workgroups and scanned
// again, a share of the chunks each, into the same lists, whose new counts go to the room of the samples (the first ones still
// have readers), and the one that finishes last makes the selection.  Nobody waits for anybody, so any number may be resident.  One
// launch where a selection, a second scan and a second selection were three, the last two of them 9 us to find that they have
// nothing to do.
// What the shares write goes through to memory (a release fence would write the whole L2 back, 512 times over: 12.5 ms for eight
// rows of 1 Mi); only the last one fences.  The row totals are not added up by the scan: its workgroups' atomics, on eight
// dies, took it from 106 to 490 us.  A call, three launches / this one, us, by rows that are scanned again with the second
// threshold: 8 rows of 200 000 slots, none 52 / 47, one 72 / 60, four 75 / 66, all 79 / 77; 8 of 1 Mi 132 / 127, 176 / 150, 200 /
// 186, 239 / 234 (2-bit codes 94 / 83, 122 / 102, 138 / 122, 152 / 146); 32 of 128 Ki, none 86 / 80, one 105 / 91, half 122 / 118, all
// 141 / 143; 64 of 128 Ki 142 / 135, 153 / 144, 200 / 194, 244 / 242; 8 rows of 1 Mi scanned again whole: one 1348 / 1315, all 1438 /
// 1441.  (Each wave waiting for its own loads, and the failed rows' own workgroups idle: all of 8 x 1 Mi 262, of 32 x 128 Ki 166, of 64
// 305.)
template <typename T>
__device__ __forceinline__ void store_through(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Chunks first, first + step, ... of a row, 64 consecutive blocks at a time, four per wave.  The next 64 are on their way while
// these are scored, across the chunks too.
template <int BITS>
__device__ __forceinline__ void rescan_chunks(const Layout& L, const uint8_t* __restrict__ kcache, const uint16_t* __restrict__ q,
                                              const int64_t n, const int row, const uint32_t from_key, const int chunk_blocks,
                                              const int nchunks, const int first, const int step, const SelectOut& so,
                                              uint32_t* __restrict__ counts) {
  constexpr int U = 4, kTpb = BITS == 4 ? 16 : 32, kStep = 16 * U;
  __shared__ QShared qs;
  __shared__ __align__(16) uint32_t opimg[64 * 8];
  __shared__ uint32_t wn[2][16];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int t = lane & 15, hd = lane >> 4;
  const int nblocks = (int)((n + kTpb - 1) / kTpb);
  const int live = (nblocks + chunk_blocks - 1) / chunk_blocks;         // chunks that hold any of the row
  for (int c = first + step * (int)threadIdx.x; c < nchunks; c += 1024 * step)
    if (c >= live) store_through(&counts[c], 0u);
  if (first >= live) return;
  const uint4* cptr = reinterpret_cast<const uint4*>(kcache + (int64_t)row * L.codes_row_bytes()) + lane;
  const uint32_t* mptr = reinterpret_cast<const uint32_t*>(kcache + L.meta_off + (int64_t)row * L.meta_row_bytes()) +
                         (BITS == 4 ? 4 * t + hd : 2 * (16 * (hd >> 1) + t) + (hd & 1));
  const float from = key_floor(from_key);
  const bool head_live = hd < L.gqa;
  auto end_of = [&](int c) { return (c + 1) * chunk_blocks < nblocks ? (c + 1) * chunk_blocks : nblocks; };
  uint4 wv[U];
  uint32_t mw[U];
  auto fetch = [&](int b0, int b1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int at = b0 + U * w + u, blk = at < b1 ? at : b1 - 1;
      wv[u] = load_stream16(&cptr[(int64_t)blk * 64]);
      mw[u] = __builtin_nontemporal_load(&mptr[(int64_t)blk * 64]);
    }
  };
  int c = first, b0 = c * chunk_blocks, turn = 0;
  uint32_t pair = query_pair(q, row, L.gqa);                // (before the codes: loads come back in order)
  asm volatile("" ::: "memory");
  fetch(b0, end_of(c));
  asm volatile("" : "+v"(pair));
  QOperand<BITS> op;
  load_query(pair, L.gqa, L.group, &qs);
  build_operand_shared<BITS>(&qs, opimg, &op);
  uint32_t base = 0;
  while (c < live) {
    const int b1 = end_of(c);
    int next_c = c, next_b = b0 + kStep;
    if (next_b >= b1) { next_c = c + step; next_b = next_c * chunk_blocks; }
    uint4 cw[U];
    uint32_t cm[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { cw[u] = wv[u]; cm[u] = mw[u]; }
    if (next_c < live) fetch(next_b, end_of(next_c));
    // the wave's slots in order, 64 at a time: lane l has the score of slot tok0 + 64 x + l
    constexpr int X = U * kTpb / 64;
    float v[X];
    if constexpr (BITS == 4) {
      float z[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        z[u] = score_block4(op, cw[u], allgather_rows(cm[u]));
        z[u] = head_live ? z[u] : -INFINITY;
      }
      v[0] = max_over_heads_scatter(z[0], z[1], z[2], z[3]);
    } else {
#pragma unroll
      for (int x = 0; x < X; ++x) {
        float z[4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const uint4 b = cw[2 * x + u], m = allgather_rows(cm[2 * x + u]);
          z[2 * u] = score_tile2(op, b.x, b.y, uint2{m.x, m.y});
          z[2 * u + 1] = score_tile2(op, b.z, b.w, uint2{m.z, m.w});
          z[2 * u] = head_live ? z[2 * u] : -INFINITY;
          z[2 * u + 1] = head_live ? z[2 * u + 1] : -INFINITY;
        }
        v[x] = max_over_heads_scatter(z[0], z[1], z[2], z[3]);
      }
    }
    const int64_t tok0 = (int64_t)(b0 + U * w) * kTpb + lane, end = (int64_t)b1 * kTpb < n ? (int64_t)b1 * kTpb : n;
    uint64_t hits[X];
    uint32_t mine = 0;
#pragma unroll
    for (int x = 0; x < X; ++x) {
      hits[x] = __builtin_amdgcn_ballot_w64(tok0 + 64 * x < end && v[x] >= from);
      mine += (uint32_t)__popcll(hits[x]);
    }
    if (lane == 0) wn[turn][w] = mine;
    __syncthreads();
    uint32_t at = base;
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const uint32_t s = wn[turn][x];
      at += x < w ? s : 0;
      base += s;
    }
    turn ^= 1;                                              // (written again two barriers from here)
    uint2* dst = so.lists + (int64_t)row * so.row_entries + (int64_t)c * chunk_blocks * kTpb;
#pragma unroll
    for (int x = 0; x < X; ++x) {
      if ((hits[x] >> lane) & 1)
        store_through(reinterpret_cast<uint64_t*>(dst + at + (uint32_t)__popcll(hits[x] & ((1ull << lane) - 1))),
                      (uint64_t)(tok0 + 64 * x) << 32 | order_key(v[x]));
      at += (uint32_t)__popcll(hits[x]);
    }
    if (next_c != c) {
      if (threadIdx.x == 0) store_through(&counts[c], base);
      base = 0;
    }
    c = next_c;
    b0 = next_b;
  }
}

constexpr int kFinishRows = 64;         // rows that tk_finish takes

template <int BITS>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void tk_finish(
    Layout L, const uint8_t* __restrict__ kcache, const uint16_t* __restrict__ q, NRes nr, int64_t chunk, int nchunks, SelRows sr,
    SelectOut so, int32_t k, int32_t* __restrict__ idx, int32_t* __restrict__ count) {
  __shared__ uint32_t wsum[16], s_flag;
  __shared__ uint32_t s_total[kFinishRows];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, rows = L.rows, own = (int)blockIdx.x;
  auto want_of = [&](int row) { return sr.want[row / L.n_kv_heads]; };
  if (own < rows && !tk_resolve_emit_body<1024>(chunk, nchunks, want_of(own), so, k, idx, count, false, own, false)) return;
  for (int x = w; x < rows; x += 16) {                    // a wave per row, all of its counts in flight
    uint32_t n[kSelectMaxChunks / 64], sum = 0;
#pragma unroll
    for (int i = 0; i < kSelectMaxChunks / 64; ++i) {
      const int c = i * 64 + lane;
      n[i] = c < nchunks ? so.ncand[(int64_t)x * kSelectMaxChunks + c] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kSelectMaxChunks / 64; ++i) sum += n[i];
    sum = wave_sum(sum);
    if (lane == 0) s_total[x] = sum;
  }
  __syncthreads();
  const bool lacks = lane < rows && want_of(lane) > 0 && s_total[lane] < (uint32_t)want_of(lane);
  uint64_t failed = __builtin_amdgcn_ballot_w64(lacks);
  if (failed == 0) return;
  // the failed rows in turn, their own workgroups behind the others: this one is number `at` of the `of` that share its row
  const int others = (int)gridDim.x - rows, many = (int)__builtin_popcountll(failed), helpers = others + many;
  const int h = own >= rows ? own - rows : others + (int)__builtin_popcountll(failed & ((1ull << own) - 1));
  const int at = h / many, of = (helpers - h % many + many - 1) / many;
  for (int x = h % many; x > 0; --x) failed &= failed - 1;
  const int row = (int)__builtin_ctzll(failed);
  // the second threshold if the first scan counted enough slots at or above it, else none
  const uint32_t above = tid < nchunks ? so.n1[(int64_t)row * kSelectMaxChunks + tid] : 0u;
  uint32_t all;
  block_scan_excl<16>(above, wsum, &all);
  const uint32_t from = all >= (uint32_t)want_of(row) ? so.spec[4 * row + 2] : 0u;
  SelectOut again = so;
  again.ncand = so.samples;                                 // [rows][kSelectMaxChunks]: a row has at least 8192 samples
  rescan_chunks<BITS>(L, kcache, q, nr.n[row / L.n_kv_heads], row, from, (int)(chunk / L.tpb), nchunks, at, of, so,
                      again.ncand + (int64_t)row * kSelectMaxChunks);
  __builtin_amdgcn_s_waitcnt(0);                            // this wave's pairs and counts are in memory
  __syncthreads();
  if (tid == 0) s_flag = atomicAdd(&so.spec[4 * row + 3], 1u) == (uint32_t)(of - 1);
  __syncthreads();
  if (s_flag == 0) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  if (tid == 0) { so.spec[4 * row] = from; so.spec[4 * row + 1] = 2; }        // (2: the counts are with the samples)
  __syncthreads();
  tk_resolve_emit_body<1024>(chunk, nchunks, want_of(row), again, k, idx, count, true, row);
}

// The last launch of a selection from scores: the chunks' lists hold the slots of the keys above the sampled key K
// (t.state), the chunks' second counts (t.above) the slots equal to it.  Enough above it: the selection over the lists.
// Enough with the equal ones: all of the lists and the first equal slots.  Neither, which takes a row that its samples
// misrepresent by six deviations: the slots at or above the second key into the lists, by this workgroup - or every slot,
// should they be too few as well.  8 rows, one of them misread, by the second key / whole, us: 50 000 slots 27 -> 45 / 185,
// 98 304 27 -> - / 165, 1 Mi 37 -> 220 / 1380.
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void tk_resolve_scores(
    const float* __restrict__ vals, int64_t stride, int64_t chunk, int nchunks, int n_kv_heads, SelRows sr, TopkWs t,
    ListRoom room, int32_t k, int32_t* __restrict__ idx, int32_t* __restrict__ count, RowSelectFused fu) {
  __shared__ ResolveShared<1024> sh;
  auto& off = sh.off;
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int64_t n = sr.nsel[row / n_kv_heads], want = sr.want[row / n_kv_heads];
  const bool live = want > 0 && tid < nchunks;
  const uint32_t mine = live ? t.ncand[(int64_t)row * kMaxChunks + tid] : 0;
  const uint32_t equal = live ? t.above[(int64_t)row * 1024 + tid] : 0;
  const uint32_t before = block_scan_excl<16>(mine, sh.wsum), before_e = block_scan_excl<16>(equal, sh.wsum);
  uint32_t* eoff = sh.h;                                    // equal slots in the chunks before
  off[tid] = before;
  eoff[tid] = before_e;
  if (tid == 1023) { off[1024] = before + mine; eoff[1024] = before_e + equal; }
  const bool fits = __syncthreads_and(mine <= (uint32_t)room.pair_chunk);
  uint32_t total = off[1024];
  const uint32_t with_equal = total + eoff[1024];
  const bool misread = want > 0 && with_equal < (uint32_t)want;
  uint32_t K = want > 0 ? t.state[4 * row] : 0;
  const float* v = vals + (int64_t)row * stride;
  bool in_pairs = fits;
  if (misread) {
    in_pairs = room.slots == nullptr;
    K = t.state[4 * row + 2];
    for (;;) {
      __syncthreads();                                      // off and eoff have been read
      for (int c = tid >> 6; c < 1024; c += 16) {           // a wave per chunk, in slot order
        const int64_t c0 = (int64_t)c * chunk, c1 = c0 + chunk < n ? c0 + chunk : n;
        uint32_t m = 0;
        for (int64_t s0 = c0; s0 < c1; s0 += 16 * 64) {
          uint32_t key[16];
#pragma unroll
          for (int x = 0; x < 16; ++x) key[x] = order_key(v[s0 + x * 64 + lane < c1 ? s0 + x * 64 + lane : c1 - 1]);
#pragma unroll
          for (int x = 0; x < 16; ++x) {
            const uint32_t slot = (uint32_t)(s0 + x * 64 + lane);
            const bool hit = slot < c1 && key[x] >= K;
            const uint64_t hits = __ballot(hit);
            const uint32_t at = m + (uint32_t)__popcll(hits & ((1ull << lane) - 1));
            if (hit && in_pairs) room.pairs[row * room.pair_row + c * chunk + at] = uint2{key[x], slot};
            else if (hit) room.slots[row * room.slot_row + c * chunk + at] = slot;
            m += (uint32_t)__popcll(hits);
          }
        }
        if (lane == 0) sh.h[c] = m;
      }
      __syncthreads();
      const uint32_t listed = sh.h[tid], first = block_scan_excl<16>(listed, sh.wsum);
      off[tid] = first;
      if (tid == 1023) off[1024] = first + listed;
      __syncthreads();
      total = off[1024];
      if (total >= (uint32_t)want) break;
      K = 0;
    }
  }
  if (fu.spec != nullptr) {                                 // the figures of hca_score_topk's report and monitor
    for (int c = tid; c < fu.nchunks; c += 1024)
      fu.ncand[(int64_t)row * kSelectMaxChunks + c] = c == 0 && want > 0 ? (misread ? total : with_equal) : 0u;
    if (tid == 0) {
      fu.spec[4 * row + 1] = misread;
      if (want > 0 && fu.mon != nullptr) {
        uint32_t* m = fu.mon + 4 * row;
        m[0] += 1;
        m[1] = with_equal < m[1] ? with_equal : m[1];
        m[2] = with_equal > m[2] ? with_equal : m[2];
        m[3] += misread;
      }
    }
  }
  if (want <= 0) {
    if (tid == 0) count[row] = 0;
    return;
  }
  const PairList pairs{room.pairs + row * room.pair_row};
  const SlotList slots{room.slots + row * room.slot_row, v};
  const int64_t list_chunk = misread ? chunk : room.pair_chunk;
  if (total >= (uint32_t)want) {
    __syncthreads();                                        // eoff has been read
    // (a second key of 0 lets the key 0 in, which a register could not tell from no pair)
    if (in_pairs && total <= (uint32_t)kHeldPairs && !(misread && K == 0))
      tk_resolve_pairs<1024, true>(sh, list_chunk, nchunks, want, pairs, K, k, idx, count, row, total);
    else if (in_pairs)
      tk_resolve_pairs<1024, false>(sh, list_chunk, nchunks, want, pairs, K, k, idx, count, row, total);
    else
      tk_resolve_pairs<1024, false>(sh, chunk, nchunks, want, slots, K, k, idx, count, row, total);
    return;
  }
  // a wave per chunk, in slot order: from the row itself while equal slots are still to take, then from the lists
  const uint32_t req = (uint32_t)want - total;
  const uint64_t lt = (1ull << lane) - 1;
  int32_t* out = idx + (int64_t)row * k;
  if (tid == 0) count[row] = (int32_t)want;
  for (int c = tid >> 6; c < nchunks; c += 16) {
    uint32_t pg = off[c], pe = eoff[c];
    if (pe >= req || eoff[c + 1] == pe) {
      const uint32_t m = off[c + 1] - pg, e = pe < req ? pe : req;
      for (uint32_t i = lane; i < m; i += 64)
        out[pg + e + i] = (int32_t)(in_pairs ? pairs.slot(c * room.pair_chunk + i) : slots.slot(c * chunk + i));
      continue;
    }
    const int64_t c0 = (int64_t)c * chunk, c1 = c0 + chunk < n ? c0 + chunk : n;
    for (int64_t s0 = c0; s0 < c1; s0 += 16 * 64) {
      uint32_t key[16];
#pragma unroll
      for (int x = 0; x < 16; ++x) key[x] = order_key(v[s0 + x * 64 + lane < c1 ? s0 + x * 64 + lane : c1 - 1]);
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const bool live = s0 + x * 64 + lane < c1, fg = live && key[x] > K, fe = live && key[x] == K;
        const uint64_t mg = __ballot(fg), me = __ballot(fe);
        const uint32_t gb = pg + (uint32_t)__popcll(mg & lt), eb = pe + (uint32_t)__popcll(me & lt);
        if (fg) out[gb + (eb < req ? eb : req)] = (int32_t)(s0 + x * 64 + lane);
        else if (fe && eb < req) out[gb + eb] = (int32_t)(s0 + x * 64 + lane);
        pg += (uint32_t)__popcll(mg);
        pe += (uint32_t)__popcll(me);
      }
    }
  }
}

// The selections of two layers in one launch (the step driver's paired form): workgroups [0, rows) take the
// first layer, [rows, 2 rows) the second.
struct ResolveSide {
  int64_t chunk;
  int32_t nchunks;
  int64_t want[kMaxBatch];
  SelectOut so;
  int32_t* idx;
  int32_t* count;
};
template <int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT == 512 ? 8 : 4))) void tk_resolve_emit_pair(ResolveSide a, ResolveSide b, int rows, int n_kv_heads,
                                                           int32_t k, bool only_failed) {
  const bool first = (int)blockIdx.x < rows;                // (the body stands once: its scalars fill the registers)
  const int row = first ? (int)blockIdx.x : (int)blockIdx.x - rows, seq = row / n_kv_heads;
  SelectOut so;
  so.spec = first ? a.so.spec : b.so.spec;
  so.ncand = first ? a.so.ncand : b.so.ncand;
  so.n1 = first ? a.so.n1 : b.so.n1;
  so.lists = first ? a.so.lists : b.so.lists;
  so.row_entries = first ? a.so.row_entries : b.so.row_entries;
  so.mon = first ? a.so.mon : b.so.mon;
  tk_resolve_emit_body<NT>(first ? a.chunk : b.chunk, first ? a.nchunks : b.nchunks, first ? a.want[seq] : b.want[seq], so,
                           k, first ? a.idx : b.idx, first ? a.count : b.count, only_failed, row);
}

namespace {
struct FusedPlan {
  SelRows sr;
  SelectOut so;
  TopkWs t;
  int64_t chunk;
  int nchunks;
};
int32_t fused_plan(const Layout& L, const NRes& nr, int64_t nmax, int32_t k, void* ws, FusedPlan* f) {
  for (int b = 0; b < kMaxBatch; ++b) { f->sr.nsel[b] = 0; f->sr.want[b] = -1; }
  for (int b = 0; b < L.batch; ++b) {
    f->sr.nsel[b] = nr.n[b];
    f->sr.want[b] = nr.n[b] < k ? nr.n[b] : k;
    if (f->sr.want[b] == 0) f->sr.want[b] = -1;
  }
  topk_carve(&f->t, ws, L.rows, L.cap);
  const int bpw = select_scan_bpw(L, nmax > 0 ? nmax : 1);
  if (bpw == 0) return HCA_ERR_CAPACITY;
  f->chunk = (int64_t)4 * bpw * L.tpb;
  const int64_t nblocks = (nmax + L.tpb - 1) / L.tpb;
  f->nchunks = (int)((nblocks + 4 * bpw - 1) / (4 * bpw));
  if (f->nchunks < 1) f->nchunks = 1;
  if (f->nchunks > kSelectMaxChunks || (int64_t)f->nchunks * f->chunk > f->t.row_entries) return HCA_ERR_CAPACITY;
  f->so = SelectOut{f->t.spec, f->t.ncand, f->t.above, f->t.cand, f->t.samples, f->t.row_entries, select_sample_count(nmax, k),
                    f->t.mon};
  return HCA_OK;
}
}  // namespace

// The fused selection in three parts, each on any stream ordered after the one before.
// 1. threshold from the sample.  The row lengths may be those before the step's token is appended: slots past
//    them are not sampled, and the estimate does not need the one more slot.
int32_t launch_select_threshold(const Layout& L, const void* kcache, const void* q, const NRes& nr, int64_t nmax,
                                int32_t k, void* ws, hipStream_t st) {
  FusedPlan f;
  int32_t rc = fused_plan(L, nr, nmax, k, ws, &f);
  if (rc != HCA_OK || nmax == 0) return rc;
  return launch_select_sample(L, kcache, q, nr, k, f.so, st);
}

// The parts of the fused selection as a decode step strings them together on one stream: (a) the sampling alone
// and (b) threshold from the samples + append of the step's key, as launches of their own for the step's first
// layers; (c) the selecting scan of a layer carrying (b) for the next layer and (a) for the one after it (lengths
// before those layers' own appends: the one more slot does not matter to the estimate and is not read).
// (nmax, nmax_before, next_nmax: the longest row at the lengths before the step's append - the sampling of a layer
// and its threshold must agree on the sample count, which depends on it.)
int32_t launch_select_samples(const Layout& L, const void* kcache, const void* q, const NRes& nr, int64_t nmax,
                              int32_t k, void* ws, hipStream_t st) {
  TopkWs t;
  topk_carve(&t, ws, L.rows, L.cap);
  SelectOut so{t.spec, t.ncand, t.above, t.cand, t.samples, t.row_entries, select_sample_count(nmax, k)};
  return launch_select_sample_scores(L, kcache, q, nr, so, st);
}

int32_t launch_select_threshold_append(const Layout& L, void* kcache, const void* k_new, const NRes& nr_before,
                                       int64_t nmax_before, float* acc, int32_t* pos, const NRes& vrow0, int32_t k,
                                       void* ws, hipStream_t st) {
  TopkWs t;
  topk_carve(&t, ws, L.rows, L.cap);
  SelectOut so{t.spec, t.ncand, t.above, t.cand, t.samples, t.row_entries, select_sample_count(nmax_before, k)};
  return launch_select_rank_append(L, kcache, k_new, nr_before, acc, pos, vrow0, k, so, st);
}

SelectOut select_view(const Layout& L, void* ws, int64_t nmax_before, int32_t k) {
  TopkWs t;
  topk_carve(&t, ws, L.rows, L.cap);
  return SelectOut{t.spec, t.ncand, t.above, t.cand, t.samples, t.row_entries, select_sample_count(nmax_before, k)};
}

int32_t launch_select_scan_step(const Layout& L, const void* kcache, const void* q, const NRes& nr, int64_t nmax,
                                int32_t k, void* ws, hipStream_t st, uint64_t* stamps, const SelectStepNext& nx) {
  FusedPlan f;
  const int32_t rc = fused_plan(L, nr, nmax, k, ws, &f);
  if (rc != HCA_OK) return rc;
  return launch_select_step(L, kcache, q, nr, nmax, f.so, st, stamps, nx);
}

int32_t launch_select_scan_step_pair(const Layout& L, const void* const kcache[2], const void* const q[2],
                                     const NRes nr[2], const int64_t nmax[2], int32_t k, void* const ws[2], hipStream_t st,
                                     uint64_t* const stamps[2], const SelectStepNext nx[2], hipEvent_t done) {
  SelectOut so[2];
  for (int i = 0; i < 2; ++i) {
    FusedPlan f;
    const int32_t rc = fused_plan(L, nr[i], nmax[i], k, ws[i], &f);
    if (rc != HCA_OK) return rc;
    so[i] = f.so;
  }
  return launch_select_step_pair(L, kcache, q, nr, nmax, so, stamps, nx, st, done);
}

// 2. the selecting scan
int32_t launch_select_begin(const Layout& L, const void* kcache, const void* q, const NRes& nr, int64_t nmax, int32_t k,
                            void* ws, hipStream_t st, uint64_t* stamps) {
  FusedPlan f;
  int32_t rc = fused_plan(L, nr, nmax, k, ws, &f);
  if (rc != HCA_OK || nmax == 0) return rc;
  return launch_select_scan(L, kcache, q, nr, nmax, f.so, false, st, stamps);
}

// 3. the selection over the lists, then,
// for rows whose sampled threshold left too few pairs, a scan with every slot a candidate and the selection
// again (both launches return at once for every other row).
int32_t launch_select_finish(const Layout& L, const void* kcache, const void* q, const NRes& nr, int64_t nmax, int32_t k,
                             int32_t* idx, int32_t* count, void* ws, hipStream_t st, int wg) {
  FusedPlan f;
  int32_t rc = fused_plan(L, nr, nmax, k, ws, &f);
  if (rc != HCA_OK) return rc;
  const auto form = wg == 256 ? tk_resolve_emit<256> : wg == 512 ? tk_resolve_emit<512> : tk_resolve_emit<1024>;
  form<<<L.rows, wg, 0, st>>>(f.chunk, f.nchunks, L.n_kv_heads, f.sr, f.so, k, idx, count, false);
  if (nmax > 0) {
    rc = launch_select_scan(L, kcache, q, nr, nmax, f.so, true, st);
    if (rc != HCA_OK) return rc;
    form<<<L.rows, wg, 0, st>>>(f.chunk, f.nchunks, L.n_kv_heads, f.sr, f.so, k, idx, count, true);
  }
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// The same in one launch, for a call that has the chip for itself (beside another stream's scan the workgroups for failed
// rows would wait for room; there the step driver's three small launches stay): a workgroup per compute unit in all.  With
// two per unit the last of them begin when the first have ended, and the launch took 26 us for 16.
static int32_t launch_select_finish_call(const Layout& L, const void* kcache, const void* q, const NRes& nr, int64_t nmax,
                                         int32_t k, int32_t* idx, int32_t* count, void* ws, hipStream_t st) {
  FusedPlan f;
  const int32_t rc = fused_plan(L, nr, nmax, k, ws, &f);
  if (rc != HCA_OK) return rc;
  const int64_t chunks = (int64_t)f.nchunks * L.rows;
  if (L.rows > kFinishRows) return launch_select_finish(L, kcache, q, nr, nmax, k, idx, count, ws, st, 1024);
  const unsigned wgs = (unsigned)(L.rows + (chunks < 256 - L.rows ? chunks : 256 - L.rows));       // one per compute unit
  const auto form = L.bits == 4 ? tk_finish<4> : tk_finish<2>;
  form<<<wgs, 1024, 0, st>>>(L, (const uint8_t*)kcache, (const uint16_t*)q, nr, f.chunk, f.nchunks, f.sr, f.so, k, idx, count);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// The same for the two layers of a paired scan launch: three launches for the two of them.
int32_t launch_select_finish_pair(const Layout& L, const void* const kcache[2], const void* const q[2], const NRes nr[2],
                                  const int64_t nmax[2], int32_t k, int32_t* const idx[2], int32_t* const count[2],
                                  void* const ws[2], hipStream_t st, int wg) {
  FusedPlan f[2];
  ResolveSide rs[2];
  for (int i = 0; i < 2; ++i) {
    const int32_t rc = fused_plan(L, nr[i], nmax[i], k, ws[i], &f[i]);
    if (rc != HCA_OK) return rc;
    rs[i].chunk = f[i].chunk;
    rs[i].nchunks = f[i].nchunks;
    for (int b = 0; b < kMaxBatch; ++b) rs[i].want[b] = f[i].sr.want[b];
    rs[i].so = f[i].so;
    rs[i].idx = idx[i];
    rs[i].count = count[i];
  }
  int32_t rc = HCA_OK;
  const auto form = wg == 256 ? tk_resolve_emit_pair<256> : wg == 512 ? tk_resolve_emit_pair<512> : tk_resolve_emit_pair<1024>;
  form<<<2 * L.rows, wg, 0, st>>>(rs[0], rs[1], L.rows, L.n_kv_heads, k, false);
  if (nmax[0] > 0 && nmax[1] > 0) {
    const SelectOut so2[2] = {f[0].so, f[1].so};
    rc = launch_select_rescan_pair(L, kcache, q, nr, nmax, so2, st);
    if (rc != HCA_OK) return rc;
    // the selection for rows that had to be scanned again - almost never any - in the four-wave form: beside a running
    // scan the 1024-thread form would wait for a compute unit to drain just to find that it has nothing to do
    tk_resolve_emit_pair<256><<<2 * L.rows, 256, 0, st>>>(rs[0], rs[1], L.rows, L.n_kv_heads, k, true);
  }
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// Top-k of long rows from their scores in three or four launches: a key from samples, the lists of the slots above it, the
// selection over them.  Bound by the launches' latency and one pass over the scores.
static int32_t launch_topk_sampled(const Layout& L, const float* scores, const NRes& nr, int64_t nmax, const SelRows& sr,
                                   int32_t k, int32_t* idx, int32_t* count, const TopkWs& t, ListRoom room,
                                   const RowSelectFused& fu, hipStream_t st) {
  int64_t chunk;
  int32_t nchunks;
  chunk_geometry(nmax, &chunk, &nchunks);
  if (room.slots == nullptr) room.pair_chunk = chunk;
  else if ((room.pair_chunk = room.pair_row / nchunks) > chunk) room.pair_chunk = chunk;
  // (the samples' keys, where they need a place, in that of the row's pairs, which are written later; a row has more room
  // for pairs than samples)
  const int32_t rc = launch_topk_sample_rank(scores, L.cap, L.rows, L.n_kv_heads, nr, nmax, k, select_sample_count(nmax, k),
                                             reinterpret_cast<uint32_t*>(room.pairs), 2 * room.pair_row, t.state, st);
  if (rc != HCA_OK) return rc;
  tk_collect_sampled<<<dim3((unsigned)nchunks, (unsigned)L.rows), 256, 0, st>>>(scores, L.cap, chunk, L.n_kv_heads, sr, t, room);
  tk_resolve_scores<<<L.rows, 1024, 0, st>>>(scores, L.cap, chunk, nchunks, L.n_kv_heads, sr, t, room, k, idx, count, fu);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// Rows up to which, and slots in all rows below which, hca_score_topk writes the scores and selects from them - four launches
// - instead of sampling and scanning the codes for a threshold and looking for rows to scan again - six.  What the scores
// cost is 8 bytes per slot.  The call by the six / these four, k = 2048, 4-bit (2-bit) codes, us: 1 row of 65 536 36 / 34 (39
// / 36), of 131 072 36 / 38 (39 / 38); 8 rows of 41 000 41 / 38 (42 / 38), of 65 536 41 / 39 (42 / 39), of 100 000 44.5 / 43.7
// (43.5 / 42.1), of 131 072 45.4 / 46.8 (43.3 / 44.1); 16 of 65 536 46.5 / 45.4 (43.7 / 42.8), of 80 000 49.5 / 51.1 (45.1 /
// 46.1); 32 of 41 000 51.5 / 51.4 (46.7 / 46.3).
constexpr int64_t kScoresMax = 98304, kScoresAll = 1200000;

int32_t launch_score_topk(const Layout& L, const void* kcache, const void* q, const NRes& nr, int64_t nmax, int32_t k,
                          int32_t* idx, int32_t* count, void* ws, hipStream_t st) {
  if (nmax > 0 && nmax <= kRowSelectMax) {
    // short rows: every score into the room of the candidate lists (8 B per slot there, 4 needed), then one launch
    FusedPlan f;
    int32_t rc = fused_plan(L, nr, nmax, k, ws, &f);
    if (rc != HCA_OK) return rc;
    float* scores = reinterpret_cast<float*>(f.t.cand);
    rc = launch_score(L, kcache, q, nr, nmax, scores, nullptr, st);
    if (rc != HCA_OK) return rc;
    return launch_row_select(scores, L.cap, L.rows, L.n_kv_heads, f.sr, nmax, k, idx, count,
                             RowSelectFused{f.t.spec, f.t.ncand, f.t.mon, f.nchunks}, st);
  }
  if (nmax > kRowSelectMax && nmax <= kScoresMax && L.rows * nmax < kScoresAll && select_sample_count(nmax, k) <= 16384 &&
      select_lists_fit(nmax, k)) {
    // rows of medium length: the scores into the first half of the room of the lists, the lists' slots into the second, and
    // the lists' (key, slot) pairs, as far as they fit - where the row's best are not crowded in a chunk, all of them - into
    // the room of the samples (by slots alone, a dependent load per pair, 8 rows of 1 Mi scores take 54 us for 43)
    FusedPlan f;
    int32_t rc = fused_plan(L, nr, nmax, k, ws, &f);
    if (rc != HCA_OK) return rc;
    float* scores = reinterpret_cast<float*>(f.t.cand);
    rc = launch_score(L, kcache, q, nr, nmax, scores, nullptr, st);
    if (rc != HCA_OK) return rc;
    const ListRoom room{reinterpret_cast<uint2*>(f.t.samples), reinterpret_cast<uint32_t*>(f.t.cand) + L.rows * f.t.row_entries,
                        kSampleMax / 2, 0, f.t.row_entries};
    return launch_topk_sampled(L, scores, nr, nmax, f.sr, k, idx, count, f.t, room,
                               RowSelectFused{f.t.spec, f.t.ncand, f.t.mon, f.nchunks}, st);
  }
  int32_t rc = launch_select_threshold(L, kcache, q, nr, nmax, k, ws, st);
  if (rc != HCA_OK) return rc;
  rc = launch_select_begin(L, kcache, q, nr, nmax, k, ws, st, nullptr);
  if (rc != HCA_OK) return rc;
  if (tuning().select_wg > 0 && tuning().select_wg != 1024)
    return launch_select_finish(L, kcache, q, nr, nmax, k, idx, count, ws, st, tuning().select_wg);
  return launch_select_finish_call(L, kcache, q, nr, nmax, k, idx, count, ws, st);
}

// What the last fused selection on this workspace did, per row: pairs that passed the threshold of the scan that
// produced the result, and whether that scan was the second, unthresholded one.
__global__ __launch_bounds__(256) void tk_select_report(TopkWs t, int nchunks, int32_t* __restrict__ candidates,
                                                        int32_t* __restrict__ rescanned) {
  __shared__ uint32_t wsum[4];
  const int row = blockIdx.x;
  uint32_t v = 0;
  const uint32_t* counts = t.spec[4 * row + 1] == 2 ? t.samples : t.ncand;      // (of a second scan by tk_finish: with the samples)
  for (int c = threadIdx.x; c < nchunks; c += 256) v += counts[(int64_t)row * kMaxChunks + c];
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    candidates[row] = (int32_t)(wsum[0] + wsum[1] + wsum[2] + wsum[3]);
    rescanned[row] = t.spec[4 * row + 1] != 0;
  }
}

int32_t launch_select_report(const Layout& L, const NRes& nr, int64_t nmax, void* ws, int32_t* candidates,
                             int32_t* rescanned, hipStream_t st) {
  FusedPlan f;
  const int32_t rc = fused_plan(L, nr, nmax, 1, ws, &f);
  if (rc != HCA_OK) return rc;
  tk_select_report<<<L.rows, 256, 0, st>>>(f.t, nmax > 0 ? f.nchunks : 0, candidates, rescanned);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// The running figures of the fused selections on a workspace (mon above), copied out and / or started afresh.
__global__ void tk_select_monitor(uint32_t* __restrict__ mon, int rows, int32_t* __restrict__ out, int reset) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * 4) return;
  if (out != nullptr) out[i] = (int32_t)mon[i];
  if (reset) mon[i] = (i & 3) == 1 ? 0x7fffffffu : 0u;
}

int32_t launch_select_monitor(const Layout& L, void* ws, int32_t* out, int reset, hipStream_t st) {
  TopkWs t;
  topk_carve(&t, ws, L.rows, L.cap);
  tk_select_monitor<<<(L.rows * 4 + 255) / 256, 256, 0, st>>>(t.mon, L.rows, out, reset);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// ---------------------------------------------------------------------------------------
// Cumulative-weight selection (Sec. 3.2, Eq. 4): the shortest prefix of the descending order whose
// softmax weight reaches tau.  Weights are integers (fixed-order fp32 arithmetic, see tp_weight), so
// the histogram sums below are exact and independent of the order in which atomics land.  The
// radix walk is the top-k one with two running totals: it stops in the first bin / digit / equal-key
// group where the weight reaches the target or the slot count reaches k_max.

// Integer weight of a logit u <= 0 relative to the row maximum: about exp(u) * 2^31.
//   t = u * log2(e); below -64 -> 0; fl = floor(t); f = t - fl in [0, 1) (exact);
//   p = 2^f by a degree-6 polynomial in Horner form with fused multiply-adds, c_k = (ln 2)^k / k!;
//   mant = (uint64)(p * 2^31) (truncated); w = mant >> -fl.
// p < 2 (the polynomial at f = 1 is 1.99999), so mant has 32 bits and w, at most 2^31, is 0 from -fl = 32 on.
__device__ __forceinline__ uint32_t tp_weight(float u) {
  const float t = u * 1.44269504f;
  if (!(t >= -32.0f)) return 0;
  const float fl = floorf(t);
  const float f = t - fl;
  float p = 1.5403530e-4f;
  p = fmaf(p, f, 1.3333558e-3f);
  p = fmaf(p, f, 9.6181291e-3f);
  p = fmaf(p, f, 5.5504109e-2f);
  p = fmaf(p, f, 2.4022651e-1f);
  p = fmaf(p, f, 6.9314718e-1f);
  p = fmaf(p, f, 1.0f);
  const uint32_t mant = (uint32_t)(p * 2147483648.0f), sh = (uint32_t)(-fl);
  return sh >= 32 ? 0 : mant >> sh;
}

// Bins of the cumulative walk, from the row maximum down: every slot's bin number is the sum of two steps that fall with
// its score.  The coarse one has 24 steps per factor of two in weight, down to 2^-64 of the maximum.  The fine one has
// 512 over the window in which most of the row lies (tp_rowmax, tp_hist): a row whose weights are nearly equal spans a
// fraction of one coarse step, and without the window nearly all its slots lie in the bin to be resolved, by one workgroup
// over lists that no longer fit its LDS.  Per call, key bins of 12 bits / 32 steps per factor of two / both kinds, 4096 to
// select: 8 rows of 131 072 scores with a spread of 0.1, 64 / 209 / 44 us, with a spread of 11, 64 / 42 / 42; 8 x 500 000
// with 11, 65 / 52 / 55.  More fine steps make the histograms' flush longer, with 256 a bin in the middle of a flat row of
// 500 000 slots no longer fits LDS (118 -> 362 us).
// The bins only steer the walk; any bin number that grows with the key gives the same selection.
constexpr int kTpBins = 2048;
constexpr int kTpFine = kTpBins / 4;
struct TpBin {
  float m, sm;           // the row maximum's logit, the softmax scale
  float top, per_unit;   // the window's upper end and the fine steps per unit of score (0: no window)
  __device__ __forceinline__ uint32_t operator()(float f) const {
    const uint32_t coarse = (uint32_t)__builtin_amdgcn_fmed3f((f * sm - m) * (-1.44269504f * (kTpBins - kTpFine) / 64.0f), 0.0f,
                                                              (float)(kTpBins - kTpFine - 1));
    const uint32_t fine = (uint32_t)__builtin_amdgcn_fmed3f((top - f) * per_unit, 0.0f, (float)kTpFine);
    return (uint32_t)(kTpBins - 1) - coarse - fine;
  }
};

// Row maximum of every group of chunks, as an order key (in `above`, the room of the chunk counts), the largest and the
// smallest score of each of the group's first two waves (in `coff`, the room of the chunk prefixes), and clean counters
// for the histogram pass.  span: the difference of scores beyond which a weight is less than 2^-64 of the larger one; a
// smallest score takes no account of those, a mask's lowest value must not widen the window.
__global__ __launch_bounds__(256) void tp_rowmax(const float* __restrict__ vals, int64_t stride, int64_t chunk,
                                                 int n_kv_heads, SelRows sr, float span, TopkWs t) {
  __shared__ float wmax[4];
  const int row = blockIdx.y;
  if (sr.want[row / n_kv_heads] <= 0) return;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < kTpBins; i += gridDim.x * 256) {
    t.pcount[(int64_t)row * kBins12 + i] = 0;
    t.pmass[(int64_t)row * kBins12 + i] = 0;
  }
  const int64_t nsel = sr.nsel[row / n_kv_heads];
  const int64_t c0 = (int64_t)blockIdx.x * chunk;
  int64_t c1 = c0 + chunk;
  if (c1 > nsel) c1 = nsel;
  const float* v = vals + (int64_t)row * stride;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float hi = -INFINITY, lo = INFINITY;
  for (int64_t s0 = c0; s0 < c1; s0 += 4096) {
    float f[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const int64_t j = s0 + x * 256 + threadIdx.x;
      f[x] = v[j < c1 ? j : c1 - 1];
    }
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      if (s0 + x * 256 + threadIdx.x >= c1) f[x] = -INFINITY;
      hi = fmaxf(hi, f[x]);
    }
    if (w < 2) {
#pragma unroll
      for (int x = 0; x < 16; ++x)
        if (f[x] > hi - span) lo = fminf(lo, f[x]);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float oh = __shfl_xor(hi, o), ol = __shfl_xor(lo, o), most = fmaxf(hi, oh), cut = most - span;
    lo = fminf(hi > cut ? fmaxf(lo, cut) : INFINITY, oh > cut ? fmaxf(ol, cut) : INFINITY);
    hi = most;
  }
  if ((threadIdx.x & 63) == 0) {
    wmax[w] = hi;
    if (w < 2) reinterpret_cast<float2*>(t.coff)[(int64_t)row * 1024 + 2 * blockIdx.x + w] = float2{hi, lo};
  }
  __syncthreads();
  if (threadIdx.x == 0)
    t.above[(int64_t)row * 1024 + blockIdx.x] =
        c0 < c1 ? order_key(fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]))) : 0u;
}

// Histogram of slot counts and integer weights, both in one 64-bit LDS counter per bin: up to 2^15 slots' weights of at most
// 2^31 stay below bit 47, the slots are counted from there on.  Bound by the counters and, level with them, by the weights'
// arithmetic; with two counters and 64-bit weights 8 rows of 500 003 slots took 13.5 us.
constexpr int kTpCountBit = 47, kTpCountMax = 1 << 15;
template <int NT>
__global__ __launch_bounds__(NT) void tp_hist(const float* __restrict__ vals, int64_t stride, int64_t chunk, int64_t group,
                                              int groups, int n_kv_heads, SelRows sr, float sm_scale, float span, TopkWs t) {
  __shared__ uint32_t wmax[NT / 64];
  __shared__ unsigned long long lm[kTpBins];
  __shared__ float s_top, s_low;
  const int row = blockIdx.y;
  if (sr.want[row / n_kv_heads] <= 0) return;
  const int64_t nsel = sr.nsel[row / n_kv_heads];
  const int64_t c0 = (int64_t)blockIdx.x * chunk;
  if (c0 >= nsel) return;
  int64_t c1 = c0 + chunk;
  if (c1 > nsel) c1 = nsel;
  const float* v = vals + (int64_t)row * stride;
  float f[16];
  auto load = [&](int64_t s0) {
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const int64_t j = s0 + x * NT + threadIdx.x;
      f[x] = v[j < c1 ? j : c1 - 1];
    }
  };
  load(c0);                                                 // on their way while the bins are laid out
  for (int i = threadIdx.x; i < kTpBins; i += NT) lm[i] = 0;
  uint32_t kmax = 0;
  for (int c = threadIdx.x; c < groups; c += NT) {
    const uint32_t x = t.above[(int64_t)row * 1024 + c];
    kmax = x > kmax ? x : kmax;
  }
  kmax = wave_max(kmax);
  const int lane = threadIdx.x & 63;
  if (lane == 0) wmax[threadIdx.x >> 6] = kmax;
  if (threadIdx.x >> 6 == 1) {
    // The window: of up to sixteen waves of tp_rowmax, spread over the row, the lower quartile of the largest scores and
    // the upper quartile of the smallest, waves that weigh nothing left out.  A few outliers either way do not move it, and
    // what lies outside has the coarse steps.
    const int pairs = 2 * (int)((nsel + group - 1) / group);
    const int ns = pairs < 16 ? pairs : 16;
    const float2 p = reinterpret_cast<const float2*>(t.coff)[(int64_t)row * 1024 + (lane < ns ? lane : 0) * pairs / ns];
    float most = p.x;
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) most = fmaxf(most, __shfl_xor(most, o));
    most = __shfl(most, 0);                                 // (lanes from 16 on hold pair 0 again)
    const uint64_t counts = __ballot(lane < ns && p.x > most - span);
    const int quarter = __popcll(counts) / 4;
    int below = 0, over = 0;
    for (uint64_t left = counts; left != 0; left &= left - 1) {
      const int i = __builtin_ctzll(left);
      const float oh = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p.x), i));
      const float ol = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p.y), i));
      below += oh < p.x || (oh == p.x && i < lane);
      over += ol > p.y || (ol == p.y && i < lane);
    }
    if (lane == 0) { s_top = -INFINITY; s_low = INFINITY; }
    __builtin_amdgcn_wave_barrier();
    if ((counts >> lane & 1) && below == quarter) s_top = p.x;
    if ((counts >> lane & 1) && over == quarter) s_low = p.y;
  }
  __syncthreads();
  for (int x = 0; x < NT / 64; ++x) if (wmax[x] > kmax) kmax = wmax[x];
  const float m = key_to_float(kmax) * sm_scale;
  const float per = (float)kTpFine / (s_top - s_low);
  const bool window = s_top > s_low && per < INFINITY;
  const TpBin bin_of{m, sm_scale, window ? s_top : 0.0f, window ? per : 0.0f};
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    t.prow[4 * row] = kmax;
    reinterpret_cast<float2*>(t.pstate)[4 * row + 1] = float2{bin_of.top, bin_of.per_unit};
  }
  for (int64_t s0 = c0; s0 < c1; s0 += 16 * NT) {
    if (s0 != c0) load(s0);
#pragma unroll
    for (int x = 0; x < 16; ++x)
      if (s0 + x * NT + threadIdx.x < c1) {
        const uint32_t b = bin_of(f[x]);
        // bin 0 weighs nothing and may hold nearly the whole row: it is not counted (its slots are the row's others)
        const uint64_t one = tp_weight(f[x] * sm_scale - m) | (b != 0 ? 1ull << kTpCountBit : 0ull);
        if (one) atomicAdd(&lm[b], (unsigned long long)one);
      }
    if (s0 + 16 * NT >= c1 || (s0 + 16 * NT - c0) % kTpCountMax == 0) {       // the last slots, or no room for more
      __syncthreads();
      for (int i = threadIdx.x; i < kTpBins; i += NT) {
        const unsigned long long both = lm[i];
        const uint32_t c = (uint32_t)(both >> kTpCountBit);
        const unsigned long long mm = both & ((1ull << kTpCountBit) - 1);
        if (c) atomicAdd(&t.pcount[(int64_t)row * kBins12 + i], c);
        if (mm) atomicAdd(reinterpret_cast<unsigned long long*>(&t.pmass[(int64_t)row * kBins12 + i]), mm);
        lm[i] = 0;
      }
      __syncthreads();
    }
  }
}

// Z, Theta, and the first bin (from the top) in which the running weight reaches Theta or the running count reaches
// k_max - found by every workgroup from the finished histogram, 24 KB from L2, instead of in a launch of its own - and
// then the ordered lists of the slots in or above that bin.
__global__ __launch_bounds__(256) void tp_collect(const float* __restrict__ vals, int64_t stride, int64_t chunk,
                                                  int n_kv_heads, SelRows sr, float sm_scale, uint64_t tau_fix, bool tau_one,
                                                  uint32_t k_max, TopkWs t, uint64_t* __restrict__ mass_out) {
  __shared__ uint64_t wsum64[4];
  __shared__ uint32_t wsum[4], s_bin, s_first[2];
  const int row = blockIdx.y;
  const bool writer = blockIdx.x == 0;
  if (sr.want[row / n_kv_heads] <= 0) {
    if (mass_out != nullptr && writer && threadIdx.x < 2) mass_out[2 * row + threadIdx.x] = 0;
    return;
  }
  collect_chunk<false>(vals, stride, chunk, sr.nsel[row / n_kv_heads], row, t, [&](uint32_t* first, uint32_t* last) {
    const float2 window = reinterpret_cast<const float2*>(t.pstate)[4 * row + 1];
    const uint32_t kmax = t.prow[4 * row];
    constexpr int BPT = kTpBins / 256;
    uint32_t hc[BPT], csum = 0;
    uint64_t hm[BPT], msum = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int b = kTpBins - 1 - (BPT * threadIdx.x + i);
      hc[i] = t.pcount[(int64_t)row * kBins12 + b];
      hm[i] = t.pmass[(int64_t)row * kBins12 + b];
      csum += hc[i];
      msum += hm[i];
    }
    uint64_t Z;
    uint64_t run_m = block_scan_excl<4>(msum, wsum64, &Z);
    uint32_t run_c = block_scan_excl<4>(csum, wsum);
    uint64_t theta = tau_one ? Z : __umul64hi(Z, tau_fix);
    if (theta < 1) theta = 1;
    if (threadIdx.x == 255) hc[BPT - 1] = (uint32_t)sr.nsel[row / n_kv_heads] - (run_c + csum);     // bin 0
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const bool before = run_m < theta && run_c < k_max;
      const bool after = run_m + hm[i] >= theta || run_c + hc[i] >= k_max;
      if (before && after && hc[i] > 0) {
        s_bin = (uint32_t)(kTpBins - 1 - (BPT * threadIdx.x + i));       // b*
        if (writer) {
          t.pstate[4 * row] = theta - run_m;                              // weight still to reach inside the bin
          t.prow[4 * row + 1] = k_max - run_c;                            // slots still allowed
        }
      }
      run_m += hm[i];
      run_c += hc[i];
    }
    if (writer && threadIdx.x == 0 && mass_out != nullptr) { mass_out[2 * row] = theta; mass_out[2 * row + 1] = Z; }
    __syncthreads();
    const TpBin bin_of{key_to_float(kmax) * sm_scale, sm_scale, window.x, window.y};
    // the smallest key of the bin (wave 0) and of the bins above it (wave 1), 64 keys at a time: the pass over the row and
    // the resolve stage then compare keys and compute no bins
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (w < 2) {
      const uint32_t bin = s_bin + w;
      uint32_t below = order_key(-INFINITY) - 1, found = kmax + 1;      // the row maximum lies in the top bin
      while (found - below > 1) {
        const uint32_t step = (found - below + 63) / 64, key = below + step * (lane + 1);
        const bool yes = key - below >= found - below || bin_of(key_to_float(key)) >= bin;
        const int at = __builtin_ctzll(__builtin_amdgcn_ballot_w64(yes) | 1ull << 63);
        if (step * (at + 1) < found - below) found = below + step * (at + 1);
        below += step * at;
      }
      if (lane == 0) s_first[w] = bin == 0 ? 0u : found;
    }
    __syncthreads();
    *first = s_first[0];
    *last = s_first[1] - 1;
    if (writer && threadIdx.x == 0) { t.state[4 * row + 2] = *first; t.state[4 * row + 3] = *last; }
  });
}

// no resident slot anywhere: only the per-row (Theta, Z) report has to be cleared
__global__ void tp_no_mass(uint64_t* __restrict__ mass_out, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) mass_out[i] = 0;
}

// One workgroup per row: finishes the walk inside bin b* (digits of the distance from the bin's smallest key, then the
// group of equal keys, whose members all weigh the same) and builds the chunk offsets for the ordered emit.
__global__ __launch_bounds__(1024) void tp_resolve(int64_t chunk, int nchunks, int n_kv_heads, SelRows sr, float sm_scale,
                                                   TopkWs t) {
  __shared__ uint32_t h[1024], e[1024], cnt[1024], wsum[16], wmin[16], wmax[16];
  __shared__ unsigned long long hm[1024];
  __shared__ uint64_t wsum64[16];
  __shared__ uint32_t s_digit, s_krem, s_n, s_eq;
  __shared__ uint64_t s_mrem;
  __shared__ uint2 lc[kResolveLds];
  const int row = blockIdx.x;
  if (sr.want[row / n_kv_heads] <= 0) return;
  const uint32_t last = t.state[4 * row + 3];               // (the lists hold no key below the bin)
  const uint2* cand = t.cand + (int64_t)row * t.row_entries;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float m = key_to_float(t.prow[4 * row]) * sm_scale;
  uint32_t krem = t.prow[4 * row + 1];
  uint64_t mrem = t.pstate[4 * row];
  cnt[tid] = tid < nchunks ? t.ncand[(int64_t)row * kMaxChunks + tid] : 0;
  if (tid == 0) s_n = 0;
  __syncthreads();
  // f(key, slot, hit) over every list entry of the row, hit = the entry exists and lies in bin b*; f is called by all lanes
  // of a wave together.  Each wave takes 8 chunks per step and fetches the first 128 entries of all of them in one batch
  // of loads, so a step costs one memory round trip; longer lists follow, 8 loads in flight.  Rows of up to 8 chunks: the
  // waves share a chunk's list.
  auto stretch = [&](auto&& f, int c, uint32_t from, uint32_t step) {
    const uint32_t mc = cnt[c];
    for (uint32_t i0 = from + lane; i0 < mc + lane; i0 += step) {
      uint2 x[8];
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        x[v] = uint2{0, 0};
        if (i0 + 64 * v < mc) x[v] = cand[(int64_t)c * chunk + i0 + 64 * v];
      }
#pragma unroll
      for (int v = 0; v < 8; ++v) f(x[v].x, x[v].y, i0 + 64 * v < mc && x[v].x <= last);
    }
  };
  auto sweep = [&](auto&& f) {
    if (nchunks <= 8) {
      const int parts = 16 / nchunks;
      if (wv < parts * nchunks) stretch(f, wv % nchunks, 512u * (uint32_t)(wv / nchunks), 512u * (uint32_t)parts);
      return;
    }
    for (int c0 = 0; c0 < nchunks; c0 += 128) {
      uint2 ent[16];
      bool has[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int c = c0 + (u >> 1) * 16 + wv;
        const uint32_t i = (uint32_t)(64 * (u & 1) + lane);
        has[u] = c < nchunks && i < cnt[c < nchunks ? c : 0];
        ent[u] = uint2{0, 0};
        if (has[u]) ent[u] = cand[(int64_t)c * chunk + i];
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) f(ent[u].x, ent[u].y, has[u] && ent[u].x <= last);
#pragma unroll 1
      for (int u = 0; u < 8; ++u)
        if (c0 + u * 16 + wv < nchunks) stretch(f, c0 + u * 16 + wv, 128u, 512u);
    }
  };
  uint32_t lo = 0xffffffffu, hi = 0;                        // smallest and largest key of the bin
  sweep([&](uint32_t key, uint32_t slot, bool hit) {
    if (hit) { lo = key < lo ? key : lo; hi = key > hi ? key : hi; }
    lds_append(&s_n, lc, (uint32_t)kResolveLds, key, slot, hit);
  });
  lo = wave_min(lo);
  hi = wave_max(hi);
  if (lane == 0) { wmin[wv] = lo; wmax[wv] = hi; }
  __syncthreads();
  for (int x = 0; x < 16; ++x) { lo = wmin[x] < lo ? wmin[x] : lo; hi = wmax[x] > hi ? wmax[x] : hi; }
  const uint32_t nst = s_n;
  const bool staged = nst <= (uint32_t)kResolveLds;
  auto visit = [&](auto&& f) {
    if (staged) {
      for (uint32_t i0 = 0; i0 < nst; i0 += 1024) {
        const bool hit = i0 + tid < nst;
        const uint2 x = lc[hit ? i0 + tid : 0];
        f(x.x, x.y, hit);
      }
    } else {
      sweep(f);
    }
  };
  uint32_t cnt_eq = 0, pd = 0;
  int left = 32 - __clz((int)((hi - lo) | 1u));             // 1 .. 32
  bool first = true;
  if (nst <= kDirectRank) {
    // a few keys: each is compared with all others, eight threads to a key, instead of two to four rounds of digits
    const uint32_t i = tid & (kDirectRank - 1), share = tid / kDirectRank, each = kDirectRank / (1024 / kDirectRank);
    if (tid < (int)kDirectRank) {
      h[tid] = 0;
      e[tid] = 0;
      hm[tid] = 0;
      hm[kDirectRank + tid] = i < nst ? tp_weight(key_to_float(lc[i].x) * sm_scale - m) : 0;
    }
    __syncthreads();
    if (i < nst) {
      const uint32_t ki = lc[i].x;
      uint32_t gt = 0, eq = 0;
      uint64_t over = 0;
      for (uint32_t j = share * each; j < (share + 1) * each && j < nst; ++j) {
        const uint32_t kj = lc[j].x;
        gt += kj > ki;
        eq += kj == ki;
        over += kj > ki ? hm[kDirectRank + j] : 0;
      }
      if (gt) atomicAdd(&h[i], gt);
      if (eq) atomicAdd(&e[i], eq);
      if (over) atomicAdd(&hm[i], (unsigned long long)over);
    }
    __syncthreads();
    if (tid < (int)nst) {
      const uint32_t run_c = h[tid], eq = e[tid];
      const uint64_t run_m = hm[tid];
      if (run_m < mrem && run_c < krem && (run_m + hm[kDirectRank + tid] * eq >= mrem || run_c + eq >= krem)) {
        s_digit = lc[tid].x - lo;                           // equal keys write equal values
        s_eq = eq;
        s_mrem = mrem - run_m;
        s_krem = krem - run_c;
      }
    }
    __syncthreads();
    pd = s_digit;
    cnt_eq = s_eq;
    mrem = s_mrem;
    krem = s_krem;
    left = 0;
    __syncthreads();
  }
  // the distances from lo, 10 bits at a time from the top: pd = the digits found, left = the bits below them
  while (left > 0) {                                        // uniform over the workgroup
    const int width = left > 10 ? 10 : left, ns = left - width;
    h[tid] = 0;
    hm[tid] = 0;
    __syncthreads();
    visit([&](uint32_t key, uint32_t, bool hit) {
      const uint32_t d = key - lo;
      const bool in = hit && (first || (d >> left) == pd);
      const uint64_t w = in ? tp_weight(key_to_float(key) * sm_scale - m) : 0;
      lds_count_mass(h, hm, (d >> ns) & ((1u << width) - 1u), key, w, in, !staged);
    });
    __syncthreads();
    const uint32_t mine_c = h[1023 - tid];                  // thread tid owns digit 1023 - tid
    const uint64_t mine_m = hm[1023 - tid];
    const uint32_t run_c = block_scan_excl<16>(mine_c, wsum);
    const uint64_t run_m = block_scan_excl<16>(mine_m, wsum64);
    const bool before = run_m < mrem && run_c < krem;
    const bool after = run_m + mine_m >= mrem || run_c + mine_c >= krem;
    if (before && after && mine_c > 0) {
      s_digit = (uint32_t)(1023 - tid);
      s_eq = mine_c;
      s_mrem = mrem - run_m;
      s_krem = krem - run_c;
    }
    __syncthreads();
    pd = first ? s_digit : ((pd << width) | s_digit);
    cnt_eq = s_eq;
    mrem = s_mrem;
    krem = s_krem;
    left = ns;
    first = false;
    __syncthreads();
  }
  const uint32_t T = lo + pd;
  // the cnt_eq slots with key == T all weigh w_T: take the least r with r * w_T >= mrem, within the
  // count limit
  const uint64_t wT = tp_weight(key_to_float(T) * sm_scale - m);
  uint64_t need = wT > 0 ? (mrem + wT - 1) / wT : (uint64_t)cnt_eq;
  if (need > krem) need = krem;
  if (need > cnt_eq) need = cnt_eq;
  const uint32_t req = (uint32_t)need;
  h[tid] = 0;
  e[tid] = 0;
  __syncthreads();
  visit([&](uint32_t key, uint32_t slot, bool hit) {
    lds_count(h, slot / (uint32_t)chunk, hit && key > T, !staged);
    lds_count(e, slot / (uint32_t)chunk, hit && key == T, !staged);
  });
  __syncthreads();
  const uint32_t g = (tid < nchunks) ? t.above[(int64_t)row * 1024 + tid] + h[tid] : 0;
  const uint32_t q = (tid < nchunks) ? e[tid] : 0;
  const uint32_t og = block_scan_excl<16>(g, wsum);
  const uint32_t oe = block_scan_excl<16>(q, wsum);
  if (tid < nchunks) {
    t.coff[((int64_t)row * nchunks + tid) * 2] = og;
    t.coff[((int64_t)row * nchunks + tid) * 2 + 1] = oe;
  }
  if (tid == nchunks - 1) t.prow[4 * row + 2] = og + g + req;      // selected slots: all above T plus req of the equal ones
  if (tid == 0) { t.state[4 * row] = T; t.state[4 * row + 1] = req; }
}

int32_t launch_topp(const Layout& L, const float* sel, const NRes& nr, int64_t nmax, float sm_scale, double tau,
                    int32_t k_max, int32_t* idx, int32_t* count, uint64_t* mass_opt, void* ws, hipStream_t st) {
  SelRows sr;
  for (int b = 0; b < kMaxBatch; ++b) { sr.nsel[b] = 0; sr.want[b] = -1; }
  for (int b = 0; b < L.batch; ++b) {
    sr.nsel[b] = nr.n[b];
    sr.want[b] = nr.n[b] > 0 ? k_max : -1;
  }
  TopkWs t;
  topk_carve(&t, ws, L.rows, L.cap);
  int64_t chunk;
  int32_t nchunks;
  chunk_geometry(nmax, &chunk, &nchunks);
  dim3 g((unsigned)nchunks, (unsigned)L.rows);
  const bool tau_one = tau >= 1.0;
  const uint64_t tau_fix = tau_one ? 0 : (uint64_t)ldexp(tau, 64);
  if (nmax > 0) {
    dim3 gh((unsigned)((nchunks + 1) / 2), (unsigned)L.rows);
    const float span = 44.3614196f / sm_scale;               // 64 ln 2 in scores: lower ones weigh nothing
    tp_rowmax<<<gh, 256, 0, st>>>(sel, L.cap, 2 * chunk, L.n_kv_heads, sr, span, t);
    // one batch of loads per thread; each workgroup flushes its bins with global atomics, so the larger ones where they fill
    // the chip.  256 threads and two batches / 512 / 1024, the whole chain of calls: 8 rows of 500 003 slots 153.2 / 149.8 /
    // 146.9 us, 32 of 130 000 151.9 / 148.8 / 147.7, 8 of 300 001 170.8 / 168.0 / 168.6, of 64 000 76.8 / 74.0 / 76.1
    if ((nchunks + 3) / 4 * L.rows >= 192)
      tp_hist<1024><<<dim3((unsigned)((nchunks + 3) / 4), (unsigned)L.rows), 1024, 0, st>>>(
          sel, L.cap, 4 * chunk, 2 * chunk, (int)gh.x, L.n_kv_heads, sr, sm_scale, span, t);
    else
      tp_hist<512><<<gh, 512, 0, st>>>(sel, L.cap, 2 * chunk, 2 * chunk, (int)gh.x, L.n_kv_heads, sr, sm_scale, span, t);
    tp_collect<<<g, 256, 0, st>>>(sel, L.cap, chunk, L.n_kv_heads, sr, sm_scale, tau_fix, tau_one, (uint32_t)k_max, t, mass_opt);
    tp_resolve<<<L.rows, 1024, 0, st>>>(chunk, nchunks, L.n_kv_heads, sr, sm_scale, t);
  } else if (mass_opt != nullptr) {
    tp_no_mass<<<(unsigned)((2 * L.rows + 255) / 256), 256, 0, st>>>(mass_opt, 2 * L.rows);
  }
  tk_emit_lists<<<g, 256, 0, st>>>(chunk, nchunks, L.n_kv_heads, sr, t, k_max, idx, count, true);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

size_t topk_hist_bytes(int rows) { return (size_t)rows * kBins12 * 4; }

int32_t launch_topk(const Layout& L, const float* sel, const NRes& nr, int64_t nmax, int32_t k,
                    int32_t* idx, int32_t* count, void* ws, hipStream_t st, bool hist_clean, int64_t list_cap) {
  SelRows sr;
  for (int b = 0; b < kMaxBatch; ++b) { sr.nsel[b] = 0; sr.want[b] = -1; }
  for (int b = 0; b < L.batch; ++b) {
    sr.nsel[b] = nr.n[b];
    sr.want[b] = nr.n[b] < k ? nr.n[b] : k;
    if (sr.want[b] == 0) sr.want[b] = -1;
  }
  if (nmax <= kRowSelectMax)
    return launch_row_select(sel, L.cap, L.rows, L.n_kv_heads, sr, nmax, k, idx, count, RowSelectFused{}, st);
  TopkWs t;
  topk_carve(&t, ws, L.rows, list_cap > 0 ? list_cap : L.cap);
  int64_t chunk;
  int32_t nchunks;
  chunk_geometry(nmax, &chunk, &nchunks);
  dim3 g((unsigned)nchunks, (unsigned)L.rows);
  // Where the sampled form's lists fit the selection's registers and one workgroup per row can rank the samples.  Per call,
  // the five launches below / its three or four, 8 rows, us: normal scores, 50 000 slots and k = 1024 42 / 27, 300 000 and
  // 1024 37 / 30, 4096 48 / 31, 500 000 and 8192 54 / 38, 1 Mi and 4096 48 / 41, 8192 52 / 47; in runs of 64 500 000 52 -
  // 100 / 38, 1 Mi 53 - 104 / 44 - 47; all equal 674 - 1170 / 30 - 41; 99 % masked 44 - 920 / 30 - 44.  4 Mi slots in one
  // row, 32 768 samples by one workgroup, 53 / 57.
  if (select_sample_count(nmax, k) <= 16384 && select_lists_fit(nmax, k))
    return launch_topk_sampled(L, sel, nr, nmax, sr, k, idx, count, t, ListRoom{t.cand, nullptr, t.row_entries, 0, 0}, RowSelectFused{}, st);
  if (nmax > 0) {
    const int64_t nz = (int64_t)L.rows * kBins12;
    // the histogram sits at the start of the workspace; tk_findbin clears what it reads, so a caller
    // that zeroed it once and uses the workspace for nothing else (the step driver) skips this launch
    if (!hist_clean) tk_zero<<<(unsigned)((nz + 255) / 256), 256, 0, st>>>(t.hist, nz);
    // fewer, larger workgroups for the histogram: each flushes its bins with global atomics, and
    // atomics to one address serialise
    dim3 gh((unsigned)((nchunks + 3) / 4), (unsigned)L.rows);
    tk_hist<<<gh, 256, 0, st>>>(sel, L.cap, 4 * chunk, L.n_kv_heads, sr, t);
    tk_findbin<<<L.rows, 256, 0, st>>>(L.n_kv_heads, sr, t);
    tk_collect<<<g, 256, 0, st>>>(sel, L.cap, chunk, L.n_kv_heads, sr, t);
    tk_resolve<<<L.rows, 1024, 0, st>>>(chunk, nchunks, L.n_kv_heads, sr, t);
  }
  tk_emit_lists<<<g, 256, 0, st>>>(chunk, nchunks, L.n_kv_heads, sr, t, k, idx, count, false);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// What hca_topk itself touches of its workspace when the candidate lists are sized for rows of at most
// `list_cap` slots: everything of topk_carve up to and including the lists.
static size_t topk_only_bytes(int rows, int64_t list_cap) {
  size_t b = 0;
  b += align_up((int64_t)rows * kBins12 * 4, 256);
  b += align_up((int64_t)rows * kMaxChunks * 4, 256);
  b += align_up((int64_t)rows * 4 * 4, 256);
  b += align_up((int64_t)rows * 1024 * 4, 256);
  b += align_up((int64_t)rows * 1024 * 2 * 4, 256);
  b += align_up((int64_t)rows * list_entries_per_row(list_cap) * 8, 256);
  return b;
}

}  // namespace hca

// ---- hca_topk without a workspace argument --------------------------------------------------------------
// The scratch memory of the top-k kernels (histogram, per-chunk counts and offsets, candidate lists) as a
// file-scope device array instead of a caller's workspace, for callers that may not allocate.  Every device the
// library runs on holds its own copy of the array at its own address; in host code the array's name is only a
// handle for hipGetSymbolAddress, never a device address.
constexpr size_t kTopkScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kTopkScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];     // device address of `scratch` on each device, once known

// Address of the current device's copy of `scratch` (looked up on the first call on that device).
int32_t scratch_address(void** out) {
  int dev = 0;
  HCA_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return HCA_ERR_UNSUPPORTED;
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    HCA_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (p == nullptr) return hca::hip_fail(hipErrorInvalidSymbol);
    g_scratch_ptr[dev].store(p, std::memory_order_release);      // racing first calls store the same address
  }
  *out = p;
  return HCA_OK;
}
}  // namespace

extern "C" int32_t hca_topk_noalloc(const hca_shape* shape, const float* sel, const int64_t* n_resident, int32_t k,
                                    int32_t* idx, int32_t* count, void* stream) {
  using namespace hca;
  Layout L;
  int32_t rc = make_layout(shape, &L);
  if (rc != HCA_OK) return rc;
  if (sel == nullptr || idx == nullptr || count == nullptr) return HCA_ERR_BAD_ARG;
  if (k < 1 || k > L.cap) return HCA_ERR_CAPACITY;
  NRes nr;
  int64_t nmax;
  rc = load_nres(L, n_resident, &nr, &nmax);
  if (rc != HCA_OK) return rc;
  // the lists are sized for the longest resident row, not for the capacity: the limit is on what is scanned
  const int64_t list_cap = nmax > 0 ? nmax : 1;
  if (topk_only_bytes(L.rows, list_cap) > kTopkScratchBytes) return HCA_ERR_CAPACITY;
  void* ws = nullptr;
  rc = scratch_address(&ws);
  if (rc != HCA_OK) return rc;
  // the array keeps the previous call's contents: launch_topk clears the histogram with a fill kernel
  // (hist_clean = false) and every other region is written before it is read
  return launch_topk(L, sel, nr, nmax, k, idx, count, ws, (hipStream_t)stream, false, list_cap);
}
