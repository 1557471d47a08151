// Step 3b: gather of the selected value rows (pinned host memory and / or an HBM slice) and the
// softmax-weighted sum over the selected set (Eq. 5), plus the accumulated-score update.
#include "hca_internal.h"

namespace hca {

constexpr int kChunk = kAttendChunk;  // selected tokens per workgroup of the partial kernel
// Most entries of a one-stream attend that reads values across the host link itself: in all, and of them in host memory.
constexpr int64_t kDirectEntries = 16384, kDirectHostEntries = 4096;

struct AttendWs {
  uint16_t* vstage;  // [rows][k][128] fp16
  float* logit;      // [rows][4][k]
  float* pmz;        // [rows][nsplit][4][2]  (max, sum) per chunk
  float* py;         // [rows][nsplit][4][128]
};

static int nsplit_of(int64_t k) { return (int)((k + kChunk - 1) / kChunk); }

size_t attend_workspace_bytes(const Layout& L, int64_t k) {
  const int64_t ns = nsplit_of(k);
  size_t b = 0;
  b += align_up((int64_t)L.rows * k * kHeadDim * 2, 256);
  b += align_up((int64_t)L.rows * 4 * k * 4, 256);
  b += align_up((int64_t)L.rows * ns * 4 * 2 * 4, 256);
  b += align_up((int64_t)L.rows * ns * 4 * kHeadDim * 4, 256);
  return b;
}

static void carve(AttendWs* a, void* ws, const Layout& L, int64_t k) {
  const int64_t ns = nsplit_of(k);
  uint8_t* w = (uint8_t*)ws;
  a->vstage = (uint16_t*)w; w += align_up((int64_t)L.rows * k * kHeadDim * 2, 256);
  a->logit = (float*)w;     w += align_up((int64_t)L.rows * 4 * k * 4, 256);
  a->pmz = (float*)w;       w += align_up((int64_t)L.rows * ns * 4 * 2 * 4, 256);
  a->py = (float*)w;
}

// 16 threads move one 256-byte value row; rows below n_host_rows are read straight from
// pinned host memory over the host link (zero-copy), the others from the HBM slice.  For host rows the grid
// is deliberately small and persistent: the host link saturates with a few hundred KiB in
// flight, and more outstanding host reads than that only clog the memory pipeline for the
// HBM-bound kernels that run beside the gather.
// Rows in HBM want the opposite, every read in flight at once: 2048 rows for each of 32 (sequence, KV head) pairs,
// 16.8 MB, take 10.7 us in one sweep of 1024 workgroups and 59.5 us through the 64 of the host grid; 8192 rows x 8:
// 9.2 us against 58.3.
// SPLIT: both kinds in one launch, each with the grid it wants - workgroups below host_wgs take the host rows, the
// others the HBM rows; each skips the other kind's entries (4 bytes of position read twice per entry).  1024 rows x 8
// pairs, half of them in HBM: 24.5 us against 26.0 through the host grid alone (18.4 of it is the link).
template <int UNROLL, bool SPLIT>
__global__ __launch_bounds__(256) void gather_values(const int32_t* __restrict__ idx, const int32_t* __restrict__ count,
                                                     int32_t k, const int32_t* __restrict__ pos, int64_t cap,
                                                     const uint4* __restrict__ v_host, int64_t host_stride,
                                                     int64_t n_host_rows, const uint4* __restrict__ v_hbm,
                                                     int64_t hbm_stride, uint4* __restrict__ vstage,
                                                     int wgs, int host_wgs, uint64_t* __restrict__ stamps, int first,
                                                     uint32_t* __restrict__ gpu_seq, uint32_t seq) {
  const int row = blockIdx.y, wg = blockIdx.x;
  // hybrid value side: the kernel before this one on the stream left the host's inputs in pinned memory; a
  // kernel starts only when its predecessor's stores are visible, so the first thing this one does is tell the host
  if (gpu_seq != nullptr && row == 0 && wg == 0 && threadIdx.x == 0)
    __hip_atomic_store(gpu_seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  // optional profiling: every workgroup leaves its start and end time (constant-rate wall clock); beyond the buffer's pairs
  // it leaves its end alone, where that is later than what its pair holds
  const int64_t number = (int64_t)row * wgs + wg;
  uint64_t* stamp = stamps ? stamps + number % kGatherStampPairs * 2 : nullptr;
  if (stamp && threadIdx.x == 0 && number < kGatherStampPairs) stamp[0] = wall_clock64();
  const int cnt = count[row];
  const int part = threadIdx.x & 15;
  const bool host_role = wg < host_wgs;                    // SPLIT only
  const int first_wg = SPLIT && !host_role ? host_wgs : 0;
  // value rows per sweep of the row's workgroups (of this kind)
  const int64_t step = (int64_t)(SPLIT ? (host_role ? host_wgs : wgs - host_wgs) : wgs) * 16;
  // entries below `first` are not fetched (their values are summed where they live, on the host)
  for (int64_t i0 = (int64_t)first + (int64_t)(wg - first_wg) * 16 + (threadIdx.x >> 4); i0 < cnt; i0 += step * UNROLL) {
    uint4 v[UNROLL];
    bool mine[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int64_t i = i0 + u * step;
      mine[u] = i < cnt;
      if (mine[u]) {
        const int32_t slot = idx[(int64_t)row * k + i];
        const int64_t vr = pos[(int64_t)row * cap + slot];
        if (SPLIT && (vr < n_host_rows) != host_role) { mine[u] = false; continue; }
        const uint4* src = (vr < n_host_rows) ? v_host + ((int64_t)row * host_stride + vr) * 16
                                              : v_hbm + ((int64_t)row * hbm_stride + (vr - n_host_rows)) * 16;
        // read-once rows, write-once staging: non-temporal both ways, so that neither side displaces or
        // queues behind what the HBM-bound kernels beside the gather keep in the caches
        const v4i t4 = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(src + part));
        v[u] = uint4{(uint32_t)t4.x, (uint32_t)t4.y, (uint32_t)t4.z, (uint32_t)t4.w};
      }
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int64_t i = i0 + u * step;
      if (mine[u]) {
        const v4i t4 = {(int)v[u].x, (int)v[u].y, (int)v[u].z, (int)v[u].w};
        __builtin_nontemporal_store(t4, reinterpret_cast<v4i*>(vstage + ((int64_t)row * k + i) * 16 + part));
      }
    }
  }
  if (stamp) {
    __syncthreads();
    if (threadIdx.x == 0) atomicMax((unsigned long long*)&stamp[1], (unsigned long long)wall_clock64());
  }
}

// Shared memory of one chunk (256 selected tokens, up to 4 query heads) of the partial kernels.
struct PartialShared {
  float lg[4][kChunk];          // logits, then exp(logit - chunk max)
  float red[4][4][kHeadDim];
  float hm[4], hz[4];
};

// Writes the neutral partial of an empty chunk.
__device__ __forceinline__ void partial_empty(float* pmz, float* py) {
  if (threadIdx.x < 4) { pmz[2 * threadIdx.x] = -INFINITY; pmz[2 * threadIdx.x + 1] = 0.f; }
  for (int c = threadIdx.x; c < 4 * kHeadDim; c += 256) py[c] = 0.f;
}

// The first half of the value rows a lane will need: entry 64 w + 4 x + sub of the chunk, 16 bytes (part) of each, x < 8.
// They depend on nothing but the keep-list, so they are asked for before the logits are formed.  Past the chunk's end the
// last row is asked for again: it is in the cache (leaving those loads out costs a branch each, 9.6 -> 10.3 us for 65 rows
// x 8 from the host).
struct ValueRows { uint4 v[8]; };
// value.at(i): where entry i's row is, all of them looked up before the first is asked for; value(r): the load.
template <typename V>
__device__ __forceinline__ void value_rows(const V& value, int x0, int nvalid, ValueRows* out) {
  const int w = threadIdx.x >> 6, sub = (threadIdx.x & 63) >> 4;
  int32_t r[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    const int i = 64 * w + 4 * (x0 + x) + sub;
    r[x] = value.at(i < nvalid ? i : nvalid - 1);
  }
#pragma unroll
  for (int x = 0; x < 8; ++x) out->v[x] = value(r[x]);
}
struct StagedValues {                // the staging area: in the chunk's order
  const uint4* vs;
  __device__ __forceinline__ int32_t at(int i) const { return i; }
  __device__ __forceinline__ uint4 operator()(int32_t i) const { return vs[(int64_t)i * 16]; }
};

// What the last stage of a row with a single chunk needs: it writes the result itself and no merge follows.
struct RowEnd {
  float* y = nullptr;          // null: more than one chunk, the partial sums go to the workspace
  float* acc = nullptr;
  const float* lse = nullptr;
  const int32_t* idx = nullptr;
  int gqa = 0;
  int64_t cap = 0;
};

// Steps 2 and 3 of a chunk, after its logits sit in ps.lg (and a __syncthreads()): per-head chunk
// max / exponentials / sum, then the weighted sum of the value rows.  value: 16 bytes (this lane's part) of an entry's
// row; rows0: the first eight of them, already on their way.
template <bool VALUES, typename V>
__device__ __forceinline__ void partial_softmax_sum(PartialShared& ps, const AttendWs& a, int row, int i0, int nvalid,
                                                    int32_t k, float* pmz, float* py, const V& value, const ValueRows& rows0,
                                                    const RowEnd& end) {
  auto& lg = ps.lg;
  auto& red = ps.red;
  auto& hm = ps.hm;
  auto& hz = ps.hz;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  ValueRows rows1;
  if constexpr (VALUES) value_rows(value, 8, nvalid, &rows1);
  // 2. per head (wave w = head w): chunk max, exponentials, chunk sum
  {
    float l[4], m = -INFINITY;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      l[x] = lane + 64 * x < nvalid ? lg[w][lane + 64 * x] : -INFINITY;
      m = fmaxf(m, l[x]);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    float z = 0.f;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int i = lane + 64 * x;
      if (i < nvalid) {
        if (end.y == nullptr) a.logit[((int64_t)row * 4 + w) * k + i0 + i] = l[x];
        const float p = expf(l[x] - m);
        lg[w][i] = p;
        z += p;
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) z += __shfl_xor(z, o);
    if (lane == 0) {
      hm[w] = m;
      // (the only chunk of its row, weights not renormalised: the merge's normaliser)
      hz[w] = end.lse != nullptr && w < end.gqa ? expf(end.lse[(int64_t)row * end.gqa + w] - m) : z;
    }
  }
  __syncthreads();
  if constexpr (!VALUES) {   // weights only: the chunk's (max, sum) pairs and the stored logits are all that is needed
    if (threadIdx.x < 4) { pmz[2 * threadIdx.x] = hm[threadIdx.x]; pmz[2 * threadIdx.x + 1] = hz[threadIdx.x]; }
    return;
  }

  // 3. weighted value sum.  Wave w owns tokens [64w, 64w+64) of the chunk; one load instruction
  //    fetches 4 rows (lane>>4 picks the row, lane&15 its 16-byte part).
  float acc[4][8];
#pragma unroll
  for (int h = 0; h < 4; ++h)
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[h][c] = 0.f;
  const int part = lane & 15, sub = lane >> 4;
  auto add = [&](const ValueRows& rows, int x0) {
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int i = 64 * w + 4 * (x0 + x) + sub;
      if (i < nvalid) {
        const uint32_t wd[4] = {rows.v[x].x, rows.v[x].y, rows.v[x].z, rows.v[x].w};
        float v[8];
#pragma unroll
        for (int c = 0; c < 4; ++c) { v[2 * c] = h2f(wd[c] & 0xffffu); v[2 * c + 1] = h2f(wd[c] >> 16); }
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const float p = lg[h][i];
#pragma unroll
          for (int c = 0; c < 8; ++c) acc[h][c] = fmaf(p, v[c], acc[h][c]);
        }
      }
    }
  };
  add(rows0, 0);
  add(rows1, 8);
#pragma unroll
  for (int h = 0; h < 4; ++h)
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float x = acc[h][c];
      x += __shfl_xor(x, 16);
      x += __shfl_xor(x, 32);
      acc[h][c] = x;
    }
  if (sub == 0) {
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int c = 0; c < 8; ++c) red[w][h][8 * part + c] = acc[h][c];
  }
  __syncthreads();
  for (int c = threadIdx.x; c < 4 * kHeadDim; c += 256) {
    const int h = c >> 7, d = c & 127;
    const float sum = (red[0][h][d] + red[1][h][d]) + (red[2][h][d] + red[3][h][d]);
    if (end.y == nullptr) py[c] = sum;
    else if (h < end.gqa) end.y[((int64_t)row * end.gqa + h) * kHeadDim + d] = sum / hz[h];
  }
  if (end.y == nullptr) {
    if (threadIdx.x < 4) { pmz[2 * threadIdx.x] = hm[threadIdx.x]; pmz[2 * threadIdx.x + 1] = hz[threadIdx.x]; }
  } else if (end.acc != nullptr && (int)threadIdx.x < nvalid) {
    float wsum = 0.f;
    for (int h = 0; h < end.gqa; ++h) wsum += fmaxf(lg[h][threadIdx.x] / hz[h], 1e-30f);
    end.acc[(int64_t)row * end.cap + end.idx[(int64_t)row * k + threadIdx.x]] += wsum;
  }
}

// Where the value rows of a launch come from: the staging area that a gather filled, or the stores themselves.
struct ValueSource {
  const int32_t* pos = nullptr;      // null: staged
  const uint4* v_host = nullptr;
  const uint4* v_hbm = nullptr;
  int64_t host_stride = 0, hbm_stride = 0, n_host_rows = 0;
};

struct DirectValues {
  const ValueSource& src;
  const int32_t* vrow;               // of the chunk's entries, in LDS
  int row, part;
  __device__ __forceinline__ int32_t at(int i) const { return vrow[i]; }
  __device__ __forceinline__ uint4 operator()(int32_t vr) const {
    return (vr < src.n_host_rows ? src.v_host + ((int64_t)row * src.host_stride + vr) * 16
                                 : src.v_hbm + ((int64_t)row * src.hbm_stride + (vr - src.n_host_rows)) * 16)[part];
  }
};

// Bound by latency: one workgroup per 256 selected tokens, a chain of dependent loads (slots, codes; positions, values) and
// a few microseconds of arithmetic.  So everything that can be asked for early is: slots, query and
// count together, the value rows' numbers before the codes (loads come back in order: behind them the values waited, 16.4 us
// in the kernel for 14.3 at 2048 x 32), the value rows before the logits.  DIRECT: the value rows are read where they live, no
// gather and no staging area.  A row's only chunk (k <= 256) finishes the row.  One head, 256 tokens: 9 us where gather, attend
// and merge took 20; 2048 tokens x 32 pairs in HBM: 22 us for attend and merge where gather, attend and merge took 34.
template <int BITS, bool VALUES = true, bool DIRECT = false>
__device__ __forceinline__ bool attend_partial_body(PartialShared& ps, QShared& sh, const Layout& L,
                                                    const uint8_t* __restrict__ kcache, const uint16_t* __restrict__ q,
                                                    const int32_t* __restrict__ idx, const int32_t* __restrict__ count,
                                                    int32_t k, float sm_scale, const AttendWs& a, int nsplit,
                                                    const int split, const ValueSource& vsrc = ValueSource{},
                                                    const RowEnd& end = RowEnd{}) {
  __shared__ int32_t s_slot[kChunk];
  __shared__ int32_t s_vrow[DIRECT ? kChunk : 1];
  __shared__ __align__(16) uint32_t opimg[64 * 8];
  auto& lg = ps.lg;
  const int row = blockIdx.y;
  const int i0 = split * kChunk;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int t = lane & 15, j = lane >> 4;
  // slot, query and count are asked for together.  (Past the list's end the slot is whatever memory held: not looked up)
  int32_t my_slot = idx[(int64_t)row * k + (i0 + tid < k ? i0 + tid : k - 1)];
  uint32_t pair = query_pair(q, row, L.gqa);
  const int cnt = count[row];
  s_slot[tid] = my_slot;
  float* pmz = a.pmz + (((int64_t)row * nsplit + split) * 4) * 2;
  float* py = a.py + (((int64_t)row * nsplit + split) * 4) * kHeadDim;
  if (i0 >= cnt) {  // empty chunk: neutral partial
    if (end.y == nullptr) partial_empty(pmz, py);
    else for (int c = tid; c < L.gqa * kHeadDim; c += 256) end.y[(int64_t)row * L.gqa * kHeadDim + c] = 0.f;
    return false;
  }
  const int nvalid = (cnt - i0 < kChunk) ? cnt - i0 : kChunk;
  // the value rows' numbers before the codes: the values, which wait for them, are then on their way with the codes
  int32_t my_vrow = 0;
  if constexpr (DIRECT) my_vrow = vsrc.pos[(int64_t)row * L.cap + (tid < nvalid ? my_slot : 0)];
  const auto value = [&] {
    if constexpr (DIRECT) return DirectValues{vsrc, s_vrow, row, lane & 15};
    else return StagedValues{reinterpret_cast<const uint4*>(a.vstage) + ((int64_t)row * k + i0) * 16 + (lane & 15)};
  }();
  ValueRows rows0;
  if constexpr (VALUES && !DIRECT) value_rows(value, 0, nvalid, &rows0);
  asm volatile("" : "+v"(pair));                            // (the query is not waited for before)
  load_query(pair, L.gqa, L.group, &sh);                           // (ends with a barrier)
  const uint8_t* crow = kcache + (int64_t)row * L.codes_row_bytes();
  const uint8_t* mrow = kcache + L.meta_off + (int64_t)row * L.meta_row_bytes();

  // 1. logits of the chunk: wave w scores tiles w, w+4, w+8, w+12 (16 selected tokens each).
  //    All code / meta pieces are asked for first, so that the wave has its
  //    whole share of the random reads in flight at once.
  {
    uint4 wv[4], mv[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int at = (w + 4 * x) * 16 + t;
      const int64_t slot = s_slot[at < nvalid ? at : nvalid - 1];
      if constexpr (BITS == 4) {
        const int64_t blk = slot >> 4;
        const int tl = (int)(slot & 15);
        wv[x] = *reinterpret_cast<const uint4*>(crow + blk * kBlockBytes + (tl + 16 * j) * 16);
        mv[x] = *reinterpret_cast<const uint4*>(mrow + blk * kMetaBytes + tl * 16);
      } else {
        const int64_t blk = slot >> 5;
        const int u = (int)((slot >> 4) & 1), tl = (int)(slot & 15);
        const uint2 c = *reinterpret_cast<const uint2*>(crow + blk * kBlockBytes + (tl + 16 * j) * 16 + 8 * u);
        const uint2 m = *reinterpret_cast<const uint2*>(mrow + blk * kMetaBytes + (16 * u + tl) * 8);
        wv[x] = uint4{c.x, c.y, 0, 0};
        mv[x] = uint4{m.x, m.y, 0, 0};
      }
    }
    QOperand<BITS> op;
    build_operand_shared<BITS>(&sh, opimg, &op);
    if constexpr (DIRECT) {
      s_vrow[tid] = my_vrow;
      __syncthreads();
      if constexpr (VALUES) value_rows(value, 0, nvalid, &rows0);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      float zv;
      if constexpr (BITS == 4) zv = score_block4(op, wv[x], mv[x]);
      else zv = score_tile2(op, wv[x].x, wv[x].y, uint2{mv[x].x, mv[x].y});
      // lane (t, hd = j) holds z~ of head j for selected token (w + 4x)*16 + t
      lg[j][(w + 4 * x) * 16 + t] = zv * sm_scale;
    }
  }
  __syncthreads();

  partial_softmax_sum<VALUES>(ps, a, row, i0, nvalid, k, pmz, py, value, rows0, end);
  return true;
}

// split0: the first chunk of the launch (chunks below it belong to the host share)
template <int BITS, bool VALUES = true, bool DIRECT = false>
__global__ __launch_bounds__(256) void attend_partial(Layout L, const uint8_t* __restrict__ kcache,
                                                      const uint16_t* __restrict__ q, const int32_t* __restrict__ idx,
                                                      const int32_t* __restrict__ count, int32_t k, float sm_scale,
                                                      AttendWs a, int nsplit, int split0, ValueSource vsrc, RowEnd end) {
  __shared__ QShared sh;
  __shared__ PartialShared ps;
  attend_partial_body<BITS, VALUES, DIRECT>(ps, sh, L, kcache, q, idx, count, k, sm_scale, a, nsplit,
                                            (int)blockIdx.x + split0, vsrc, end);
}

// The chunks of the host share: logits, chunk (max, sum) and stored logits as for any chunk (the merge and the
// accumulated scores need them), no value rows; instead every entry's exp(logit - chunk max) per head and its
// value-row number go to pinned host memory.  An entry whose value row is not in the host store (rows >=
// n_host_rows live in the HBM slice: the newest tokens) is summed here, into the chunk's device-side partial,
// and is handed to the host as "nothing to add".
template <int BITS>
__global__ __launch_bounds__(256) void attend_host_chunks(Layout L, const uint8_t* __restrict__ kcache,
                                                          const uint16_t* __restrict__ q, const int32_t* __restrict__ idx,
                                                          const int32_t* __restrict__ count, int32_t k,
                                                          const int32_t* __restrict__ pos, int64_t n_host_rows,
                                                          const uint16_t* __restrict__ v_hbm, int64_t hbm_stride,
                                                          float sm_scale, AttendWs a, int nsplit, HostShare hs) {
  __shared__ QShared sh;
  __shared__ PartialShared ps;
  __shared__ int32_t vr[kChunk];
  __shared__ int n_dev;
  const int row = blockIdx.y, split = blockIdx.x;
  const int tid = threadIdx.x;
  float* out_p = hs.p + ((int64_t)row * hs.chunks + split) * 4 * kChunk;
  int32_t* out_v = hs.vrow + ((int64_t)row * hs.chunks + split) * kChunk;
  float* py = a.py + (((int64_t)row * nsplit + split) * 4) * kHeadDim;
  if (tid == 0) n_dev = 0;
  const bool live_chunk = attend_partial_body<BITS, false>(ps, sh, L, kcache, q, idx, count, k, sm_scale, a, nsplit, split);
  if (!live_chunk) {                  // nothing selected here: partial_empty has written the neutral partial
    out_v[tid] = -1;
#pragma unroll
    for (int h = 0; h < 4; ++h) out_p[h * kChunk + tid] = 0.f;
    return;
  }
  // ps.lg now holds exp(logit - chunk max) of the chunk's live entries
  const int cnt = count[row];
  const int i0 = split * kChunk;
  const int nvalid = (cnt - i0 < kChunk) ? cnt - i0 : kChunk;
  int32_t r = -1;
  bool on_dev = false;
  if (tid < nvalid) {
    const int32_t slot = idx[(int64_t)row * k + i0 + tid];
    const int32_t v = pos[(int64_t)row * L.cap + slot];
    on_dev = v >= n_host_rows;
    r = on_dev ? -1 : v;
    vr[tid] = on_dev ? (int32_t)(v - n_host_rows) : -1;
    if (on_dev) atomicAdd(&n_dev, 1);
  } else {
    vr[tid] = -1;
  }
  out_v[tid] = r;
#pragma unroll
  for (int h = 0; h < 4; ++h) out_p[h * kChunk + tid] = (tid < nvalid && h < L.gqa) ? ps.lg[h][tid] : 0.f;
  __syncthreads();
  // device-side partial of the chunk: the entries that the host cannot reach (usually none)
  for (int c = tid; c < 4 * kHeadDim; c += 256) {
    const int h = c >> 7, d = c & 127;
    float s = 0.f;
    if (n_dev > 0 && h < L.gqa) {
      for (int i = 0; i < nvalid; ++i) {
        const int32_t x = vr[i];
        if (x >= 0) s = fmaf(ps.lg[h][i], h2f(v_hbm[((int64_t)row * hbm_stride + x) * kHeadDim + d]), s);
      }
    }
    py[c] = s;
  }
}

// Table entry of one (group, centroid): the G query heads of the KV head, adjacent in memory.
template <int G>
__device__ __forceinline__ void load_entry(const float* p, float (&e)[G]) {
  if constexpr (G == 4) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    e[0] = v.x; e[1] = v.y; e[2] = v.z; e[3] = v.w;
  } else if constexpr (G == 2) {
    const float2 v = *reinterpret_cast<const float2*>(p);
    e[0] = v.x; e[1] = v.y;
  } else {
    e[0] = p[0];
  }
}

// Codebook form: the logit of a selected token is the sum over the groups of the table entries
// its indices select (Eq. 3), added exactly on the table's power-of-two grid (the exponents that the
// scan left behind the table in `lut`).  Thread i of the chunk owns selected token i0 + i.
// EARLY: the first value rows are asked for before the table reads: what a workgroup wants that has a compute unit for
// itself (200 x 128 13.2 -> 9.7 us for attend alone).  It costs registers - three waves per SIMD instead of four in the narrow form -
// and loads come back in order, so that table reads wait for the values: launches of more workgroups than compute units ask
// for them behind the logits in the narrow form (2048 x 64, 64 centroids: 22.7 us, 23.5 with EARLY; wide, 4096 x 128, 1024: 149 and 143).
template <int G, bool WIDE, bool EARLY>
__global__ __launch_bounds__(256) void vq_attend_partial(int g, int c, int64_t cap, const uint8_t* __restrict__ pcache,
                                                         const float* __restrict__ lut, const int32_t* __restrict__ idx,
                                                         const int32_t* __restrict__ count, int32_t k, float sm_scale,
                                                         AttendWs a, int nsplit, RowEnd end) {
  __shared__ PartialShared ps;
  __shared__ int32_t s_slot[kChunk];
  const int row = blockIdx.y, split = blockIdx.x;
  const int i0 = split * kChunk;
  s_slot[threadIdx.x] = idx[(int64_t)row * k + (i0 + (int)threadIdx.x < k ? i0 + (int)threadIdx.x : k - 1)];    // with the count
  const int cnt = count[row];
  float* pmz = a.pmz + (((int64_t)row * nsplit + split) * 4) * 2;
  float* py = a.py + (((int64_t)row * nsplit + split) * 4) * kHeadDim;
  if (i0 >= cnt) {
    if (end.y == nullptr) partial_empty(pmz, py);
    else for (int c = threadIdx.x; c < G * kHeadDim; c += 256) end.y[(int64_t)row * G * kHeadDim + c] = 0.f;
    return;
  }
  const int nvalid = (cnt - i0 < kChunk) ? cnt - i0 : kChunk;
  const StagedValues value{reinterpret_cast<const uint4*>(a.vstage) + ((int64_t)row * k + i0) * 16 + (threadIdx.x & 15)};
  ValueRows rows0;
  __syncthreads();
  if constexpr (EARLY) value_rows(value, 0, nvalid, &rows0);
  {
    const int i = threadIdx.x;
    const int64_t slot = s_slot[i < nvalid ? i : nvalid - 1];
    const uint8_t* pr = pcache + ((int64_t)row * cap + slot) * g;                  // narrow form: the slot's record
    const uint16_t* pw = reinterpret_cast<const uint16_t*>(pcache);
    const int64_t tiles = vq_tiles(cap);
    const float* T = lut + (int64_t)row * g * c * G;
    const int32_t* sexp = reinterpret_cast<const int32_t*>(lut + (int64_t)gridDim.y * g * (c * G + 4)) + row * 4;
    int s[G], zi[G];
#pragma unroll
    for (int h = 0; h < G; ++h) { s[h] = sexp[h]; zi[h] = 0; }
    for (int i16 = 0; i16 < g; i16 += 16) {
      int64_t ent[16];                          // entry number in the table of this row
      if constexpr (WIDE) {                     // 16-bit indices, group-major tiles; table [group][centroid]
#pragma unroll
        for (int b = 0; b < 16; ++b) {
          const int code = (int)pw[vq_wide_at(g, tiles, row, slot, i16 + b)];
          ent[b] = (int64_t)(i16 + b) * c + code;
        }
      } else {                                  // byte indices, rotated by the slot number; table [centroid][group]
        const uint4 pv = *reinterpret_cast<const uint4*>(pr + i16);
        const uint32_t wd[4] = {pv.x, pv.y, pv.z, pv.w};
#pragma unroll
        for (int b = 0; b < 16; ++b)
          ent[b] = (int64_t)((wd[b >> 2] >> (8 * (b & 3))) & 255u) * g + vq_group_at(i16 + b, slot);
      }
      float e[16][G];
#pragma unroll
      for (int b = 0; b < 16; ++b)              // 16 independent table reads in flight
        load_entry<G>(T + ent[b] * G, e[b]);
#pragma unroll
      for (int b = 0; b < 16; ++b)
#pragma unroll
        for (int h = 0; h < G; ++h) zi[h] += vq_fix(e[b][h], s[h]);
    }
    float z[G];
#pragma unroll
    for (int h = 0; h < G; ++h) z[h] = ldexpf((float)zi[h], -s[h]);
#pragma unroll
    for (int h = 0; h < 4; ++h) ps.lg[h][i] = h < G ? z[h < G ? h : 0] * sm_scale : 0.f;
  }
  if constexpr (!EARLY) value_rows(value, 0, nvalid, &rows0);
  __syncthreads();
  partial_softmax_sum<true>(ps, a, row, i0, nvalid, k, pmz, py, value, rows0, end);
}

// The row's maximum (fm) and normaliser (fz) per head from its chunks' (max, sum) pairs, and every chunk's factor
// exp(chunk max - row max); one thread per (chunk, head), 256 of them, nsplit <= 64.  The sum runs over the chunks in
// ascending order of a tree, 16 chunks per wave.  With lse the normaliser is exp(lse - row max).  Ends with a barrier.
__device__ __forceinline__ void merge_chunks(const float* __restrict__ pmz, int nsplit, const float* __restrict__ lse, int gqa,
                                             float (&fm)[4], float (&fz)[4], float (&wgt)[4][64]) {
  __shared__ float wm[4][4], wz[4][4];
  const int h = threadIdx.x & 3, sp = threadIdx.x >> 2, w = threadIdx.x >> 6;
  if (nsplit <= 16) {          // up to 4096 selected: the first wave's share, nothing to exchange (0.5 us less)
    if (w == 0) {
      float2 v{-INFINITY, 0.f};
      if (sp < nsplit) v = reinterpret_cast<const float2*>(pmz)[threadIdx.x];
      float m = v.x;
#pragma unroll
      for (int o = 4; o <= 32; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
      const float e = v.x == -INFINITY ? 0.f : expf(v.x - m);
      wgt[h][sp] = e;
      float z = e * v.y;
#pragma unroll
      for (int o = 4; o <= 32; o <<= 1) z += __shfl_xor(z, o);
      if (lse != nullptr && h < gqa) z = expf(lse[h] - m);
      if (threadIdx.x < 4) { fm[h] = m; fz[h] = z; }
    }
    __syncthreads();
    return;
  }
  float2 v{-INFINITY, 0.f};
  if (sp < nsplit) v = reinterpret_cast<const float2*>(pmz)[threadIdx.x];   // index = split*4 + head
  float m = v.x;
#pragma unroll
  for (int o = 4; o <= 32; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) < 4) wm[w][h] = m;
  __syncthreads();
  m = fmaxf(fmaxf(wm[0][h], wm[1][h]), fmaxf(wm[2][h], wm[3][h]));
  const float e = v.x == -INFINITY ? 0.f : expf(v.x - m);
  wgt[h][sp] = e;
  float z = e * v.y;
#pragma unroll
  for (int o = 4; o <= 32; o <<= 1) z += __shfl_xor(z, o);
  if ((threadIdx.x & 63) < 4) wz[w][h] = z;
  __syncthreads();
  if (threadIdx.x < 4) {
    z = (wz[0][h] + wz[1][h]) + (wz[2][h] + wz[3][h]);
    // global normalisation: sum_i exp(l_i - m) v_i / exp(lse - m)
    if (lse != nullptr && h < gqa) z = expf(lse[h] - m);
    fm[h] = m;
    fz[h] = z;
  }
  __syncthreads();
}

// Workgroup 0 of a row merges the chunk partials into y; workgroups 1.. add the final softmax
// weights of their 256 selected tokens to the accumulated scores.
// With `lse` (log of the softmax denominator over ALL resident tokens, per query head) the weights are the
// paper's own, exp(l_i - lse), not renormalised over the selected set (Sec. 3.2, Eq. 5).
__global__ __launch_bounds__(256) void attend_merge(Layout L, const int32_t* __restrict__ idx,
                                                    const int32_t* __restrict__ count, int32_t k, AttendWs a,
                                                    int nsplit, float* __restrict__ y, float* __restrict__ acc,
                                                    const float* __restrict__ lse, HostShare hs) {
  __shared__ float fm[4], fz[4];
  __shared__ float wgt[4][64];  // nsplit <= 64
  const int row = blockIdx.y;
  const int cnt = count[row];
  const float* pmz = a.pmz + ((int64_t)row * nsplit * 4) * 2;
  merge_chunks(pmz, nsplit, lse != nullptr ? lse + (int64_t)row * L.gqa : nullptr, L.gqa, fm, fz, wgt);
  if (blockIdx.x == 0) {
    if (hs.chunks > 0) {
      // the host's partial sums of this row: wait, a bounded number of polls, until the host has stored this
      // step's sequence number (it never stores an older one afterwards)
      if (threadIdx.x == 0) {
        int polls = 0;
        while ((int32_t)(__hip_atomic_load(hs.host_seq + row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) - hs.seq) < 0) {
          if (++polls >= hs.spin_limit) {
            __hip_atomic_store(hs.err, hs.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            break;
          }
          __builtin_amdgcn_s_sleep(20);
        }
      }
      __syncthreads();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");       // nothing read below may come from before the flag
    }
    for (int c = threadIdx.x; c < L.gqa * kHeadDim; c += 256) {
      const int h = c >> 7, d = c & 127;
      float s = 0.f;
      // chunks of the host share: device-side partial (entries the host cannot reach) + the host's partial.  A load over
      // the host link takes 1.5 us: all of a batch are asked for before the first is used (one after another, 14 chunks
      // made a merge of four layers of 1 Mi tokens 42 - 75 us; now 25 - 31, the four layers 719 -> 672 us)
      const int nh = hs.chunks < nsplit ? hs.chunks : nsplit;
      for (int s0 = 0; s0 < nh; s0 += 16) {
        float hv[16], dv[16];
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          const int sp = s0 + x < nh ? s0 + x : nh - 1;
          hv[x] = __builtin_nontemporal_load(&hs.py[(((int64_t)row * hs.chunks + sp) * 4 + h) * kHeadDim + d]);
          dv[x] = a.py[((int64_t)row * nsplit * 4 + sp * 4 + h) * kHeadDim + d];
        }
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          const float e = s0 + x < nh ? wgt[h][s0 + x] : 0.f;
          if (e != 0.f) s = fmaf(e, dv[x] + hv[x], s);
        }
      }
      const float* src = a.py + ((int64_t)row * nsplit * 4 + h) * kHeadDim + d;
      for (int s0 = hs.chunks; s0 < nsplit; s0 += 16) {      // 16 independent loads per batch
        float v[16];
#pragma unroll
        for (int x = 0; x < 16; ++x) v[x] = (s0 + x < nsplit) ? src[(int64_t)(s0 + x) * 4 * kHeadDim] : 0.f;
#pragma unroll
        for (int x = 0; x < 16; ++x)
          if (s0 + x < nsplit) s = fmaf(wgt[h][s0 + x], v[x], s);
      }
      y[((int64_t)row * L.gqa + h) * kHeadDim + d] = cnt > 0 ? s / fz[h] : 0.f;
    }
  } else if (acc != nullptr) {
    const int i = (blockIdx.x - 1) * 256 + threadIdx.x;
    if (i < cnt) {
      float wsum = 0.f;
      for (int h = 0; h < L.gqa; ++h) {
        const float p = expf(a.logit[((int64_t)row * 4 + h) * k + i] - fm[h]) / fz[h];
        wsum += fmaxf(p, 1e-30f);
      }
      acc[(int64_t)row * L.cap + idx[(int64_t)row * k + i]] += wsum;
    }
  }
}

// Small per-thread ring of events for the stream fork / join around the gather.
static hipEvent_t next_event(hipError_t* err) {
  thread_local hipEvent_t ring[32];
  thread_local bool made[32] = {false};
  thread_local int cur = 0;
  const int i = cur;
  cur = (cur + 1) & 31;
  *err = hipSuccess;
  if (!made[i]) {
    *err = hipEventCreateWithFlags(&ring[i], hipEventDisableTiming);
    if (*err != hipSuccess) return nullptr;
    made[i] = true;
  }
  return ring[i];
}

int32_t launch_gather(const Layout& L, const int32_t* idx, const int32_t* count, int32_t k, const int32_t* pos,
                      const void* v_host, int64_t host_stride, int64_t n_host_rows, const void* v_hbm,
                      int64_t hbm_stride, void* ws, hipStream_t st, uint64_t* stamps, int first_entry,
                      const Tuning* tune, const HostShare* hs) {
  AttendWs a;
  carve(&a, ws, L, k);
  uint32_t* gpu_seq = hs != nullptr ? hs->gpu_seq : nullptr;
  const uint32_t seq = hs != nullptr ? hs->seq : 0u;
  const Tuning& tn = tune != nullptr ? *tune : tuning();
  const int64_t entries = (int64_t)k - first_entry;
  int64_t wgs = ((int64_t)k + 15) / 16;                  // one workgroup per 16 rows at most
  // per (sequence, KV head).  About 64 workgroups in total keep enough reads in flight to fill the host
  // link; more only take queue entries in the memory system away from the HBM-bound kernels beside it.
  int64_t lim = tn.gather_wgs > 0 ? tn.gather_wgs : (L.rows >= 64 ? 1 : 64 / L.rows);
  if (wgs > lim) wgs = lim;
  // Rows in HBM: one sweep, a row per thread while that is at most 1024 workgroups (64 rows: 2.6 us, 3.4 with four per
  // thread), else every thread's four rows in flight together.  Where the store is shared between host
  // and HBM the launch has both kinds of workgroups, unless the HBM slice is only the few rows of the appended
  // tokens (less than a sixteenth of the host rows) or the launch is small: then the host kind takes them along (half of
  // the values in HBM, both kinds / one: 64 x 128 25.3 / 24.3 us, 512 x 8 13.9 / 13.6; 256 x 32 24.7 / 25.8, 512 x 32 44 / 47,
  // 2048 x 8 44 / 45; three quarters in HBM: 100 x 32 8.0 / 8.7, 1024 x 8 15.5 / 16.2, 256 x 49 21.6 / 27.1).
  const int64_t wide = entries > 0 ? (entries + 63) / 64 : 1, rows16 = entries > 0 ? (entries + 15) / 16 : 1;
  const bool no_host = v_host == nullptr || n_host_rows == 0;
  const bool split = !no_host && v_hbm != nullptr && hbm_stride > n_host_rows / 16 && entries > 64 &&
                     entries * L.rows >= (L.rows >= 16 ? 3072 : 8192) && tn.gather_wgs == 0;
  const int64_t host_wgs = wgs;
  if (no_host && tn.gather_wgs == 0) wgs = rows16 * L.rows <= 1024 ? rows16 : wide;
  else if (split) wgs += wide;
  dim3 g((unsigned)wgs, (unsigned)L.rows);
  const uint4 *vh = (const uint4*)v_host, *vd = (const uint4*)v_hbm;
#define HCA_GATHER_S(U, S)                                                                                            \
  gather_values<U, S><<<g, 256, 0, st>>>(idx, count, k, pos, L.cap, vh, host_stride, n_host_rows, vd, hbm_stride, \
                                         (uint4*)a.vstage, (int)wgs, (int)host_wgs, stamps, first_entry, gpu_seq, seq)
#define HCA_GATHER(U) do { if (split) HCA_GATHER_S(U, true); else HCA_GATHER_S(U, false); } while (0)
  if (tn.gather_unroll >= 4) HCA_GATHER(4);
  else if (tn.gather_unroll >= 2) HCA_GATHER(2);
  else HCA_GATHER(1);
#undef HCA_GATHER
#undef HCA_GATHER_S
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

static int32_t attend_launches(const Layout& L, const void* kcache, const void* q, const int32_t* idx,
                               const int32_t* count, int32_t k, float sm_scale, float* y, float* acc_opt,
                               void* ws, hipStream_t st, const float* lse, const HostShare* hs, const ValueSource& vsrc) {
  AttendWs a;
  carve(&a, ws, L, k);
  const int ns = nsplit_of(k);
  if (ns > 64) return HCA_ERR_CAPACITY;
  HostShare h0;
  if (hs != nullptr) h0 = *hs;
  if (h0.chunks > ns) h0.chunks = ns;
  // one chunk per row: no merge, the chunk's workgroup writes the row's results (a launch of 4 us less)
  RowEnd end;
  if (ns == 1 && h0.chunks == 0) end = RowEnd{y, acc_opt, lse, idx, L.gqa, L.cap};
  if (ns - h0.chunks > 0) {            // the chunks whose value rows are not the host's to sum
    dim3 gp((unsigned)(ns - h0.chunks), (unsigned)L.rows);
#define HCA_PARTIAL(B, D) attend_partial<B, true, D><<<gp, 256, 0, st>>>(L, (const uint8_t*)kcache, (const uint16_t*)q, idx, count, k, sm_scale, a, ns, h0.chunks, vsrc, end)
    if (vsrc.pos != nullptr) {
      if (L.bits == 4) HCA_PARTIAL(4, true);
      else HCA_PARTIAL(2, true);
    } else {
      if (L.bits == 4) HCA_PARTIAL(4, false);
      else HCA_PARTIAL(2, false);
    }
#undef HCA_PARTIAL
  }
  if (end.y == nullptr) {
    dim3 gm((unsigned)(1 + (acc_opt ? ns : 0)), (unsigned)L.rows);
    attend_merge<<<gm, 256, 0, st>>>(L, idx, count, k, a, ns, y, acc_opt, lse, h0);
  }
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

int32_t launch_attend_gathered(const Layout& L, const void* kcache, const void* q, const int32_t* idx,
                               const int32_t* count, int32_t k, float sm_scale, float* y, float* acc_opt,
                               void* ws, hipStream_t st, const float* lse, const HostShare* hs) {
  return attend_launches(L, kcache, q, idx, count, k, sm_scale, y, acc_opt, ws, st, lse, hs, ValueSource{});
}

int host_share_chunks(int32_t k, int want) {
  const int ns = nsplit_of(k);
  return want < 0 ? 0 : (want > ns ? ns : want);
}
size_t host_share_p_bytes(const Layout& L, int chunks) { return (size_t)L.rows * chunks * 4 * kChunk * sizeof(float); }
size_t host_share_vrow_bytes(const Layout& L, int chunks) { return (size_t)L.rows * chunks * kChunk * sizeof(int32_t); }
size_t host_share_py_bytes(const Layout& L, int chunks) { return (size_t)L.rows * chunks * 4 * kHeadDim * sizeof(float); }

int32_t launch_attend_host_chunks(const Layout& L, const void* kcache, const void* q, const int32_t* idx,
                                  const int32_t* count, int32_t k, const int32_t* pos, int64_t n_host_rows,
                                  const void* v_hbm, int64_t hbm_stride, float sm_scale, void* ws, const HostShare& hs,
                                  hipStream_t st) {
  AttendWs a;
  carve(&a, ws, L, k);
  const int ns = nsplit_of(k);
  if (ns > 64 || hs.chunks < 1 || hs.chunks > ns) return HCA_ERR_CAPACITY;
  dim3 gp((unsigned)hs.chunks, (unsigned)L.rows);
  if (L.bits == 4)
    attend_host_chunks<4><<<gp, 256, 0, st>>>(L, (const uint8_t*)kcache, (const uint16_t*)q, idx, count, k, pos,
                                              n_host_rows, (const uint16_t*)v_hbm, hbm_stride, sm_scale, a, ns, hs);
  else
    attend_host_chunks<2><<<gp, 256, 0, st>>>(L, (const uint8_t*)kcache, (const uint16_t*)q, idx, count, k, pos,
                                              n_host_rows, (const uint16_t*)v_hbm, hbm_stride, sm_scale, a, ns, hs);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

int32_t launch_vq_attend_gathered(const Layout& L, int g, int c, const uint8_t* pcache, const float* lut,
                                  const int32_t* idx, const int32_t* count, int32_t k, float sm_scale, float* y,
                                  float* acc_opt, void* ws, hipStream_t st) {
  AttendWs a;
  carve(&a, ws, L, k);
  const int ns = nsplit_of(k);
  if (ns > 64) return HCA_ERR_CAPACITY;
  dim3 gp((unsigned)ns, (unsigned)L.rows);
  RowEnd end;
  if (ns == 1) end = RowEnd{y, acc_opt, nullptr, idx, L.gqa, L.cap};
  const bool early = (int64_t)ns * L.rows <= 256 || vq_is_wide(L, g, c);
#define HCA_VQ_P(GQ, W, E) vq_attend_partial<GQ, W, E><<<gp, 256, 0, st>>>(g, c, L.cap, pcache, lut, idx, count, k, sm_scale, a, ns, end)
#define HCA_VQ_PARTIAL(GQ)                                                                                               \
  do {                                                                                                                   \
    if (vq_is_wide(L, g, c)) { if (early) HCA_VQ_P(GQ, true, true); else HCA_VQ_P(GQ, true, false); }                    \
    else { if (early) HCA_VQ_P(GQ, false, true); else HCA_VQ_P(GQ, false, false); }                                      \
  } while (0)
  if (L.gqa == 4) HCA_VQ_PARTIAL(4);
  else if (L.gqa == 2) HCA_VQ_PARTIAL(2);
  else HCA_VQ_PARTIAL(1);
#undef HCA_VQ_PARTIAL
#undef HCA_VQ_P
  if (end.y == nullptr) {
    dim3 gm((unsigned)(1 + (acc_opt ? ns : 0)), (unsigned)L.rows);
    attend_merge<<<gm, 256, 0, st>>>(L, idx, count, k, a, ns, y, acc_opt, nullptr, HostShare{});
  }
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// The paper's split (Sec. 3.2 "CPU part", Sec. 3.3 "Communication overhead"): only the selected tokens'
// value-row numbers and weights leave the GPU (2 bytes per weight), the host forms the weighted sum.
// One workgroup per chunk of 256 selected tokens merges the chunk (max, sum) pairs of the row and writes
// fp16 weights [row * G + h][k], value rows [row][k] and, optionally, the accumulated scores.
__global__ __launch_bounds__(256) void weights_finalize(Layout L, const int32_t* __restrict__ idx,
                                                        const int32_t* __restrict__ count, int32_t k,
                                                        const int32_t* __restrict__ pos, AttendWs a, int nsplit,
                                                        const float* __restrict__ lse, uint16_t* __restrict__ w_out,
                                                        int32_t* __restrict__ vrow_out, float* __restrict__ acc) {
  __shared__ float fm[4], fz[4];
  __shared__ float wgt[4][64];
  const int row = blockIdx.y;
  const int cnt = count[row];
  merge_chunks(a.pmz + ((int64_t)row * nsplit * 4) * 2, nsplit, lse != nullptr ? lse + (int64_t)row * L.gqa : nullptr, L.gqa,
               fm, fz, wgt);
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= k) return;
  const bool live = i < cnt;
  float wsum = 0.f;
  for (int h = 0; h < L.gqa; ++h) {
    const float p = live ? expf(a.logit[((int64_t)row * 4 + h) * k + i] - fm[h]) / fz[h] : 0.f;
    w_out[((int64_t)row * L.gqa + h) * k + i] = f2h_bits(p);
    wsum += fmaxf(p, 1e-30f);
  }
  const int32_t slot = live ? idx[(int64_t)row * k + i] : 0;
  vrow_out[(int64_t)row * k + i] = live ? pos[(int64_t)row * L.cap + slot] : -1;
  if (live && acc != nullptr) acc[(int64_t)row * L.cap + slot] += wsum;
}

int32_t launch_attend_weights(const Layout& L, const void* kcache, const void* q, const int32_t* idx,
                              const int32_t* count, int32_t k, const int32_t* pos, float sm_scale, const float* lse,
                              void* w_out, int32_t* vrow_out, float* acc_opt, void* ws, hipStream_t st) {
  AttendWs a;
  carve(&a, ws, L, k);
  const int ns = nsplit_of(k);
  if (ns > 64) return HCA_ERR_CAPACITY;
  dim3 gp((unsigned)ns, (unsigned)L.rows);
  if (L.bits == 4)
    attend_partial<4, false><<<gp, 256, 0, st>>>(L, (const uint8_t*)kcache, (const uint16_t*)q, idx, count, k, sm_scale, a, ns, 0, ValueSource{}, RowEnd{});
  else
    attend_partial<2, false><<<gp, 256, 0, st>>>(L, (const uint8_t*)kcache, (const uint16_t*)q, idx, count, k, sm_scale, a, ns, 0, ValueSource{}, RowEnd{});
  weights_finalize<<<gp, 256, 0, st>>>(L, idx, count, k, pos, a, ns, lse, (uint16_t*)w_out, vrow_out, acc_opt);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

int32_t launch_attend(const Layout& L, const void* kcache, const void* q, const int32_t* idx,
                      const int32_t* count, int32_t k, const int32_t* pos, const void* v_host,
                      int64_t host_stride, int64_t n_host_rows, const void* v_hbm, int64_t hbm_stride,
                      float sm_scale, float* y, float* acc_opt, void* ws, hipStream_t gst, hipStream_t st) {
  if (nsplit_of(k) > 64) return HCA_ERR_CAPACITY;
  // On one stream nothing overlaps the gather, so the attend can read the value rows where they live: without host rows
  // always (4096 rows x 32 pairs: 27 us for the call against 42 through the staging area), with them while few are read
  // there.  Alone, direct / staged: 512 x 8 from the host 31 / 38 us, 128 x 32 26 / 36, 2048 x 8 88 / 96; half of the values
  // in HBM: 1024 x 8 31 / 41.  But a read per thread clogs the memory pipeline for what runs on other streams, which the
  // gather's few workgroups do not: a scan of 8 x 1 Mi keys, 123 us, takes 133, 143, 250 and 128 us beside these four.
  // A caller that shapes the gather (hca_tune, "gather_wgs") gets the gather.
  const bool no_host = v_host == nullptr || n_host_rows == 0;
  const int64_t entries = (int64_t)k * L.rows;
  const double host_part = v_hbm == nullptr ? 1.0 : (double)n_host_rows / ((double)n_host_rows + (double)hbm_stride);
  const bool few = entries <= kDirectEntries && entries * host_part <= kDirectHostEntries;
  if (gst == st && (no_host || few) && tuning().gather_wgs == 0) {
    const ValueSource vsrc{pos, (const uint4*)v_host, (const uint4*)v_hbm, host_stride, hbm_stride, n_host_rows};
    return attend_launches(L, kcache, q, idx, count, k, sm_scale, y, acc_opt, ws, st, nullptr, nullptr, vsrc);
  }
  if (gst != st) {
    hipError_t e;
    hipEvent_t ev = next_event(&e);
    if (e != hipSuccess) return hip_fail(e);
    HCA_HIP(hipEventRecord(ev, st));
    HCA_HIP(hipStreamWaitEvent(gst, ev, 0));
  }
  int32_t rc = launch_gather(L, idx, count, k, pos, v_host, host_stride, n_host_rows, v_hbm, hbm_stride, ws, gst);
  if (rc != HCA_OK) return rc;
  if (gst != st) {
    hipError_t e;
    hipEvent_t ev = next_event(&e);
    if (e != hipSuccess) return hip_fail(e);
    HCA_HIP(hipEventRecord(ev, gst));
    HCA_HIP(hipStreamWaitEvent(st, ev, 0));
  }
  return launch_attend_gathered(L, kcache, q, idx, count, k, sm_scale, y, acc_opt, ws, st);
}

}  // namespace hca
