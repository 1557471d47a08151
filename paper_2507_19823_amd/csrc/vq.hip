// Codebook form of the key path: grouped vector quantisation (Sec. 3.1) and the table-lookup
// scores of Sec. 3.2, Eq. 3.  A token is one centroid index per group (a byte: c <= 256), the query
// becomes a table T[centroid][group][query head of the KV head] that sits in LDS while a workgroup
// scans its share of the index matrix.  The host-side trainer is at the end of the file.
//
// Two storage forms.  Narrow (c <= 256 and the table of a KV head within 128 KiB): byte indices, table in
// LDS - everything said above.  Wide (up to c = 8192, the paper's own size, Fig. 4 / Table 4a): 16-bit
// indices stored group-major in tiles of 16 Ki slots (vq_wide_at in hca_device.h) and a table kept
// group-major too; a workgroup scans a share of the slots and brings the table through LDS one slice of groups at a
// time (vq_scan_wide_kernel).
//
// Narrow index rows are stored rotated: byte p of the record of slot j holds the index of group
// 16 * (p / 16) + (p + j) % 16  (vq_byte_of / vq_group_at in hca_device.h).  A thread of the scan reads
// its token's bytes in storage order, so at any moment the 16 lanes that share one pass of a 16-byte
// LDS read are on 16 different groups, and because a group's entries sit 16 bytes apart within a
// centroid's 256-byte line those lanes hit 16 different sets of 4 banks whatever their indices are.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <thread>
#include <vector>

#include "hca_internal.h"

namespace hca {

// ------------------------------------------------------------------------------- assign ---
// One wave = 64 tokens x GPW consecutive groups (4 for bulk calls; 1 for blocks of a few thousand tokens, which
// would otherwise leave most of the chip without a wave).  Every centroid read is wave-uniform (scalar loads),
// the running minimum is per lane.  distance: e = x - c; d = fmaf(e, e, d) over the group's channels in ascending
// order from d = 0; the first smallest wins.
template <int DBAR, bool WIDE, int GPW>
__global__ __launch_bounds__(256) void vq_assign_kernel(int g, int c, int n_kv_heads, int64_t cap,
                                                        const float* __restrict__ centroids,
                                                        uint8_t* __restrict__ pcache, const uint16_t* __restrict__ k_new,
                                                        int64_t T, NRes nr, float* __restrict__ acc,
                                                        int32_t* __restrict__ pos, NRes vrow0) {
  const int row = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int g0 = __builtin_amdgcn_readfirstlane((int)(blockIdx.z * 4 + (threadIdx.x >> 6))) * GPW;   // first group
  if (g0 >= g) return;
  const int64_t tt = (int64_t)blockIdx.x * 64 + lane;
  const bool live = tt < T;
  const int64_t tc = live ? tt : T - 1;
  // the wave's GPW * DBAR channels of this lane's token
  float x[GPW][DBAR];
  {
    const uint16_t* src = k_new + ((int64_t)row * T + tc) * kHeadDim + g0 * DBAR;
    constexpr int NW32 = GPW * DBAR / 2;                  // dwords: 8, 4, 2 or 1
    uint32_t wd[NW32];
    if constexpr (NW32 == 8) {
      const uint4 a = reinterpret_cast<const uint4*>(src)[0], b = reinterpret_cast<const uint4*>(src)[1];
      wd[0] = a.x; wd[1] = a.y; wd[2] = a.z; wd[3] = a.w; wd[4] = b.x; wd[5] = b.y; wd[6] = b.z; wd[7] = b.w;
    } else if constexpr (NW32 == 4) {
      const uint4 a = reinterpret_cast<const uint4*>(src)[0];
      wd[0] = a.x; wd[1] = a.y; wd[2] = a.z; wd[3] = a.w;
    } else if constexpr (NW32 == 2) {
      const uint2 a = reinterpret_cast<const uint2*>(src)[0];
      wd[0] = a.x; wd[1] = a.y;
    } else {
      wd[0] = reinterpret_cast<const uint32_t*>(src)[0];
    }
#pragma unroll
    for (int i = 0; i < NW32; ++i) {
      const int ch = 2 * i;
      x[ch / DBAR][ch % DBAR] = h2f(wd[i] & 0xffffu);
      x[(ch + 1) / DBAR][(ch + 1) % DBAR] = h2f(wd[i] >> 16);
    }
  }
  const float* cb = centroids + ((int64_t)(row % n_kv_heads) * g + g0) * c * DBAR;
  int win[GPW];
#pragma unroll
  for (int u = 0; u < GPW; ++u) {
    const float* cg = cb + (int64_t)u * c * DBAR;
    float bd = INFINITY;
    int best = 0;
    for (int cc = 0; cc < c; ++cc) {
      float d = 0.f;
#pragma unroll
      for (int dd = 0; dd < DBAR; ++dd) {
        const float e = x[u][dd] - cg[cc * DBAR + dd];
        d = fmaf(e, e, d);
      }
      if (d < bd || cc == 0) { bd = d; best = cc; }
    }
    win[u] = best;
  }
  if (!live) return;
  const int b = row / n_kv_heads;
  const int64_t slot = nr.n[b] + tt;
  if constexpr (WIDE) {
    uint16_t* pw = reinterpret_cast<uint16_t*>(pcache);
    const int64_t tiles = vq_tiles(cap);
#pragma unroll
    for (int u = 0; u < GPW; ++u) pw[vq_wide_at(g, tiles, row, slot, g0 + u)] = (uint16_t)win[u];
  } else {
    uint8_t* rec = pcache + ((int64_t)row * cap + slot) * g;
#pragma unroll
    for (int u = 0; u < GPW; ++u) rec[vq_byte_of(g0 + u, slot)] = (uint8_t)win[u];
  }
  if (g0 == 0) {
    if (acc != nullptr) acc[(int64_t)row * cap + slot] = 0.0f;
    if (pos != nullptr) pos[(int64_t)row * cap + slot] = (int32_t)(vrow0.n[b] + tt);
  }
}

// Bulk calls (a prefill block, a whole context): the matrix cores find, for every token, the few centroids that can
// be the nearest one, and only those go through the exact distance chain of vq_assign_kernel - the same index, bit
// for bit.
//   e(c) = |c|^2 / 2 - x.c  (= (distance - |x|^2) / 2) comes out of v_mfma_f32_32x32x16_f16, 32 centroids x 32 tokens
//   per instruction, with every factor an fp16 number so that the 16 products are exact in fp32:
//     k 0..3   A = -hi(c_d)            B = x_d        hi(c) = fp16(c), lo(c) = fp16(c - hi(c))
//     k 4..7   A = -lo(c_d)            B = x_d        (x is fp16 as it arrives)
//     k 8..10  A = h1, h2, h3          B = 1          h = fp32 |c|^2 / 2 cut into three fp16 pieces
//   Errors of e(c), for S = |x|^2 + max_c |c|^2 < 2^15 (so that no piece overflows fp16; fp16 denormals are kept by the
//   instruction) and with s(c) = |x|^2 + |c|^2: c_d - hi - lo is at most 2^-22 |c_d| + 2^-25, h loses at most
//   2^-33 of itself + 2^-25, the fp32 |c|^2 chain 4 u |c|^2 (u = 2^-24), and the instruction's 15 additions at
//   most 2^-23 each of sum |terms| <= 2.01 s(c) whatever their order and rounding: together below
//   E(c) = 2^-17.9 s(c) + 2^-23.  The exact chain d(c) itself is within 7 u d of the truth.
//   Let c1 have the smallest e as computed and c* be the winner of the exact chain (first smallest d): then
//   e(c*) <= e(c1) + E(c*) + E(c1) + 7.5 u d(c1) as computed.  Both lie near x: d(c*) <= (1 + 15 u) d(c1), and
//   d(c1) = |x|^2 + 2 e(c1) is known up to 2 E(c1) <= 2^-16.9 S + 2^-22, so that |c| <= |x| + sqrt(d2) for both, d2 an
//   upper bound of d(c1), and  S' = |x|^2 + (|x| + sqrt(d2))^2  bounds both s(c), however far away other centroids
//   are.  With  delta = 2^-17 S' + 2^-21 - one and a half times the sum of the errors -  e(c*) <= e(c1) + 2 delta.
//   (S in the place of S' sent 19 % of normal tokens to the queue below at two channels and 8192 centroids, and 86 %
//   where one channel has eight times the other's scale; S' sends 0.7 % and 10 %.)
//   One pass takes the minimum of e over every block of centroids and half wave (eight v_min3 per instruction) and
//   keeps the smallest ones per token, each with its block's number in the low mantissa bits (4 more per block): a
//   v_and_or, v_med3 and v_min in place of compares and selects.  That moves a value by less than 2^-16 of itself, so a
//   block counts as a candidate up to  m1 + 2.1 delta + 2^-14.9 |m1|  (m1 the smallest).  The exact chain then runs over
//   the 16 rows of a tile that the half wave holds, both halves sharing the work, for one block per token and now and
//   then two.  Tokens with more blocks in question than were kept, or with S out of range, are noted in an LDS queue
//   and go through the exact chain of every centroid at the end.  (|m1| < 1.01 S moves d2 by at most 2^-15 S more.)
// What bounds it is the vector ALU's issue (a second pass of products with the threshold folded in, a sign test and a
// list of candidates in the loop took twice the instructions): 12.9 per matrix instruction with everything, 79 % of
// the issue slots, the matrix cores 46 % busy.  16 Ki tokens x 8 KV heads against 8192 centroids: 1.09 ms (2.44 in two
// passes).
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ _Float16 am_f16(float v) { return (_Float16)v; }

// The A operands of one centroid (k blocks 0 and 1 of its row) and |c|^2.
template <int DBAR>
__device__ __forceinline__ void am_operands(const float (&cv)[DBAR], v8h* ra0, v8h* ra1, float* norm2) {
  const _Float16 zero = (_Float16)0.f;
  _Float16 hi[4] = {zero, zero, zero, zero}, lo[4] = {zero, zero, zero, zero};
  float nn = 0.f;
#pragma unroll
  for (int d = 0; d < DBAR; ++d) {
    nn = fmaf(cv[d], cv[d], nn);
    hi[d] = am_f16(-cv[d]);
    lo[d] = am_f16(-cv[d] - (float)hi[d]);
  }
  const float hh = 0.5f * nn;
  const _Float16 h1 = am_f16(hh);
  const float r1 = hh - (float)h1;
  const _Float16 h2 = am_f16(r1);
  const _Float16 h3 = am_f16(r1 - (float)h2);
  *ra0 = v8h{hi[0], hi[1], hi[2], hi[3], lo[0], lo[1], lo[2], lo[3]};
  *ra1 = v8h{h1, h2, h3, zero, zero, zero, zero, zero};
  *norm2 = nn;
}
// past the codebook: never among the smallest
__device__ __forceinline__ void am_no_centroid(v8h* ra0, v8h* ra1) {
  const _Float16 zero = (_Float16)0.f;
  *ra0 = v8h{zero, zero, zero, zero, zero, zero, zero, zero};
  *ra1 = v8h{(_Float16)65504.f, zero, zero, zero, zero, zero, zero, zero};
}
// The B operand of this lane's k block for a token's channels (pairs of fp16 as they lie in memory) and |x|^2.
template <int DBAR>
__device__ __forceinline__ v8h am_token(const uint32_t (&xw)[DBAR / 2], int kb, float* norm2) {
  const _Float16 one = (_Float16)1.f, zero = (_Float16)0.f;
  _Float16 xh[4] = {zero, zero, zero, zero};
  float n2 = 0.f;
#pragma unroll
  for (int d = 0; d < DBAR / 2; ++d) {
    const v2h pair = __builtin_bit_cast(v2h, xw[d]);
    n2 = __builtin_amdgcn_fdot2(pair, pair, n2, false);     // (only a bound is needed of it)
    xh[2 * d] = pair[0];
    xh[2 * d + 1] = pair[1];
  }
  *norm2 = n2;
  return kb == 0 ? v8h{xh[0], xh[1], xh[2], xh[3], xh[0], xh[1], xh[2], xh[3]}
                 : v8h{one, one, one, zero, zero, zero, zero, zero};
}
// The smaller of two numbers as one instruction: fminf spends another to quiet each operand that may be a signalling NaN.
// (NaNs only come from tokens or centroids out of range, which the caller finds by S.)  16 Ki tokens x 8 KV heads against
// 8192 centroids: 1168 us with fminf, 1092 with it.
__device__ __forceinline__ float am_min(float a, float b) { return __builtin_elementwise_minimum(a, b); }
__device__ __forceinline__ float am_max(float a, float b) { return __builtin_elementwise_maximum(a, b); }
// v with the bits of `mask` replaced by those of n (mask in a vector register: one instruction with n in a scalar one)
__device__ __forceinline__ float am_number(float v, uint32_t n, uint32_t mask) {
  return __uint_as_float((n & mask) | (__float_as_uint(v) & ~mask));
}
// How far above the smallest value a block can still hold the winner (m1: the smallest value with its block number in it,
// S = |x|^2 + max |c|^2 in range).
__device__ __forceinline__ float am_limit(float m1, float x2, float S) {
  const float d2 = am_max(2.f * m1 + x2 + (5e-5f * S + 9.5367431640625e-7f), 0.f);
  const float near = 2.f * x2 + d2 + 2.f * __builtin_amdgcn_sqrtf(x2 * d2);
  const float delta = am_min(near, S) * 7.62939453125e-6f + 4.76837158203125e-7f;      // 2^-17 S' + 2^-21
  return m1 + (2.1f * delta + 3.3e-5f * fabsf(m1));
}
// (value of the lower half, value of the upper half) of a wave, on every lane of a column
struct Halves { uint32_t lo, hi; };
__device__ __forceinline__ Halves halves_of(uint32_t v) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return Halves{r[0], r[1]};
}
// (distance, index) as one number that orders by distance, then by index; distances are never negative
__device__ __forceinline__ uint64_t am_key(float dist, int ci) { return (uint64_t)__float_as_uint(dist) << 32 | (uint32_t)ci; }
constexpr uint64_t kAmNoKey = ~0ull;

// The exact chain over every centroid of a group for N tokens, by LANES neighbouring lanes (y = which of them): the
// winners of the ascending scan of vq_assign_kernel, which starts from centroid 0 whatever its distance - no finite
// distance at all, or a first distance that is not a number, leave it the winner.
template <int DBAR, int LANES, int N>
__device__ __forceinline__ void am_exhaustive_of(const uint16_t* const (&src)[N], const float* cg, int c, int y, int (&win)[N]) {
  float x[N][DBAR], bd[N];
  int bi[N], first_nan[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
#pragma unroll
    for (int d = 0; d < DBAR; ++d) x[i][d] = h2f(src[i][d]);
    bd[i] = INFINITY;
    bi[i] = 0x7fffffff;
    first_nan[i] = 0;
  }
  for (int c0 = y; c0 < c; c0 += 4 * LANES) {               // four centroids in flight
    float cv[4][DBAR];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int d = 0; d < DBAR; ++d) cv[u][d] = cg[(c0 + u * LANES < c ? c0 + u * LANES : c0) * DBAR + d];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < N; ++i) {
        float dist = 0.f;
#pragma unroll
        for (int d = 0; d < DBAR; ++d) {
          const float e = x[i][d] - cv[u][d];
          dist = fmaf(e, e, dist);
        }
        if (c0 + u * LANES < c && dist < bd[i]) { bd[i] = dist; bi[i] = c0 + u * LANES; }
        if (c0 == 0 && u == 0) first_nan[i] = dist != dist;
      }
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
#pragma unroll
    for (int o = LANES / 2; o >= 1; o >>= 1) {
      const float od = __shfl_xor(bd[i], o);
      const int ob = __shfl_xor(bi[i], o);
      first_nan[i] |= __shfl_xor(first_nan[i], o);
      if (od < bd[i] || (od == bd[i] && ob < bi[i])) { bd[i] = od; bi[i] = ob; }
    }
    win[i] = (bi[i] == 0x7fffffff || first_nan[i]) ? 0 : bi[i];
  }
}
template <int DBAR, int LANES>
__device__ __forceinline__ int am_exhaustive(const uint16_t* src, const float* cg, int c, int y) {
  const uint16_t* const one[1] = {src};
  int win[1];
  am_exhaustive_of<DBAR, LANES, 1>(one, cg, c, y, win);
  return win[0];
}

// More than 256 centroids, and blocks of few tokens against 96 and more.  One workgroup of 8 waves = 1024 tokens x one group; a wave holds
// 128 tokens (four 32-token B operands) against centroids that pass through LDS 512 at a time (A operands only,
// double-buffered, one barrier per chunk).  kAmBlock: tiles of 32 centroids per block, two beyond 2048 centroids (128 blocks
// at 8192, half the bookkeeping), else one (half the rows to look into).  The three smallest values are kept, so two
// blocks per half wave can be looked into.
constexpr int kAmChunk = 512;       // centroids per LDS chunk

template <int DBAR, int kAmBlock, bool WIDE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void vq_assign_mfma_kernel(
    int g, int c, int n_kv_heads, int64_t cap, const float* __restrict__ centroids, uint8_t* __restrict__ pcache,
    const uint16_t* __restrict__ k_new, int64_t T, NRes nr, float* __restrict__ acc, int32_t* __restrict__ pos,
    NRes vrow0) {
  constexpr int TT = 4;
  // A operands: [buffer][tile of 32 centroids][k block 0 / 1][row] x 8 fp16
  __shared__ __align__(16) v8h sA[2][kAmChunk / 32][2][32];
  __shared__ float s_cmax[8];
  __shared__ uint16_t s_queue[1024];
  __shared__ uint32_t s_nq;
  const int row = blockIdx.y, grp = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int col = lane & 31, kb = lane >> 5;
  const int64_t wg0 = (int64_t)blockIdx.x * 1024, tok0 = wg0 + w * 128;
  const int b = row / n_kv_heads;
  const float* cg = centroids + ((int64_t)(row % n_kv_heads) * g + grp) * c * DBAR;
  const v16f zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto channels_of = [&](int64_t t) { return k_new + ((int64_t)row * T + (t < T ? t : T - 1)) * kHeadDim + grp * DBAR; };
  auto load_x = [&](int tt, uint32_t (&xw)[DBAR / 2]) {
    const uint16_t* src = channels_of(tok0 + 32 * tt + col);
#pragma unroll
    for (int d = 0; d < DBAR / 2; ++d) xw[d] = (uint32_t)src[2 * d] | (uint32_t)src[2 * d + 1] << 16;
  };
  const bool wave_live = tok0 < T;                          // (a wave without tokens only helps with the operands)
  float x2[TT];
  v8h bop[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    uint32_t xw[DBAR / 2];
    load_x(tt, xw);
    bop[tt] = am_token<DBAR>(xw, kb, &x2[tt]);
  }

  const int nchunk = (c + kAmChunk - 1) / kAmChunk;
  float cv[DBAR];                    // this thread's centroid of the chunk on its way to LDS
  float mycmax = 0.f;
  auto fetch = [&](int ch) {
    const int cc = ch * kAmChunk + tid;
#pragma unroll
    for (int d = 0; d < DBAR; ++d) cv[d] = cg[(int64_t)(cc < c ? cc : 0) * DBAR + d];
  };
  auto commit = [&](int ch) {
    v8h ra0, ra1;
    am_no_centroid(&ra0, &ra1);
    if (ch * kAmChunk + tid < c) {
      float nn;
      am_operands<DBAR>(cv, &ra0, &ra1, &nn);
      mycmax = nn < INFINITY ? fmaxf(mycmax, nn) : INFINITY;     // not finite or not a number: no token is in range
    }
    sA[ch & 1][tid >> 5][0][tid & 31] = ra0;
    sA[ch & 1][tid >> 5][1][tid & 31] = ra1;
  };
  auto blocks_of = [&](int ch) {
    const int left = c - ch * kAmChunk;
    return ((left < kAmChunk ? left : kAmChunk) + 32 * kAmBlock - 1) / (32 * kAmBlock);
  };

  float m1[TT], m2[TT], m3[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) { m1[tt] = INFINITY; m2[tt] = INFINITY; m3[tt] = INFINITY; }
  uint32_t number = 127;
  asm volatile("" : "+v"(number));
  if (tid == 0) s_nq = 0;
  fetch(0);
  commit(0);
  __syncthreads();
  for (int ch = 0; ch < nchunk; ++ch) {
    const int buf = ch & 1;
    if (ch + 1 < nchunk) fetch(ch + 1);
    if (wave_live) {
      const int nblk = blocks_of(ch);
      for (int bl = 0; bl < nblk; ++bl) {
        float tm[TT];
#pragma unroll
        for (int u = 0; u < kAmBlock; ++u) {
          const v8h a = sA[buf][bl * kAmBlock + u][kb][col];
          v16f d[TT];
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) d[tt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bop[tt], zero16, 0, 0, 0);
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) {
            float mm = u == 0 ? am_min(d[tt][14], d[tt][15]) : am_min(am_min(tm[tt], d[tt][14]), d[tt][15]);
#pragma unroll
            for (int j = 0; j < 14; j += 2) mm = am_min(am_min(mm, d[tt][j]), d[tt][j + 1]);
            tm[tt] = mm;
          }
        }
        const uint32_t blk = (uint32_t)(ch * (kAmChunk / 32 / kAmBlock) + bl);
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          const float pk = am_number(tm[tt], blk, number);
          m3[tt] = __builtin_amdgcn_fmed3f(m2[tt], m3[tt], pk);
          m2[tt] = __builtin_amdgcn_fmed3f(m1[tt], m2[tt], pk);
          m1[tt] = am_min(m1[tt], pk);
        }
      }
    }
    if (ch + 1 < nchunk) commit(ch + 1);
    __syncthreads();
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mycmax = fmaxf(mycmax, __shfl_xor(mycmax, o));
  if (lane == 0) s_cmax[w] = mycmax;
  __syncthreads();
  float cmax2 = s_cmax[0];
#pragma unroll
  for (int x = 1; x < 8; ++x) cmax2 = fmaxf(cmax2, s_cmax[x]);

  auto put = [&](int64_t t, int win) {
    if (t >= T) return;
    const int64_t slot = nr.n[b] + t;
    if constexpr (WIDE) reinterpret_cast<uint16_t*>(pcache)[vq_wide_at(g, vq_tiles(cap), row, slot, grp)] = (uint16_t)win;
    else pcache[((int64_t)row * cap + slot) * g + vq_byte_of(grp, slot)] = (uint8_t)win;
    if (grp == 0) {
      if (acc != nullptr) acc[(int64_t)row * cap + slot] = 0.0f;
      if (pos != nullptr) pos[(int64_t)row * cap + slot] = (int32_t)(vrow0.n[b] + t);
    }
  };
  if (wave_live) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const float S = x2[tt] + cmax2;
      const Halves a1 = halves_of(__float_as_uint(m1[tt])), a2 = halves_of(__float_as_uint(m2[tt])),
                   a3 = halves_of(__float_as_uint(m3[tt]));
      const float lim = am_limit(fminf(__uint_as_float(a1.lo), __uint_as_float(a1.hi)), x2[tt], S);
      // the token's candidates, one byte each (block, 255: none): smallest of the lower half, of the upper half, then
      // the second smallest
      auto cand = [&](uint32_t v) { return __uint_as_float(v) <= lim ? (v & 127u) : 255u; };
      uint32_t todo = cand(a1.lo) | cand(a1.hi) << 8 | cand(a2.lo) << 16 | cand(a2.hi) << 24;
      // (a column past the last token holds a copy of that token, up to 127 of them, and has nothing to look up)
      const bool real = tok0 + 32 * tt + col < T;
      const bool queue = real && (!(S < 32768.f) || __uint_as_float(a3.lo) <= lim || __uint_as_float(a3.hi) <= lim);
      if (queue || !real) todo = 0xffffffffu;
      uint64_t best = kAmNoKey;
      float x[DBAR];
      {
        uint32_t xw[DBAR / 2];
        load_x(tt, xw);
#pragma unroll
        for (int d = 0; d < DBAR; ++d) x[d] = h2f((xw[d >> 1] >> (16 * (d & 1))) & 0xffffu);
      }
      while (__builtin_amdgcn_ballot_w64(todo != 0xffffffffu) != 0) {
        if (todo != 0xffffffffu) {
          const int which = (int)__builtin_ctz(~((todo & 0x80808080u) | 0x7f7f7f7fu)) >> 3;    // first byte below 128
          const int blk = (int)((todo >> (8 * which)) & 127u), half = which & 1;
          todo |= 0xffu << (8 * which);
          // rows of a 32 x 32 result held by a half: 8 (j / 4) + 4 half + j % 4, j < 16; this lane takes j = 8 kb ..
          float rd = INFINITY;
          int ri = 0x7fffffff;
#pragma unroll
          for (int u = 0; u < kAmBlock; ++u) {
            const int c0 = (blk * kAmBlock + u) * 32 + 16 * kb + 4 * half;
            float cc[8][DBAR];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int ci = c0 + 8 * (j >> 2) + (j & 3);
#pragma unroll
              for (int d = 0; d < DBAR; ++d) cc[j][d] = cg[(int64_t)(ci < c ? ci : 0) * DBAR + d];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int ci = c0 + 8 * (j >> 2) + (j & 3);
              float dist = 0.f;
#pragma unroll
              for (int d = 0; d < DBAR; ++d) {
                const float e = x[d] - cc[j][d];
                dist = fmaf(e, e, dist);
              }
              if (ci < c && dist < rd) { rd = dist; ri = ci; }
            }
          }
          const uint64_t key = am_key(rd, ri);
          if (key < best) best = key;
        }
      }
      const Halves bh = halves_of((uint32_t)(best >> 32)), bl = halves_of((uint32_t)best);
      const uint64_t k0 = (uint64_t)bh.lo << 32 | bl.lo, k1 = (uint64_t)bh.hi << 32 | bl.hi;
      if (kb == 0) {
        if (queue) s_queue[atomicAdd(&s_nq, 1u)] = (uint16_t)(w * 128 + 32 * tt + col);
        else put(tok0 + 32 * tt + col, (int)(uint32_t)(k0 < k1 ? k0 : k1));
      }
    }
  }
  __syncthreads();
  for (uint32_t e = w; e < s_nq; e += 8) {                   // one wave per queued token
    const int64_t t = wg0 + s_queue[e];
    const int win = am_exhaustive<DBAR, 64>(channels_of(t), cg, c, lane);
    if (lane == 0) put(t, win);
  }
}

// At most 256 centroids: at most eight tiles cover a group, so a group's operands (and the centroids themselves, for the
// exact chain) sit in LDS at once.  A workgroup of four waves takes 256 tokens through sixteen consecutive groups: the
// next group's centroids are fetched, split and stored to the other LDS buffer meanwhile (one thread per centroid), one
// barrier per group, and the sixteen index bytes of a token leave as one 16-byte store (narrow form).  A block is half of
// a tile's rows in a half wave; two values are kept, a token with rivals in another block (a few in a thousand) goes to
// the queue.
// Bound by the issue of the vector ALU (97 % of its slots at 64 Ki tokens x 8 KV heads and 256 centroids, 30 instructions per
// product of two tiles, at the 1.93 GHz that the power limit leaves): the two minima of 16 blocks of products, half of it, and
// one block's exact chain per token.  Every lane decides about one token - the two tiles' halves change places
// in one swap each - so that the limit and the chain's set-up are paid once per token, not once per half wave.
// 64 Ki tokens x 8 KV heads against 256 centroids: 311 -> 239 us (0.99 ms in the vector form), 64 centroids: 178 -> 128
// (0.25); two channels: 586 -> 433, 335 -> 193.
constexpr int kAsCodewords = 256;

// largest of a wave's numbers, none of them negative: their bits compare like them
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max(uint32_t v) {
  const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
  return o > v ? o : v;
}
__device__ __forceinline__ float wave_max_nonneg(float f) {
  uint32_t v = __float_as_uint(f);
  v = dpp_max<0xB1>(v);               // quad_perm [1,0,3,2]
  v = dpp_max<0x4E>(v);               // quad_perm [2,3,0,1]
  v = dpp_max<0x141>(v);              // row_half_mirror
  v = dpp_max<0x140>(v);              // row_mirror
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = a[0] > a[1] ? a[0] : a[1];
  const Halves h = halves_of(v);
  return __uint_as_float(h.lo > h.hi ? h.lo : h.hi);
}

// NT: tiles of 32 centroids (2, 4 or 8)
template <int DBAR, bool WIDE, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void vq_assign_small_c_kernel(
    int g, int c, int n_kv_heads, int64_t cap, const float* __restrict__ centroids, uint8_t* __restrict__ pcache,
    const uint16_t* __restrict__ k_new, int64_t T, NRes nr, float* __restrict__ acc, int32_t* __restrict__ pos,
    NRes vrow0) {
  constexpr int kGroups = 16;         // groups per workgroup
  constexpr int TT = 2;               // 32-token tiles per wave
  constexpr int kCen = NT * 32;
  __shared__ __align__(16) v8h sA[2][NT][2][32];
  __shared__ __align__(16) float sC[2][kCen + 12][DBAR];        // centroids, the tiles' rows shifted (cen_at)
  __shared__ float s_cmax[2][4];
  __shared__ __align__(16) uint8_t s_win[WIDE ? 1 : 256][kGroups];         // narrow form: a token's sixteen record bytes
  __shared__ uint16_t s_queue[512];                             // (token, group) pairs left to the exhaustive chain
  __shared__ uint32_t s_added[kGroups];                         // how many of them each group added
  const int row = blockIdx.y, g0 = blockIdx.z * kGroups;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int col = lane & 31, kb = lane >> 5;
  const int64_t wg0 = (int64_t)blockIdx.x * 256, tok0 = wg0 + w * 64;
  const int b = row / n_kv_heads;
  const float* cb = centroids + ((int64_t)(row % n_kv_heads) * g + g0) * c * DBAR;
  const v16f zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // row r of tile t: 16 lanes that read the same row of their halves in any of the eight tiles are on different banks
  // (at four channels; a row is 4 banks, the halves are 16 apart)
  auto cen_at = [](int t, int r) { return t * 32 + r + (t & 3) + (t >> 2) * 8; };
  // one centroid of a group per thread: fetched to registers, later split into operands and stored
  float cv[DBAR];
  auto fetch = [&](int gi) {
    const float* p = cb + ((int64_t)gi * c + (tid < c ? tid : 0)) * DBAR;
#pragma unroll
    for (int d = 0; d < DBAR; ++d) cv[d] = p[d];
  };
  auto commit = [&](int buf) {
    float nn = 0.f;
    if (kCen == 256 || w * 64 < kCen) {
      v8h ra0, ra1;
      am_no_centroid(&ra0, &ra1);
      if (tid < c) am_operands<DBAR>(cv, &ra0, &ra1, &nn);
      sA[buf][tid >> 5][0][tid & 31] = ra0;
      sA[buf][tid >> 5][1][tid & 31] = ra1;
      // past the codebook: a distance of infinity, never the smallest
#pragma unroll
      for (int d = 0; d < DBAR; ++d) sC[buf][cen_at(tid >> 5, tid & 31)][d] = tid < c ? cv[d] : INFINITY;
    }
    const float m = wave_max_nonneg(nn < INFINITY ? nn : INFINITY);     // not finite or not a number: no token is in range
    if (lane == 0) s_cmax[buf][w] = m;
  };
  // this lane's own token (lane 32 tt + col has column col of the wave's tile tt): 16 bytes of it as they lie in memory,
  // the channels of two or four groups, the next group's first, and the 16 bytes after them.  (A load per group asks for
  // every line of the keys sixteen times, and beyond 16 Ki tokens x 8 KV heads not out of L2: with few centroids that is
  // what bounds the launch.  32 Ki x 8 against 64 centroids: 100 us with 8 bytes per load, 73 with 16.)
  constexpr int kPer = 8 / DBAR;
  const int64_t mine = tok0 + lane;
  const uint4* xsrc =
      reinterpret_cast<const uint4*>(k_new + ((int64_t)row * T + (mine < T ? mine : T - 1)) * kHeadDim + g0 * DBAR);
  uint4 xq = xsrc[0], xnext = xq;
  // the winner of token `tok` (of the workgroup's 256) in group gi
  auto put = [&](int tok, int gi, int win) {
    const int64_t t = wg0 + tok;
    if constexpr (WIDE) {
      if (t < T) reinterpret_cast<uint16_t*>(pcache)[vq_wide_at(g, vq_tiles(cap), row, nr.n[b] + t, g0 + gi)] = (uint16_t)win;
    } else {
      s_win[tok][(gi - (int)(nr.n[b] + t)) & 15] = (uint8_t)win;
    }
  };
  fetch(0);
  commit(0);
  if (tid < kGroups) s_added[tid] = 0;
  __syncthreads();
  // entries in the queue when a group begins.  Every wave keeps it for itself, from counts that no longer change: a wave
  // still deciding about group gi reads s_added[gi] while another may already be appending to s_added[gi + 1], and all of
  // them decide the same - the branch below holds a barrier
  uint32_t queued = 0;
  for (int gi = 0; gi < kGroups; ++gi) {
    const int buf = gi & 1;
    float x2 = 0.f, x[DBAR];
    v8h bop[TT];
    {
      uint32_t xt[TT][DBAR / 2];
#pragma unroll
      for (int d = 0; d < DBAR / 2; ++d) {
        const uint32_t xw = d == 0 ? xq.x : xq.y;
        const v2h pair = __builtin_bit_cast(v2h, xw);
        x2 = __builtin_amdgcn_fdot2(pair, pair, x2, false);
        x[2 * d] = h2f(xw & 0xffffu);
        x[2 * d + 1] = h2f(xw >> 16);
        const Halves h = halves_of(xw);
        xt[0][d] = h.lo;
        xt[1][d] = h.hi;
      }
      float unused;
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) bop[tt] = am_token<DBAR>(xt[tt], kb, &unused);
    }
    if (gi + 1 < kGroups) fetch(gi + 1);
    if (gi % kPer == 0 && gi + kPer < kGroups) xnext = xsrc[gi / kPer + 1];
    float m1[TT], m2[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) { m1[tt] = INFINITY; m2[tt] = INFINITY; }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      // the empty asm statements keep the tiles in order: the scheduler would start all products at once and spill
      v8h a = sA[buf][t][kb][col];
      asm volatile("" : "+v"(a));
      v16f d[TT];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) d[tt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bop[tt], zero16, 0, 0, 0);
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {                       // the half wave's first and last eight rows
          float tm = am_min(d[tt][8 * q], d[tt][8 * q + 1]);
#pragma unroll
          for (int j = 2; j < 8; j += 2) tm = am_min(am_min(tm, d[tt][8 * q + j]), d[tt][8 * q + j + 1]);
          const float pk = am_number(tm, (uint32_t)(2 * t + q), 15u);
          m2[tt] = __builtin_amdgcn_fmed3f(m1[tt], m2[tt], pk);
          m1[tt] = am_min(m1[tt], pk);
        }
        asm volatile("" : "+v"(m1[tt]));
      }
    }
    const float cmax2 = am_max(am_max(s_cmax[buf][0], s_cmax[buf][1]), am_max(s_cmax[buf][2], s_cmax[buf][3]));
    if (gi + 1 < kGroups) commit(buf ^ 1);
    // every lane decides about its own token: its tile's values of the lower and of the upper half wave in one swap
    static_assert(TT == 2, "a token per lane");
    const auto p1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(m1[0]), __float_as_uint(m1[1]), false, false);
    const auto p2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(m2[0]), __float_as_uint(m2[1]), false, false);
    const float f0 = __uint_as_float(p1[0]), f1 = __uint_as_float(p1[1]);
    const bool upper = f1 < f0;
    const float S = x2 + cmax2;
    const float lim = am_limit(upper ? f1 : f0, x2, S);
    // a second block within the limit, or values that say nothing (and a token: past the last there are copies of it)
    const float next = am_min(am_min(__uint_as_float(p2[0]), __uint_as_float(p2[1])), am_max(f0, f1));
    const bool queue = mine < T && (next <= lim || !(S < 32768.f));
    // rows of a 32 x 32 result held by a half: 8 (j / 4) + 4 half + j % 4, j < 16; block 2 t + q has j = 8 q .. 8 q + 7
    const uint32_t blk = (upper ? p1[1] : p1[0]) & 15u;
    const int tile = (int)(blk >> 1) & (NT - 1), r0 = 16 * (int)(blk & 1u) + (upper ? 4 : 0);
    typedef float cen_t __attribute__((ext_vector_type(DBAR)));
    const cen_t* cen = reinterpret_cast<const cen_t*>(sC[buf][cen_at(tile, r0)]);
    float bd = 0.f;
    int bj = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int r = 8 * (j >> 2) + (j & 3);
      const cen_t cv = cen[r];
      float dist = 0.f;
#pragma unroll
      for (int d = 0; d < DBAR; ++d) {
        const float e = x[d] - cv[d];
        dist = fmaf(e, e, dist);
      }
      if (j == 0 || dist < bd) { bd = dist; bj = r; }
    }
    if (gi % kPer == kPer - 1) xq = xnext;
    else xq = DBAR == 4 ? uint4{xq.z, xq.w, 0, 0} : uint4{xq.y, xq.z, xq.w, 0};
    const int tok = w * 64 + lane;
    if (queue) s_queue[queued + atomicAdd(&s_added[gi], 1u)] = (uint16_t)(tok | gi << 8);
    else put(tok, gi, tile * 32 + r0 + bj);
    __syncthreads();
    queued += s_added[gi];
    if (queued > 256 || gi + 1 == kGroups) {                // no room for another group's 256 tokens, or the end
      for (uint32_t e = tid >> 3; e < queued; e += 32) {    // eight lanes per queued token
        const int tok = s_queue[e] & 255, qi = s_queue[e] >> 8;
        const int64_t t = wg0 + tok;
        const int win = am_exhaustive<DBAR, 8>(k_new + ((int64_t)row * T + (t < T ? t : T - 1)) * kHeadDim + (g0 + qi) * DBAR,
                                               cb + (int64_t)qi * c * DBAR, c, tid & 7);
        if ((tid & 7) == 0) put(tok, qi, win);
      }
      __syncthreads();                                      // the entries have been read, and s_win is complete
      queued = 0;
    }
  }
  const int64_t t = wg0 + tid;
  if (t >= T) return;
  const int64_t slot = nr.n[b] + t;
  if constexpr (!WIDE)
    *reinterpret_cast<uint4*>(pcache + ((int64_t)row * cap + slot) * g + g0) = *reinterpret_cast<const uint4*>(s_win[tid]);
  if (g0 == 0) {
    if (acc != nullptr) acc[(int64_t)row * cap + slot] = 0.0f;
    if (pos != nullptr) pos[(int64_t)row * cap + slot] = (int32_t)(vrow0.n[b] + t);
  }
}

// Thousands of centroids and enough tokens per workgroup: the same shortlist and the same winner, but each wave looks at
// the few blocks of centroids that its tokens are near.  One workgroup of 16 waves = up to 16 Ki tokens x one group.
//   Order.  Tokens and centroids are each put in the order of a nested grid of quantiles (cells_order): every channel in
//   turn cuts each cell into equal parts, more parts where the spread is wider.  32 neighbours of that order lie close
//   together: 32 tokens are one B operand, 32 centroids one block with a bounding box.  The sorted tokens live in registers
//   (their numbers), the sorted centroids in LDS as (fp16, fp16 of twice the rest) per channel, 16 bytes at four channels,
//   so that 8192 of them fit; |c|^2 / 2 is formed from the same bytes when a block is multiplied.
//   Search, per 32 tokens: the distance from the tokens' box to every block's box (a lane has four blocks); the blocks at
//   the least distance are multiplied; then each block whose distance does not exceed the worst token's upper bound is
//   tested token by token (two blocks at once, one per half wave) and multiplied if it can still hold any token's winner.
//   The products' accumulator starts from |x|^2 / 2, so the results are d(c) / 2 and the blocks' numbers in the low 8 bits
//   cost 2^-15 of d, not of |x|^2.
//   Errors, for S and s(c) as above: with p = hi^2 / 2 rounded to fp16 and q = fp16(rest of it + hi lo), the pieces lose at most
//   2^-20.3 s(c) + 2^-21.3, sixteen additions 2^-17.6 s(c): E(c) = 2^-17.3 s(c) + 2^-21.3, and cells_limit takes 1.4 times that.
//   Emulated against 64 bits (1500 tokens and their 24 nearest of 8192, two and four channels: normal; one channel, or all,
//   20 - 40 times as wide; centroids next to tokens), root mean square, vq_assign_mfma_kernel's form as 1: the products 0.75 -
//   1.07, with the blocks' numbers in their low bits 0.016 - 0.12.
//   A box can be passed over when its squared distance exceeds 1.002 times the upper bound that cells_bound gives: gaps
//   are fp16 differences (2^-11 each), boxes are rounded outwards, the chain's own error is 2^-20.
//   The candidates' distances come from the two halves in LDS, in 32 bits; only where the second best is within the
//   error of the halves (one token in ten thousand and fewer) does the exact chain decide.  Tokens with three blocks of a
//   half wave in question go through the exact chain of all near blocks, out-of-range ones of every centroid (settle).
// Bound by the issue of the vector ALU (88 % of its slots by the counters): 16 Ki normal tokens x 8 KV heads, 32 groups, c =
// 8192: per 32 tokens 20 of 256 blocks are multiplied and 1730 vector instructions issued.  A call of that 1120 us in
// vq_assign_mfma_kernel, 454 here (with the waves left to the order of age 60 more).
constexpr int kCellTokens = 16384, kCellBins = 4096;

__device__ __forceinline__ v2h cells_min(v2h a, v2h b) { return __builtin_elementwise_minimum(a, b); }
__device__ __forceinline__ v2h cells_max(v2h a, v2h b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ uint32_t cells_bits(v2h v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ v2h cells_pair(uint32_t v) { return __builtin_bit_cast(v2h, v); }

// min over the 32 lanes of a half wave (every lane gets it); packed fp16
template <int CTRL> __device__ __forceinline__ uint32_t cells_dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}
template <class Op> __device__ __forceinline__ uint32_t cells_over_half(uint32_t v, Op op) {
  v = op(v, cells_dpp<0xB1>(v));
  v = op(v, cells_dpp<0x4E>(v));
  v = op(v, cells_dpp<0x141>(v));
  v = op(v, cells_dpp<0x140>(v));
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return op(a[0], a[1]);
}

__device__ __forceinline__ float cells_sum(float v) {
  dpp_steps([&](auto&& shift) { v += __uint_as_float(shift(0u, __float_as_uint(v))); });
  return __uint_as_float(wave_last(__float_as_uint(v)));
}

// Positions of n items in the order of the nested grid: item number i * 1024 + thread has channels value(i, d).  Cells of
// a round are cut at exact ranks; inside a bin (a 16th to a 256th of the channel's softsign-scaled range) items stay in any order.
// hist: twice kCellBins words of LDS, one histogram for even and one for odd rounds; the caller synchronises before reusing it.
template <int P, int DBAR, class Value>
__device__ __forceinline__ void cells_order(Value value, int n, const float (&mu)[DBAR], const float (&sd)[DBAR], uint32_t* hist,
                                            uint32_t* s_wave, int (&pos)[P]) {
  const int tid = threadIdx.x;
  int nb[DBAR];
  {
    float v[DBAR];
#pragma unroll
    for (int d = 0; d < DBAR; ++d) { nb[d] = 0; v[d] = sd[d]; }
    for (int cells = 32; cells < n; cells *= 2) {            // the widest channel is halved
      float top = v[0];
#pragma unroll
      for (int d = 1; d < DBAR; ++d) top = fmaxf(top, v[d]);
      bool done = false;
#pragma unroll
      for (int d = 0; d < DBAR; ++d)
        if (!done && (v[d] >= top || d == DBAR - 1)) { ++nb[d]; v[d] *= 0.5f; done = true; }
    }
  }
#pragma unroll
  for (int i = 0; i < P; ++i) pos[i] = i * 1024 + tid;
  int logn = 0;
  bool first = true;
  uint4* hz = reinterpret_cast<uint4*>(hist) + tid;          // this thread's bins of this round's histogram
  uint4* hn = hz + kCellBins / 4;
  hz[0] = uint4{0, 0, 0, 0};
  hn[0] = uint4{0, 0, 0, 0};
  __syncthreads();
#pragma unroll
  for (int d = 0; d < DBAR; ++d) {
    const int bits = __builtin_amdgcn_readfirstlane(nb[d]);
    if (bits == 0) continue;
    const int lb = 12 - logn < 8 ? 12 - logn : 8;
    const float half = 0.5f * (float)(1 << lb), last = (float)((1 << lb) - 1);
    const float inv = sd[d] > 0.f ? __builtin_amdgcn_rcpf(sd[d]) : 0.f;
    const float parts = (float)(1 << logn) / (float)((n + 31) >> 5);
    uint32_t* bins = reinterpret_cast<uint32_t*>(hz - tid);
    // four items at a time, so that their updates are in flight together
#pragma unroll
    for (int i0 = 0; i0 < P; i0 += 4) {
      if (i0 * 1024 >= n) continue;
      uint32_t key[4], rank[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u;
        const float v = (value(i, d) - mu[d]) * inv;
        const float f = fminf(fmaxf(fmaf(v * __builtin_amdgcn_rcpf(1.f + fabsf(v)), half, half), 0.f), last);
        int node = first ? 0 : (int)((float)(pos[i] >> 5) * parts);      // cells are cut between 32s, which are never in two
        node = node < (1 << logn) - 1 ? node : (1 << logn) - 1;
        key[u] = (uint32_t)node << lb | (uint32_t)f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        rank[u] = 0;
        if ((i0 + u) * 1024 + tid < n) rank[u] = atomicAdd(&bins[key[u]], 1u);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) pos[i0 + u] = (int)(key[u] | rank[u] << 12);
    }
    __syncthreads();
    uint4 a = hz[0];
    const uint32_t own = a.x + a.y + a.z + a.w, inc = wave_scan_incl(own);
    if ((tid & 63) == 63) s_wave[tid >> 6] = inc;
    hn[0] = uint4{0, 0, 0, 0};                               // (read before the last barrier)
    __syncthreads();
    uint32_t run = inc - own, t;
    {
      const uint32_t before = wave_scan_incl((tid & 63) < 16 ? s_wave[tid & 15] : 0u);        // lane x: of waves 0 .. x
      if (tid >= 64) run += (uint32_t)__builtin_amdgcn_readlane((int)before, __builtin_amdgcn_readfirstlane((tid >> 6) - 1));
    }
    t = a.x; a.x = run; run += t;
    t = a.y; a.y = run; run += t;
    t = a.z; a.z = run; run += t;
    a.w = run;
    hz[0] = a;
    __syncthreads();
#pragma unroll
    for (int i0 = 0; i0 < P; i0 += 4) {
      if (i0 * 1024 >= n) continue;
#pragma unroll
      for (int u = 0; u < 4; ++u)        // (past the last item: key and rank 0, a position nobody reads)
        pos[i0 + u] = (int)(bins[pos[i0 + u] & (kCellBins - 1)] + ((uint32_t)pos[i0 + u] >> 12));
    }
    uint4* swap = hz;
    hz = hn;
    hn = swap;
    logn += bits;
    first = false;
  }
}

// Mean and mean distance from it of the items' channels (a few items far away hardly move either).
template <int P, int DBAR, class Value>
__device__ __forceinline__ void cells_moments(Value value, int n, float (&mu)[DBAR], float (&sd)[DBAR], float* s_stat) {
  const int tid = threadIdx.x;
  if (tid < 2 * DBAR) s_stat[tid] = 0.f;
  __syncthreads();
  auto mean = [&](int at, auto&& of, float (&out)[DBAR]) {
#pragma unroll
    for (int d = 0; d < DBAR; ++d) {
      float a = 0.f;
#pragma unroll
      for (int i = 0; i < P; ++i) {
        if (i * 1024 >= n) continue;
        a += i * 1024 + tid < n ? of(value(i, d), d) : 0.f;
      }
      a = cells_sum(a);
      if ((tid & 63) == 0) atomicAdd(&s_stat[at + d], a);
    }
    __syncthreads();
#pragma unroll
    for (int d = 0; d < DBAR; ++d) out[d] = s_stat[at + d] / (float)n;
  };
  mean(0, [&](float v, int) { return v; }, mu);
  mean(DBAR, [&](float v, int d) { return fabsf(v - mu[d]); }, sd);
}

// As am_limit, of a value that is half a squared distance with a number in its low 8 bits.
// Upper bound of the squared distance: first with S, then with what that says of the centroid, |c|^2 <= 2 |x|^2 + 2 d, however
// far away others are.
__device__ __forceinline__ float cells_bound(float m1, float x2, float S) {
  const float d0 = am_max(fmaf(2.0002f, m1, fmaf(5e-5f, S, 1e-6f)), 0.f);
  return am_max(fmaf(2.0002f, m1, fmaf(5e-5f, am_min(S, fmaf(3.f, x2, 2.f * d0)), 1e-6f)), 0.f);
}
__device__ __forceinline__ float cells_limit(float m1, float x2, float S) {
  const float d2 = cells_bound(m1, x2, S);
  const float near = 2.f * x2 + d2 + 2.f * __builtin_amdgcn_sqrtf(x2 * d2);
  return m1 + (2.1f * (am_min(near, S) * 9e-6f + 7e-7f) + 6.6e-5f * fabsf(m1));
}

// LDS bytes: operands, their centroids' numbers, boxes; before that (tokens and centroids being ordered) the histogram and the token list.
__host__ __device__ constexpr size_t cells_lds(int c, int dbar) {
  const size_t pad = (size_t)(c + 31) / 32 * 32, need = pad * 4 * dbar + pad * 2 + pad / 32 * 4 * dbar;
  return need > kCellBins * 8 + kCellTokens * 2 ? need : kCellBins * 8 + kCellTokens * 2;
}

template <int DBAR>
__global__ __launch_bounds__(1024) void vq_assign_cells_kernel(int g, int c, int n_kv_heads, int rows, int64_t cap,
                                                                const float* __restrict__ centroids,
                                                                uint16_t* __restrict__ pcache,
                                                                const uint16_t* __restrict__ k_new, int64_t T, int chunk,
                                                                NRes nr, float* __restrict__ acc, int32_t* __restrict__ pos_out,
                                                                NRes vrow0) {
  constexpr int H = DBAR / 2;                                // dwords of a token's channels
  constexpr int kTokPer = kCellTokens / 1024, kCenPer = 8, kBlkPer = 4;
  typedef uint32_t op_t __attribute__((ext_vector_type(DBAR)));        // hi pairs, then pairs of twice the rest
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ float s_stat[2 * DBAR];
  constexpr uint32_t kQueue = 512;
  __shared__ uint32_t s_cmax, s_done, s_queued;
  __shared__ uint16_t s_queue[kQueue];
  __shared__ uint32_t s_wave[16];
  __shared__ uint8_t s_ids[16 * 256 + 32];                   // each wave's list of blocks (stale entries are blocks too)
  // workgroup x serves row x % rows: with eight rows all groups of a row, which share its tokens' lines, run on one die
  const int row = blockIdx.x % rows, rest = blockIdx.x / rows;
  const int grp = rest % g;
  const int64_t first = (int64_t)(rest / g) * chunk;
  const int n = (int)(T - first < chunk ? T - first : chunk);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int col = lane & 31, kb = lane >> 5;
  const int b = row / n_kv_heads;
  const float* cg = centroids + ((int64_t)(row % n_kv_heads) * g + grp) * c * DBAR;
  const uint16_t* keys = k_new + ((int64_t)row * T + first) * kHeadDim + grp * DBAR;
  const int cpad = (c + 31) & ~31, nblk = cpad >> 5;
  op_t* s_op = reinterpret_cast<op_t*>(lds_raw);
  uint16_t* s_perm = reinterpret_cast<uint16_t*>(lds_raw + (size_t)cpad * sizeof(op_t));
  op_t* s_box = reinterpret_cast<op_t*>(lds_raw + (size_t)cpad * (sizeof(op_t) + 2));    // lower corner, upper corner
  uint32_t* hist = reinterpret_cast<uint32_t*>(lds_raw);
  uint16_t* s_list = reinterpret_cast<uint16_t*>(lds_raw + kCellBins * 8);
  const int64_t slot0 = nr.n[b] + first;
  if (grp == 0) {
    for (int t = tid; t < n; t += 1024) {
      if (acc != nullptr) acc[(int64_t)row * cap + slot0 + t] = 0.0f;
      if (pos_out != nullptr) pos_out[(int64_t)row * cap + slot0 + t] = (int32_t)(vrow0.n[b] + first + t);
    }
  }
  if (tid == 0) { s_cmax = 0; s_done = 0; s_queued = 0; }
  for (int i = tid; i < 16 * 256 + 32; i += 1024) s_ids[i] = 0;
  // the codebook's lines are asked for while the tokens are put in order
  const float warm = cg[(size_t)tid * 32 < (size_t)c * DBAR ? tid * 32 : 0];
  auto words_of = [&](int t, uint32_t (&xw)[H]) {
    const uint16_t* src = keys + (int64_t)t * kHeadDim;
#pragma unroll
    for (int d = 0; d < H; ++d) xw[d] = (uint32_t)src[2 * d] | (uint32_t)src[2 * d + 1] << 16;
  };

  // the tokens' order: this wave takes the 32-token tiles tile_of(0), tile_of(1), ...; lane (col, kb) keeps the tokens of column col of
  // its tiles 4 j + kb (low half of lst[j]) and 4 j + 2 + kb
  const int tiles = (n + 31) >> 5, mine = (tiles + 15) >> 4;
  auto tile_of = [&](int k) { return 16 * k + ((w + 5 * k) & 15); };
  uint32_t lst[8];
  {
    uint32_t xw[kTokPer][H];
    int pos[kTokPer];
#pragma unroll
    for (int i = 0; i < kTokPer; ++i)
      words_of(i * 1024 + tid < n ? i * 1024 + tid : n - 1, xw[i]);
    float mu[DBAR], sd[DBAR];
    auto value = [&](int i, int d) { return h2f((xw[i][d >> 1] >> (16 * (d & 1))) & 0xffffu); };
    cells_moments<kTokPer, DBAR>(value, n, mu, sd, s_stat);
    cells_order<kTokPer, DBAR>(value, n, mu, sd, hist, s_wave, pos);
#pragma unroll
    for (int i = 0; i < kTokPer; ++i)
      if (i * 1024 + tid < n) s_list[pos[i]] = (uint16_t)(i * 1024 + tid);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      lst[j] = 0;
      if (4 * j < mine) {
        const int p0 = tile_of(4 * j + kb) * 32 + col, p1 = tile_of(4 * j + 2 + kb) * 32 + col;
        lst[j] = (uint32_t)s_list[p0 < n ? p0 : n - 1] | (uint32_t)s_list[p1 < n ? p1 : n - 1] << 16;
      }
    }
    __syncthreads();
  }
  asm volatile("" ::"v"(warm));
  {
    float cv[kCenPer][DBAR];
    int pos[kCenPer];
    float most = 0.f;
#pragma unroll
    for (int i = 0; i < kCenPer; ++i) {
      const int ci = i * 1024 + tid < c ? i * 1024 + tid : c - 1;
      float nn = 0.f;
#pragma unroll
      for (int d = 0; d < DBAR; ++d) { cv[i][d] = cg[(int64_t)ci * DBAR + d]; nn = fmaf(cv[i][d], cv[i][d], nn); }
      most = nn < INFINITY ? fmaxf(most, nn) : INFINITY;     // not finite or not a number: no token is in range
    }
    most = wave_max_nonneg(most);
    if (lane == 0) atomicMax(&s_cmax, __float_as_uint(most));
    float mu[DBAR], sd[DBAR];
    auto value = [&](int i, int d) { return cv[i][d]; };
    cells_moments<kCenPer, DBAR>(value, c, mu, sd, s_stat);
    cells_order<kCenPer, DBAR>(value, c, mu, sd, hist, s_wave, pos);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kCenPer; ++i) {
      if (i * 1024 + tid < c) {
        op_t o;
#pragma unroll
        for (int d = 0; d < H; ++d) {
          const _Float16 h0 = am_f16(cv[i][2 * d]), h1 = am_f16(cv[i][2 * d + 1]);
          o[d] = cells_bits(v2h{h0, h1});
          o[H + d] = cells_bits(v2h{am_f16(2.f * (cv[i][2 * d] - (float)h0)), am_f16(2.f * (cv[i][2 * d + 1] - (float)h1))});
        }
        const int last = pos[i] == c - 1 ? cpad : pos[i] + 1;          // the last one also fills up its block
        for (int p = pos[i]; p < last; ++p) {
          s_op[p] = o;
          s_perm[p] = (uint16_t)(i * 1024 + tid);
        }
      }
    }
    __syncthreads();
  }
  // the two halves of a channel as one number (2^-21.6 of it off the centroid)
  auto channel = [&](const op_t& o, int d) {
    const v2h hi = cells_pair(o[d >> 1]), lo = cells_pair(o[H + (d >> 1)]);
    return fmaf((float)lo[d & 1], 0.5f, (float)hi[d & 1]);
  };
  for (int blk = 2 * w + kb; blk < nblk + (nblk & 1); blk += 32) {
    const op_t o = s_op[(blk < nblk ? blk : nblk - 1) * 32 + col];
    op_t box;
#pragma unroll
    for (int d = 0; d < H; ++d) {
      v2h lo, hi;
#pragma unroll
      for (int e = 0; e < 2; ++e) {                          // corners rounded outwards: 2^-10 covers fp16 and the halves
        const float v = channel(o, 2 * d + e), slack = fmaf(fabsf(v), 9.765625e-4f, 9.5367431640625e-7f);
        lo[e] = am_f16(v - slack);
        hi[e] = am_f16(v + slack);
      }
      box[d] = cells_over_half(cells_bits(lo), [](uint32_t a, uint32_t z) { return cells_bits(cells_min(cells_pair(a), cells_pair(z))); });
      box[H + d] = cells_over_half(cells_bits(hi), [](uint32_t a, uint32_t z) { return cells_bits(cells_max(cells_pair(a), cells_pair(z))); });
    }
    if (col == 0 && blk < nblk) s_box[blk] = box;
  }
  __syncthreads();
  const float cmax2 = __uint_as_float(s_cmax);
  // squared distance between [alo, ahi] and a box, per channel pair in fp16
  const v2h zero2 = {(_Float16)0.f, (_Float16)0.f};
  auto gap2 = [&](const uint32_t (&alo)[H], const uint32_t (&ahi)[H], const op_t& box) {
    float s = 0.f;
#pragma unroll
    for (int d = 0; d < H; ++d) {
      const v2h q = cells_max(cells_max(cells_pair(box[d]) - cells_pair(ahi[d]), cells_pair(alo[d]) - cells_pair(box[H + d])), zero2);
      s = __builtin_amdgcn_fdot2(q, q, s, false);
    }
    return s;
  };
  op_t mybox[kBlkPer];                                       // of blocks lane, lane + 64, ...
#pragma unroll
  for (int i = 0; i < kBlkPer; ++i) mybox[i] = s_box[lane + 64 * i < nblk ? lane + 64 * i : nblk - 1];
  const v2h kS = kb ? v2h{(_Float16)0.5f, (_Float16)0.5f} : zero2, kO = kb ? zero2 : v2h{(_Float16)1.f, (_Float16)1.f};
  uint32_t number = 255;
  asm volatile("" : "+v"(number));
  float minus = -1.f;                                        // (opaque: fma with fp16 operands, one instruction, and no conversion and subtraction)
  asm volatile("" : "+s"(minus));
  uint32_t turn[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) turn[j] = (uint32_t)(j + col) & 3u;

  auto put = [&](int t, int win) { pcache[vq_wide_at(g, vq_tiles(cap), row, slot0 + t, grp)] = (uint16_t)win; };
  // the numbers of the blocks with lb in (low, high] into the wave's list, ascending; how many
  auto list = [&](const float (&lb)[kBlkPer], float low, float high) {
    int count = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int i = 0; i < kBlkPer; ++i) {
      const bool in_list = lb[i] > low && lb[i] <= high && lane + 64 * i < nblk;
      const uint64_t ball = __builtin_amdgcn_ballot_w64(in_list);
      const int at = count + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(ball >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ball, 0));
      if (in_list) s_ids[w * 256 + at] = (uint8_t)(lane + 64 * i);
      count += (int)__builtin_popcountll(ball);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return count;
  };
  // The exact chain over every centroid that can win, by the whole wave: those of the nearest block, then of the blocks
  // within the distance that this leaves.  Out of order in memory each costs a line of its own: of more blocks than an
  // eighth (two channels: a quarter) all centroids in their order, and for a token out of range, two such tokens at a time.
  // 8 x 16 Ki tokens that all end here, c = 8192, us, every centroid for one token at a time / this: 8 points 1024 times each
  // 17 300 / 14 300 (by blocks, 32 of them, 20 000), with two channels 29 100 / 13 400; 64 points 128 times 17 100 / 7700; all on one
  // line 9300 / 1760; 16 dense clusters 3710 / 2370.
  constexpr int kFew = DBAR == 4 ? 8 : 4;
  int waiting = -1;                                          // a token that waits for a second one
  auto in_order = [&](int t0, int t1) {
    const uint16_t* const src[2] = {keys + (int64_t)t0 * kHeadDim, keys + (int64_t)t1 * kHeadDim};
    int win[2];
    am_exhaustive_of<DBAR, 64, 2>(src, cg, c, lane, win);
    if (lane == 0) { put(t0, win[0]); put(t1, win[1]); }
  };
  auto settle = [&](int t) {
    uint32_t xw[H];
    words_of(t, xw);
    float x2 = 0.f, lb[kBlkPer], least = INFINITY;
#pragma unroll
    for (int d = 0; d < H; ++d) x2 = __builtin_amdgcn_fdot2(cells_pair(xw[d]), cells_pair(xw[d]), x2, false);
    bool by_blocks = x2 + cmax2 < 32768.f;
#pragma unroll
    for (int i = 0; i < kBlkPer; ++i) {
      lb[i] = by_blocks && lane + 64 * i < nblk ? gap2(xw, xw, mybox[i]) : INFINITY;
      least = am_min(least, lb[i]);
    }
    least = __uint_as_float(wave_min(__float_as_uint(least)));
    uint64_t key = kAmNoKey;
    float low = -1.f, high = least;
    for (int round = 0; round < 2 && by_blocks; ++round) {
      const int count = list(lb, low, high);
      if (count * kFew >= nblk) { by_blocks = false; break; }
      for (int from = 0; from < count; from += 8) {          // a block per half wave, four of each in flight
        int ci[4];
        float cv[4][DBAR];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int at = from + 2 * u + kb;
          ci[u] = s_perm[s_ids[w * 256 + (at < count ? at : count - 1)] * 32 + col];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int d = 0; d < DBAR; ++d) cv[u][d] = cg[(int64_t)ci[u] * DBAR + d];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float dist = 0.f;
#pragma unroll
          for (int d = 0; d < DBAR; ++d) {
            const float e = h2f((xw[d >> 1] >> (16 * (d & 1))) & 0xffffu) - cv[u][d];
            dist = fmaf(e, e, dist);
          }
          const uint64_t kk = am_key(dist, ci[u]);
          if (kk < key) key = kk;
        }
      }
      // a box further away than the best so far (1.002 and 1e-6: as for the tiles' boxes) holds no winner
      low = least;
      high = fmaf(1.002f, __uint_as_float(wave_min((uint32_t)(key >> 32))), 1e-6f);
    }
    if (!by_blocks) {
      if (waiting >= 0) in_order(waiting, t);
      waiting = waiting >= 0 ? -1 : t;
      return;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const uint64_t other = (uint64_t)__shfl_xor((uint32_t)(key >> 32), o) << 32 | __shfl_xor((uint32_t)key, o);
      if (other < key) key = other;
    }
    if (lane == 0) put(t, (int)(uint32_t)key);
  };
  auto token_of = [&](int k) {                               // of this column in tile k of the wave (4 j .. 4 j + 3: lst[0])
    const Halves h = halves_of(k & 2 ? lst[0] >> 16 : lst[0] & 0xffffu);
    return (int)(k & 1 ? h.hi : h.lo);
  };
  int tok = 0;
  uint32_t xw[H];
  if (mine > 0) {
    tok = token_of(0);
    words_of(tok, xw);
  }
  for (int k = 0; k < mine; ++k) {
    const int t = tok;
    uint32_t x01[H];
#pragma unroll
    for (int d = 0; d < H; ++d) x01[d] = xw[d];
    if (k + 1 < mine) {                                      // the next tile's channels
      if (((k + 1) & 3) == 0) {
#pragma unroll
        for (int j = 0; j < 7; ++j) lst[j] = lst[j + 1];
      }
      tok = token_of(k + 1);
      words_of(tok, xw);
    }
    const bool real = tile_of(k) * 32 + col < n;
    if (tile_of(k) >= tiles) continue;
    // waves behind the workgroup's average go first: left to the order of age, the last wave of a SIMD ends alone
    uint32_t done = 0;
    if (lane == 0) done = atomicAdd(&s_done, 1u);
    if (16u * (uint32_t)k < (uint32_t)__builtin_amdgcn_readfirstlane((int)done)) __builtin_amdgcn_s_setprio(2);
    else __builtin_amdgcn_s_setprio(0);
    float x2 = 0.f;
#pragma unroll
    for (int d = 0; d < H; ++d) x2 = __builtin_amdgcn_fdot2(cells_pair(x01[d]), cells_pair(x01[d]), x2, false);
    const float S = x2 + cmax2;
    const bool in = S < 32768.f;
    float m1 = INFINITY, m2 = INFINITY, m3 = INFINITY;
    if (__builtin_amdgcn_ballot_w64(in) != 0) {
      v8h bop;
      {
        const v2h one = {(_Float16)1.f, (_Float16)1.f};
        v2h r[4] = {zero2, zero2, zero2, zero2};
#pragma unroll
        for (int d = 0; d < H; ++d) {
          r[d] = kb ? one : -cells_pair(x01[d]);
          r[H + d] = kb ? one : cells_pair(x01[d]) * v2h{(_Float16)-0.5f, (_Float16)-0.5f};
        }
        bop = v8h{r[0][0], r[0][1], r[1][0], r[1][1], r[2][0], r[2][1], r[3][0], r[3][1]};
      }
      const float hx = 0.5f * x2;
      const v16f start = {hx, hx, hx, hx, hx, hx, hx, hx, hx, hx, hx, hx, hx, hx, hx, hx};
      auto multiply = [&](const op_t& o, int blk) {
        v2h r[4] = {zero2, zero2, zero2, zero2};
#pragma unroll
        for (int d = 0; d < H; ++d) {                        // k block 0: hi, 2 lo; k block 1: hi^2 / 2 in two pieces, with hi lo
          const v2h hi = cells_pair(o[d]), lo = cells_pair(o[H + d]);
          const v2h m = __builtin_elementwise_fma(hi, kS, kO);
          r[d] = hi * m;
          r[H + d] = __builtin_elementwise_fma(lo, m, __builtin_elementwise_fma(hi, m, -r[d]));
        }
        const v8h a = {r[0][0], r[0][1], r[1][0], r[1][1], r[2][0], r[2][1], r[3][0], r[3][1]};
        const v16f d = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bop, start, 0, 0, 0);
        float mm = am_min(d[14], d[15]);
#pragma unroll
        for (int j = 0; j < 14; j += 2) mm = am_min(am_min(mm, d[j]), d[j + 1]);
        const float pk = am_number(mm, (uint32_t)blk, number);
        m3 = __builtin_amdgcn_fmed3f(m2, m3, pk);
        m2 = __builtin_amdgcn_fmed3f(m1, m2, pk);
        m1 = am_min(m1, pk);
      };
      // blocks of this wave's list, from number `from` on, whose bits in `which` are set; each operand is read while the one
      // before it is multiplied
      const uint8_t* ids = s_ids + w * 256;
      auto multiply_all = [&](int from, uint32_t which) {
        const int mine = ids[from + (lane & 31)];
        int blk = __builtin_amdgcn_readlane(mine, __builtin_ctz(which));
        op_t o = s_op[blk * 32 + col];
        for (;;) {
          which &= which - 1;
          const int after = which != 0 ? __builtin_amdgcn_readlane(mine, __builtin_ctz(which)) : blk;
          const op_t next = s_op[after * 32 + col];
          multiply(o, blk);
          if (which == 0) break;
          o = next;
          blk = after;
        }
      };
      // the tile's box, over the tokens in range
      uint32_t tlo[H], thi[H];
      float lb[kBlkPer];
#pragma unroll
      for (int d = 0; d < H; ++d) {
        tlo[d] = cells_over_half(in ? x01[d] : 0x7bff7bffu, [](uint32_t a, uint32_t z) { return cells_bits(cells_min(cells_pair(a), cells_pair(z))); });
        thi[d] = cells_over_half(in ? x01[d] : 0xfbfffbffu, [](uint32_t a, uint32_t z) { return cells_bits(cells_max(cells_pair(a), cells_pair(z))); });
      }
#pragma unroll
      for (int i = 0; i < kBlkPer; ++i) lb[i] = gap2(tlo, thi, mybox[i]);
      if (nblk <= 192) lb[3] = INFINITY;
      if (nblk <= 128) lb[2] = INFINITY;
      if (nblk <= 64) lb[1] = INFINITY;
      const float least = __uint_as_float(wave_min(__float_as_uint(am_min(am_min(lb[0], lb[1]), am_min(lb[2], lb[3])))));
      for (int count = list(lb, -1.f, least), from = 0; from < count; from += 32)
        multiply_all(from, count - from >= 32 ? ~0u : (1u << (count - from)) - 1u);
      // twice: the blocks within half the distance of the worst token's bound, and, with that bound lowered by them, the others.
      // Sixteen blocks are tested at a time, two per product of boxes and tokens
      float low = least;
      for (int round = 0; round < 2; ++round) {
        float d2;
        auto bound = [&]() {
          const Halves h = halves_of(__float_as_uint(m1));
          d2 = in ? 1.002f * cells_bound(am_min(__uint_as_float(h.lo), __uint_as_float(h.hi)), x2, S) : 0.f;
        };
        bound();
        const float high = __uint_as_float(wave_max(__float_as_uint(d2))) * (round == 0 ? 0.25f : 1.f);
        const int count = list(lb, low, high);
        low = am_max(low, high);
        for (int from = 0; from < count; from += 16) {
          const int left = count - from;
          uint32_t hits = 0;
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            if (8 * half >= left) continue;
            op_t box[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) box[u] = s_box[ids[from + 8 * half + 2 * u + kb]];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const uint64_t hit = __builtin_amdgcn_ballot_w64(gap2(x01, x01, box[u]) <= d2);
              hits |= ((uint32_t)hit != 0 ? 1u : 0u) << (8 * half + 2 * u) | ((hit >> 32) != 0 ? 2u : 0u) << (8 * half + 2 * u);
            }
          }
          if (left < 16) hits &= (1u << left) - 1u;
          if (hits != 0) {
            multiply_all(from, hits);
            bound();
          }
        }
      }
    }

    // candidates as in vq_assign_mfma_kernel: the smallest of each half, then the second smallest
    const Halves a1 = halves_of(__float_as_uint(m1)), a2 = halves_of(__float_as_uint(m2)), a3 = halves_of(__float_as_uint(m3));
    const float lim = cells_limit(am_min(__uint_as_float(a1.lo), __uint_as_float(a1.hi)), x2, S);
    const uint32_t blocks = (a1.lo & 255u) | (a1.hi & 255u) << 8 | (a2.lo & 255u) << 16 | a2.hi << 24;
    auto below = [&](uint32_t v) { return __uint_as_float(v) <= lim ? 1u : 0u; };
    const bool queue = real && (!in || below(a3.lo) != 0 || below(a3.hi) != 0);
    const uint32_t mask = queue || !real ? 0u : below(a1.lo) | below(a1.hi) << 1 | below(a2.lo) << 2 | below(a2.hi) << 3;
    float bd = INFINITY, sd = INFINITY, xf[DBAR];
#pragma unroll
    for (int d = 0; d < DBAR; ++d) xf[d] = h2f((x01[d >> 1] >> (16 * (d & 1))) & 0xffffu);
    uint32_t bp = 0;
    // rows of a 32 x 32 result held by a half: 8 (j / 4) + 4 half + j % 4, j < 16; this lane takes j = 8 kb .. (each
    // lane begins with another one of four neighbours: they are on different banks)
    auto place = [&](uint32_t which) { return ((blocks >> (8 * which)) & 255u) * 32 + 16 * kb + 4 * (which & 1u); };
    for (uint32_t left = mask; __builtin_amdgcn_ballot_w64(left != 0) != 0;) {
      if (left != 0) {
        const uint32_t which = (uint32_t)__builtin_ctz(left), base = place(which);
        left &= left - 1;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const op_t o = s_op[base + turn[j & 3] + 8 * (j >> 2)];
          float dist = 0.f;
#pragma unroll
          for (int d = 0; d < DBAR; ++d) {
            const v2h hi = cells_pair(o[d >> 1]), lo = cells_pair(o[H + (d >> 1)]);
            const float e = fmaf((float)lo[d & 1], -0.5f, fmaf((float)hi[d & 1], minus, xf[d]));
            dist = fmaf(e, e, dist);
          }
          sd = __builtin_amdgcn_fmed3f(bd, sd, dist);
          bp = dist < bd ? which * 8 + j : bp;
          bd = am_min(bd, dist);
        }
      }
    }
    bp = place(bp >> 3) + ((bp + col) & 3u) + 2 * (bp & 4u);
    const Halves hb = halves_of(__float_as_uint(bd)), hs = halves_of(__float_as_uint(sd)), hp = halves_of(bp);
    const float b0 = __uint_as_float(hb.lo), b1 = __uint_as_float(hb.hi), best = am_min(b0, b1);
    const float next = am_min(am_max(b0, b1), am_min(__uint_as_float(hs.lo), __uint_as_float(hs.hi)));
    int win = s_perm[b1 < b0 ? hp.hi : hp.lo];
    // what that leaves undecided: the halves are 2^-20.9 |c| off the centroid, and this chain and the exact one 2^-22 of the result
    // off theirs: with r the distance, r^2 is off by less than 2^-21 r^2 + 2^-19.9 r (|x| + r) + 2^-23 r
    const float ax = __builtin_amdgcn_sqrtf(x2), r = __builtin_amdgcn_sqrtf(best) + fmaf(ax, 9.5367431640625e-7f, 5.9604644775390625e-8f);
    const bool close = mask != 0 && !(next - best > r * fmaf(ax, 2.9e-6f, fmaf(r, 5e-6f, 6e-7f)));
    if (__builtin_amdgcn_ballot_w64(close) != 0) {
      uint64_t key = kAmNoKey;
      for (uint32_t left = close ? mask : 0u; __builtin_amdgcn_ballot_w64(left != 0) != 0;) {
        if (left != 0) {
          const uint32_t base = place((uint32_t)__builtin_ctz(left));
          left &= left - 1;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int ci = s_perm[base + (j & 3) + 8 * (j >> 2)];
            float dist = 0.f;
#pragma unroll
            for (int d = 0; d < DBAR; ++d) {
              const float e = xf[d] - cg[(int64_t)ci * DBAR + d];
              dist = fmaf(e, e, dist);
            }
            const uint64_t kk = am_key(dist, ci);
            if (kk < key) key = kk;
          }
        }
      }
      const Halves kh = halves_of((uint32_t)(key >> 32)), kl = halves_of((uint32_t)key);
      const uint64_t k0 = (uint64_t)kh.lo << 32 | kl.lo, k1 = (uint64_t)kh.hi << 32 | kl.hi;
      if (close) win = (int)(uint32_t)(k0 < k1 ? k0 : k1);
    }
    if (kb == 0 && real && !queue) put(t, win);
    // the others: at the end, shared by all waves, as far as the queue has room
    uint32_t place_in_queue = kQueue;
    if (queue && kb == 0) {
      place_in_queue = atomicAdd(&s_queued, 1u);
      if (place_in_queue < kQueue) s_queue[place_in_queue] = (uint16_t)t;
    }
    for (uint64_t left = __builtin_amdgcn_ballot_w64(queue && kb == 0 && place_in_queue >= kQueue); left != 0; left &= left - 1)
      settle(__builtin_amdgcn_readlane(t, (int)__builtin_ctzll(left)));
  }
  __syncthreads();
  const int queued = s_queued < kQueue ? (int)s_queued : (int)kQueue;
  for (int e = w; e < queued; e += 16) settle(s_queue[e]);
  if (waiting >= 0) in_order(waiting, waiting);
}

// Few tokens per call (decode appends): one workgroup of four waves per (token, row, 4 / SPLIT groups).  SPLIT waves
// share a group, each takes a part of its centroids and spreads it over its lanes (lane, lane + 64, ...; four distances
// in flight per lane); the lanes' candidates, then the waves', are reduced by (distance, index): the smaller distance
// wins, equal distances go to the lower index - the same winner as the ascending scan with a strict comparison.
// Bound by the latency of a lane's chain of loads: with all four waves on one group the append of one token x 8 KV heads takes 8 us at 8192
// centroids instead of 25.
template <int DBAR, bool WIDE, int SPLIT>
__global__ __launch_bounds__(256) void vq_assign_small_kernel(int g, int c, int n_kv_heads, int64_t cap,
                                                              const float* __restrict__ centroids,
                                                              uint8_t* __restrict__ pcache,
                                                              const uint16_t* __restrict__ k_new, int64_t T, NRes nr,
                                                              float* __restrict__ acc, int32_t* __restrict__ pos,
                                                              NRes vrow0) {
  __shared__ float s_d[4];
  __shared__ int s_i[4];
  const int row = blockIdx.y;
  const int64_t tt = blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int b = row / n_kv_heads;
  const int64_t slot = nr.n[b] + tt;
  const uint16_t* src = k_new + ((int64_t)row * T + tt) * kHeadDim;
  const float* cb = centroids + (int64_t)(row % n_kv_heads) * g * c * DBAR;
  const int i = blockIdx.z * (4 / SPLIT) + w / SPLIT;
  float x[DBAR];
#pragma unroll
  for (int dd = 0; dd < DBAR; ++dd) x[dd] = h2f(src[i * DBAR + dd]);
  float bd = INFINITY;
  int best = 0x7fffffff;
  for (int c0 = 256 * (w % SPLIT) + lane; c0 < c; c0 += 256 * SPLIT) {
    float cv[4][DBAR];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int cc = c0 + 64 * u < c ? c0 + 64 * u : c0;
      const float* p = cb + ((int64_t)i * c + cc) * DBAR;
#pragma unroll
      for (int dd = 0; dd < DBAR; ++dd) cv[u][dd] = p[dd];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int cc = c0 + 64 * u;
      if (cc < c) {
        float d = 0.f;
#pragma unroll
        for (int dd = 0; dd < DBAR; ++dd) {
          const float e = x[dd] - cv[u][dd];
          d = fmaf(e, e, d);
        }
        if (d < bd || best == 0x7fffffff) { bd = d; best = cc; }
      }
    }
  }
  auto take = [&](float od, int ob) {
    if (ob != 0x7fffffff && (best == 0x7fffffff || od < bd || (od == bd && ob < best))) { bd = od; best = ob; }
  };
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) take(__shfl_xor(bd, o), __shfl_xor(best, o));
  if constexpr (SPLIT > 1) {
    if (lane == 0) { s_d[w] = bd; s_i[w] = best; }
    __syncthreads();
    if (w % SPLIT == 0)
      for (int y = 1; y < SPLIT; ++y) take(s_d[w + y], s_i[w + y]);
  }
  if (lane == 0 && w % SPLIT == 0) {
    if constexpr (WIDE) reinterpret_cast<uint16_t*>(pcache)[vq_wide_at(g, vq_tiles(cap), row, slot, i)] = (uint16_t)best;
    else pcache[((int64_t)row * cap + slot) * g + vq_byte_of(i, slot)] = (uint8_t)best;
  }
  if (threadIdx.x == 0 && blockIdx.z == 0) {
    if (acc != nullptr) acc[(int64_t)row * cap + slot] = 0.0f;
    if (pos != nullptr) pos[(int64_t)row * cap + slot] = (int32_t)(vrow0.n[b] + tt);
  }
}

// -------------------------------------------------------------------------------- table ---
// T[row][cc][i][h] (narrow form; T[row][i][cc][h] in the wide form) = qbar_i . C[i][cc] for the G query heads of the row: t = 0; t = fmaf(q, c, t) over
// the group's channels in ascending order.  grid (g, rows), centroids spread over the threads.  The workgroup also
// leaves the largest magnitude of its group's entries, per head, in amax[row][i][4] for the scan.
// PER: centroids in flight per thread.  8 rows, c = 8192, one -> eight: 15.3 -> 12.2 us; a codebook of at most 256 has one per
// thread and wants the registers for more workgroups (128 rows, c = 64, the call that fills the table and scans 100 slots:
// 14.0 us with eight, 13.0 with one).
template <int G, int DBAR, int PER>
__global__ __launch_bounds__(256) void vq_lut_kernel(int g, int c, int n_kv_heads, bool wide,
                                                     const float* __restrict__ centroids,
                                                     const uint16_t* __restrict__ q, float* __restrict__ lut,
                                                     float* __restrict__ amax) {
  __shared__ float wmax[4][4];
  const int i = blockIdx.x, row = blockIdx.y;
  float m[G];
#pragma unroll
  for (int h = 0; h < G; ++h) m[h] = 0.f;
  float qv[G][DBAR];
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int dd = 0; dd < DBAR; ++dd) qv[h][dd] = h2f(q[((int64_t)row * G + h) * kHeadDim + i * DBAR + dd]);
  const float* cb = centroids + ((int64_t)(row % n_kv_heads) * g + i) * c * DBAR;
  for (int c0 = threadIdx.x; c0 < c; c0 += PER * 256) {
    float cv[PER][DBAR];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
#pragma unroll
      for (int dd = 0; dd < DBAR; ++dd) cv[u][dd] = cb[(int64_t)(c0 + 256 * u < c ? c0 + 256 * u : c0) * DBAR + dd];
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int cc = c0 + 256 * u;
      if (cc >= c) break;
      float* out = lut + (wide ? ((int64_t)row * g + i) * c + cc : ((int64_t)row * c + cc) * g + i) * G;
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float t = 0.f;
#pragma unroll
        for (int dd = 0; dd < DBAR; ++dd) t = fmaf(qv[h][dd], cv[u][dd], t);
        out[h] = t;
        m[h] = fmaxf(m[h], fabsf(t));
      }
    }
  }
#pragma unroll
  for (int h = 0; h < G; ++h) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m[h] = fmaxf(m[h], __shfl_xor(m[h], o));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6][h] = m[h];
  }
  __syncthreads();
  if (threadIdx.x < G)
    amax[((int64_t)row * g + i) * 4 + threadIdx.x] = fmaxf(fmaxf(wmax[0][threadIdx.x], wmax[1][threadIdx.x]),
                                                           fmaxf(wmax[2][threadIdx.x], wmax[3][threadIdx.x]));
}

// --------------------------------------------------------------------------------- scan ---
template <int G> struct EntryT;
template <> struct EntryT<4> { using type = float4; using fix = int4; };
template <> struct EntryT<2> { using type = float2; using fix = int2; };
template <> struct EntryT<1> { using type = float; using fix = int; };

template <int G>
__device__ __forceinline__ typename EntryT<G>::fix entry_fix(const typename EntryT<G>::type& e, const int* s) {
  typename EntryT<G>::fix r;
  if constexpr (G == 4) {
    r.x = vq_fix(e.x, s[0]); r.y = vq_fix(e.y, s[1]); r.z = vq_fix(e.z, s[2]); r.w = vq_fix(e.w, s[3]);
  } else if constexpr (G == 2) {
    r.x = vq_fix(e.x, s[0]); r.y = vq_fix(e.y, s[1]);
  } else {
    r = vq_fix(e, s[0]);
  }
  return r;
}
template <int G>
__device__ __forceinline__ void entry_add2(int (&z)[G], const typename EntryT<G>::fix& a,
                                           const typename EntryT<G>::fix& b) {
  if constexpr (G == 4) {
    z[0] = z[0] + a.x + b.x; z[1] = z[1] + a.y + b.y; z[2] = z[2] + a.z + b.z; z[3] = z[3] + a.w + b.w;
  } else if constexpr (G == 2) {
    z[0] = z[0] + a.x + b.x; z[1] = z[1] + a.y + b.y;
  } else {
    z[0] = z[0] + a + b;
  }
}

// Eq. 3.  One workgroup of 1024 threads reduces the per-group maxima to the largest magnitude of each
// query head's table and copies the row's table (c * g entries of G floats) into LDS on that head's
// power-of-two grid (24 bits for the largest entry, vq_fix).  Then each thread scores one
// token at a time: NG index bytes (two or four 16-byte loads; a wave reads 64 consecutive tokens = 2 or
// 4 KiB in one piece, the next token's bytes are on their way while this one's are looked up), NG table
// reads, an exact integer sum - so the order of the additions is free and two entries go into one
// three-operand add - and one conversion back to fp32.  With the largest supported table (128 KiB) one
// workgroup fits a compute unit, so the launch has about one workgroup per unit and each takes an
// equal share of the row.  Shares start at multiples of 1024 slots: a thread's tokens all have its own
// lane number modulo 16, which makes the rotation of the index bytes a per-thread constant.
template <int G, int NG>
__global__ __launch_bounds__(1024) void vq_scan_kernel(int c, int64_t cap, const uint8_t* __restrict__ pcache,
                                                       float* __restrict__ lut, NRes nr, int n_kv_heads,
                                                       int64_t per_wg, float* __restrict__ sel, float* __restrict__ z_out) {
  using E = typename EntryT<G>::type;
  using F = typename EntryT<G>::fix;
  constexpr int ES = 4 * G;                              // bytes per table entry
  constexpr int kAhead = 1;                              // tokens whose index bytes are in flight per thread (deeper: slower)
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ int sexp[4];
  const int row = blockIdx.y;
  const int64_t n = nr.n[row / n_kv_heads];
  const int64_t j0 = (int64_t)blockIdx.x * per_wg;
  if (j0 >= n) return;
  int64_t j1 = j0 + per_wg;
  if (j1 > n) j1 = n;
  const uint8_t* prow = pcache + (int64_t)row * cap * NG;
  int64_t j = j0 + threadIdx.x;
  uint4 nx[kAhead][NG / 16];                             // the index bytes of this thread's next kAhead tokens
#pragma unroll
  for (int d = 0; d < kAhead; ++d)
    if (j + 1024 * d < j1) {
#pragma unroll
      for (int v = 0; v < NG / 16; ++v) nx[d][v] = reinterpret_cast<const uint4*>(prow + (j + 1024 * d) * NG)[v];
    }
  {
    // exponents of the heads' grids from the per-group maxima the table kernel left behind the table
    float* tail = lut + (int64_t)gridDim.y * NG * c * G;
    if (threadIdx.x < 64) {
      const float* am = tail + (int64_t)row * NG * 4;
      const int h = threadIdx.x & 3, part = threadIdx.x >> 2;          // 16 lanes per head
      float m = 0.f;
      if (h < G)
        for (int i = part; i < NG; i += 16) m = fmaxf(m, am[i * 4 + h]);
#pragma unroll
      for (int o = 32; o >= 4; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
      if (threadIdx.x < G) {
        const int s = vq_grid_exponent(m);
        sexp[threadIdx.x] = s;
        if (blockIdx.x == 0)                             // kept for the attend kernels
          reinterpret_cast<int32_t*>(tail + (int64_t)gridDim.y * NG * 4)[row * 4 + threadIdx.x] = s;
      }
    }
    __syncthreads();
    int s[G];
#pragma unroll
    for (int h = 0; h < G; ++h) s[h] = sexp[h];
    const E* src = reinterpret_cast<const E*>(lut) + (int64_t)row * NG * c;
    F* tabi = reinterpret_cast<F*>(lds_raw);
    for (int i = threadIdx.x; i < NG * c; i += 1024) tabi[i] = entry_fix<G>(src[i], s);
    __syncthreads();
  }
  int sx[G];
#pragma unroll
  for (int h = 0; h < G; ++h) sx[h] = -sexp[h];
  const uint32_t l16 = threadIdx.x & 15u;
  uint32_t off[16];
#pragma unroll
  for (int b = 0; b < 16; ++b) off[b] = ((b + l16) & 15u) * ES;
  for (; j < j1; j += 1024 * kAhead) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
      const int64_t jj = j + 1024 * d;
      if (jj >= j1) break;
      uint4 pw[NG / 16];
#pragma unroll
      for (int v = 0; v < NG / 16; ++v) pw[v] = nx[d][v];
      if (jj + 1024 * kAhead < j1) {
#pragma unroll
        for (int v = 0; v < NG / 16; ++v)
          nx[d][v] = reinterpret_cast<const uint4*>(prow + (jj + 1024 * kAhead) * NG)[v];
      }
      int zi[G];
#pragma unroll
      for (int h = 0; h < G; ++h) zi[h] = 0;
#pragma unroll
      for (int v = 0; v < NG / 16; ++v) {
        const uint32_t wd[4] = {pw[v].x, pw[v].y, pw[v].z, pw[v].w};
        F e[16];                                         // sixteen table reads in flight
#pragma unroll
        for (int b = 0; b < 16; ++b) {
          const uint32_t code = (wd[b >> 2] >> (8 * (b & 3))) & 255u;
          e[b] = *reinterpret_cast<const F*>(lds_raw + code * (NG * ES) + off[b] + 16 * v * ES);
        }
#pragma unroll
        for (int b = 0; b < 16; b += 2) entry_add2<G>(zi, e[b], e[b + 1]);
      }
      float z[G];
#pragma unroll
      for (int h = 0; h < G; ++h) z[h] = ldexpf((float)zi[h], sx[h]);
      float best = z[0];
#pragma unroll
      for (int h = 1; h < G; ++h) best = fmaxf(best, z[h]);
      sel[(int64_t)row * cap + jj] = best;
      if (z_out != nullptr) {
#pragma unroll
        for (int h = 0; h < G; ++h) z_out[((int64_t)row * G + h) * cap + jj] = z[h];
      }
    }
  }
}

// The grid exponents of a row's heads from the table's per-group maxima, into sexp and, by one workgroup, behind the maxima.
template <int G>
__device__ __forceinline__ void vq_row_exponents(float* __restrict__ lut, int g, int c, int rows, int row, bool writer,
                                                 int* sexp) {
  float* tail = lut + (int64_t)rows * g * c * G;
  if (threadIdx.x < 64) {
    const float* am = tail + (int64_t)row * g * 4;
    const int h = threadIdx.x & 3, part = threadIdx.x >> 2;
    float m = 0.f;
    if (h < G)
      for (int i = part; i < g; i += 16) m = fmaxf(m, am[i * 4 + h]);
#pragma unroll
    for (int o = 32; o >= 4; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if (threadIdx.x < G) {
      const int s = vq_grid_exponent(m);
      sexp[threadIdx.x] = s;
      if (writer) reinterpret_cast<int32_t*>(tail + (int64_t)rows * g * 4)[row * 4 + threadIdx.x] = s;
    }
  }
}

// Eq. 3 for the wide form (16-bit indices, a table larger than LDS).  One workgroup of 1024 threads scans a share
// of up to NQ * 4096 slots, per thread NQ quads of consecutive slots with their running integer sums in registers,
// and walks through the groups a slice at a time: gps groups whose entries (gps * c * G * 4 bytes <= 128 KiB) are
// copied from the group-major table into LDS on their heads' grids, then looked up with the share's indices of
// those groups.  The table is re-read once per share: full lines from L2, instead of one L2 request per token and
// group.
// Bound by the refills and the lookups, which take turns.  So the shares are equal and as many as compute units (8 rows x
// 300 Ki slots, c = 8192, entries on the grid at the refill: 157 us with a tile of 16 Ki slots per workgroup, 152 of
// them, 118 with 256 shares), and there a thread asks for its whole part of a slice, eight 16-byte entries, when it has
// finished its own lookups and before it waits for the others' (99 us; asked for before the lookups, 118: the indices
// queue behind it).
// RAW: the slice as it lies in memory, straight into LDS, and on the heads' grids at every lookup - where there are not many
// more lookups than entries (scan_wide_launch).  What is left of a slice then: 1.2 us of refill, and the lookups, whose
// vector instructions (18 of each with four heads, 7 without RAW) take as long as a share has slots: at that size, 93 us in
// the kernel, the vector ALU issues in 49 % of the clocks, LDS is busy in 28 % (two thirds of it bank conflicts).
template <int G, int NQ, bool RAW>
__global__ __launch_bounds__(1024) void vq_scan_wide_kernel(int g, int c, int gps, int64_t cap, int64_t per_wg,
                                                             const uint16_t* __restrict__ pcache,
                                                             float* __restrict__ lut, NRes nr, int n_kv_heads, int rows,
                                                             float* __restrict__ sel, float* __restrict__ z_out) {
  using E = typename EntryT<G>::type;
  using F = typename EntryT<G>::fix;
  constexpr int kPer = 128 / (int)sizeof(E);              // entries of a slice per thread,
  constexpr int kGo = NQ <= 3 ? kPer : kPer / 4;          // and how many of them are in flight: what the registers allow
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ int sexp[4];
  // workgroup x serves row x % rows: consecutive workgroups go to the eight dies in turn, so with eight rows
  // every row is scanned by one die and its table (4 MiB at c = 8192, four query heads) stays in that die's L2
  const int row = blockIdx.x % rows;
  const int64_t share = blockIdx.x / rows;
  const int64_t n = nr.n[row / n_kv_heads];
  const int64_t t0 = share * per_wg;
  if (t0 >= n) return;
  const int64_t t1 = t0 + per_wg < n ? t0 + per_wg : n;
  using T = typename std::conditional<RAW, E, F>::type;
  T* tab = reinterpret_cast<T*>(lds_raw);
  const E* trow = reinterpret_cast<const E*>(lut) + (int64_t)row * g * c;
  const int ne = gps * c;                                 // entries of a slice, at most 1024 * kPer
  E nt[RAW ? 1 : kGo];
  auto fetch = [&](int g0, int u0) {
    const E* src = trow + (int64_t)g0 * c;
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));                           // addresses formed here, not kept over the lookups
#pragma unroll
    for (int u = 0; u < kGo; ++u)
      if (1024 * (u0 + u) < ne) nt[u] = (src + 1024 * (u0 + u))[t < (uint32_t)(ne - 1024 * (u0 + u)) ? t : 0u];
  };
  vq_row_exponents<G>(lut, g, c, rows, row, share == 0, sexp);
  __syncthreads();
  int s[G];
#pragma unroll
  for (int h = 0; h < G; ++h) s[h] = __builtin_amdgcn_readfirstlane(sexp[h]);
  const int64_t tiles = vq_tiles(cap);
  // quad q of a thread is the four slots from t0 + (threadIdx.x + 1024 q) * 4.  Shares start at multiples of 256
  // slots, so the quads of a wave lie in one tile and are scanned or left out together
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const uint16_t* ip[NQ];
  int nq = 0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int64_t j = t0 + 256 * w + 4096 * q;
    if (j < t1) nq = q + 1;
    ip[q] = pcache + vq_wide_at(g, tiles, row, j < t1 ? j : t0, 0);
  }
  int zi[NQ][4][G];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int h = 0; h < G; ++h) zi[q][tt][h] = 0;
  // the indices of the next group are fetched while the current group is looked up (and while the next slice
  // of the table is brought in), so no slice waits for HBM; read once: kept out of the way of the table in L2
  v2i nx[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) nx[q] = __builtin_nontemporal_load(reinterpret_cast<const v2i*>(ip[q]) + lane);
  const uint32_t last = (uint32_t)(c - 1);
  for (int g0 = 0; g0 < g; g0 += gps) {
    if constexpr (RAW) {
      __syncthreads();                                    // the previous slice's lookups are done
      // sixteen bytes per lane, a wave's 1 KiB in one piece behind a common address.  (A slice is a multiple of 16 bytes:
      // one group with four heads, an even number of groups with two, four or more with one)
      const unsigned char* src = reinterpret_cast<const unsigned char*>(trow + (int64_t)g0 * c);
      const int n16 = (gps < g - g0 ? gps : g - g0) * c * (int)sizeof(E) / 16;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int at = 1024 * u + 64 * w;
        if (at + lane < n16)
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + (int64_t)(at + lane) * 16),
                                           (__attribute__((address_space(3))) void*)(lds_raw + at * 16), 16, 0, 0);
      }
      __builtin_amdgcn_s_waitcnt(0x0f70);                 // vmcnt(0): they are in LDS
      __syncthreads();
    } else {
      fetch(g0, 0);
      __syncthreads();                                    // the previous slice's lookups are done
#pragma unroll
      for (int u0 = 0; u0 < kPer; u0 += kGo) {
        if (u0 > 0) fetch(g0, u0);
#pragma unroll
        for (int u = 0; u < kGo; ++u)
          if (1024 * (u0 + u) < ne && threadIdx.x < (uint32_t)(ne - 1024 * (u0 + u)))
            tab[threadIdx.x + 1024 * (u0 + u)] = entry_fix<G>(nt[u], s);
      }
      __syncthreads();
    }
    for (int gl = 0; gl < gps; ++gl) {
      v2i cur[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) cur[q] = nx[q];
      if (g0 + gl + 1 < g) {
        const int64_t off = (int64_t)(g0 + gl + 1) * kVqTile;
#pragma unroll
        for (int q = 0; q < NQ; ++q) nx[q] = __builtin_nontemporal_load(reinterpret_cast<const v2i*>(ip[q] + off) + lane);
      }
      const T* tg = tab + gl * c;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        if (q >= nq) continue;
        T raw[4];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
          const uint32_t code = ((uint32_t)(tt < 2 ? cur[q].x : cur[q].y) >> (16 * (tt & 1))) & 0xffffu;
          raw[tt] = tg[code < last ? code : last];        // slots past n hold whatever memory held
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
          F e;
          if constexpr (RAW) e = entry_fix<G>(raw[tt], s);
          else e = raw[tt];
          if constexpr (G == 4) { zi[q][tt][0] += e.x; zi[q][tt][1] += e.y; zi[q][tt][2] += e.z; zi[q][tt][3] += e.w; }
          else if constexpr (G == 2) { zi[q][tt][0] += e.x; zi[q][tt][1] += e.y; }
          else { zi[q][tt][0] += e; }
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      const int64_t j = t0 + ((int64_t)threadIdx.x + 1024 * q) * 4 + tt;
      if (j >= t1) break;
      float z[G];
#pragma unroll
      for (int h = 0; h < G; ++h) z[h] = ldexpf((float)zi[q][tt][h], -s[h]);
      float best = z[0];
#pragma unroll
      for (int h = 1; h < G; ++h) best = fmaxf(best, z[h]);
      sel[(int64_t)row * cap + j] = best;
      if (z_out != nullptr) {
#pragma unroll
        for (int h = 0; h < G; ++h) z_out[((int64_t)row * G + h) * cap + j] = z[h];
      }
    }
  }
}

// The wide scan of few slots: every entry where it lies, in L2, instead of the whole table through every compute unit's
// LDS, whose 30 to 100 us do not fall with the number of slots.  A thread per slot, eight groups' indices and then their
// entries in flight; rows on dies as above.  Bound by the rate at which L2 answers scattered lines:
// 8 rows of 24 000 slots, c = 8192, table included: 97 -> 42 us.
template <int G>
__global__ __launch_bounds__(256) void vq_scan_direct_kernel(int g, int c, int64_t cap, const uint16_t* __restrict__ pcache,
                                                             float* __restrict__ lut, NRes nr, int n_kv_heads, int rows,
                                                             float* __restrict__ sel, float* __restrict__ z_out) {
  using E = typename EntryT<G>::type;
  using F = typename EntryT<G>::fix;
  __shared__ int sexp[4];
  const int row = blockIdx.x % rows;
  const int64_t n = nr.n[row / n_kv_heads], t0 = (int64_t)(blockIdx.x / rows) * 256;
  if (t0 >= n) return;
  const E* trow = reinterpret_cast<const E*>(lut) + (int64_t)row * g * c;
  const int64_t j = t0 + threadIdx.x < n ? t0 + threadIdx.x : n - 1;
  const uint16_t* ip = pcache + vq_wide_at(g, vq_tiles(cap), row, j, 0);
  constexpr int U = 8;
  uint32_t nx[U];
#pragma unroll
  for (int u = 0; u < U; ++u) nx[u] = ip[(int64_t)u * kVqTile];
  vq_row_exponents<G>(lut, g, c, rows, row, t0 == 0, sexp);
  __syncthreads();
  int s[G];
#pragma unroll
  for (int h = 0; h < G; ++h) s[h] = __builtin_amdgcn_readfirstlane(sexp[h]);
  int zi[G];
#pragma unroll
  for (int h = 0; h < G; ++h) zi[h] = 0;
  const uint32_t last = (uint32_t)(c - 1);
  for (int g0 = 0; g0 < g; g0 += U) {
    E e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) e[u] = trow[(int64_t)(g0 + u) * c + (nx[u] < last ? nx[u] : last)];
    if (g0 + U < g) {
#pragma unroll
      for (int u = 0; u < U; ++u) nx[u] = ip[(int64_t)(g0 + U + u) * kVqTile];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const F f = entry_fix<G>(e[u], s);
      if constexpr (G == 4) { zi[0] += f.x; zi[1] += f.y; zi[2] += f.z; zi[3] += f.w; }
      else if constexpr (G == 2) { zi[0] += f.x; zi[1] += f.y; }
      else { zi[0] += f; }
    }
  }
  if (t0 + threadIdx.x >= n) return;
  float z[G];
#pragma unroll
  for (int h = 0; h < G; ++h) z[h] = ldexpf((float)zi[h], -s[h]);
  float best = z[0];
#pragma unroll
  for (int h = 1; h < G; ++h) best = fmaxf(best, z[h]);
  sel[(int64_t)row * cap + j] = best;
  if (z_out != nullptr) {
#pragma unroll
    for (int h = 0; h < G; ++h) z_out[((int64_t)row * G + h) * cap + j] = z[h];
  }
}

// Canonical export of the index rows for tests: out[row][slot][group], slots < n_resident.
__global__ __launch_bounds__(256) void vq_export_kernel(int g, int64_t cap, const uint8_t* __restrict__ pcache, NRes nr,
                                                        int n_kv_heads, uint8_t* __restrict__ out) {
  const int row = blockIdx.y;
  const int64_t n = nr.n[row / n_kv_heads];
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t slot = gid / g;
  const int i = (int)(gid % g);
  if (slot >= n) return;
  out[((int64_t)row * cap + slot) * g + i] = pcache[((int64_t)row * cap + slot) * g + vq_byte_of(i, slot)];
}

__global__ __launch_bounds__(256) void vq_export_wide_kernel(int g, int64_t cap, const uint16_t* __restrict__ pcache,
                                                             NRes nr, int n_kv_heads, uint16_t* __restrict__ out) {
  const int row = blockIdx.y;
  const int64_t n = nr.n[row / n_kv_heads];
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (gid >= n * g) return;
  const int64_t slot = gid / g;
  const int i = (int)(gid % g);
  out[(int64_t)row * cap * g + gid] = pcache[vq_wide_at(g, vq_tiles(cap), row, slot, i)];
}

// More than 256 centroids: the shortlist always from 257 tokens on, below by estimates in us of the vector form and of
// vq_assign_mfma_kernel, fitted to 500 such sizes (none picked more than 6 % slower than the better of the two).  A
// workgroup of the latter walks the codebook for up to 1024 tokens, two of them per compute unit at a time; with few tokens
// most of its waves only help with the operands, and a launch of many (KV head, group) pairs is faster in the vector form,
// whose waves take 64 tokens each.  Measured, mfma / vector: 8 rows, 32 groups, c = 8192, 9 tokens 0.25; 32 rows, 64 groups,
// 64 tokens: c = 257 1.66, 700 1.03, 1024 0.87; 128 rows, 64 groups, 64 tokens: c = 1024 1.71, 2048 1.47; 128 tokens: 512
// 1.32, 1024 0.99; 256 tokens: 257 1.31, 400 0.98.
static bool assign_by_shortlist(int rows, int g, int c, int64_t T) {
  if (T > 256) return true;
  const double pairs = (double)rows * g, waves = pairs * (double)((T + 63) / 64);
  const double alone = g == 64 ? 0.058 : 0.089, each = g == 64 ? 1.38e-5 : 1.99e-5;      // per centroid: one wave; per wave
  const double vec = c * (waves * each > alone ? waves * each : alone);
  const double mfma = (pairs > 420 ? pairs : 420) * (0.0108 + 1.1e-5 * c) * (1.0 + T / 940.0);
  return mfma < vec;
}

// 33 to 256 centroids: the least of three estimates in us, each fitted to the form's own times at 3500 sizes (1 to 56 rows,
// 33 to 256 centroids, 64 to 60 000 tokens; of 3187 calls above 13 us the pick is 6 % or more off the best form in 31 and 15 %
// or more in 3).  The vector form takes all centroids of a group in a chain, per 64 tokens and group a wave: flat to four
// waves per SIMD, a step at more than the eight that fit.  The tiles' and the shortlist's workgroups (16 groups of 256
// tokens; one group of 1024) come in rounds of 256.  Per call, vector / tiles / shortlist, us: 8 rows, 32 groups, c = 256,
// 256 tokens 27 / 34 / 12, 1000 27 / 35 / 14, 2000 41 / 35 / 20, 4000 69 / 36 / 34; c = 128, 1000 15 / 26 / 13, 4000 37 / 27
// / 30; 64 groups, c = 96, 1500 20 / 25 / 30; c = 128, 1100 22 / 25 / 32; 1 row, 64 groups, c = 256, 9000 39 / 37 / 30; c = 33,
// 4 rows, 32 groups, 33 000 44 / 49 / -; 32 rows, 64 groups, 64 tokens, c = 256 19 / - / 26.  The shortlist's single index
// bytes crowd the L2s beyond a million of them (1 row, 32 groups, c = 256, 33 000 tokens 48, tiles 41; 8 rows 573 / 232), and
// for fewer than 96 centroids it is never the best.
enum class AssignForm { kVector, kTiles, kShortlist, kCells };

// Tokens per workgroup of vq_assign_cells_kernel: as many workgroups as compute units where the blocks allow it.
static int assign_cells_chunk(int rows, int g, int64_t T) {
  const int64_t pairs = (int64_t)rows * g;
  int64_t parts = pairs < 256 ? 256 / pairs : 1;
  if ((T + parts - 1) / parts < 1024) parts = (T + 1023) / 1024;
  const int64_t least = (T + kCellTokens - 1) / kCellTokens;
  if (parts < least) parts = least;
  return (int)align_up((T + parts - 1) / parts, 32);
}

// More than 256 centroids and tokens: vq_assign_cells_kernel against vq_assign_mfma_kernel by estimates in us, fitted to 600
// sizes (1 to 49 rows, 1024 to 8192 centroids, 256 to 33 000 tokens; half of them within 2.5 %, nineteen in twenty within 8 %).  A
// workgroup of the former pays for two orderings before its first token, and what it multiplies grows with less than the
// codebook; the 4 % are for what the fit does not see.  Measured, mfma / cells: 8 rows, 32 groups, c = 8192: 1000 tokens
// 108 / 97 us, 2000 177 / 128, 4000 311 / 182, 16 384 1120 / 454; c = 4096: 4000 163 / 143, 16 384 610 / 389; c = 2048:
// 16 384 350 / 332; 24 rows, c = 8192: 1000 tokens 229 / 255; 64 groups, 8 rows: c = 8192, 512 102 / 69, 16 384 2213 / 414; c =
// 2048: 512 34 / 50, 2000 92 / 82, 16 384 646 / 357.  Of 75 sizes the pick is 5 % or more off the better form in three, 10 % at
// most (8 rows, c = 8192, 1000 tokens).
static bool assign_by_cells(int rows, int g, int c, int64_t T) {
  const int chunk = assign_cells_chunk(rows, g, T);
  const double pairs = (double)rows * g, n = (double)(T < chunk ? T : chunk) / 1000, k = (double)c / 1000;
  const double rounds = ceil(pairs * (double)((T + chunk - 1) / chunk) / 256);
  const double part = T < 1024 ? (double)T / 1024 : 1.0;
  double turns = pairs * (double)((T + 1023) / 1024) / 512;
  double cells, mfma;
  if (g == 32) {
    cells = 6.5 + rounds * (23.3 + 0.93 * k + 14.1 * n + 2.22 * n * sqrt(k) + 4.0 * sqrt(n) * k);
    mfma = 11.5 + (turns > 0.56 ? turns : 0.56) * (8.2 + 17.1 * k) * (0.37 + 0.63 * part);
  } else {
    cells = 5.8 + rounds * (13.5 + 1.35 * k + 8.08 * n + 1.37 * n * sqrt(k) + 0.62 * sqrt(n) * k);
    mfma = 11.3 + (turns > 0.62 ? turns : 0.62) * (6.3 + 19.0 * k) * (0.34 + 0.66 * part);
  }
  return 1.04 * cells < mfma;
}

static AssignForm assign_form(int rows, int g, int c, int64_t T) {
  if (T <= 8 || c <= 32) return AssignForm::kVector;
  if (c > kAsCodewords && T > 256 && assign_by_cells(rows, g, c, T)) return AssignForm::kCells;
  if (c > kAsCodewords) return assign_by_shortlist(rows, g, c, T) ? AssignForm::kShortlist : AssignForm::kVector;
  const bool four = g == 32;                                // channels per centroid, else two
  const auto rounds = [](int64_t workgroups) { return (double)((workgroups + 255) / 256); };
  const double w = (double)rows * g * (double)((T + 63) / 64) / 1024;                    // waves per SIMD
  const double vec = four ? 3.6 + (c + 8.7) * (w <= 8 ? fmax(0.081, 0.0121 * w + 0.044) : w <= 64 ? 0.149 + 0.0126 * (w - 8) : 0.014 * w)
                          : 4.0 + (c + 11.5) * (w <= 8 ? fmax(0.056, 0.0077 * w + 0.0386) : w <= 64 ? 0.115 + 0.0095 * (w - 8) : 0.0104 * w);
  double tiles = 1e30, mfma = 1e30;
  if (T >= 256) {
    const double x = rounds((int64_t)rows * (g / 16) * ((T + 255) / 256));
    if (c <= 64) tiles = four ? (x <= 8 ? 19.3 + 1.6 * x + 0.62 * x * x : 10.5 + 7.7 * x) : fmax(20.5, 10.5 + 5.5 * x);
    else if (c <= 128) tiles = four ? fmax(26.0, 12.5 + 8.7 * x) : fmax(25.0, 13.0 + 7.6 * x);
    else tiles = four ? fmax(35.5, 21.0 + 11.8 * x) : fmax(36.0, 20.5 + 11.5 * x);
  }
  if (c >= 96 && (int64_t)rows * g * T <= 1050000) {
    const double x = rounds((int64_t)rows * g * ((T + 1023) / 1024)), part = T < 1024 ? (double)T / 1024 : 1.0, k = log2(c / 32.0);
    mfma = four ? 6.0 + (3.8 + 1.2 * k) * x * (0.3 + 0.7 * part) : 6.5 + (3.8 + 1.3 * k) * x * (0.27 + 0.73 * part);
  }
  if (mfma < vec && mfma < tiles) return AssignForm::kShortlist;
  return tiles < vec ? AssignForm::kTiles : AssignForm::kVector;
}

int32_t launch_vq_assign(const Layout& L, int g, int c, const float* centroids, uint8_t* pcache, const void* k_new,
                         int64_t T, const NRes& nr, float* acc_opt, int32_t* pos_opt, const NRes& vrow0, hipStream_t st) {
  if (T == 0) return HCA_OK;
  const uint16_t* kn = (const uint16_t*)k_new;
  const bool wide = vq_is_wide(L, g, c);
#define HCA_ASSIGN_T(SPLIT)                                                                                           \
  do {                                                                                                                \
    dim3 gs((unsigned)T, (unsigned)L.rows, (unsigned)(g / (4 / SPLIT)));                                               \
    if (g == 32 && wide) vq_assign_small_kernel<4, true, SPLIT><<<gs, 256, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0); \
    else if (g == 32) vq_assign_small_kernel<4, false, SPLIT><<<gs, 256, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0);   \
    else if (wide) vq_assign_small_kernel<2, true, SPLIT><<<gs, 256, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0);      \
    else vq_assign_small_kernel<2, false, SPLIT><<<gs, 256, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0);               \
  } while (0)
#define HCA_ASSIGN_B(GPW, GRID)                                                                                       \
  do {                                                                                                                \
    if (g == 32 && wide) vq_assign_kernel<4, true, GPW><<<GRID, 256, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0); \
    else if (g == 32) vq_assign_kernel<4, false, GPW><<<GRID, 256, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0);   \
    else if (wide) vq_assign_kernel<2, true, GPW><<<GRID, 256, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0);      \
    else vq_assign_kernel<2, false, GPW><<<GRID, 256, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0);               \
  } while (0)
  const AssignForm form = assign_form(L.rows, g, c, T);
  if (form == AssignForm::kTiles) {
    dim3 gm((unsigned)((T + 255) / 256), (unsigned)L.rows, (unsigned)(g / 16));
#define HCA_ASSIGN_SC(D, W, NT) vq_assign_small_c_kernel<D, W, NT><<<gm, 256, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0)
#define HCA_ASSIGN_SCN(D, W)                                                                                          \
  do {                                                                                                                \
    if (c <= 64) HCA_ASSIGN_SC(D, W, 2); else if (c <= 128) HCA_ASSIGN_SC(D, W, 4); else HCA_ASSIGN_SC(D, W, 8);      \
  } while (0)
    if (g == 32 && wide) HCA_ASSIGN_SCN(4, true);
    else if (g == 32) HCA_ASSIGN_SCN(4, false);
    else if (wide) HCA_ASSIGN_SCN(2, true);
    else HCA_ASSIGN_SCN(2, false);
#undef HCA_ASSIGN_SCN
#undef HCA_ASSIGN_SC
  } else if (form == AssignForm::kCells) {
    const int chunk = assign_cells_chunk(L.rows, g, T);
    const unsigned wgs = (unsigned)(L.rows * g * ((T + chunk - 1) / chunk));
#define HCA_ASSIGN_CELLS(D)                                                                                           \
  do {                                                                                                                \
    static std::atomic<uint64_t> opted{0};                /* one per instantiation */                                 \
    const int32_t rc = lds_opt_in(reinterpret_cast<const void*>(&vq_assign_cells_kernel<D>), (int)cells_lds(8192, D), &opted); \
    if (rc != HCA_OK) return rc;                                                                                      \
    vq_assign_cells_kernel<D><<<wgs, 1024, cells_lds(c, D), st>>>(g, c, L.n_kv_heads, L.rows, L.cap, centroids, (uint16_t*)pcache, kn, T, chunk, nr, acc_opt, pos_opt, vrow0); \
  } while (0)
    if (g == 32) HCA_ASSIGN_CELLS(4); else HCA_ASSIGN_CELLS(2);
#undef HCA_ASSIGN_CELLS
  } else if (form == AssignForm::kShortlist) {
    // a block or a context: shortlist on the matrix cores, exact chain on the shortlist
    dim3 gm((unsigned)((T + 1023) / 1024), (unsigned)L.rows, (unsigned)g);
#define HCA_ASSIGN_M(D, BT, W) vq_assign_mfma_kernel<D, BT, W><<<gm, 512, 0, st>>>(g, c, L.n_kv_heads, L.cap, centroids, pcache, kn, T, nr, acc_opt, pos_opt, vrow0)
    if (g == 32 && c > 2048) HCA_ASSIGN_M(4, 2, true);
    else if (g == 32 && wide) HCA_ASSIGN_M(4, 1, true);
    else if (g == 32) HCA_ASSIGN_M(4, 1, false);
    else if (c > 2048) HCA_ASSIGN_M(2, 2, true);
    else if (wide) HCA_ASSIGN_M(2, 1, true);
    else HCA_ASSIGN_M(2, 1, false);
#undef HCA_ASSIGN_M
  } else if (T <= 8) {                              // decode appends: parallel over centroids, not over tokens
    // four waves on a group shorten a wave's chain of loads but are four times as many workgroups: while those of the
    // other form fill the chip once, or the codebook is long.  Times of the other form over this one: 64 workgroups of it
    // 1.3 (c = 1024), 2.5 (8192); 256: 1.07, 1.9; 512: 0.9 - 1.02 (1024), 0.91 (2048), 1.08 (4096); 1024: 0.74, 0.96,
    // 1.04, 1.0 (8192); 2048: 0.64, 0.8, 0.96, 1.12; 4096: 0.99 (8192) and less.
    const int64_t wgs = T * L.rows * (g / 4);
    if (c >= 1024 && (wgs <= 256 || (c >= 4096 && 4 * wgs <= c))) HCA_ASSIGN_T(4);
    else HCA_ASSIGN_T(1);
  } else if ((T + 63) / 64 * L.rows * (g / 4) < 16 * 1024) {
    // a block of a few thousand tokens: with four groups per wave the launch would have at most a few waves per
    // SIMD (the chip has 1024 of them); one group per wave gives four times as many
    dim3 grid((unsigned)((T + 63) / 64), (unsigned)L.rows, (unsigned)(g / 4));
    HCA_ASSIGN_B(1, grid);
  } else {
    dim3 grid((unsigned)((T + 63) / 64), (unsigned)L.rows, (unsigned)(g / 16));
    HCA_ASSIGN_B(4, grid);
  }
#undef HCA_ASSIGN_B
#undef HCA_ASSIGN_T
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

// Whether the wide scan looks its entries up where they lie: by an estimate of both in us.  The form through LDS takes as
// long as the whole table takes to pass through it; a lookup in L2 takes 1.7 to 4 us per million while a die's tables fit
// its L2 (rows go to the eight dies in turn), 9.5 beyond.  Measured, through LDS / directly, table included: 8 rows of four
// heads, 32 groups, c = 8192: 4000 slots 99 / 28, 24 000 97 / 42, 60 000 98 / 81, 90 000 100 / 109; c = 4096: 4000 63 / 21,
// 40 000 63 / 50, 60 000 64 / 69; c = 1024: 4000 30 / 14, 24 000 30 / 25, 40 000 30 / 34; c = 300: 23 / 12, 23 / 16, 23 / 21;
// 64 groups, c = 8192: 187 / 43, 182 / 77, 183 / 169 (60 000); 32 rows, c = 8192: 4000 128 / 73, 12 000 125 / 142;
// 3 rows, c = 8192: 40 000 98 / 41, 131 000 95 / 98; 1 row: 262 000 95 / 50, 500 000 96 / 81, 1 Mi 100 / 149.
static bool scan_directly(int rows, int g, int c, int gqa, int64_t nmax) {
  const double table = (double)c * g * gqa * 4 / (1 << 20), lookups = (double)rows * (double)nmax * g * 1e-6;
  const double on_die = table * (rows % 8 == 0 ? rows / 8 : rows);
  const double rate = on_die <= 0.3 ? 1.7 : on_die <= 0.6 ? 2.6 : on_die <= 4.0 ? 3.9 : on_die <= 8.0 ? 5.7 : 9.5;
  return 12.0 + 4.0 * table + rate * lookups < 12.0 + 0.36 * g + 17.0 * table;
}

template <int G>
static int32_t scan_wide_launch(const Layout& L, int g, int c, const uint8_t* pcache, float* lut, const NRes& nr,
                                int64_t nmax, float* sel, float* z_opt, hipStream_t st) {
  if (scan_directly(L.rows, g, c, G, nmax)) {
    vq_scan_direct_kernel<G><<<(unsigned)((nmax + 255) / 256 * L.rows), 256, 0, st>>>(
        g, c, L.cap, (const uint16_t*)pcache, lut, nr, L.n_kv_heads, L.rows, sel, z_opt);
    HCA_HIP(hipGetLastError());
    return HCA_OK;
  }
  int gps = 1;                                      // groups per LDS slice: the most that fit 128 KiB
  while (gps * 2 <= g && (int64_t)gps * 2 * c * G * 4 <= 128 * 1024) gps *= 2;
  const size_t lds = (size_t)gps * c * G * 4;
  // Equal shares, as many as compute units or a multiple, of at most 12 Ki slots where that gives one share per
  // unit: three quads leave registers for a whole slice in flight.  Else 16 Ki, with a quarter of a slice in flight,
  // as a larger share has fewer refills.  8 rows, c = 8192, score call with table, before -> now: n = 1000 165 -> 101 us,
  // 300 000 175 -> 107, 400 000 178 -> 145, 530 000 329 -> 260, 1 Mi 347 -> 296 (c = 1024: 65 -> 31, 78 -> 52, 81 -> 61,
  // 139 -> 90, 174 -> 145; one query head per KV head, c = 8192, 1 Mi: 250 -> 162).
  const int64_t units = L.rows < 256 ? 256 / L.rows : 1;
  const bool one = nmax <= units * 12 * 1024;
  const int64_t turns = one ? 1 : (nmax + units * 16 * 1024 - 1) / (units * 16 * 1024);
  // The table's entries straight into LDS (RAW): no registers between, a refill takes 1.2 us for 2.1, but each lookup puts its
  // entry on the grid instead of each refill.  Measured, as it was / RAW, table included, by slots of a share per
  // centroid: four heads, 8 rows x 32 groups: c = 8192, 0.28 99 / 87 us, 0.6 102 / 92, 1.16 106 / 104; c = 6000, 1.6 90 / 94; c =
  // 3000, 1.6 59 / 59, 3.2 70 / 77; c = 1024, 4.8 38 / 44.  Two heads: c = 8192, 1.16 86 / 70, 2 (1 Mi) 180 / 168; c = 4096, 2.3 60
  // / 55, 3.8 (64 groups) 127 / 131; c = 2048, 4.6 47 / 48; c = 1024, 9.2 40 / 45.  One head: c = 8192, 1.16 68 / 52, 2 163 / 142;
  // c = 300, 8 27 / 24, 32 36 / 34, 52 (64 groups) 88 / 90.
  const double per_centroid = (double)nmax / (double)(units * turns * c);
  const bool raw = per_centroid <= (G == 4 ? 1.3 : G == 2 ? 3.5 : 40.0) && (one || G < 4) && ((uintptr_t)lut & 15) == 0;
  int64_t per_wg = align_up((nmax + units * turns - 1) / (units * turns), 256);
  if (per_wg < 2048) per_wg = 2048;
  const int64_t shares = (nmax + per_wg - 1) / per_wg;
#define HCA_WIDE(NQ, RAW)                                                                                                \
  {                                                                                                                      \
    if (lds > 64 * 1024) {                                                                                               \
      static std::atomic<uint64_t> opted{0};                /* one per instantiation */                                  \
      const int32_t rc = lds_opt_in(reinterpret_cast<const void*>(&vq_scan_wide_kernel<G, NQ, RAW>), 128 * 1024, &opted); \
      if (rc != HCA_OK) return rc;                          /* + 16 B static */                                          \
    }                                                                                                                    \
    vq_scan_wide_kernel<G, NQ, RAW><<<(unsigned)(shares * L.rows), 1024, lds, st>>>(                                     \
        g, c, gps, L.cap, per_wg, (const uint16_t*)pcache, lut, nr, L.n_kv_heads, L.rows, sel, z_opt);                   \
  }
  if constexpr (G < 4) {
    if (raw && !one) HCA_WIDE(4, true)
  }
  if (raw && one) HCA_WIDE(3, true)
  else if (!raw && one) HCA_WIDE(3, false)
  else if (!raw) HCA_WIDE(4, false)
#undef HCA_WIDE
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

template <int G, int NG>
static int32_t scan_launch(const Layout& L, int c, const uint8_t* pcache, float* lut, const NRes& nr,
                           int64_t nmax, float* sel, float* z_opt, hipStream_t st) {
  const size_t lds = (size_t)NG * c * G * 4;
  if (lds > 64 * 1024) {                            // tables beyond 64 KiB need the opt-in, once per device
    static std::atomic<uint64_t> opted{0};          // one per instantiation
    const int32_t rc = lds_opt_in(reinterpret_cast<const void*>(&vq_scan_kernel<G, NG>), 128 * 1024, &opted);   // + 272 B static
    if (rc != HCA_OK) return rc;
  }
  // about one workgroup per compute unit, each with at least 1024 tokens, shares a multiple of 1024
  int64_t per_row = 256 / L.rows;
  if (per_row < 1) per_row = 1;
  int64_t per_wg = align_up((nmax + per_row - 1) / per_row, 1024);
  const int64_t chunks = (nmax + per_wg - 1) / per_wg;
  dim3 grid((unsigned)chunks, (unsigned)L.rows);
  vq_scan_kernel<G, NG><<<grid, 1024, lds, st>>>(c, L.cap, pcache, lut, nr, L.n_kv_heads, per_wg, sel, z_opt);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

int32_t launch_vq_score(const Layout& L, int g, int c, const float* centroids, const uint8_t* pcache, const void* q,
                        const NRes& nr, int64_t nmax, float* lut, float* sel, float* z_opt, hipStream_t st) {
  const uint16_t* qq = (const uint16_t*)q;
  dim3 gl((unsigned)g, (unsigned)L.rows);
  float* amax = lut + (int64_t)L.rows * g * c * L.gqa;   // [rows][g][4], then the exponents [rows][4]
#define HCA_LUT_P(G, D, PER) vq_lut_kernel<G, D, PER><<<gl, 256, 0, st>>>(g, c, L.n_kv_heads, vq_is_wide(L, g, c), centroids, qq, lut, amax)
#define HCA_LUT(G, D) do { if (c <= 256) HCA_LUT_P(G, D, 1); else HCA_LUT_P(G, D, 8); } while (0)
  if (g == 32) {
    if (L.gqa == 4) HCA_LUT(4, 4); else if (L.gqa == 2) HCA_LUT(2, 4); else HCA_LUT(1, 4);
  } else {
    if (L.gqa == 4) HCA_LUT(4, 2); else if (L.gqa == 2) HCA_LUT(2, 2); else HCA_LUT(1, 2);
  }
#undef HCA_LUT
#undef HCA_LUT_P
  HCA_HIP(hipGetLastError());
  if (nmax == 0) return HCA_OK;
  if (vq_is_wide(L, g, c)) {
    if (L.gqa == 4) return scan_wide_launch<4>(L, g, c, pcache, lut, nr, nmax, sel, z_opt, st);
    if (L.gqa == 2) return scan_wide_launch<2>(L, g, c, pcache, lut, nr, nmax, sel, z_opt, st);
    return scan_wide_launch<1>(L, g, c, pcache, lut, nr, nmax, sel, z_opt, st);
  }
  if (g == 32) {
    if (L.gqa == 4) return scan_launch<4, 32>(L, c, pcache, lut, nr, nmax, sel, z_opt, st);
    if (L.gqa == 2) return scan_launch<2, 32>(L, c, pcache, lut, nr, nmax, sel, z_opt, st);
    return scan_launch<1, 32>(L, c, pcache, lut, nr, nmax, sel, z_opt, st);
  }
  if (L.gqa == 4) return scan_launch<4, 64>(L, c, pcache, lut, nr, nmax, sel, z_opt, st);
  if (L.gqa == 2) return scan_launch<2, 64>(L, c, pcache, lut, nr, nmax, sel, z_opt, st);
  return scan_launch<1, 64>(L, c, pcache, lut, nr, nmax, sel, z_opt, st);
}

// Shape checks shared by the entry points: the uniform-code fields of the shape are not used here.
static int32_t vq_layout(const hca_shape* shape, const hca_vq_codebook* cb, Layout* L, bool need_centroids) {
  if (shape == nullptr || cb == nullptr) return HCA_ERR_BAD_ARG;
  hca_shape s = *shape;
  s.bits = 4;
  s.group = 32;
  int32_t rc = make_layout(&s, L);
  if (rc != HCA_OK) return rc;
  if (cb->groups != 32 && cb->groups != 64) return HCA_ERR_UNSUPPORTED;
  if (cb->codewords < 1) return HCA_ERR_BAD_ARG;
  if (cb->codewords > 8192) return HCA_ERR_UNSUPPORTED;
  if (need_centroids && cb->centroids == nullptr) return HCA_ERR_BAD_ARG;
  return HCA_OK;
}

// ------------------------------------------------------------------------------ trainer ---
// Lloyd's k-means, one codebook per group (or one for the pooled sub-vectors), codebooks spread over
// host threads.  Within a codebook everything runs in pool order, so the result does not depend on
// the number of threads.
static void train_one(const uint16_t* kval, int64_t nval, int D, int g, int c, int dbar, bool shared, int b,
                      const int32_t* init, int iters, float* cb, double* iner, std::atomic<int>* bad) {
  const int64_t npool = shared ? nval * g : nval;
  std::vector<float> x((size_t)npool * dbar);
  auto half = [](uint16_t h) -> float {
    _Float16 v;
    std::memcpy(&v, &h, 2);
    return (float)v;
  };
  for (int64_t p = 0; p < npool; ++p) {
    const int64_t t = shared ? p / g : p;
    const int i = shared ? (int)(p % g) : b;
    for (int dd = 0; dd < dbar; ++dd) x[(size_t)p * dbar + dd] = half(kval[t * D + i * dbar + dd]);
  }
  for (int cc = 0; cc < c; ++cc) {
    int64_t s = init[cc];
    if (s < 0 || s >= npool) { bad->store(1); s = 0; }
    std::memcpy(cb + (size_t)cc * dbar, &x[(size_t)s * dbar], sizeof(float) * dbar);
  }
  std::vector<double> sum((size_t)c * dbar);
  std::vector<int64_t> cnt((size_t)c);
  for (int it = 0; it <= iters; ++it) {
    std::fill(sum.begin(), sum.end(), 0.0);
    std::fill(cnt.begin(), cnt.end(), (int64_t)0);
    double obj = 0.0;
    for (int64_t p = 0; p < npool; ++p) {
      const float* xp = &x[(size_t)p * dbar];
      int best = 0;
      float bd = 0.f;
      for (int cc = 0; cc < c; ++cc) {
        const float* cv = cb + (size_t)cc * dbar;
        float d = 0.f;
        for (int dd = 0; dd < dbar; ++dd) {
          const float e = xp[dd] - cv[dd];
          d = std::fmaf(e, e, d);
        }
        if (cc == 0 || d < bd) { bd = d; best = cc; }
      }
      obj += (double)bd;
      cnt[best] += 1;
      for (int dd = 0; dd < dbar; ++dd) sum[(size_t)best * dbar + dd] += (double)xp[dd];
    }
    iner[it] = obj;
    if (it == iters) break;
    for (int cc = 0; cc < c; ++cc)
      if (cnt[cc] > 0)
        for (int dd = 0; dd < dbar; ++dd) cb[(size_t)cc * dbar + dd] = (float)(sum[(size_t)cc * dbar + dd] / (double)cnt[cc]);
  }
}

}  // namespace hca

using namespace hca;

extern "C" {

size_t hca_vq_pcache_bytes(const hca_shape* shape, const hca_vq_codebook* cb) {
  Layout L;
  if (vq_layout(shape, cb, &L, false) != HCA_OK) return 0;
  if (vq_is_wide(L, cb->groups, cb->codewords))      // whole tiles of 16 Ki slots
    return (size_t)L.rows * (size_t)vq_tiles(L.cap) * kVqTile * (size_t)cb->groups * 2;
  return (size_t)L.rows * (size_t)L.cap * (size_t)cb->groups;
}

size_t hca_vq_workspace_bytes(const hca_shape* shape, const hca_vq_codebook* cb, int64_t k_max, int64_t m_max) {
  Layout L;
  if (vq_layout(shape, cb, &L, false) != HCA_OK) return 0;
  hca_shape s = *shape;      // the hca_vq_* calls lay the workspace out as the 4-bit uniform path does
  s.bits = 4;
  s.group = 32;
  return hca_workspace_bytes(&s, k_max, m_max);
}

size_t hca_vq_lut_bytes(const hca_shape* shape, const hca_vq_codebook* cb) {
  Layout L;
  if (vq_layout(shape, cb, &L, false) != HCA_OK) return 0;
  return (size_t)L.rows * cb->groups * cb->codewords * L.gqa * 4 + (size_t)L.rows * (cb->groups + 1) * 4 * sizeof(int32_t);
}

int32_t hca_vq_train(const void* kval_f16, int64_t n_val, int32_t head_dim, int32_t groups, int32_t codewords,
                     const int32_t* init, int32_t iters, int32_t shared, float* centroids, double* inertia_opt) {
  if (kval_f16 == nullptr || init == nullptr || centroids == nullptr) return HCA_ERR_BAD_ARG;
  if (head_dim < 1 || groups < 1 || head_dim % groups != 0 || codewords < 1 || n_val < 1 || iters < 0)
    return HCA_ERR_BAD_ARG;
  const int dbar = head_dim / groups;
  const int ncb = shared ? 1 : groups;
  std::vector<double> iner((size_t)ncb * (iters + 1), 0.0);
  std::atomic<int> bad{0};
  std::atomic<int> next{0};
  auto work = [&]() {
    for (int b = next.fetch_add(1); b < ncb; b = next.fetch_add(1))
      train_one((const uint16_t*)kval_f16, n_val, head_dim, groups, codewords, dbar, shared != 0, b,
                init + (size_t)b * codewords, iters, centroids + (size_t)b * codewords * dbar,
                &iner[(size_t)b * (iters + 1)], &bad);
  };
  unsigned nt = std::thread::hardware_concurrency();
  if (nt < 1) nt = 1;
  if (nt > 16) nt = 16;
  if ((int)nt > ncb) nt = (unsigned)ncb;
  std::vector<std::thread> pool;
  for (unsigned t = 1; t < nt; ++t) pool.emplace_back(work);
  work();
  for (auto& th : pool) th.join();
  if (shared)
    for (int i = 1; i < groups; ++i)
      std::memcpy(centroids + (size_t)i * codewords * dbar, centroids, sizeof(float) * (size_t)codewords * dbar);
  if (inertia_opt != nullptr)
    for (int it = 0; it <= iters; ++it) {
      double s = 0.0;
      for (int b = 0; b < ncb; ++b) s += iner[(size_t)b * (iters + 1) + it];
      inertia_opt[it] = s;
    }
  return bad.load() ? HCA_ERR_BAD_ARG : HCA_OK;
}

int32_t hca_vq_assign(const hca_shape* shape, const hca_vq_codebook* cb, void* pcache, const void* k_new_f16,
                      int64_t T, const int64_t* n_resident, float* acc_opt, int32_t* pos_opt,
                      const int64_t* value_row0, void* stream) {
  Layout L;
  int32_t rc = vq_layout(shape, cb, &L, true);
  if (rc != HCA_OK) return rc;
  if (pcache == nullptr || T < 0 || (T > 0 && k_new_f16 == nullptr)) return HCA_ERR_BAD_ARG;
  NRes nr, vrow0;
  int64_t nmax;
  rc = load_nres(L, n_resident, &nr, &nmax);
  if (rc != HCA_OK) return rc;
  for (int b = 0; b < L.batch; ++b)
    if (nr.n[b] + T > L.cap) return HCA_ERR_CAPACITY;
  for (int b = 0; b < kMaxBatch; ++b) vrow0.n[b] = 0;
  for (int b = 0; b < L.batch; ++b) vrow0.n[b] = value_row0 ? value_row0[b] : nr.n[b];
  return launch_vq_assign(L, cb->groups, cb->codewords, cb->centroids, (uint8_t*)pcache, k_new_f16, T, nr, acc_opt,
                          pos_opt, vrow0, (hipStream_t)stream);
}

int32_t hca_vq_score(const hca_shape* shape, const hca_vq_codebook* cb, const void* pcache, const void* q_f16,
                     const int64_t* n_resident, float* lut, float* sel, float* z_opt, void* stream) {
  Layout L;
  int32_t rc = vq_layout(shape, cb, &L, true);
  if (rc != HCA_OK) return rc;
  if (pcache == nullptr || q_f16 == nullptr || lut == nullptr || sel == nullptr) return HCA_ERR_BAD_ARG;
  NRes nr;
  int64_t nmax;
  rc = load_nres(L, n_resident, &nr, &nmax);
  if (rc != HCA_OK) return rc;
  return launch_vq_score(L, cb->groups, cb->codewords, cb->centroids, (const uint8_t*)pcache, q_f16, nr, nmax, lut,
                         sel, z_opt, (hipStream_t)stream);
}

int32_t hca_vq_export_pcache(const hca_shape* shape, const hca_vq_codebook* cb, const void* pcache,
                             const int64_t* n_resident, void* indices, void* stream) {
  Layout L;
  int32_t rc = vq_layout(shape, cb, &L, false);
  if (rc != HCA_OK) return rc;
  if (pcache == nullptr || indices == nullptr) return HCA_ERR_BAD_ARG;
  NRes nr;
  int64_t nmax;
  rc = load_nres(L, n_resident, &nr, &nmax);
  if (rc != HCA_OK) return rc;
  if (nmax == 0) return HCA_OK;
  dim3 grid((unsigned)((nmax * cb->groups + 255) / 256), (unsigned)L.rows);
  if (vq_is_wide(L, cb->groups, cb->codewords))
    vq_export_wide_kernel<<<grid, 256, 0, (hipStream_t)stream>>>(cb->groups, L.cap, (const uint16_t*)pcache, nr,
                                                                 L.n_kv_heads, (uint16_t*)indices);
  else
    vq_export_kernel<<<grid, 256, 0, (hipStream_t)stream>>>(cb->groups, L.cap, (const uint8_t*)pcache, nr, L.n_kv_heads,
                                                            (uint8_t*)indices);
  HCA_HIP(hipGetLastError());
  return HCA_OK;
}

int32_t hca_vq_attend_gathered(const hca_shape* shape, const hca_vq_codebook* cb, const void* pcache,
                               const float* lut, const int32_t* idx, const int32_t* count, int32_t k,
                               float sm_scale, float* y, float* acc_opt, void* workspace, void* stream) {
  Layout L;
  int32_t rc = vq_layout(shape, cb, &L, false);
  if (rc != HCA_OK) return rc;
  if (pcache == nullptr || lut == nullptr || idx == nullptr || count == nullptr || y == nullptr ||
      workspace == nullptr)
    return HCA_ERR_BAD_ARG;
  if (k < 1 || k > L.cap || k > 64 * 256) return HCA_ERR_CAPACITY;
  return launch_vq_attend_gathered(L, cb->groups, cb->codewords, (const uint8_t*)pcache, lut, idx, count, k, sm_scale,
                                   y, acc_opt, workspace, (hipStream_t)stream);
}

int32_t hca_vq_evict(const hca_shape* shape, const hca_vq_codebook* cb, void* pcache, float* acc, int32_t* pos,
                     const int64_t* n_resident, int64_t M, int64_t n_protect, int32_t* kept_opt, void* workspace,
                     void* pcache_dst, float* acc_dst, int32_t* pos_dst, void* stream) {
  Layout L;
  int32_t rc = vq_layout(shape, cb, &L, false);
  if (rc != HCA_OK) return rc;
  if (pcache == nullptr || acc == nullptr || pos == nullptr || workspace == nullptr) return HCA_ERR_BAD_ARG;
  const bool oop = pcache_dst != nullptr || acc_dst != nullptr || pos_dst != nullptr;
  if (oop && (pcache_dst == nullptr || acc_dst == nullptr || pos_dst == nullptr)) return HCA_ERR_BAD_ARG;
  if (oop && (pcache_dst == pcache || acc_dst == acc || pos_dst == pos)) return HCA_ERR_BAD_ARG;
  if (M < 1 || M > L.cap || n_protect < 0 || n_protect > M) return HCA_ERR_CAPACITY;
  NRes nr;
  int64_t nmax;
  rc = load_nres(L, n_resident, &nr, &nmax);
  if (rc != HCA_OK) return rc;
  return launch_vq_evict(L, cb->groups, cb->codewords, (uint8_t*)pcache, acc, pos, nr, nmax, M, n_protect, kept_opt,
                         workspace, (uint8_t*)pcache_dst, acc_dst, pos_dst, (hipStream_t)stream);
}

}  // extern "C"
