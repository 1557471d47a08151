// Device-side building blocks shared by the HIP kernels of libhca: the tiled key-cache
// layout, the fixed-point query operand and the MFMA scoring of one 1 KiB code block.
// gfx950 only (wave64, v_mfma_i32_16x16x64_i8).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hca {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));

constexpr int kHeadDim = 128;
constexpr int kBlockBytes = 1024;  // one code block = 64 lanes x 16 B
constexpr int kMetaBytes = 256;    // scales + zeros of one code block
constexpr int kMaxBatch = 64;

// Key cache in HBM.  A row (sequence, KV head) is a sequence of code blocks followed, in a
// second region, by the matching meta blocks.
//   4-bit / group 32: a block holds 16 tokens.  Lane l = t + 16*j (t token, j in 0..3) owns
//     bytes [16*l, 16*l+16): two 8-byte slots m = 0, 1; slot m packs channels
//     [32*(2m + j/2) + 16*(j%2), +16), two codes per byte, low nibble first.
//     Meta of token t: 16 B at 16*t = fp16 scale[0..3], zero[0..3].
//   2-bit / group 64: a block holds 32 tokens = two 16-token tiles u = 0, 1.  Lane l owns
//     bytes [16*l, +16): tile u at +8*u, slot m at +4*m; slot m packs channels
//     [64*m + 16*j, +16), four codes per byte, lowest bits first.
//     Meta of token (u, t): 8 B at 8*(16*u + t) = fp16 scale[0..1], zero[0..1].
// With this order one global_load_dwordx4 per lane fetches a whole block, fully coalesced,
// and every lane already holds the bytes it feeds to the matrix core.
struct Layout {
  int32_t bits, group, ng, tpb;  // ng groups per token, tpb tokens per block
  int32_t rows, gqa, batch, n_kv_heads;
  int64_t cap, nblk;             // capacity (tokens) and blocks per row
  int64_t meta_off;              // byte offset of the meta region
  __host__ __device__ int64_t codes_row_bytes() const { return nblk * kBlockBytes; }
  __host__ __device__ int64_t meta_row_bytes() const { return nblk * kMetaBytes; }
  __host__ __device__ int64_t total_bytes() const {
    return (int64_t)rows * (codes_row_bytes() + meta_row_bytes());
  }
};

struct NRes {  // resident tokens per sequence, passed by value to kernels
  int64_t n[kMaxBatch];
};

__device__ __forceinline__ float h2f(uint32_t bits16) {
  return (float)__builtin_bit_cast(_Float16, (unsigned short)(bits16 & 0xffffu));
}
__device__ __forceinline__ unsigned short f2h_bits(float x) {
  return __builtin_bit_cast(unsigned short, (_Float16)x);  // v_cvt_f16_f32, round to nearest even
}

// Codebook form: where the index of group `grp` sits in the stored record of slot `slot`, and back.
__device__ __forceinline__ int vq_byte_of(int grp, int64_t slot) {
  return (grp & ~15) | ((grp - (int)slot) & 15);
}
__device__ __forceinline__ int vq_group_at(int byte, int64_t slot) {
  return (byte & ~15) | ((byte + (int)slot) & 15);
}
// Wide codebook form: 16-bit indices, stored in tiles of kVqTile slots, group-major inside a tile
// (uint16 [row][tile][group][kVqTile]), so that the scan, which handles one group (or a few) at a time, reads
// each group's indices of its tile in one piece.  Position of (row, slot, group) in uint16 units:
constexpr int kVqTile = 16384;
__host__ __device__ __forceinline__ int64_t vq_tiles(int64_t cap) { return (cap + kVqTile - 1) / kVqTile; }
__host__ __device__ __forceinline__ int64_t vq_wide_at(int g, int64_t tiles, int64_t row, int64_t slot, int grp) {
  return ((row * tiles + slot / kVqTile) * g + grp) * kVqTile + slot % kVqTile;
}
// Power-of-two grid of one query head's table: s = 23 - floor(log2(largest magnitude)) (0 for an all-zero
// table), entry -> rint(entry * 2^s), at most 2^24 in magnitude, so that 64 of them add up exactly in 32 bits.
__device__ __forceinline__ int vq_grid_exponent(float amax) {
  return amax == 0.f ? 0 : 23 - ilogbf(amax);
}
__device__ __forceinline__ int vq_fix(float t, int s) { return (int)rintf(ldexpf(t, s)); }

// Order-preserving map float -> uint32 (larger float <=> larger key), -0 treated as +0.
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u << 1) == 0) u = 0;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// ---------------------------------------------------------------------------------------
// Query operand.  Each query head is mapped to fixed point, qfx = rint(q * 2^s) with
// s = 13 - floor(log2(max|q|)), split into a low and a high signed byte (qfx = lo + 256*hi).
// The A operand of the 16x16x64 i8 MFMA has 16 rows = 4 heads x 4 sub-rows; a sub-row is
// (byte piece, group selector) and carries the piece on the channels of its group and 0
// elsewhere, so one MFMA yields the per-group integer dot products of 16 tokens x 4 heads.
struct QShared {           // LDS image of the query of one row (4 heads)
  int16_t qfx[4][kHeadDim];
  int32_t qsum[4][4];      // per head, per group: sum of qfx
  int32_t sexp[4];
};

template <int BITS>
struct QOperand {
  v4i a[2];       // A operand of MFMA m = 0, 1
  float qf[4];    // (float) sum of qfx over group g, for head lane/16
  float unscale;  // 2^-s of head lane/16
  float nzero;    // -0.0f, opaque to the compiler (see zero_term)
};

// zero_g * Q_g rounded once, as a fused multiply-add with the addend -0.0f (x * y + (-0) == x * y for all finite
// x, y, signs of zero included): in this form the fp16 -> fp32 conversion of `zero` rides inside v_fma_mix_f32
// instead of costing an instruction of its own.  The addend is kept opaque so that it is not folded back.
__device__ __forceinline__ float zero_term(uint32_t zero_bits16, float qf, float nzero) {
  return __builtin_fmaf(h2f(zero_bits16), qf, nzero);
}

// channel held in byte x (0..15) of the B operand of MFMA m by a lane of k-group j
template <int BITS>
__device__ __forceinline__ int operand_channel(int m, int j, int x) {
  const int i = x >> 2, y = x & 3;
  if (BITS == 4) {
    const int idx = ((i >> 1) << 3) + 2 * y + (i & 1);
    return 32 * (2 * m + (j >> 1)) + 16 * (j & 1) + idx;
  } else {
    return 64 * m + 16 * j + 4 * y + i;
  }
}

__device__ __forceinline__ float wave_max(float v);
template <int CTRL> __device__ __forceinline__ int query_dpp(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
// This lane's two channels of head w of the row (past the last head: of that one), for query_on_grid and load_query below:
// asked for as early as the caller likes.
__device__ __forceinline__ uint32_t query_pair(const uint16_t* __restrict__ q, int row, int gqa) {
  const int w = threadIdx.x >> 6;
  return reinterpret_cast<const uint32_t*>(q + ((int64_t)row * gqa + (w < gqa ? w : gqa - 1)) * kHeadDim)[threadIdx.x & 63];
}
// Computes the fixed-point query of a row into LDS.  Called by all threads of the block
// (at least 256); wave w < 4 handles query head w of the row.  A barrier has to follow.
__device__ __forceinline__ void query_on_grid(uint32_t pair, int gqa, int group, QShared* sh) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (w >= gqa) pair = 0;
  const float x0 = h2f(pair & 0xffffu), x1 = h2f(pair >> 16);
  const float amax = wave_max(fmaxf(fabsf(x0), fabsf(x1)));
  int s = 0;
  if (amax != 0.f) s = 13 - ilogbf(amax);
  if (w < 4) {                       // workgroups larger than four waves: the extra waves only take the barrier
    const int16_t v0 = (int16_t)(int)rintf(ldexpf(x0, s)), v1 = (int16_t)(int)rintf(ldexpf(x1, s));
    reinterpret_cast<uint32_t*>(sh->qfx[w])[lane] = (uint16_t)v0 | (uint32_t)(uint16_t)v1 << 16;
    if (lane == 0) sh->sexp[w] = s;
    // a row of 16 lanes holds 32 channels; a group is one, two or four rows (16 threads that added a group each from LDS,
    // behind a barrier of their own, took 1 us more)
    int sum = v0 + v1;
    sum += query_dpp<0xB1>(sum);     // quad_perm [1,0,3,2]
    sum += query_dpp<0x4E>(sum);     // quad_perm [2,3,0,1]
    sum += query_dpp<0x141>(sum);    // row_half_mirror
    sum += query_dpp<0x140>(sum);    // row_mirror
    int rows[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) rows[r] = __builtin_amdgcn_readlane(sum, 16 * r);
    const int per = group >> 5, g = lane >> 4;       // rows per group
    int acc = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc += r >= g * per && r < (g + 1) * per ? rows[r] : 0;
    if ((lane & 15) == 0) sh->qsum[w][g] = acc;
  }
}
__device__ __forceinline__ void load_query(uint32_t pair, int gqa, int group, QShared* sh) {
  query_on_grid(pair, gqa, group, sh);
  __syncthreads();
}
__device__ __forceinline__ void load_query(const uint16_t* __restrict__ q, int row, int gqa, int group,
                                           QShared* sh) {
  load_query(query_pair(q, row, gqa), gqa, group, sh);
}

template <int BITS>
__device__ __forceinline__ void build_operand(const QShared* sh, QOperand<BITS>* op) {
  const int lane = threadIdx.x & 63;
  const int r = lane & 15, j = lane >> 4;       // A operand: row r, k-group j
  const int head = r >> 2, sub = r & 3;
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    int regs[4] = {0, 0, 0, 0};
    bool active;
    int piece;
    if (BITS == 4) { piece = sub & 1; active = ((sub >> 1) == (j >> 1)); }
    else           { piece = sub & 1; active = (sub < 2); }
    if (active) {
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const int v = sh->qfx[head][operand_channel<BITS>(m, j, x)];
        const int lo = ((v + 128) & 255) - 128;
        const int hi = (v - lo) / 256;
        const int b = (piece ? hi : lo) & 255;
        regs[x >> 2] |= b << (8 * (x & 3));
      }
    }
    op->a[m] = v4i{regs[0], regs[1], regs[2], regs[3]};
  }
  const int hd = lane >> 4;                      // epilogue: this lane scores head hd
#pragma unroll
  for (int g = 0; g < 4; ++g) op->qf[g] = (float)sh->qsum[hd][g];
  op->unscale = ldexpf(1.0f, -sh->sexp[hd]);
  float nz = -0.0f;
  asm volatile("" : "+v"(nz));
  op->nzero = nz;
}

// The same operand built once per workgroup of four waves instead of once per wave (every wave of a scan
// workgroup uses the same query): wave w forms two of the eight operand dwords of every lane, the image goes
// through LDS (img: 64 lanes x 8 dwords).  To be called by all 256 threads; contains a barrier.
template <int BITS>
__device__ __forceinline__ void build_operand_shared(const QShared* sh, uint32_t* img, QOperand<BITS>* op) {
  const int lane = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3;
  const int r = lane & 15, j = lane >> 4;
  const int head = r >> 2, sub = r & 3;
  const int m = w >> 1;
  const int piece = sub & 1;
  const bool active = BITS == 4 ? ((sub >> 1) == (j >> 1)) : (sub < 2);
#pragma unroll
  for (int dd = 0; dd < 2; ++dd) {
    const int i = 2 * (w & 1) + dd;
    int reg = 0;
    if (active) {
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        const int v = sh->qfx[head][operand_channel<BITS>(m, j, 4 * i + y)];
        const int lo = ((v + 128) & 255) - 128;
        const int hi = (v - lo) / 256;
        reg |= ((piece ? hi : lo) & 255) << (8 * y);
      }
    }
    img[lane * 8 + 4 * m + i] = (uint32_t)reg;
  }
  __syncthreads();
  const v4i* im = reinterpret_cast<const v4i*>(img + lane * 8);
  op->a[0] = im[0];
  op->a[1] = im[1];
  const int hd = lane >> 4;
#pragma unroll
  for (int g = 0; g < 4; ++g) op->qf[g] = (float)sh->qsum[hd][g];
  op->unscale = ldexpf(1.0f, -sh->sexp[hd]);
  float nz = -0.0f;
  asm volatile("" : "+v"(nz));
  op->nzero = nz;
}

__device__ __forceinline__ v4i mfma_i8(v4i a, v4i b, v4i c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// 4-bit: scores the 16 tokens of one block.  w = this lane's 16 code bytes, mw = the meta of
// token lane%16.  Returns z~ of (token lane%16, head lane/16).
__device__ __forceinline__ float score_block4(const QOperand<4>& op, uint4 w, uint4 mw) {
  const v4i zero = {0, 0, 0, 0};
  const uint32_t M = 0x0f0f0f0fu;
  v4i b0 = {(int)(w.x & M), (int)((w.x >> 4) & M), (int)(w.y & M), (int)((w.y >> 4) & M)};
  v4i b1 = {(int)(w.z & M), (int)((w.z >> 4) & M), (int)(w.w & M), (int)((w.w >> 4) & M)};
  v4i d0 = mfma_i8(op.a[0], b0, zero);   // rows: lo/hi of group 0, lo/hi of group 1
  v4i d1 = mfma_i8(op.a[1], b1, zero);   // rows: lo/hi of group 2, lo/hi of group 3
  const float t0 = fmaf(h2f(mw.x), (float)(d0.y * 256 + d0.x), zero_term(mw.z, op.qf[0], op.nzero));
  const float t1 = fmaf(h2f(mw.x >> 16), (float)(d0.w * 256 + d0.z), zero_term(mw.z >> 16, op.qf[1], op.nzero));
  const float t2 = fmaf(h2f(mw.y), (float)(d1.y * 256 + d1.x), zero_term(mw.w, op.qf[2], op.nzero));
  const float t3 = fmaf(h2f(mw.y >> 16), (float)(d1.w * 256 + d1.z), zero_term(mw.w >> 16, op.qf[3], op.nzero));
  const float a = t0 + t1, b = t2 + t3;
  return (a + b) * op.unscale;
}

// 2-bit: scores one 16-token tile.  c0, c1 = this lane's 4 code bytes of slot 0 and 1;
// mw = meta of the token (scale0|scale1<<16, zero0|zero1<<16).
__device__ __forceinline__ float score_tile2(const QOperand<2>& op, uint32_t c0, uint32_t c1, uint2 mw) {
  const v4i zero = {0, 0, 0, 0};
  const uint32_t M = 0x03030303u;
  v4i b0 = {(int)(c0 & M), (int)((c0 >> 2) & M), (int)((c0 >> 4) & M), (int)((c0 >> 6) & M)};
  v4i b1 = {(int)(c1 & M), (int)((c1 >> 2) & M), (int)((c1 >> 4) & M), (int)((c1 >> 6) & M)};
  v4i d0 = mfma_i8(op.a[0], b0, zero);   // rows: lo, hi of group 0
  v4i d1 = mfma_i8(op.a[1], b1, zero);   // rows: lo, hi of group 1
  const float t0 = fmaf(h2f(mw.x), (float)(d0.y * 256 + d0.x), zero_term(mw.y, op.qf[0], op.nzero));
  const float t1 = fmaf(h2f(mw.x >> 16), (float)(d1.y * 256 + d1.x), zero_term(mw.y >> 16, op.qf[1], op.nzero));
  return (t0 + t1) * op.unscale;
}

// max of two finite floats (plain v_max_f32: the inputs are never NaN, so no canonicalisation)
__device__ __forceinline__ float fmax_raw(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// max over the four 16-lane rows of a wave (the four query heads of a token), result on every lane
__device__ __forceinline__ float max_over_heads(float x) {
  const uint32_t xi = __float_as_uint(x);
  const auto r16 = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);   // rows {0,1} and {2,3}
  const float m = fmax_raw(__uint_as_float(r16[0]), __uint_as_float(r16[1]));
  const uint32_t mi = __float_as_uint(m);
  const auto r32 = __builtin_amdgcn_permlane32_swap(mi, mi, false, false);   // halves
  return fmax_raw(__uint_as_float(r32[0]), __uint_as_float(r32[1]));
}

// Four values per lane, one per 16-token tile (z0..z3: the score of this lane's (token, head) in tiles 0..3): returns,
// on the lanes of row r, the maximum over the four rows (= the token's four query heads) of tile r's values - the
// reduction and the hand-over of tile r to row r in three swaps and three maxima.
__device__ __forceinline__ float max_over_heads_scatter(float z0, float z1, float z2, float z3) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(z0), __float_as_uint(z2), false, false);
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(z1), __float_as_uint(z3), false, false);
  // p[0] = [z0.r0 z0.r1 z2.r0 z2.r1], p[1] = [z0.r2 z0.r3 z2.r2 z2.r3]: maxima over the row pairs (0,2), (1,3)
  const float m02 = fmax_raw(__uint_as_float(p[0]), __uint_as_float(p[1]));
  const float m13 = fmax_raw(__uint_as_float(q[0]), __uint_as_float(q[1]));
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(m02), __float_as_uint(m13), false, false);
  // r[0] = [m02.r0 m13.r0 m02.r2 m13.r2], r[1] = [m02.r1 m13.r1 m02.r3 m13.r3]
  return fmax_raw(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// 16-byte load with the non-temporal hint: the code stream is read once per decode step and
// should not displace anything in the caches.
__device__ __forceinline__ uint4 load_stream16(const uint4* p) {
  const v4i v = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p));
  return uint4{(uint32_t)v.x, (uint32_t)v.y, (uint32_t)v.z, (uint32_t)v.w};
}

// All-gather over the four 16-lane rows of a wave: returns, on every lane, the values that the
// lanes of the same column hold in rows 0..3.
__device__ __forceinline__ uint4 allgather_rows(uint32_t v) {
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);        // [r0 r0 r2 r2], [r1 r1 r3 r3]
  const auto b = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);  // r0 everywhere, r2 everywhere
  const auto c = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);  // r1 everywhere, r3 everywhere
  return uint4{b[0], c[0], b[1], c[1]};
}

// The float whose order key is `key`, or -inf for keys below those of all finite floats (0: "no threshold"):
// v >= key_floor(key) <=> order_key(v) >= key for every finite v (-0 and +0 share a key and compare equal).
__device__ __forceinline__ float key_floor(uint32_t key) {
  if (key <= 0x007fffffu) return -INFINITY;
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// ---- wave-wide scans and reductions by DPP: six dependent vector instructions where six __shfl_up or __shfl_xor go through
// the LDS crossbar.  Called by all 64 lanes.  (With the workgroup scans reading the
// waves' sums at once: cumulative-weight selection and attend over 8 x 500 003 tokens 157.4 -> 155.0 us, eviction 126.2 -> 124.9.)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or(uint32_t other, uint32_t v) {      // `other` where no lane is shifted in
  return (uint32_t)__builtin_amdgcn_update_dpp((int)other, (int)v, CTRL, ROWS, 0xf, false);
}
// f(shift) for the six steps after which lane 63 has seen every lane (lane l: lanes 0 .. l)
template <typename F>
__device__ __forceinline__ void dpp_steps(F&& f) {
  f([](uint32_t o, uint32_t v) { return dpp_or<0x111, 0xf>(o, v); });         // row_shr:1
  f([](uint32_t o, uint32_t v) { return dpp_or<0x112, 0xf>(o, v); });         // row_shr:2
  f([](uint32_t o, uint32_t v) { return dpp_or<0x114, 0xf>(o, v); });         // row_shr:4
  f([](uint32_t o, uint32_t v) { return dpp_or<0x118, 0xf>(o, v); });         // row_shr:8
  f([](uint32_t o, uint32_t v) { return dpp_or<0x142, 0xa>(o, v); });         // row_bcast:15 into rows 1 and 3
  f([](uint32_t o, uint32_t v) { return dpp_or<0x143, 0xc>(o, v); });         // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t v) {
  dpp_steps([&](auto&& shift) { v += shift(0u, v); });
  return v;
}
__device__ __forceinline__ uint64_t wave_scan_incl(uint64_t v) {
  dpp_steps([&](auto&& shift) {
    const uint32_t lo = shift(0u, (uint32_t)v), hi = shift(0u, (uint32_t)(v >> 32));
    v += (uint64_t)hi << 32 | lo;
  });
  return v;
}
__device__ __forceinline__ uint32_t wave_last(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return wave_last(wave_scan_incl(v)); }
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  dpp_steps([&](auto&& shift) { const uint32_t o = shift(v, v); v = o < v ? o : v; });
  return wave_last(v);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  dpp_steps([&](auto&& shift) { const uint32_t o = shift(v, v); v = o > v ? o : v; });
  return wave_last(v);
}
__device__ __forceinline__ float wave_min(float v) {
  dpp_steps([&](auto&& shift) { const uint32_t b = __float_as_uint(v); v = fminf(v, __uint_as_float(shift(b, b))); });
  return __uint_as_float(wave_last(__float_as_uint(v)));
}
__device__ __forceinline__ float wave_max(float v) {
  dpp_steps([&](auto&& shift) { const uint32_t b = __float_as_uint(v); v = fmaxf(v, __uint_as_float(shift(b, b))); });
  return __uint_as_float(wave_last(__float_as_uint(v)));
}
// exclusive prefix sum of one value per thread over a workgroup of NW waves; *total (optional) gets the sum
template <int NW, typename T>
__device__ __forceinline__ T block_scan_excl(T v, T* wsum /*[NW]*/, T* total = nullptr) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const T inc = wave_scan_incl(v);
  if ((threadIdx.x & 63) == 63) wsum[w] = inc;
  __syncthreads();
  T base = 0, all = 0;
#pragma unroll
  for (int x = 0; x < NW; ++x) {
    const T s = wsum[x];
    base += x < w ? s : 0;
    all += s;
  }
  if (total != nullptr) *total = all;
  __syncthreads();
  return base + inc - v;
}

}  // namespace hca
