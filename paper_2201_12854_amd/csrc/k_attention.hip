// Attention stages of the MCA forward pass on gfx950:
//   scores + row softmax statistics + column max   (softmax(a Q K^T), a = 1/8, and the
//                                                    per-block part of max A[:, j], Eq. 8/9;
//                                                    or of the column sum (mean rule), or
//                                                    every probability (median rule))
//   Y = A H~                                        ("Y = AH", Sec. "Self-Attention
//                                                    Mechanisms"; Eq. 5 outer sum)
// Both kernels compute a probability the same way, A = exp2(fma(q . k, log2(e)/8, -c))
// with the row normaliser c written by the score pass. A is never written to memory
// (except under the median rule).
//
// Tiling: one block = 4 waves = 64 queries of one (batch row, head), a wave owning 16
// queries (the streaming kernels: 128 queries, 32 per wave in two 16-query tiles). Keys
// come in tiles of 64 staged in LDS; 16x16 MFMA tiles (bf16 16x16x32 or fp32 16x16x4).
// The score pass computes S = Q K^T (its layout and reductions are described with the
// kernels). The output pass computes S^T = K Q^T, so lane l holds the scores of query
// (l % 16) for keys 16 s + 4 (l / 16) + i (s, i = 0..3): exactly the A-operand layout of
// the P V MFMA, with no data movement between the two products.
//
// Variants by padded length:
//   resident (up to 64 NT keys, NT <= 4 for bf16, 2 for fp32): every K (and H~) tile of
//     the sequence is loaded at once behind one barrier and all scores stay in registers,
//     so the statistics and the column max come from a single pass;
//   score pass up to 8 key tiles: K tiles streamed through two LDS buffers, every score
//     kept in registers, still a single pass;
//   streaming (longer sequences): tiles are double buffered in LDS with the next tile
//     prefetched into registers; the score pass sweeps twice (per-lane statistics, then
//     the column statistic). The bf16 kernels use 32x32x16 MFMA tiles and direct loads to
//     LDS (k_scores_stream32, k_attn_stream32; large grids of 5 to 8 key tiles keep the
//     16x16 output pass).
// Local-window attention (Sec. "Longformer": a window of w keys around each token and a
// global first token): query q attends key k < len when |q - k| <= w / 2, or q = 0, or
// k = 0; the other scores are masked like padded keys. The column max is then taken of
// |S_q| A[q, k], |S_q| the number of keys query q attends (the count rule's per-row factor
// n of Eq. 9), and the streaming variants visit only the key tiles a query tile's window
// reaches, plus tile 0 (float32, and rows of up to 8 key tiles: all tiles for the tile holding
// query 0; the bfloat16 streaming kernels take query 0's other keys apart, far_from).
//
// Rows past the padded length are read from the last row instead of being zero-filled:
// their scores are masked and their probabilities are exactly 0. Tile loads are
// unconditional (a tile index past the last valid tile is clamped to it), which keeps the
// tiles in registers and the load stream free of divergent branches.
#include <type_traits>

#include "mca_device.h"
#include "mca_kernels.h"

namespace mca {
namespace {

constexpr int kThreads = 256;
constexpr int kTile = 64;                // queries per block and keys per tile
// bf16 tiles in LDS: rows of 64 elements (128 bytes, no padding) whose eight 16-byte
// chunks are permuted per row, chunk c of row r stored at chunk c ^ (r & 7). gfx950 serves a
// wave's 16-byte LDS accesses in four cycles, and its transposing 8-byte reads in two, only
// when the lanes served together fall in distinct banks; with this permutation that holds
// for the three accesses to a tile (a bank-conflict probe measured each): the fragment
// reads of Q K^T (16 consecutive rows, one chunk), the transposing reads of P V (rows
// 4 g + i, one pair of chunks) and the row stores. Unpermuted 128-byte rows serialise the
// fragment reads four ways, 144-byte rows two ways.
constexpr int kStrideBf = kDHead;
// The streaming output pass keeps its H~ tiles unpermuted in 160-byte rows instead (also
// conflict-free for the transposing reads): there the four column groups of a read are
// constant offsets from one address, where the permutation would need a register per group
// and take the kernel past the register count that allows three waves per SIMD.
constexpr int kStrideBfWide = kDHead + 16;
// element offset of (row, col) in a bf16 tile; col a multiple of 4 (an 8-byte piece)
__device__ __forceinline__ int kv_at(int row, int col) {
  return row * kStrideBf + ((((col >> 3) ^ (row & 7)) << 3) | (col & 7));
}
constexpr int kStrideF = kDHead + 4;     // LDS row stride of fp32 tiles (elements)

template <int BF> struct Elem { using T = float; };
template <> struct Elem<1> { using T = uint16_t; };
template <int BF> constexpr int stride_of() { return BF ? kStrideBf : kStrideF; }

// ------------------------------------------------------------------ Q fragments
// The wave's 16 queries as the B operand of S^T = K Q^T.
template <int BF> struct QFrag;
template <> struct QFrag<1> { bf16x8_t v[2]; };   // d = 32 ks + 8 g + (0..7)
template <> struct QFrag<0> { float v[16]; };      // d = 16 g + t

__device__ __forceinline__ void load_qfrag(QFrag<1>& f, const uint16_t* qrow, int g) {
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
    f.v[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(qrow + 32 * ks + 8 * g));
}

__device__ __forceinline__ void load_qfrag(QFrag<0>& f, const float* qrow, int g) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float4 u = *reinterpret_cast<const float4*>(qrow + 16 * g + 4 * c);
    f.v[4 * c + 0] = u.x;
    f.v[4 * c + 1] = u.y;
    f.v[4 * c + 2] = u.z;
    f.v[4 * c + 3] = u.w;
  }
}

// ------------------------------------------------------------------ tiles in flight
// A 64-row x 64-column tile of a [*, d_out] matrix (the head's column slice) held in
// registers between its global load and its LDS store: 16-byte vectors v0, v1 (bf16) or
// v0..v3 (fp32) per thread; vector v of the tile is row v / R, chunk v % R (R vectors per
// row). Rows past the padded length read as zeros. (Plain members, no arrays: the tiles
// are carried across loop iterations and must stay in registers.)
struct TileRegs {
  uint4 v0, v1, v2, v3;
};

// The loads go through a buffer descriptor built per tile in scalar registers: its base is
// the tile's first row and its size ends with the head's slice of the last valid row, so
// the per-lane offset (row within the tile times the row pitch, plus the chunk) is the
// same for every tile and no per-tile address arithmetic runs on the vector units; the
// hardware range check returns zeros for rows at or past n (whose keys are masked).
constexpr int kBufWord3 = 0x00020000;  // gfx9 descriptor word 3: 32-bit data format

// The descriptor of the tile whose first row is key0: with r = min(n - key0, 64) valid rows
// its size is (r - 1) pitch + 64 elements, and 0 when r <= 0 (the pitch, d_out elements, is
// at least 256 of them, so the max() below needs no branch).
template <int BF>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* base, int64_t ld, int key0, int n) {
  constexpr int ES = (int)sizeof(typename Elem<BF>::T);
  const int bytes = max((min(n - key0, kTile) - 1) * (int)ld * ES + kDHead * ES, 0);
  return __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char*>(static_cast<const char*>(base) + (int64_t)key0 * ld * ES), 0, bytes, kBufWord3);
}

// vector v of the tile
template <int BF>
__device__ __forceinline__ uint4 tile_vec_load(__amdgpu_buffer_rsrc_t rs, int64_t ld, int v) {
  constexpr int R = BF ? 8 : 16;
  constexpr int ES = (int)sizeof(typename Elem<BF>::T);
  const int off = (v / R) * (int)ld * ES + (v % R) * 16;
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
}

template <int BF>
__device__ __forceinline__ TileRegs tile_load(const void* base, int64_t ld, int key0, int n, int tid) {
  const __amdgpu_buffer_rsrc_t rs = tile_rsrc<BF>(base, ld, key0, n);
  TileRegs t;
  t.v0 = tile_vec_load<BF>(rs, ld, tid);
  t.v1 = tile_vec_load<BF>(rs, ld, tid + kThreads);
  if constexpr (!BF) {
    t.v2 = tile_vec_load<BF>(rs, ld, tid + 2 * kThreads);
    t.v3 = tile_vec_load<BF>(rs, ld, tid + 3 * kThreads);
  } else {
    t.v2 = t.v3 = make_uint4(0, 0, 0, 0);
  }
  return t;
}

// row-major LDS tile [key][d]
template <int BF>
__device__ __forceinline__ void tile_vec_store(uint4 u, typename Elem<BF>::T* lds, int v) {
  constexpr int R = BF ? 8 : 16;
  if constexpr (BF) *reinterpret_cast<uint4*>(lds + kv_at(v / R, (v % R) * 8)) = u;
  else *reinterpret_cast<uint4*>(lds + (v / R) * kStrideF + (v % R) * 4) = u;
}

template <int BF>
__device__ __forceinline__ void tile_store(const TileRegs& t, typename Elem<BF>::T* lds, int tid) {
  tile_vec_store<BF>(t.v0, lds, tid);
  tile_vec_store<BF>(t.v1, lds, tid + kThreads);
  if constexpr (!BF) {
    tile_vec_store<BF>(t.v2, lds, tid + 2 * kThreads);
    tile_vec_store<BF>(t.v3, lds, tid + 3 * kThreads);
  }
}

// H~ tiles are stored like K tiles, row-major [key][column]; the P V MFMA reads its B
// operand (8 keys of one column per lane) with the transposing LDS read below.
template <int BF, bool WIDE = false>
__device__ __forceinline__ void tile_store_v(const TileRegs& t, typename Elem<BF>::T* lds, int tid) {
  if constexpr (BF && WIDE) {
    *reinterpret_cast<uint4*>(lds + (tid / 8) * kStrideBfWide + (tid % 8) * 8) = t.v0;
    *reinterpret_cast<uint4*>(lds + (tid / 8 + kThreads / 8) * kStrideBfWide + (tid % 8) * 8) = t.v1;
  } else {
    tile_store<BF>(t, lds, tid);
  }
}

// ds_read_b64_tr_b16 (gfx950). Within each row of 16 lanes, every lane supplies the address
// of 4 consecutive 16-bit elements; lane i receives, as its element k (k = 0..3), element
// i % 4 of the 4 addressed by lane 4 k + i / 4 of its row. Lane s addressing
// V[kb + s / 4][d0 + 4 (s % 4)] of a row-major tile therefore gives lane i the column
// V[kb .. kb + 3][d0 + i].
typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16_t lds_v4i16_t;

__device__ __forceinline__ uint2 lds_read_tr16(const uint16_t* p) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)p));
}

// ------------------------------------------------------------------ score tile
// acc[s][i] = (K Q^T)[key 16 s + 4 g + i][query l % 16] for the 64 keys in LDS.
__device__ __forceinline__ void score_tile(f32x4_t acc[4], const uint16_t* Ks, const QFrag<1>& q,
                                           int r16, int g) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    acc[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(Ks + kv_at(16 * s + r16, 32 * ks + 8 * g));
      acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, q.v[ks], acc[s], 0, 0, 0);
    }
  }
}

__device__ __forceinline__ void score_tile(f32x4_t acc[4], const float* Ks, const QFrag<0>& q,
                                           int r16, int g) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    acc[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const float* krow = Ks + (16 * s + r16) * kStrideF + 16 * g;
#pragma unroll
    for (int t = 0; t < 16; ++t)
      acc[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(krow[t], q.v[t], acc[s], 0, 0, 0);
  }
}

// Logits in base-2 units: a (q . k) log2(e) with a = 1/sqrt(64), the rounded constant
// log2(e) / 8, so that softmax needs only exp2 (one hardware instruction):
// exp(a x - m) = exp2(a log2(e) x - m log2(e)). An attention probability is
// A = exp2(fma(dot, log2(e) / 8, -c)) with the row's c = M + log2(sum of exp2(logit - M)).
constexpr float kLog2eOver8 = (float)(1.4426950408889634 / 8.0);
__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }  // exp2(-inf) = 0

// max of floats on the VALU max instructions, without the operand canonicalisation the
// compiler adds around fmaxf: v_max_f32 and the three-input v_max3_f32. The operands are
// scores, statistics and probabilities (finite or -inf), whose maximum is exact.
__device__ __forceinline__ float vmax(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float vmax3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

__device__ __forceinline__ int valid_len(const FwdParams& p, int b) {
  int len = p.seq_lens ? p.seq_lens[b] : p.n;
  return min(max(len, 1), p.n);
}

// P V for one 64-key tile: acc holds the probabilities (S^T layout), Vs the H~ tile.
__device__ __forceinline__ void pv_tile(f32x4_t y[4], const f32x4_t acc[4], const uint16_t* Vs, int r16, int g) {
  // 32 keys per MFMA: k-slots 0..3 = keys 32 pp + 4 g + (0..3), 4..7 = keys 32 pp + 16 + 4 g + (0..3)
#pragma unroll
  for (int pp = 0; pp < 2; ++pp) {
    const uint4 pa = make_uint4(pack_bf16x2(acc[2 * pp][0], acc[2 * pp][1]), pack_bf16x2(acc[2 * pp][2], acc[2 * pp][3]),
                                pack_bf16x2(acc[2 * pp + 1][0], acc[2 * pp + 1][1]),
                                pack_bf16x2(acc[2 * pp + 1][2], acc[2 * pp + 1][3]));
    const bf16x8_t a = __builtin_bit_cast(bf16x8_t, pa);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      // lane (g, r16) addresses key 32 pp + 4 g + r16 / 4, columns 16 c + 4 (r16 % 4) .. + 3
      // rows 32 pp + 4 g + r16 / 4 and 16 further (the same permutation: it depends on row & 7)
      const uint16_t* vrow = Vs + kv_at(32 * pp + 4 * g + (r16 >> 2), 16 * c + 4 * (r16 & 3));
      const uint2 lo = lds_read_tr16(vrow);
      const uint2 hi = lds_read_tr16(vrow + 16 * kStrideBf);
      const bf16x8_t bv = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
      y[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bv, y[c], 0, 0, 0);
    }
  }
}

__device__ __forceinline__ void pv_tile(f32x4_t y[4], const f32x4_t acc[4], const float* Vs, int r16, int g) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* vrow = Vs + (16 * s + 4 * g + i) * kStrideF + r16;
#pragma unroll
      for (int c = 0; c < 4; ++c) y[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(acc[s][i], vrow[16 * c], y[c], 0, 0, 0);
    }
}

struct BlockCtx {
  int qt, h, b, tid, wave, lane, r16, g, n, d_out, len, q, ntl;
  int half;       // local window: keys within half of the query (0: full attention)
  int tlo, thi;   // key tiles visited: 0, then tlo .. thi (tlo >= 1)
  int klo, kspan; // local window: the lane's query attends keys klo .. klo + kspan, and key 0
};

// One-dimensional grid of qtiles * H * B blocks. Consecutive blocks go to the 8 XCDs in
// turn, each with its own L2; the query tiles of one (batch row, head) read the same K
// (and H~) tile, so they are placed 8 block ids apart, on the same XCD, and the second
// read hits its L2 (when H * B is a multiple of 8; otherwise in plain order).
__device__ __forceinline__ BlockCtx block_ctx(const FwdParams& p) {
  BlockCtx c;
  const int bid = blockIdx.x, Q = p.qtiles, P = p.H * p.B;
  int pair;
  if (P % 8 == 0) {
    const int G = 8 * Q, w = bid % G;
    pair = bid / G * 8 + w % 8;
    c.qt = w / 8;
  } else {
    pair = bid / Q;
    c.qt = bid % Q;
  }
  c.h = pair % p.H;
  c.b = pair / p.H;
  c.tid = threadIdx.x;
  c.wave = c.tid >> 6;
  c.lane = c.tid & 63;
  c.r16 = c.lane & 15;
  c.g = c.lane >> 4;
  c.n = p.n;
  c.d_out = p.d_out;
  c.len = valid_len(p, c.b);
  c.q = c.qt * kTile + c.wave * 16 + c.r16;
  c.ntl = (c.len + kTile - 1) / kTile;  // tiles past the valid length are all masked
  c.half = p.band_half;
  c.tlo = 1;
  c.thi = c.ntl - 1;
  c.klo = 0;
  c.kspan = 0;
  if (c.half > 0) {  // the window cut to the valid keys; every valid key for query 0
    int lo = c.q == 0 ? 0 : max(0, c.q - c.half);
    int hi = c.q == 0 ? c.len - 1 : min(c.len - 1, c.q + c.half);
    if (hi < lo) lo = hi = 1 << 30;  // a padded query past the window's reach: key 0 only
    c.klo = lo;
    c.kspan = hi - lo;
  }
  if (c.half > 0 && c.qt > 0) {  // the window of queries q0 .. q0 + 63
    const int q0 = c.qt * kTile;
    c.tlo = max(1, max(q0 - c.half, 0) / kTile);
    c.thi = min(c.ntl - 1, (q0 + kTile - 1 + c.half) / kTile);
  }
  return c;
}

// Key tiles a block visits, in order: tile 0, then tlo .. thi.
__device__ __forceinline__ int tile_count(const BlockCtx& c) { return 1 + max(0, c.thi - c.tlo + 1); }
__device__ __forceinline__ int tile_at(const BlockCtx& c, int idx) { return idx == 0 ? 0 : c.tlo + idx - 1; }

// Key e = 16 s + 4 g + i of tile kt (lim = len - 64 kt) is attended by the lane's query:
// a valid key (full attention), or a key in klo .. klo + kspan or key 0 (local window; one
// unsigned compare per key).
template <bool BAND>
__device__ __forceinline__ bool key_ok(const BlockCtx& c, int kt, int lim, int s, int i) {
  const int e = 16 * s + 4 * c.g + i;
  if constexpr (BAND) {
    const bool in = (unsigned)(kt * kTile + e - c.klo) <= (unsigned)c.kspan;
    return (s == 0 && i == 0) ? (in || (kt == 0 && c.g == 0)) : in;
  } else {
    return lim >= kTile || e < lim;
  }
}

// The same for the output pass's probabilities (S^T layout): masked keys get 0.
template <bool BAND>
__device__ __forceinline__ void mask_tile(f32x4_t acc[4], const BlockCtx& c, int kt, int lim) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (!key_ok<BAND>(c, kt, lim, s, i)) acc[s][i] = 0.f;
}

// Writes Y rows of the wave's queries: y[cc][i] = Y[query 4 g + i][column 16 cc + l % 16].
__device__ __forceinline__ void store_y(const FwdParams& p, const BlockCtx& c, const f32x4_t y[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = c.qt * kTile + c.wave * 16 + 4 * c.g + i;
    if (row < c.n) {
      float* yrow = p.Y + ((int64_t)c.b * c.n + row) * c.d_out + c.h * kDHead + c.r16;
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) yrow[16 * cc] = y[cc][i];
    }
  }
}

// ------------------------------------------------------------------ score pass
// The score pass computes S = Q K^T (Q as the MFMA A operand): lane (g, r16) of a wave
// holds the scores of its queries qw + 4 g + i (i < 4, qw = the wave's first query) with
// keys 16 s + r16 of each tile, so the statistics of a query row reduce over the 16 lanes
// of a lane row and the column max of a key reduces over four values in registers and the
// four lane rows. Softmax statistics are kept per query as c = M + log2(sum of exp2(logit -
// M)), so that A = exp2(dot a log2(e) - c) (one fma, one exp2; the output pass computes A
// the same way), and the column max is taken on t = dot a log2(e) - c before a single exp2
// per key: m = exp2(max t) = max A, because exp2 is monotone.

// The wave's four queries of lane row g under a local window: each attends keys
// klo .. klo + kspan (its window cut to the valid keys; all of them for query 0) and key 0.
struct RowQ {
  int klo[4], kspan[4];
};

template <bool BAND>
__device__ __forceinline__ RowQ row_queries(const BlockCtx& c) {
  RowQ r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r.klo[i] = 0;
    r.kspan[i] = 0;
    if constexpr (BAND) {
      const int q = c.qt * kTile + c.wave * 16 + 4 * c.g + i;
      int lo = q == 0 ? 0 : max(0, q - c.half);
      int hi = q == 0 ? c.len - 1 : min(c.len - 1, q + c.half);
      if (hi < lo) lo = hi = 1 << 30;  // a padded query past the window's reach: key 0 only
      r.klo[i] = lo;
      r.kspan[i] = hi - lo;
    }
  }
  return r;
}

// Key 16 s + r16 of tile kt (lim = len - 64 kt) is attended by query i of the lane row.
template <bool BAND>
__device__ __forceinline__ bool key_ok_q(const BlockCtx& c, const RowQ& rq, int kt, int lim, int s, int i) {
  if constexpr (BAND) {
    const bool in = (unsigned)(kt * kTile + 16 * s + c.r16 - rq.klo[i]) <= (unsigned)rq.kspan[i];
    return s == 0 ? (in || (kt == 0 && c.r16 == 0)) : in;
  } else {
    return lim >= kTile || 16 * s + c.r16 < lim;
  }
}

// Masks the scores of a tile the lane's queries do not all attend (a partial last tile, a
// local window): called only for such tiles, so that full tiles pay no per-key test.
template <bool BAND>
__device__ __forceinline__ void mask_tile_q(f32x4_t acc[4], const BlockCtx& c, const RowQ& rq, int kt, int lim,
                                            float fill) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (!key_ok_q<BAND>(c, rq, kt, lim, s, i)) acc[s][i] = fill;
}

// Offset of the column-max argument of query i: c (full attention) or c - log2 |S_q|
// (local window, the count rule's per-row factor); +inf for padded queries (excluded).
template <bool BAND>
__device__ __forceinline__ float colmax_offset(const BlockCtx& c, const RowQ& rq, int i, float cq) {
  const int q = c.qt * kTile + c.wave * 16 + 4 * c.g + i;
  if (q >= c.len) return INFINITY;
  if constexpr (BAND) {
    const int nk = rq.kspan[i] + 1 + (rq.klo[i] > 0 ? 1 : 0);
    return cq - __builtin_amdgcn_logf((float)nk);
  } else {
    return cq;
  }
}

// S = Q K^T for the 64 keys in LDS: acc[s][i] = dot(query 4 g + i, key 16 s + r16).
__device__ __forceinline__ void score_tile_qk(f32x4_t acc[4], const uint16_t* Ks, const QFrag<1>& q, int r16,
                                              int g) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    acc[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const bf16x8_t b = *reinterpret_cast<const bf16x8_t*>(Ks + kv_at(16 * s + r16, 32 * ks + 8 * g));
      acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q.v[ks], b, acc[s], 0, 0, 0);
    }
  }
}

__device__ __forceinline__ void score_tile_qk(f32x4_t acc[4], const float* Ks, const QFrag<0>& q, int r16, int g) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    acc[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const float* krow = Ks + (16 * s + r16) * kStrideF + 16 * g;
#pragma unroll
    for (int t = 0; t < 16; ++t)
      acc[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(q.v[t], krow[t], acc[s], 0, 0, 0);
  }
}

// Reductions over the 16 lanes of a lane row (DPP butterflies; every lane gets the result).
template <int CTRL>
__device__ __forceinline__ float row_max_step(float v) { return vmax(v, dpp_f32<CTRL>(v)); }
__device__ __forceinline__ float row16_max_sel(float v) {
  return row_max_step<0x140>(row_max_step<0x141>(row_max_step<0x4E>(row_max_step<0xB1>(v))));
}
template <int CTRL>
__device__ __forceinline__ float row_sum_step(float v) { return v + dpp_f32<CTRL>(v); }
__device__ __forceinline__ float row16_sum(float v) {
  return row_sum_step<0x140>(row_sum_step<0x141>(row_sum_step<0x4E>(row_sum_step<0xB1>(v))));
}
// (reference, sum of exp2(logit - reference)) pairs of the 16 lanes of a row combined,
// rescaled to the larger reference; a lane with no attended key holds (-inf or a reference
// below every logit, 0).
template <int CTRL>
__device__ __forceinline__ void row_stat_step(float& M, float& L) {
  const float m2 = dpp_f32<CTRL>(M), l2 = dpp_f32<CTRL>(L);
  const float Mn = vmax(M, m2);
  const float a = M == -INFINITY ? 0.f : __fmul_rn(L, exp2_fast(__fsub_rn(M, Mn)));
  const float b = m2 == -INFINITY ? 0.f : __fmul_rn(l2, exp2_fast(__fsub_rn(m2, Mn)));
  L = a + b;
  M = Mn;
}

// Column statistic of one tile, t = dot a log2(e) - cc[i]: the max of t over the lane's four
// queries (max rule) or the sum of exp2(t) = A (mean rule), per key 16 s + r16, left in
// cml[g][r16][s] (the wave's slot of the tile) for the combination over the four lane rows
// and the four waves (col_combine).
template <int IMP>
__device__ __forceinline__ void tile_colstat(const f32x4_t acc[4], const float cc[4], float (*cml)[16][4],
                                             const BlockCtx& c) {
  float v[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if constexpr (IMP == 1) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) t += exp2_fast(__fmaf_rn(acc[s][i], kLog2eOver8, -cc[i]));
      v[s] = t;
    } else {
      float t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = __fmaf_rn(acc[s][i], kLog2eOver8, -cc[i]);
      v[s] = vmax(vmax3(t[0], t[1], t[2]), t[3]);
    }
  }
  *reinterpret_cast<float4*>(&cml[c.g][c.r16][0]) = make_float4(v[0], v[1], v[2], v[3]);
}

// The block's partial of key e (< 64) of a tile from its sixteen values (four waves x four
// lane rows) in a fixed order: exp2 of the max (max rule; SCALED: the values are dot - c / s
// and the max is multiplied by s first) or the sum (mean rule).
template <int IMP, bool SCALED = false>
__device__ __forceinline__ float col_combine(const float (*cmt)[4][16][4], int e) {
  const int r16 = e & 15, sk = e >> 4;
  float x[16];
#pragma unroll
  for (int w = 0; w < 4; ++w)
#pragma unroll
    for (int g = 0; g < 4; ++g) x[4 * w + g] = cmt[w][g][r16][sk];
  if constexpr (IMP == 1) {
    float a[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) a[w] = (x[4 * w] + x[4 * w + 1]) + (x[4 * w + 2] + x[4 * w + 3]);
    return (a[0] + a[1]) + (a[2] + a[3]);
  } else {
    const float a = vmax3(x[0], x[1], x[2]), b = vmax3(x[3], x[4], x[5]), d = vmax3(x[6], x[7], x[8]);
    const float f = vmax3(x[9], x[10], x[11]), g = vmax3(x[12], x[13], x[14]);
    const float m = vmax3(vmax3(a, b, d), vmax3(f, g, x[15]), a);
    return exp2_fast(SCALED ? __fmul_rn(m, kLog2eOver8) : m);
  }
}

// Four probabilities of queries q .. q + 3 (q a multiple of 4) of one key, at dst = the
// key's row + q: one 16-byte store when all four queries exist and the row is 16-byte
// aligned (n a multiple of 4), else one store per existing query.
__device__ __forceinline__ void store_probs4(float* dst, float a0, float a1, float a2, float a3, int q, int n) {
  if ((n & 3) == 0 && q + 3 < n) {
    *reinterpret_cast<float4*>(dst) = make_float4(a0, a1, a2, a3);
  } else {
    if (q < n) dst[0] = a0;
    if (q + 1 < n) dst[1] = a1;
    if (q + 2 < n) dst[2] = a2;
    if (q + 3 < n) dst[3] = a3;
  }
}

// Median rule: the probabilities of one tile, A = exp2(dot a log2(e) - c), into the per-key
// array acol[b n + key][h][query].
__device__ __forceinline__ void store_probs(const FwdParams& p, const BlockCtx& c, const f32x4_t acc[4], int kt,
                                            const float cq[4], int qw) {
  float* ac = p.acol + (int64_t)c.b * c.n * p.H * c.n;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int key = kt * kTile + 16 * s + c.r16;
    if (key < c.n) {
      float a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = exp2_fast(__fmaf_rn(acc[s][i], kLog2eOver8, -cq[i]));
      store_probs4(ac + ((int64_t)key * p.H + c.h) * c.n + qw, a[0], a[1], a[2], a[3], qw, c.n);
    }
  }
}

// c of query qw + 4 g + i from lane r16 = i of each lane row.
__device__ __forceinline__ void store_row_c(const FwdParams& p, const BlockCtx& c, const float cq[4]) {
  const int q = c.qt * kTile + c.wave * 16 + 4 * c.g + c.r16;
  if (c.r16 < 4 && q < c.n) {
    const float v = c.r16 == 0 ? cq[0] : c.r16 == 1 ? cq[1] : c.r16 == 2 ? cq[2] : cq[3];
    p.row_c[((int64_t)c.b * p.H + c.h) * c.n + q] = v;
  }
}

// Resident variant: all ntl <= NT tiles in LDS and all scores in registers.
template <int BF, int NT, bool BAND, int IMP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_scores_res(FwdParams p) {
  using T = typename Elem<BF>::T;
  constexpr int S = stride_of<BF>();
  __shared__ __align__(16) T Ks[NT][kTile * S];
  __shared__ __align__(16) float cm[NT][4][4][16][4];  // [tile][wave][lane row][r16][s]
  const BlockCtx c = block_ctx(p);
  const T* Qb = static_cast<const T*>(p.Q) + (int64_t)c.b * c.n * c.d_out + c.h * kDHead;
  const T* Kb = static_cast<const T*>(p.K) + (int64_t)c.b * c.n * c.d_out + c.h * kDHead;

  TileRegs kr[NT];
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) kr[kt] = tile_load<BF>(Kb, c.d_out, min(kt, c.ntl - 1) * kTile, c.n, c.tid);
  QFrag<BF> qf;
  load_qfrag(qf, Qb + (int64_t)min(c.q, c.n - 1) * c.d_out, c.g);
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
    if (kt < c.ntl) tile_store<BF>(kr[kt], Ks[kt], c.tid);
  lds_barrier();

  // scores in registers (masked keys -inf), the lane's max dot product per query
  const RowQ rq = row_queries<BAND>(c);
  f32x4_t acc[NT][4];
  float dmax[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    if (kt < c.ntl) {
      score_tile_qk(acc[kt], Ks[kt], qf, c.r16, c.g);
      const int lim = c.len - kt * kTile;
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i)  // a select per key: cheaper here than a branch per tile
          acc[kt][s][i] = key_ok_q<BAND>(c, rq, kt, lim, s, i) ? acc[kt][s][i] : -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        dmax[i] = vmax3(vmax3(dmax[i], acc[kt][0][i], acc[kt][1][i]), acc[kt][2][i], acc[kt][3][i]);
    }
  }
  // row statistics: M = the largest logit (rounding is monotone, so it is the rounded
  // largest dot product), then the sum of exp2(logit - M) over the row's 16 lanes
  float M[4], Ls[4], cq[4], cc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    M[i] = __fmul_rn(row16_max_sel(dmax[i]), kLog2eOver8);  // finite: key 0 is attended
    Ls[i] = 0.f;
  }
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    if (kt < c.ntl) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) Ls[i] += exp2_fast(__fmaf_rn(acc[kt][s][i], kLog2eOver8, -M[i]));
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    cq[i] = M[i] + __builtin_amdgcn_logf(row16_sum(Ls[i]));
    cc[i] = colmax_offset<BAND>(c, rq, i, cq[i]);
  }
  store_row_c(p, c, cq);

  // column max (or, mean rule, column sum) of the block's valid queries, every tile in its
  // own LDS slot (one barrier); median rule: every probability to acol as well
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    if (kt < c.ntl) {
      tile_colstat<IMP>(acc[kt], cc, cm[kt][c.wave], c);
      if constexpr (IMP == 2) store_probs(p, c, acc[kt], kt, cq, c.qt * kTile + c.wave * 16 + 4 * c.g);
    }
  }
  lds_barrier();
  float* part = p.colmax_part + (int64_t)c.b * c.n * p.nparts + c.h * p.qtiles + c.qt;
  for (int e = c.tid; e < c.ntl * kTile; e += kThreads) {
    const float v = col_combine<IMP>(cm[e / kTile], e % kTile);
    if (e < c.n) part[(int64_t)e * p.nparts] = v;
  }
}

// Streamed-resident variant (up to NT visited tiles, padded length <= 64 NT): K tiles are
// streamed through two LDS buffers as in the streaming variant, but every score stays in
// registers, so a single sweep over K gives the statistics and the column statistic (the
// streaming variant computes every score twice and keeps online statistics).
template <int BF, int NT, bool BAND, int IMP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_scores_rs(FwdParams p) {
  using T = typename Elem<BF>::T;
  constexpr int S = stride_of<BF>();
  __shared__ __align__(16) T Ks[2][kTile * S];
  __shared__ __align__(16) float cm[NT][4][4][16][4];  // [tile][wave][lane row][r16][s]
  const BlockCtx c = block_ctx(p);
  const T* Qb = static_cast<const T*>(p.Q) + (int64_t)c.b * c.n * c.d_out + c.h * kDHead;
  const T* Kb = static_cast<const T*>(p.K) + (int64_t)c.b * c.n * c.d_out + c.h * kDHead;
  const int nvis = tile_count(c);  // <= NT (the launch checks the padded length)
  // two K tiles in flight: the work per tile before its buffer's barrier is short
  TileRegs kr = tile_load<BF>(Kb, c.d_out, 0, c.n, c.tid);
  TileRegs kr2 = tile_load<BF>(Kb, c.d_out, tile_at(c, min(1, nvis - 1)) * kTile, c.n, c.tid);
  QFrag<BF> qf;
  load_qfrag(qf, Qb + (int64_t)min(c.q, c.n - 1) * c.d_out, c.g);
  const RowQ rq = row_queries<BAND>(c);

  // scores in registers (masked keys -inf); the t-th visited tile goes through K buffer
  // t & 1 (the barrier after its store also orders the reads of tile t - 2, consumed by
  // that tile's MFMAs, before it). The row sums are software pipelined: once the MFMAs of
  // tile t are issued, the terms of tile t - 1 are added, under a reference M that is the
  // row's largest logit in tile 0 (finite: key 0 is attended by every query). A sum of
  // positive terms keeps its relative precision when terms exceed 1; only a logit more than
  // about 127 log2 units above M overflows it, and then (or with non-finite scores) the
  // wave takes each row's largest logit as M and sums again (a wave-uniform branch).
  f32x4_t acc[NT][4];
  float M[4], Ls[4] = {0.f, 0.f, 0.f, 0.f};
  auto tile0_ref = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      M[i] = __fmul_rn(row16_max_sel(vmax(vmax3(acc[0][0][i], acc[0][1][i], acc[0][2][i]), acc[0][3][i])),
                       kLog2eOver8);
  };
  auto add_terms = [&](const f32x4_t a[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) Ls[i] += exp2_fast(__fmaf_rn(a[s][i], kLog2eOver8, -M[i]));
  };
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t < nvis) {
      const int kt = tile_at(c, t);
      T* buf = Ks[t & 1];
      tile_store<BF>(kr, buf, c.tid);
      lds_barrier();
      kr = kr2;
      kr2 = tile_load<BF>(Kb, c.d_out, tile_at(c, min(t + 2, nvis - 1)) * kTile, c.n, c.tid);
      score_tile_qk(acc[t], buf, qf, c.r16, c.g);
      const int lim = c.len - kt * kTile;
      if (BAND || lim < kTile) mask_tile_q<BAND>(acc[t], c, rq, kt, lim, -INFINITY);  // tile-uniform
      if (t > 0) {
        if (t == 1) tile0_ref();
        add_terms(acc[t - 1]);
      }
    }
  }
  if (nvis == 1) tile0_ref();
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (t == nvis - 1) add_terms(acc[t]);
  float Lr[4], cq[4], cc[4];
  bool bad = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    Lr[i] = row16_sum(Ls[i]);
    bad |= !(Lr[i] < INFINITY);
  }
  if (__any(bad)) {
    float dmax[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t < nvis) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          dmax[i] = vmax3(vmax3(dmax[i], acc[t][0][i], acc[t][1][i]), acc[t][2][i], acc[t][3][i]);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      M[i] = __fmul_rn(row16_max_sel(dmax[i]), kLog2eOver8);
      Ls[i] = 0.f;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (t < nvis) add_terms(acc[t]);
#pragma unroll
    for (int i = 0; i < 4; ++i) Lr[i] = row16_sum(Ls[i]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    cq[i] = M[i] + __builtin_amdgcn_logf(Lr[i]);
    cc[i] = colmax_offset<BAND>(c, rq, i, cq[i]);
  }
  store_row_c(p, c, cq);

  float* part = p.colmax_part + (int64_t)c.b * c.n * p.nparts + c.h * p.qtiles + c.qt;
  if (BAND) {  // valid keys of the tiles outside the window get a zero partial
    for (int key = kTile + c.tid; key < c.len; key += kThreads) {
      const int kt = key / kTile;
      if (kt < c.tlo || kt > c.thi) part[(int64_t)key * p.nparts] = 0.f;
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t < nvis) {
      tile_colstat<IMP>(acc[t], cc, cm[t][c.wave], c);
      if constexpr (IMP == 2) store_probs(p, c, acc[t], tile_at(c, t), cq, c.qt * kTile + c.wave * 16 + 4 * c.g);
    }
  }
  lds_barrier();
  for (int e = c.tid; e < nvis * kTile; e += kThreads) {
    const int t = e / kTile, k = e % kTile;
    const float v = col_combine<IMP>(cm[t], k);
    const int key = tile_at(c, t) * kTile + k;
    if (key < c.n) part[(int64_t)key * p.nparts] = v;
  }
}

// ------------------------------------------------------------------ Y = A H~
template <int BF, int NT, bool BAND>
__global__ __launch_bounds__(kThreads) void k_attn_res(FwdParams p) {
  using T = typename Elem<BF>::T;
  constexpr int S = stride_of<BF>();
  __shared__ __align__(16) T Ks[NT][kTile * S];
  __shared__ __align__(16) T Vs[NT][kTile * S];  // [key][column]
  const BlockCtx c = block_ctx(p);
  const int64_t off = (int64_t)c.b * c.n * c.d_out + c.h * kDHead;
  const T* Qb = static_cast<const T*>(p.Q) + off;
  const T* Kb = static_cast<const T*>(p.K) + off;
  const T* Vb = static_cast<const T*>(p.Henc) + off;

  TileRegs kr[NT], vr[NT];
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    kr[kt] = tile_load<BF>(Kb, c.d_out, min(kt, c.ntl - 1) * kTile, c.n, c.tid);
    vr[kt] = tile_load<BF>(Vb, c.d_out, min(kt, c.ntl - 1) * kTile, c.n, c.tid);
  }
  QFrag<BF> qf;
  load_qfrag(qf, Qb + (int64_t)min(c.q, c.n - 1) * c.d_out, c.g);
  const int64_t so = ((int64_t)c.b * p.H + c.h) * c.n + min(c.q, c.n - 1);
  const float cq = p.row_c[so];
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    if (kt < c.ntl) {
      tile_store<BF>(kr[kt], Ks[kt], c.tid);
      tile_store_v<BF>(vr[kt], Vs[kt], c.tid);
    }
  }
  lds_barrier();

  f32x4_t y[4];
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) y[cc] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    if (kt < c.ntl) {
      f32x4_t acc[4];
      score_tile(acc, Ks[kt], qf, c.r16, c.g);
      const int lim = c.len - kt * kTile;
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[s][i] = exp2_fast(__fmaf_rn(acc[s][i], kLog2eOver8, -cq));
      if (BAND || lim < kTile) mask_tile<BAND>(acc, c, kt, lim);  // tile-uniform
      pv_tile(y, acc, Vs[kt], c.r16, c.g);
    }
  }
  store_y(p, c, y);
}

// ------------------------------------------------------------------ Y = A H~, streaming
// The streaming output pass takes MT 16-query tiles per wave (64 MT queries per block):
// each K and H~ fragment read from LDS feeds MT MFMAs. With one query tile per wave the
// pass is bound by LDS reads; two cut its time by about a sixth at 4096 keys; three or
// four measured slower (fewer waves fit beside their accumulators), so MT = 2.

// Block context for blocks of QB queries (QB / 4 per wave); as block_ctx otherwise. FAR: under a
// local window the first block, too, visits only tile 0 and the tiles that its windows reach
// (far_from: the first key past them, which the kernel takes care of for query 0).
template <int QB, bool FAR = false>
__device__ __forceinline__ BlockCtx block_ctx_q(const FwdParams& p) {
  BlockCtx c;
  const int bid = blockIdx.x, Q = (p.n + QB - 1) / QB, P = p.H * p.B;
  int pair;
  if (P % 8 == 0) {  // the query tiles of a (batch row, head) on one XCD, as in block_ctx
    const int G = 8 * Q, w = bid % G;
    pair = bid / G * 8 + w % 8;
    c.qt = w / 8;
  } else {
    pair = bid / Q;
    c.qt = bid % Q;
  }
  c.h = pair % p.H;
  c.b = pair / p.H;
  c.tid = threadIdx.x;
  c.wave = c.tid >> 6;
  c.lane = c.tid & 63;
  c.r16 = c.lane & 15;
  c.g = c.lane >> 4;
  c.n = p.n;
  c.d_out = p.d_out;
  c.len = valid_len(p, c.b);
  c.q = c.qt * QB + c.wave * (QB / 4) + c.r16;  // query tile 0 of the wave; tile m is q + 16 m
  c.ntl = (c.len + kTile - 1) / kTile;
  c.half = p.band_half;
  c.tlo = 1;
  c.thi = c.ntl - 1;
  c.klo = 0;
  c.kspan = 0;
  if (c.half > 0 && (FAR || c.qt > 0)) {  // the window of queries q0 .. q0 + QB - 1
    const int q0 = c.qt * QB;
    c.tlo = max(1, max(q0 - c.half, 0) / kTile);
    c.thi = min(c.ntl - 1, (q0 + QB - 1 + c.half) / kTile);
  }
  return c;
}

// Under a local window query 0 attends every key. Where the others' windows end, one query is
// left of the block's 128: its keys from far_from on are taken on the vector units, 256 a round
// (8 x 1057 tokens, window 256: score pass 33.4 -> 25.9 us, output pass 22.2 -> 18.5; 4 x 4096,
// window 512: 168 -> 98 and 112 -> 62, which had waited for the first block's masked tiles). Thread tid reads chunk tid % 8 (8 values) of the
// rows tid / 8 + 32 r, r < 8, of a round: whole rows per eight lanes.
constexpr int kFarRows = 8;  // rows per thread and round
__device__ __forceinline__ int far_from(const BlockCtx& c) { return (c.thi + 1) * kTile; }
__device__ __forceinline__ int far_key(int k0, int tid, int r) { return k0 + (tid >> 3) + 32 * r; }

// The thread's chunks of a round's rows (past the valid ones: of the last).
__device__ __forceinline__ void far_load(u32x4_t (&v)[kFarRows], const uint16_t* base, const BlockCtx& c, int k0) {
#pragma unroll
  for (int r = 0; r < kFarRows; ++r)
    v[r] = *reinterpret_cast<const u32x4_t*>(base + (int64_t)min(far_key(k0, c.tid, r), c.len - 1) * c.d_out + 8 * (c.tid & 7));
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Query 0's dot products with the rows, summed over the eight lanes of a row (each gets them).
__device__ __forceinline__ void far_dots(float (&dot)[kFarRows], const u32x4_t& q, const u32x4_t (&k)[kFarRows]) {
#pragma unroll
  for (int r = 0; r < kFarRows; ++r) {
    float d = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      d = fmaf(bf16_lo(q[w]), bf16_lo(k[r][w]), d);
      d = fmaf(bf16_hi(q[w]), bf16_hi(k[r][w]), d);
    }
    d += dpp_f32<0xB1>(d);
    d += dpp_f32<0x4E>(d);
    dot[r] = d + dpp_f32<0x141>(d);  // the other four lanes' sum, by the mirror of eight
  }
}

// The window of query q (klo .. klo + kspan, and key 0), as block_ctx sets it for c.q.
// Under a local window: whether every key of tile kt is attended by every query q0 .. q0 +
// nq - 1 (then the tile needs no mask): the keys are below len and within half of each of
// those queries (query 0 attends every key below len). Wave-uniform arguments.
__device__ __forceinline__ bool band_tile_inside(const BlockCtx& c, int kt, int q0, int nq) {
  const int k0 = kt * kTile, k1 = k0 + kTile - 1;
  return k1 < c.len && k0 >= q0 + nq - 1 - c.half && k1 <= max(q0, 1) + c.half;
}

__device__ __forceinline__ void query_window(const BlockCtx& c, int q, int& klo, int& kspan) {
  int lo = q == 0 ? 0 : max(0, q - c.half);
  int hi = q == 0 ? c.len - 1 : min(c.len - 1, q + c.half);
  if (hi < lo) lo = hi = 1 << 30;
  klo = lo;
  kspan = hi - lo;
}

// S^T = K Q^T for MT 16-query tiles sharing each K fragment read.
template <int MT>
__device__ __forceinline__ void score_tile_m(f32x4_t acc[MT][4], const uint16_t* Ks, const QFrag<1> q[MT], int r16,
                                             int g) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m][s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(Ks + kv_at(16 * s + r16, 32 * ks + 8 * g));
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m][s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, q[m].v[ks], acc[m][s], 0, 0, 0);
    }
  }
}

template <int MT>
__device__ __forceinline__ void score_tile_m(f32x4_t acc[MT][4], const float* Ks, const QFrag<0> q[MT], int r16,
                                             int g) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m][s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const float* krow = Ks + (16 * s + r16) * kStrideF + 16 * g;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const float a = krow[t];
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, q[m].v[t], acc[m][s], 0, 0, 0);
    }
  }
}

// P V for MT query tiles sharing each H~ fragment read.
template <int MT>
__device__ __forceinline__ void pv_tile_m(f32x4_t y[MT][4], const f32x4_t acc[MT][4], const uint16_t* Vs, int r16,
                                          int g) {
#pragma unroll
  for (int pp = 0; pp < 2; ++pp) {
    bf16x8_t a[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
      a[m] = __builtin_bit_cast(bf16x8_t, make_uint4(pack_bf16x2(acc[m][2 * pp][0], acc[m][2 * pp][1]),
                                                     pack_bf16x2(acc[m][2 * pp][2], acc[m][2 * pp][3]),
                                                     pack_bf16x2(acc[m][2 * pp + 1][0], acc[m][2 * pp + 1][1]),
                                                     pack_bf16x2(acc[m][2 * pp + 1][2], acc[m][2 * pp + 1][3])));
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint16_t* vrow = Vs + (32 * pp + 4 * g + (r16 >> 2)) * kStrideBfWide + 16 * c + 4 * (r16 & 3);
      const uint2 lo = lds_read_tr16(vrow);
      const uint2 hi = lds_read_tr16(vrow + 16 * kStrideBfWide);
      const bf16x8_t bv = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
      for (int m = 0; m < MT; ++m) y[m][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], bv, y[m][c], 0, 0, 0);
    }
  }
}

template <int MT>
__device__ __forceinline__ void pv_tile_m(f32x4_t y[MT][4], const f32x4_t acc[MT][4], const float* Vs, int r16,
                                          int g) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* vrow = Vs + (16 * s + 4 * g + i) * kStrideF + r16;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float v = vrow[16 * c];
#pragma unroll
        for (int m = 0; m < MT; ++m) y[m][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(acc[m][s][i], v, y[m][c], 0, 0, 0);
      }
    }
}

// Software pipelined like the streaming score pass: iteration t issues the Q K^T MFMAs of tile
// t + 1 before the VALU work (exp2, bf16 packing) on tile t's scores and tile t's P V MFMAs.
// K and H~ tiles are double buffered in LDS with different schedules: K tile t + 1 is
// stored before iteration t's barrier (its buffer was last read by the Q K^T of tile t - 1,
// issued in iteration t - 2), H~ tile t + 1 after it (its buffer was last read by the P V of
// tile t - 1 in iteration t - 1, which every wave has finished once it passes the barrier).
// The bf16 instance (full attention) is held to 168 registers (three waves per SIMD), which it
// meets without spilling; the float32 ones need more.
template <int BF, bool BAND, int MT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu((BF && !BAND) ? 3 : 1))) void k_attn_stream(FwdParams p) {
  using T = typename Elem<BF>::T;
  constexpr int S = stride_of<BF>();
  constexpr int QB = 64 * MT;  // queries per block
  __shared__ __align__(16) T Ks[2][kTile * S];
  constexpr int SV = BF ? kStrideBfWide : kStrideF;  // H~ tiles: unpermuted rows
  __shared__ __align__(16) T Vs[2][kTile * SV];
  BlockCtx c = block_ctx_q<QB>(p);
  const int qw = __builtin_amdgcn_readfirstlane(c.qt * QB + c.wave * (QB / 4));  // the wave's first query
  const int64_t off = (int64_t)c.b * c.n * c.d_out + c.h * kDHead;
  const T* Qb = static_cast<const T*>(p.Q) + off;
  const T* Kb = static_cast<const T*>(p.K) + off;
  const T* Vb = static_cast<const T*>(p.Henc) + off;

  QFrag<BF> qf[MT];
  float cq[MT];
  int klo[MT], kspan[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int q = c.q + 16 * m;
    load_qfrag(qf[m], Qb + (int64_t)min(q, c.n - 1) * c.d_out, c.g);
    cq[m] = p.row_c[((int64_t)c.b * p.H + c.h) * c.n + min(q, c.n - 1)];
    klo[m] = 0;
    kspan[m] = 0;
    if (BAND) query_window(c, q, klo[m], kspan[m]);
  }

  f32x4_t y[MT][4];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) y[m][cc] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int nvis = tile_count(c);
  TileRegs kr = tile_load<BF>(Kb, c.d_out, 0, c.n, c.tid);
  TileRegs vr = tile_load<BF>(Vb, c.d_out, 0, c.n, c.tid);
  tile_store<BF>(kr, Ks[0], c.tid);
  tile_store_v<BF, true>(vr, Vs[0], c.tid);
  const int t1 = tile_at(c, min(1, nvis - 1)) * kTile;
  kr = tile_load<BF>(Kb, c.d_out, t1, c.n, c.tid);
  vr = tile_load<BF>(Vb, c.d_out, t1, c.n, c.tid);
  lds_barrier();
  f32x4_t accA[MT][4], accB[MT][4];
  score_tile_m<MT>(accA, Ks[0], qf, c.r16, c.g);
  auto step = [&](f32x4_t cur[MT][4], f32x4_t nxt[MT][4], int t) {
    const int kt = tile_at(c, t);
    const int lim = c.len - kt * kTile;
    // tile-uniform: masked scores give probability 0; under a window, tiles that every query
    // of the wave attends whole need no mask
    if (__builtin_expect(BAND ? !band_tile_inside(c, kt, qw, QB / 4) : lim < kTile, 0)) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        c.klo = klo[m];
        c.kspan = kspan[m];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (!key_ok<BAND>(c, kt, lim, s, i)) cur[m][s][i] = -INFINITY;
      }
    }
    const int nb = (t + 1) & 1;
    tile_store<BF>(kr, Ks[nb], c.tid);
    lds_barrier();
    tile_store_v<BF, true>(vr, Vs[nb], c.tid);
    const int next = tile_at(c, min(t + 2, nvis - 1)) * kTile;
    kr = tile_load<BF>(Kb, c.d_out, next, c.n, c.tid);
    vr = tile_load<BF>(Vb, c.d_out, next, c.n, c.tid);
    score_tile_m<MT>(nxt, Ks[nb], qf, c.r16, c.g);  // tile t + 1 (the last iteration repeats a tile, unused)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) cur[m][s][i] = exp2_fast(__fmaf_rn(cur[m][s][i], kLog2eOver8, -cq[m]));
    pv_tile_m<MT>(y, cur, Vs[t & 1], c.r16, c.g);
  };
  int t = 0;
  for (; t + 1 < nvis; t += 2) {
    step(accA, accB, t);
    step(accB, accA, t + 1);
  }
  if (t < nvis) step(accA, accB, t);
  // y[m][cc][i] = Y[query c.q - r16 + 16 m + 4 g + i][column 16 cc + r16]
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = c.qt * QB + c.wave * (QB / 4) + 16 * m + 4 * c.g + i;
      if (row < c.n) {
        float* yrow = p.Y + ((int64_t)c.b * c.n + row) * c.d_out + c.h * kDHead + c.r16;
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) yrow[16 * cc] = y[m][cc][i];
      }
    }
}

// ------------------------------------------------------------------ Y = A H~, streaming, bf16
// 32x32x16 MFMA tiles, 128 queries per block, 32 per wave. What bounds the pass is issue on
// each SIMD: a 32-key half tile costs a wave 8 MFMAs, 16 exp2, 16 fma and 8 bf16 packs. Next to
// vector work an MFMA of either shape costs about 8 issue cycles, an exp2 8, another vector
// instruction 4, so 32x32 tiles halve the matrix cores' share of the issue, but only where
// every MFMA has vector work beside it: an MFMA that waits in a run of MFMAs costs its full 32
// cycles (issue probe, per 32 scores of a lane: 586 cycles with one MFMA, two fma, two exp2 and
// a pack in turn, 771 with the MFMAs in blocks; 16x16 tiles 715 and 826). So half tile h runs
// as eight slots that are fixed in the source, each one MFMA and the vector work of two scores:
// the MFMAs are Q K^T of half tile h + 1 and P V of half tile h - 1, the vector work P of h.
// Each slot then reloads the fragment its MFMA has just used, for half tile h + 2 (K) or h (V).
//
// K and H~ tiles (64 keys) are loaded straight into LDS (no registers, no vector work), three
// buffers each: iteration t reads K tile t + 1 and H~ tile t, which have landed at its barrier,
// and starts the loads of K tile t + 2 and H~ tile t + 1 into the buffers last read in
// iteration t - 2, whose reads every wave had consumed before this barrier. 128-byte rows, the
// 16-byte chunks permuted per row so that each access is free of bank conflicts (measured per
// permutation): K chunk c of row r at c ^ ((r >> 1) & 7), H~ chunk c at c ^ 2 (r & 1) ^ 4 (r >> 1 & 1).
__device__ __forceinline__ int k32_swz(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int v32_swz(int row) { return ((row & 1) << 1) | ((row & 2) << 1); }

// One direct load of 16 bytes per lane through the buffer descriptor rs (four scalar words)
// at byte offset off: lane l's bytes land at lds + 16 l, zeros where the offset is out of
// range. As load_lds16: the kernel does the waiting, and the s_nop is M0's wait state.
__device__ __forceinline__ void buffer_load_lds16(u32x4_t rs, uint32_t off, uint32_t lds) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(off), "s"(rs), "{m0}"(lds) : "memory");
}

// Descriptor of the 32 rows from key0 on of a [*, ld] bfloat16 matrix (the head's column slice),
// as four scalar words; rows at or past n are out of range (as tile_rsrc).
__device__ __forceinline__ u32x4_t rows32_rsrc(const void* base, int ld, int key0, int n) {
  const int bytes = max((min(n - key0, 32) - 1) * ld * 2 + kDHead * 2, 0);
  const uint64_t a = (uint64_t)(uintptr_t)base + (uint64_t)((int64_t)key0 * ld * 2);
  u32x4_t w;
  w[0] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  w[1] = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
  w[2] = (uint32_t)__builtin_amdgcn_readfirstlane(bytes);
  w[3] = (uint32_t)kBufWord3;
  return w;
}

// s += b with the rounding error of the sum added to c (Knuth's two-sum).
__device__ __forceinline__ void add_carry(float& s, float& c, float b) {
  const float t = s + b, z = t - s;
  c += (s - (t - z)) + (b - z);
  s = t;
}

// Keeps the computation of x before this point and what follows behind it.
template <typename T>
__device__ __forceinline__ void pin(T& x) { asm volatile("" : "+v"(x)); }

template <bool BAND, int MT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(MT == 1 ? 3 : 2))) void k_attn_stream32(FwdParams p) {
  constexpr int QB = 128 * MT;
  constexpr int kTileElems = kTile * kDHead;
  __shared__ __align__(16) uint16_t smem[6 * kTileElems];  // three K tiles, three H~ tiles
  const BlockCtx c = block_ctx_q<QB, true>(p);
  const int wave = __builtin_amdgcn_readfirstlane(c.wave);
  const int qw = c.qt * QB + wave * 32 * MT;  // the wave's first query
  const int r32 = c.lane & 31, hf = c.lane >> 5, i16 = c.lane & 15;
  const int64_t off = (int64_t)c.b * c.n * c.d_out + c.h * kDHead;
  const uint16_t* Qb = static_cast<const uint16_t*>(p.Q) + off;
  const uint16_t* Kb = static_cast<const uint16_t*>(p.K) + off;
  const uint16_t* Vb = static_cast<const uint16_t*>(p.Henc) + off;
  const int nvis = tile_count(c);

  // the wave's direct loads of a tile: rows 8 wave + lane / 8 and 32 further, lane l filling
  // chunk position l % 8 of its row
  const int drow = 8 * wave + (c.lane >> 3);
  const uint32_t koff = (uint32_t)(drow * c.d_out * 2 + (((c.lane & 7) ^ k32_swz(drow)) << 4));
  const uint32_t voff = (uint32_t)(drow * c.d_out * 2 + (((c.lane & 7) ^ v32_swz(drow)) << 4));
  const uint32_t dst = lds_addr(smem) + 1024u * wave;
  auto load_tile = [&](const uint16_t* base, uint32_t loff, int t, int slot) __attribute__((always_inline)) {
    const int key0 = tile_at(c, min(t, nvis - 1)) * kTile;
    const uint32_t to = dst + (uint32_t)slot * (kTileElems * 2);
    buffer_load_lds16(rows32_rsrc(base, c.d_out, key0, c.n), loff, to);
    buffer_load_lds16(rows32_rsrc(base, c.d_out, key0 + 32, c.n), loff, to + 4096u);
  };
  load_tile(Kb, koff, 0, 0);

  // Q as the B operand of S^T = K Q^T: query qw + 32 m + r32, d = 16 ks + 8 hf .. + 7
  bf16x8_t qf[MT][4];
  float ncq[MT];
  int klo[MT], kspan[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int q = min(qw + 32 * m + r32, c.n - 1);
    const uint16_t* qrow = Qb + (int64_t)q * c.d_out + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) qf[m][ks] = *reinterpret_cast<const bf16x8_t*>(qrow + 16 * ks);
    ncq[m] = -p.row_c[((int64_t)c.b * p.H + c.h) * c.n + q];
    klo[m] = kspan[m] = 0;
    if (BAND) query_window(c, qw + 32 * m + r32, klo[m], kspan[m]);
  }

  load_tile(Kb, koff, 1, 1);  // not waited for before the first scores
  load_tile(Vb, voff, 0, 3);

  // fragment addresses (elements) in a tile: K row r32 (of a half tile), d = 16 ks + 8 hf; H~
  // rows 4 hf + i16 / 4 (+ 8, 16 pp, 32 per half tile), columns 32 cc + 16 (lane / 16 % 2) + 4 (i16 % 4)
  int ka[4], va[2];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) ka[ks] = r32 * kDHead + (((2 * ks + hf) ^ k32_swz(r32)) << 3);
#pragma unroll
  for (int cc = 0; cc < 2; ++cc) {
    const int row = 4 * hf + (i16 >> 2), col = 32 * cc + 16 * ((c.lane >> 4) & 1) + 4 * (i16 & 3);
    va[cc] = row * kDHead + ((((col >> 3) ^ v32_swz(row)) << 3) | (col & 7));
  }
  const uint16_t *kp[4], *vp[2];  // the lane's addresses in the tiles being read
  auto set_tiles = [&](int kslot, int vslot) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kp[ks] = smem + (ka[ks] + kslot * kTileElems);
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) vp[cc] = smem + (va[cc] + (3 + vslot) * kTileElems);
  };
  auto read_k = [&](int half, int ks) __attribute__((always_inline)) {
    return *reinterpret_cast<const bf16x8_t*>(kp[ks] + half * 32 * kDHead);
  };
  auto read_v = [&](int half, int pp, int cc) __attribute__((always_inline)) {
    const uint16_t* v = vp[cc] + (32 * half + 16 * pp) * kDHead;
    const uint2 lo = lds_read_tr16(v), hi = lds_read_tr16(v + 8 * kDHead);
    return __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
  };

  const f32x16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16_t y[MT][2], s0[MT], s1[MT];
  u32x4_t pa[MT][2], pb[MT][2];  // P of a half tile, 16 keys each, as A operands
  bf16x8_t kf[4], vf[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {  // the first P V multiplies zeros
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      y[m][i] = zero;
      pb[m][i] = u32x4_t{0u, 0u, 0u, 0u};
    }
    vf[i][0] = vf[i][1] = __builtin_bit_cast(bf16x8_t, pb[0][0]);
  }
  wait_vmcnt<4>();  // K tile 0 (and Q)
  stage_barrier();
  set_tiles(0, 0);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) kf[ks] = read_k(0, ks);
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
      s0[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[m][ks], ks == 0 ? zero : s0[m], 0, 0, 0);
    kf[ks] = read_k(1, ks);
  }

  // masked scores of half tile `half` of tile kt: reg i is key 64 kt + 32 half + 8 (i / 4) + 4 hf
  // + i % 4
  auto mask = [&](f32x16_t (&s)[MT], int kt, int half) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      // keys lo .. lo + span, one unsigned compare per score; key 0 on top
      const int lo = BAND ? klo[m] : 0, span = BAND ? kspan[m] : c.len - 1;
      const float key0 = s[m][0];
      const int base = kt * kTile + 32 * half + 4 * hf - lo;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        s[m][i] = (unsigned)(base + 8 * (i >> 2) + (i & 3)) <= (unsigned)span ? s[m][i] : -INFINITY;
      if (BAND && kt == 0 && half == 0 && hf == 0) s[m][0] = key0;
    }
  };
  // Half tile h: P of cur into pout, Q K^T of half tile h + 1 into nxt, P V of half tile h - 1
  // (pi, vf); K half tile h + 2 and H~ half tile h are `half` of the tiles that set_tiles chose.
  auto step = [&](f32x16_t (&cur)[MT], f32x16_t (&nxt)[MT], const u32x4_t (&pi)[MT][2], u32x4_t (&po)[MT][2], int half)
      __attribute__((always_inline)) {
    float e0 = 0.f, e1 = 0.f;
#pragma unroll
    for (int j = 0; j < 8 * MT; ++j) {
      const int i = j / (2 * MT), m = (j >> 1) % MT, pp = i >> 1, cc = i & 1;
      if (j % 2 == 0) {
        nxt[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qf[m][i], i == 0 ? zero : nxt[m], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);  // the reload takes the registers the MFMA has read
        if (m == MT - 1) kf[i] = read_k(half, i);
      } else {
        y[m][cc] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, pi[m][pp]), vf[pp][cc], y[m][cc],
                                                           0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (m == MT - 1) vf[pp][cc] = read_v(half, pp, cc);
      }
      const int n = j >> 3, k = j & 7;  // scores 2 k, + 1 of query tile n
      const float x0 = __fmaf_rn(cur[n][2 * k], kLog2eOver8, ncq[n]);
      const float x1 = __fmaf_rn(cur[n][2 * k + 1], kLog2eOver8, ncq[n]);
      if (j > 0) {  // the pair before: its exp2 results are not waited for
        uint32_t w = pack_bf16x2(e0, e1);
        pin(w);
        po[(j - 1) >> 3][((j - 1) >> 2) & 1][(j - 1) & 3] = w;
      }
      e0 = exp2_fast(x0);
      e1 = exp2_fast(x1);
      pin(e0);
      pin(e1);
      __builtin_amdgcn_sched_barrier(0);
    }
    po[MT - 1][1][3] = pack_bf16x2(e0, e1);
  };
  int b0 = 0, b1 = 1, b2 = 2;  // buffers of tiles t, t + 1, t + 2
#pragma clang loop unroll(disable)
  for (int t = 0; t < nvis; ++t) {
    wait_vmcnt<0>();
    stage_barrier();
    load_tile(Kb, koff, t + 2, b2);
    load_tile(Vb, voff, t + 1, 3 + b1);
    set_tiles(b1, b0);
    const int kt = tile_at(c, t);
    const bool masked = BAND ? !band_tile_inside(c, kt, qw, 32 * MT) : c.len - kt * kTile < kTile;  // wave-uniform
    if (__builtin_expect(masked, 0)) mask(s0, kt, 0);
    step(s0, s1, pb, pa, 0);
    if (__builtin_expect(masked, 0)) mask(s1, kt, 1);
    step(s1, s0, pa, pb, 1);
    const int b = b0;
    b0 = b1;
    b1 = b2;
    b2 = b;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int m = 0; m < MT; ++m)
      y[m][i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, pb[m][i >> 1]), vf[i >> 1][i & 1],
                                                            y[m][i & 1], 0, 0, 0);
  wait_vmcnt<0>();  // the trailing loads have landed before the wave ends
  if constexpr (BAND) {
    if (c.qt == 0 && far_from(c) < c.len) {  // block-uniform: query 0's far keys
      static_assert(MT == 1, "query 0 is in the wave's first query tile");
      float* ps = reinterpret_cast<float*>(smem);  // [32][64] partial sums
      const u32x4_t q0 = *reinterpret_cast<const u32x4_t*>(Qb + 8 * (c.tid & 7));
      const float ncq0 = -p.row_c[((int64_t)c.b * p.H + c.h) * c.n];
      float yf[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // columns 8 (tid % 8) .. + 7
      for (int k0 = far_from(c); k0 < c.len; k0 += kThreads) {
        u32x4_t k[kFarRows], v[kFarRows];
        far_load(k, Kb, c, k0);
        far_load(v, Vb, c, k0);
        float dot[kFarRows];
        far_dots(dot, q0, k);
#pragma unroll
        for (int r = 0; r < kFarRows; ++r) {
          if (far_key(k0, c.tid, r) < c.len) {
            const float a = exp2_fast(__fmaf_rn(dot[r], kLog2eOver8, ncq0));
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              yf[2 * w] = fmaf(a, bf16_lo(v[r][w]), yf[2 * w]);
              yf[2 * w + 1] = fmaf(a, bf16_hi(v[r][w]), yf[2 * w + 1]);
            }
          }
        }
      }
      __syncthreads();  // the tiles have been read
#pragma unroll
      for (int e = 0; e < 8; ++e) ps[8 * c.tid + e] = yf[e];
      __syncthreads();
      if (wave == 0) {
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) {
          float a = 0.f;
          for (int g = 0; g < 32; ++g) a += ps[g * kDHead + 32 * cc + r32];
          y[0][cc][0] += hf == 0 ? a : 0.f;  // query 0
        }
      }
    }
  }
  // y[m][cc][i] = Y[query qw + 32 m + 8 (i / 4) + 4 hf + i % 4][column 32 cc + r32]
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = qw + 32 * m + 8 * (i >> 2) + 4 * hf + (i & 3);
      if (row < c.n) {
        float* yrow = p.Y + ((int64_t)c.b * c.n + row) * c.d_out + c.h * kDHead + r32;
        yrow[0] = y[m][0][i];
        yrow[32] = y[m][1][i];
      }
    }
}

// ------------------------------------------------------------------ score pass, streaming, float32
// float32 rows longer than 8 key tiles: 128 queries per block, two 16-query
// tiles per wave, so that every K fragment read from LDS feeds two MFMAs and the per-tile
// work (tile loads and stores, barriers, lane swaps, partial stores) serves twice the
// queries. Two sweeps over the visited tiles: per-lane row statistics, then the column
// statistic, one partial per (key, head, 128-query tile).
//
// Both sweeps are software pipelined: the MFMAs of tile t + 1 are issued before the VALU
// work on tile t's scores, so the matrix cores and the vector units of a wave work at the
// same time (a wave's MFMA results are only read one iteration later). The loop is unrolled
// by two so that the two accumulator sets swap roles without register copies.
//
// Sweep 2 folds the row normaliser into the MFMA: its accumulators start at -c_q / s
// (s = log2(e) / 8) instead of 0, so an accumulator holds dot - c_q / s, whose maximum over
// the lane's queries needs no per-score arithmetic; the maximum over the block is scaled by
// s once per key: t = s * max(dot - c_q / s) = max(dot s - c_q) (s > 0).

// S = Q K^T of two 16-query tiles: acc[m][s][i] = dot(query 16 m + 4 g + i, key 16 s + r16)
// + init[m][i].
__device__ __forceinline__ void score_tile_qk2(f32x4_t acc[2][4], const float* Ks, const QFrag<0> q[2], int r16,
                                               int g, const f32x4_t init[2]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    acc[0][s] = init[0];
    acc[1][s] = init[1];
    const float* krow = Ks + (16 * s + r16) * kStrideF + 16 * g;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const float b = krow[t];
      acc[0][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[0].v[t], b, acc[0][s], 0, 0, 0);
      acc[1][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(q[1].v[t], b, acc[1][s], 0, 0, 0);
    }
  }
}

// IMP: the column statistic, 0 max (Eq. 8-9), 1 mean, 2 median (every probability to acol).
template <bool BAND, int IMP>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_scores_stream(FwdParams p) {
  __shared__ __align__(16) float Ks[2][kTile * kStrideF];
  // sweep 2: per tile (three in flight), per wave and lane row, the lane row's value of key
  // 16 s + r16 at [r16][s]
  __shared__ __align__(16) float cm[3][4][4][16][4];
  __shared__ int redo;
  const BlockCtx c = block_ctx_q<128>(p);
  if (c.tid == 0) redo = 0;  // seen behind the first sweep's barriers
  const float* Qb = static_cast<const float*>(p.Q) + (int64_t)c.b * c.n * c.d_out + c.h * kDHead;
  const float* Kb = static_cast<const float*>(p.K) + (int64_t)c.b * c.n * c.d_out + c.h * kDHead;
  const int qw = __builtin_amdgcn_readfirstlane(c.qt * 128 + c.wave * 32);  // the wave's first query
  QFrag<0> qf[2];
#pragma unroll
  for (int m = 0; m < 2; ++m) load_qfrag(qf[m], Qb + (int64_t)min(qw + 16 * m + c.r16, c.n - 1) * c.d_out, c.g);
  // the lane's eight queries qw + 16 m + 4 g + i in slot 4 m + i; under a local window each
  // attends keys klo .. klo + kspan and key 0
  int klo[8], kspan[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    klo[k] = 0;
    kspan[k] = 0;
    if constexpr (BAND) query_window(c, qw + 16 * (k >> 2) + 4 * c.g + (k & 3), klo[k], kspan[k]);
  }
  // masked keys of a tile the lane's queries do not all attend (called for such tiles only)
  auto mask = [&](f32x4_t acc[2][4], int kt, int lim) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          bool ok;
          if constexpr (BAND) {
            const int key = kt * kTile + 16 * s + c.r16;
            ok = (unsigned)(key - klo[4 * m + i]) <= (unsigned)kspan[4 * m + i] || key == 0;
          } else {
            ok = 16 * s + c.r16 < lim;
          }
          if (!ok) acc[m][s][i] = -INFINITY;
        }
  };
  const int nvis = tile_count(c);
  // One sweep over the visited tiles, software pipelined: K tile t + 1 is staged in LDS buffer
  // (t + 1) & 1 and its scores issued on the matrix cores before `work` runs on tile t's
  // scores. The barrier of iteration t orders the LDS stores of tile t + 1 before their reads
  // and the reads of tile t - 1 (same buffer, two iterations earlier) before those stores.
  // Every iteration does the same (the last one stages and multiplies the last tile again,
  // with results unused): one straight-line region per tile, and a barrier in every iteration
  // (sweep 2 combines the waves' values of tile t - 1 after iteration t's barrier).
  // `first` sees tile 0's scores (masked) before the loop.
  auto sweep = [&](const f32x4_t init[2], auto&& first, auto&& work) {
    TileRegs kr = tile_load<0>(Kb, c.d_out, 0, c.n, c.tid);
    tile_store<0>(kr, Ks[0], c.tid);
    kr = tile_load<0>(Kb, c.d_out, tile_at(c, min(1, nvis - 1)) * kTile, c.n, c.tid);
    lds_barrier();
    f32x4_t accA[2][4], accB[2][4];
    score_tile_qk2(accA, Ks[0], qf, c.r16, c.g, init);
    first(accA);
    auto step = [&](f32x4_t cur[2][4], f32x4_t nxt[2][4], int t) {
      const int kt = tile_at(c, t);
      const int lim = c.len - kt * kTile;
      if (BAND ? !band_tile_inside(c, kt, qw, 32) : lim < kTile) mask(cur, kt, lim);  // tile-uniform
      float* buf = Ks[(t + 1) & 1];
      tile_store<0>(kr, buf, c.tid);
      lds_barrier();
      kr = tile_load<0>(Kb, c.d_out, tile_at(c, min(t + 2, nvis - 1)) * kTile, c.n, c.tid);
      score_tile_qk2(nxt, buf, qf, c.r16, c.g, init);
      work(cur, t, kt);
    };
    int t = 0;
    for (; t + 1 < nvis; t += 2) {
      step(accA, accB, t);
      step(accB, accA, t + 1);
    }
    if (t < nvis) step(accA, accB, t);
  };

  // Sweep 1: per lane and query, a reference logit M and the sum of exp2(logit - M) over
  // the lane's keys; the 16 lanes of a row are combined at the end. M is the row's largest
  // logit in tile 0 (finite: key 0 is attended by every query), and every later term is
  // added under it, with no check per tile: the terms of a positive sum may exceed 1 without
  // losing relative precision, and only a sum of 2^128 or more (logits 127 log2 units above M)
  // overflows. If any row's sum came out non-finite (that, or non-finite scores), the block runs the
  // sweep again the careful way: terms added under the current reference as long as a tile's
  // four terms of a query sum to at most 2^16, otherwise (the first tile, and rarely later)
  // the tile redone with M raised to the running max and the sum rescaled (wave-uniform).
  constexpr float kNoMax = -1e30f;  // below every logit: no attended key seen yet
  constexpr float kRaise = 65536.f;
  float M[8], Ls[8];
  const f32x4_t zero2[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int k = 0; k < 8; ++k) Ls[k] = 0.f;
  sweep(
      zero2,
      [&](f32x4_t acc[2][4]) {
        if (BAND ? !band_tile_inside(c, 0, qw, 32) : c.len < kTile) mask(acc, 0, c.len);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int m = k >> 2, i = k & 3;
          const float dm = vmax(vmax3(acc[m][0][i], acc[m][1][i], acc[m][2][i]), acc[m][3][i]);
          M[k] = __fmul_rn(row16_max(dm), kLog2eOver8);
        }
      },
      [&](f32x4_t acc[2][4], int, int) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int m = k >> 2, i = k & 3;
          float e = exp2_fast(__fmaf_rn(acc[m][0][i], kLog2eOver8, -M[k]));
#pragma unroll
          for (int s = 1; s < 4; ++s) e += exp2_fast(__fmaf_rn(acc[m][s][i], kLog2eOver8, -M[k]));
          Ls[k] += e;
        }
      });
  bool overflow = false;  // of the row's sum: lanes' parts that are finite may add up to infinity
#pragma unroll
  for (int k = 0; k < 8; ++k) overflow |= !(row16_sum(Ls[k]) < INFINITY);
  if (overflow) redo = 1;
  lds_barrier();  // the first sweep is done with both K buffers
  if (redo) {     // block-uniform: every wave stages its share of the tiles and meets the barriers
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      M[k] = kNoMax;
      Ls[k] = 0.f;
    }
    sweep(
        zero2, [&](f32x4_t[2][4]) {},
        [&](f32x4_t acc[2][4], int, int) {
          float ts[8];
          bool raise = false;
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int m = k >> 2, i = k & 3;
            float e = exp2_fast(__fmaf_rn(acc[m][0][i], kLog2eOver8, -M[k]));
#pragma unroll
            for (int s = 1; s < 4; ++s) e += exp2_fast(__fmaf_rn(acc[m][s][i], kLog2eOver8, -M[k]));
            ts[k] = e;
            raise |= !(e <= kRaise);
          }
          if (__any(raise)) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const int m = k >> 2, i = k & 3;
              const float dm = vmax(vmax3(acc[m][0][i], acc[m][1][i], acc[m][2][i]), acc[m][3][i]);
              const float Mn = vmax(M[k], __fmul_rn(dm, kLog2eOver8));
              float e = exp2_fast(__fmaf_rn(acc[m][0][i], kLog2eOver8, -Mn));
#pragma unroll
              for (int s = 1; s < 4; ++s) e += exp2_fast(__fmaf_rn(acc[m][s][i], kLog2eOver8, -Mn));
              Ls[k] = __fmul_rn(Ls[k], exp2_fast(__fsub_rn(M[k], Mn))) + e;
              M[k] = Mn;
            }
          } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) Ls[k] += ts[k];
          }
        });
  }
  float cq[8], cc[8];
  f32x4_t dneg[2];  // sweep 2's accumulator start: -cc / s per query (-inf for padded queries)
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    float Mi = M[k], Li = Ls[k];
    row_stat_step<0xB1>(Mi, Li);
    row_stat_step<0x4E>(Mi, Li);
    row_stat_step<0x141>(Mi, Li);
    row_stat_step<0x140>(Mi, Li);
    cq[k] = Mi + __builtin_amdgcn_logf(Li);  // finite: key 0 is attended by every query
    // the column statistic's offset: c, or c - log2 |S_q| under a window; +inf for
    // padded queries (excluded)
    const int q = qw + 16 * (k >> 2) + 4 * c.g + (k & 3);
    float off = cq[k];
    if constexpr (BAND) off = cq[k] - __builtin_amdgcn_logf((float)(kspan[k] + 1 + (klo[k] > 0 ? 1 : 0)));
    cc[k] = q >= c.len ? INFINITY : off;
    dneg[k >> 2][k & 3] = -__fdiv_rn(cc[k], kLog2eOver8);
  }
  {  // c of query qw + 16 m + 4 g + i from lane r16 = 4 m + i of each lane row
    float v = cq[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) v = c.r16 == k ? cq[k] : v;
    const int q = qw + 16 * (c.r16 >> 2) + 4 * c.g + (c.r16 & 3);
    if (c.r16 < 8 && q < c.n) p.row_c[((int64_t)c.b * p.H + c.h) * c.n + q] = v;
  }

  // Sweep 2: the per-key column statistic of this block's valid queries. Each lane row of each
  // wave leaves its value of tile t's keys (over its four queries of each of the wave's two
  // query tiles) in cm[t % 3][wave][row]; after the barrier of iteration t + 1 (or the final
  // one), threads 0..63 combine the sixteen values of a key in a fixed order and store the
  // block's partial. A slot is reused three tiles later, after two more barriers.
  float* part = p.colmax_part + (int64_t)c.b * c.n * p.nparts + c.h * p.qtiles + c.qt;
  if (BAND) {  // valid keys of the tiles outside the window get a zero partial
    for (int key = kTile + c.tid; key < c.len; key += kThreads) {
      const int kt = key / kTile;
      if (kt < c.tlo || kt > c.thi) part[(int64_t)key * p.nparts] = 0.f;
    }
  }
  constexpr bool sum = IMP == 1;
  auto combine = [&](int t) {  // the block's partial of tile t's keys
    if (c.tid < kTile) {
      const float r = col_combine<IMP == 1 ? 1 : 0, true>(cm[t % 3], c.tid);
      const int key = tile_at(c, t) * kTile + c.tid;
      if (key < c.n) part[(int64_t)key * p.nparts] = r;
    }
  };
  lds_barrier();  // sweep 1 is done with both K buffers
  sweep(dneg, [&](f32x4_t[2][4]) {}, [&](f32x4_t acc[2][4], int t, int kt) {
    // the lane's eight queries per key: the max of dot - cc / s (or the sum of the
    // probabilities exp2(s (dot - cc / s))), left in cm for the combination over the lane
    // rows and waves
    float v[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if constexpr (sum) {
        float e = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) e += exp2_fast(__fmul_rn(acc[k >> 2][s][k & 3], kLog2eOver8));
        v[s] = e;
      } else {
        v[s] = vmax3(vmax3(acc[0][s][0], acc[0][s][1], acc[0][s][2]), vmax3(acc[0][s][3], acc[1][s][0], acc[1][s][1]),
                     vmax(acc[1][s][2], acc[1][s][3]));
      }
    }
    *reinterpret_cast<float4*>(&cm[t % 3][c.wave][c.g][c.r16][0]) = make_float4(v[0], v[1], v[2], v[3]);
    if constexpr (IMP == 2) {  // median rule: every probability, exp2(s (dot - cc / s))
      float* ac = p.acol + (int64_t)c.b * c.n * p.H * c.n;
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int key = kt * kTile + 16 * s + c.r16;
          if (key < c.n) {
            const int q = qw + 16 * m + 4 * c.g;
            float a[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = exp2_fast(__fmul_rn(acc[m][s][i], kLog2eOver8));
            store_probs4(ac + ((int64_t)key * p.H + c.h) * c.n + q, a[0], a[1], a[2], a[3], q, c.n);
          }
        }
    }
    if (t > 0) combine(t - 1);  // the barrier of this iteration follows every wave's tile t - 1 values
  });
  lds_barrier();
  combine(nvis - 1);
}

// ------------------------------------------------------------------ score pass, streaming, bf16
// The two sweeps of the streaming score pass on 32x32x16 MFMA tiles, 32 MT queries per wave
// (128 MT per block), with k_attn_stream32's K tiles, fragments and fixed slots.
//
// Sweep 1 takes S^T = K Q^T: a lane holds 16 keys of one query per half tile, so a query's
// reference M and running sum are one register each. A slot is one MFMA (half tile h + 1) and
// fma, exp2 and add of four scores of half tile h.
// Sweep 2 takes S = Q K^T from the same fragments: a lane holds 16 queries of one key, whose
// maximum needs eight three-input maxima and one exchange between the wave's two halves, made
// with the other waves' through LDS. Its accumulators start at -c / s. A slot is one MFMA and
// two of the maxima.
//
// What bounds it: issue on the SIMDs, and at 4096 tokens the clock, which the card lowers under
// this work (2.1 GHz reported over 5 s of passes, 2.4 in BERT-base layers), so that LDS reads and
// tile loads count beside the arithmetic: 64 queries per wave share them. K tiles
// take four buffers and load two iterations ahead, through the end of one sweep into the next.
template <bool BAND, int IMP, int MT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_scores_stream32(FwdParams p) {
  constexpr int QB = 128 * MT;
  constexpr int kTileElems = kTile * kDHead;
  __shared__ __align__(16) uint16_t smem[4 * kTileElems];
  __shared__ __align__(16) float cm[3][8][kTile];  // per tile in flight, wave and half: a value per key
  __shared__ __align__(16) float cs[4][32 * MT];   // per wave: the column statistic's offset of each query
  __shared__ int redo;
  __shared__ float far[2][16];  // query 0's far keys: sums and maxima of the lane rows
  const BlockCtx c = block_ctx_q<QB, true>(p);
  const int wave = __builtin_amdgcn_readfirstlane(c.wave);
  const int qw = c.qt * QB + wave * 32 * MT;  // the wave's first query
  const int r32 = c.lane & 31, hf = c.lane >> 5;
  const int64_t off = (int64_t)c.b * c.n * c.d_out + c.h * kDHead;
  const uint16_t* Qb = static_cast<const uint16_t*>(p.Q) + off;
  const uint16_t* Kb = static_cast<const uint16_t*>(p.K) + off;
  const int nvis = tile_count(c);

  const int drow = 8 * wave + (c.lane >> 3);
  const uint32_t koff = (uint32_t)(drow * c.d_out * 2 + (((c.lane & 7) ^ k32_swz(drow)) << 4));
  const uint32_t dst = lds_addr(smem) + 1024u * wave;
  // tile t of the sequence of sweeps (t < nvis + 3): each sweep visits the same tiles
  auto tile_mod = [&](int t) __attribute__((always_inline)) {
    while (t >= nvis) t -= nvis;  // at most three times
    return t;
  };
  auto load_tile = [&](int t, int slot) __attribute__((always_inline)) {  // t < nvis
    const int key0 = tile_at(c, t) * kTile;
    const uint32_t to = dst + (uint32_t)slot * (kTileElems * 2);
    buffer_load_lds16(rows32_rsrc(Kb, c.d_out, key0, c.n), koff, to);
    buffer_load_lds16(rows32_rsrc(Kb, c.d_out, key0 + 32, c.n), koff, to + 4096u);
  };
  int b0 = 0;  // buffer of tile t; tile t + i is in b0 + i mod 4
  load_tile(0, 0);
  load_tile(tile_mod(1), 1);
  load_tile(tile_mod(2), 2);
  if (c.tid == 0) redo = 0;

  bf16x8_t qf[MT][4];  // query qw + 32 m + r32, d = 16 ks + 8 hf .. + 7: the B (sweep 1) or A operand
  int klo[MT], kspan[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const uint16_t* qrow = Qb + (int64_t)min(qw + 32 * m + r32, c.n - 1) * c.d_out + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) qf[m][ks] = *reinterpret_cast<const bf16x8_t*>(qrow + 16 * ks);
    klo[m] = kspan[m] = 0;
    if (BAND) query_window(c, qw + 32 * m + r32, klo[m], kspan[m]);
  }
  int ka[4];  // fragment addresses (elements) in a tile
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) ka[ks] = r32 * kDHead + (((2 * ks + hf) ^ k32_swz(r32)) << 3);
  const uint16_t* kp[4];  // in the tile being read
  auto set_tile = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kp[ks] = smem + (ka[ks] + slot * kTileElems);
  };
  auto read_k = [&](int half, int ks) __attribute__((always_inline)) {
    return *reinterpret_cast<const bf16x8_t*>(kp[ks] + half * 32 * kDHead);
  };
  const f32x16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bf16x8_t kf[4];
  f32x16_t s0[MT], s1[MT];

  // One sweep over the visited tiles. Tiles 0 to 2 are in their buffers or on their way; at the
  // end those of the next sweep are. T: S^T = K Q^T (else S = Q K^T); init: the
  // accumulators' start; first(s): after the scores of tile 0's first half; work(cur, j, half):
  // the vector work of slot j; done(t, half): after a half tile's slots; mask(s, kt, half); ahead(t):
  // behind iteration t's barrier.
  auto sweep = [&](auto transposed, const f32x16_t (&init)[MT], auto&& first, auto&& mask, auto&& work, auto&& done,
                   auto&& ahead) __attribute__((always_inline)) {
    constexpr bool T = decltype(transposed)::value;
    auto mul = [&](f32x16_t (&nxt)[MT], int i, int m) __attribute__((always_inline)) {
      const f32x16_t a = i == 0 ? init[m] : nxt[m];
      nxt[m] = T ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qf[m][i], a, 0, 0, 0)
                 : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[m][i], kf[i], a, 0, 0, 0);
    };
    // half tile h: the work on cur, the scores of half tile h + 1 into nxt; K half tile h + 2 is
    // `half` of the tile that set_tile chose
    auto step = [&](f32x16_t (&cur)[MT], f32x16_t (&nxt)[MT], int half) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < 4 * MT; ++j) {
        const int i = j / MT, m = j % MT;
        mul(nxt, i, m);
        __builtin_amdgcn_sched_barrier(0);  // the reload takes the registers the MFMA has read
        if (m == MT - 1) kf[i] = read_k(half, i);
        work(cur, j, half);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    wait_vmcnt<2>();  // all but tile 2's
    stage_barrier();
    set_tile(b0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kf[ks] = read_k(0, ks);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int m = 0; m < MT; ++m) mul(s0, ks, m);
      kf[ks] = read_k(1, ks);
    }
    first(mul);
#pragma clang loop unroll(disable)
    for (int t = 0; t < nvis; ++t) {
      wait_vmcnt<2>();  // tile t + 1 has landed, tile t + 2 (and a partial's store) may be on its way
      if constexpr (!T) wait_lds();  // the values left in cm
      stage_barrier();
      load_tile(tile_mod(t + 3), (b0 + 3) & 3);  // the buffer of tile t - 1
      set_tile((b0 + 1) & 3);
      ahead(t);
      const int kt = tile_at(c, t);
      const bool masked = BAND ? !band_tile_inside(c, kt, qw, 32 * MT) : c.len - kt * kTile < kTile;  // wave-uniform
      if (__builtin_expect(masked, 0)) mask(s0, kt, 0);
      step(s0, s1, 0);
      done(t, 0);
      if (__builtin_expect(masked, 0)) mask(s1, kt, 1);
      step(s1, s0, 1);
      done(t, 1);
      b0 = (b0 + 1) & 3;
    }
  };

  // ---- sweep 1: M and the sum of exp2(logit - M) of the lane's queries, over the lane's half of
  // the keys. M is the row's largest logit in tile 0 (finite: key 0 is attended by every query);
  // the terms of a positive sum may exceed 1 without losing relative precision, and only a row
  // sum of 2^128 or more (logits 127 log2 units above M) overflows: then (or with non-finite
  // scores) the block takes each row's largest logit as M, from a sweep of its own, and sums again.
  //
  // A lane adds half of a row, so the sum is taken in levels, lest the rounding of n / 8 additions
  // into one register be left in it: the terms of a tile in Lt, four tiles in Lu, and those in
  // Ls + Lc, the rounding errors of Ls kept in Lc (add_carry). Root mean square of the sum's
  // relative error in float32, normal logits (emulated; the 16x16 kernel's order in brackets):
  // 3.7e-8 (4.7e-8) at 576 keys, 3.4e-8 (5.8e-8) at 4096, 3.3e-8 (7.4e-8) at 16384; one register
  // 1.0e-7, 2.3e-7, 4.5e-7.
  float M[MT], Ls[MT], Lc[MT], Lu[MT], Lt[MT];
  f32x16_t init[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    init[m] = zero;
    Ls[m] = Lc[m] = Lu[m] = Lt[m] = 0.f;
  }
  auto mask_t = [&](f32x16_t (&s)[MT], int kt, int half) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      // keys lo .. lo + span, one unsigned compare per score; key 0 on top
      const int lo = BAND ? klo[m] : 0, span = BAND ? kspan[m] : c.len - 1;
      const float key0 = s[m][0];
      const int base = kt * kTile + 32 * half + 4 * hf - lo;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        s[m][i] = (unsigned)(base + 8 * (i >> 2) + (i & 3)) <= (unsigned)span ? s[m][i] : -INFINITY;
      if (BAND && kt == 0 && half == 0 && hf == 0) s[m][0] = key0;
    }
  };
  auto max16 = [&](const f32x16_t& s, float v) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; i += 2) v = vmax3(v, s[i], s[i + 1]);
    return v;
  };
  auto none = [&](auto&&...) __attribute__((always_inline)) {};
  float e[4] = {0.f, 0.f, 0.f, 0.f};
  auto add_terms = [&](f32x16_t (&cur)[MT], int j, int half) __attribute__((always_inline)) {
    const int n = j >> 2, k = 4 * (j & 3);  // scores k .. k + 3 of query tile n
    float x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = __fmaf_rn(cur[n][k + u], kLog2eOver8, -M[n]);
    // the four terms of the slot before: their exp2 results are not waited for
    const int b = j == 0 ? MT - 1 : (j - 1) >> 2;
    const float sum = (e[0] + e[1]) + (e[2] + e[3]);
    // the first since Lt went into Lu (for the last query tile those of the tile before)
    if (half == 0 && (b == MT - 1 ? j == 0 : j == 4 * b + 1)) Lt[b] = sum;
    else Lt[b] += sum;
    pin(Lt[b]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      e[u] = exp2_fast(x[u]);
      pin(e[u]);
    }
  };
  auto end_tile = [&](int t, int half) __attribute__((always_inline)) {
    if (half == 0) return;
#pragma unroll
    for (int m = 0; m < MT; ++m) Lu[m] += Lt[m];
    if ((t & 3) == 3) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        add_carry(Ls[m], Lc[m], Lu[m]);
        Lu[m] = 0.f;
      }
    }
  };
  auto end_terms = [&]() __attribute__((always_inline)) {
    Lu[MT - 1] += (e[0] + e[1]) + (e[2] + e[3]);
#pragma unroll
    for (int m = 0; m < MT; ++m) add_carry(Ls[m], Lc[m], Lu[m]);
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = 0.f;
  };
  auto row_sum = [&](int m) __attribute__((always_inline)) {  // both halves of the wave
    float L = Ls[m], carry = Lc[m] + __shfl_xor(Lc[m], 32);
    add_carry(L, carry, __shfl_xor(Ls[m], 32));
    return L + carry;
  };
  using Yes = std::integral_constant<bool, true>;
  using No = std::integral_constant<bool, false>;
  sweep(
      Yes(), init,
      [&](auto&& mul) __attribute__((always_inline)) {  // M from both halves of tile 0
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
          for (int m = 0; m < MT; ++m) mul(s1, ks, m);
        if (BAND ? !band_tile_inside(c, 0, qw, 32 * MT) : c.len < kTile) {
          mask_t(s0, 0, 0);
          mask_t(s1, 0, 1);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const float v = max16(s1[m], max16(s0[m], -INFINITY));
          M[m] = __fmul_rn(vmax(v, __shfl_xor(v, 32)), kLog2eOver8);
        }
      },
      mask_t, add_terms, end_tile, none);
  end_terms();
  // query 0's keys past the tiles (its terms under m0, and their largest logit), in thread 0
  const bool has_far = BAND && c.qt == 0 && far_from(c) < c.len;  // block-uniform
  float* const part = p.colmax_part + (int64_t)c.b * c.n * p.nparts + c.h * p.qtiles + c.qt;
  // (the dot products are left in the keys' partials, by the thread that takes them up later)
  auto far_terms = [&](float& top) __attribute__((always_inline)) {
    if (c.tid == 0) far[0][0] = M[0];
    const u32x4_t q0 = *reinterpret_cast<const u32x4_t*>(Qb + 8 * (c.tid & 7));
    __syncthreads();
    const float m0 = far[0][0];
    float sum = 0.f;
    top = -INFINITY;
    for (int k0 = far_from(c); k0 < c.len; k0 += kThreads) {
      u32x4_t k[kFarRows];
      far_load(k, Kb, c, k0);
      float dot[kFarRows];
      far_dots(dot, q0, k);
#pragma unroll
      for (int r = 0; r < kFarRows; ++r) {
        const int key = far_key(k0, c.tid, r);
        if (key < c.len) {
          top = vmax(top, dot[r]);
          if ((c.tid & 7) == r) {  // one of the row's eight lanes
            sum += exp2_fast(__fmaf_rn(dot[r], kLog2eOver8, -m0));
            part[(int64_t)key * p.nparts] = dot[r];
          }
        }
      }
    }
    sum = row16_sum(sum);
    top = row16_max_sel(top);
    __syncthreads();  // every thread has m0
    if (c.r16 == 0) {
      far[0][4 * wave + c.g] = sum;
      far[1][4 * wave + c.g] = top;
    }
    __syncthreads();
    sum = row16_sum(far[0][c.r16]);
    top = row16_max_sel(far[1][c.r16]);
    __syncthreads();  // read before the next use
    return sum;
  };
  float far_top = -INFINITY;
  if (has_far) {
    const float sum = far_terms(far_top);
    if (c.tid == 0) add_carry(Ls[0], Lc[0], sum);
  }
  bool overflow = false;  // of the row's sum: two finite halves may add up to infinity
#pragma unroll
  for (int m = 0; m < MT; ++m) overflow |= !(row_sum(m) < INFINITY);
  if (overflow) redo = 1;
  lds_barrier();
  if (redo) {  // block-uniform
    float v[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      v[m] = -INFINITY;
      Ls[m] = Lc[m] = Lu[m] = Lt[m] = 0.f;
    }
    sweep(Yes(), init, none, mask_t,
          [&](f32x16_t (&cur)[MT], int j, int) __attribute__((always_inline)) {
            if (j % 4 == 0) v[j >> 2] = max16(cur[j >> 2], v[j >> 2]);
          },
          none, none);
    if (has_far && wave == 0 && r32 == 0) v[0] = vmax(v[0], far_top);
#pragma unroll
    for (int m = 0; m < MT; ++m) M[m] = __fmul_rn(vmax(v[m], __shfl_xor(v[m], 32)), kLog2eOver8);
    sweep(Yes(), init, none, mask_t, add_terms, end_tile, none);
    end_terms();
    if (has_far) {
      const float sum = far_terms(far_top);
      if (c.tid == 0) add_carry(Ls[0], Lc[0], sum);
    }
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int q = qw + 32 * m + r32;
    const float cq = M[m] + __builtin_amdgcn_logf(row_sum(m));  // finite: key 0 is attended by every query
    if (hf == 0 && q < c.n) p.row_c[((int64_t)c.b * p.H + c.h) * c.n + q] = cq;
    // the column statistic's offset: c, or c - log2 |S_q| under a window; +inf for padded
    // queries (excluded)
    float o = cq;
    if constexpr (BAND) o = cq - __builtin_amdgcn_logf((float)(kspan[m] + 1 + (klo[m] > 0 ? 1 : 0)));
    if (hf == 0) cs[wave][32 * m + r32] = -__fdiv_rn(q >= c.len ? INFINITY : o, kLog2eOver8);
  }

  // ---- sweep 2: the per-key column statistic of this block's valid queries. Each half of each
  // wave leaves its value of tile t's keys in cm[t % 3]; behind the barrier of iteration t + 1
  // (or the final one) threads 0 .. 63 combine a key's eight values in a fixed order and store
  // the block's partial. A slot is reused three tiles later, after two more barriers.
  if (BAND) {  // valid keys of the tiles outside the windows: query 0's value, or zero
    if (c.qt == 0) {
      __syncthreads();  // its offset is in cs
      for (int k0 = far_from(c); k0 < c.len; k0 += kThreads) {
        const int key = far_key(k0, c.tid, c.tid & 7);
        if (key < c.len) {
          float* a = part + (int64_t)key * p.nparts;
          *a = exp2_fast(__fmul_rn(*a + cs[0][0], kLog2eOver8));
        }
      }
    } else {
      for (int key = kTile + c.tid; key < c.len; key += kThreads) {
        const int kt = key / kTile;
        if (kt < c.tlo || kt > c.thi) part[(int64_t)key * p.nparts] = 0.f;
      }
    }
  }
  auto combine = [&](int t, int slot) __attribute__((always_inline)) {
    if (c.tid < kTile) {
      float x[8];
#pragma unroll
      for (int w = 0; w < 8; ++w) x[w] = cm[slot][w][c.tid];
      float v;
      if constexpr (IMP == 1) v = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
      else v = exp2_fast(__fmul_rn(vmax(vmax3(vmax3(x[0], x[1], x[2]), x[3], x[4]), vmax3(x[5], x[6], x[7])), kLog2eOver8));
      const int key = tile_at(c, t) * kTile + c.tid;
      if (key < c.n) part[(int64_t)key * p.nparts] = v;
    }
  };
  wave_lds_sync();
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int g = 0; g < 4; ++g) {  // queries 8 g + 4 hf .. + 3 of query tile m
      const float4 v = *reinterpret_cast<const float4*>(&cs[wave][32 * m + 8 * g + 4 * hf]);
      init[m][4 * g] = v.x;
      init[m][4 * g + 1] = v.y;
      init[m][4 * g + 2] = v.z;
      init[m][4 * g + 3] = v.w;
    }
  auto mask_q = [&](f32x16_t (&s)[MT], int kt, int half) __attribute__((always_inline)) {
    // the lane's key is attended by queries lo .. lo + span: within the window, all of them (key
    // 0, or full attention) or none (past the valid keys); and by query 0
    const int key = kt * kTile + 32 * half + r32;
    const int lo = !BAND || key == 0 ? 0 : key - c.half;
    const unsigned span = !BAND || key == 0 ? 0x7fffffffu : (unsigned)(2 * c.half);
    const float first = s[0][0];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int base = qw + 32 * m + 4 * hf - lo;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const bool ok = (BAND ? (unsigned)(base + 8 * (i >> 2) + (i & 3)) <= span : true) && key < c.len;
        s[m][i] = ok ? s[m][i] : -INFINITY;
      }
    }
    if (BAND && qw == 0 && hf == 0 && key < c.len) s[0][0] = first;
  };
  float v = IMP == 1 ? 0.f : -INFINITY;
  int slot = 0;  // t % 3
  sweep(
      No(), init, none, mask_q,
      [&](f32x16_t (&cur)[MT], int j, int) __attribute__((always_inline)) {
        const int n = j >> 2, k = 4 * (j & 3);
        if constexpr (IMP == 1) {
          float a = 0.f;
#pragma unroll
          for (int u = 0; u < 4; ++u) a += exp2_fast(__fmul_rn(cur[n][k + u], kLog2eOver8));
          v += a;
        } else {
          v = vmax3(vmax3(v, cur[n][k], cur[n][k + 1]), cur[n][k + 2], cur[n][k + 3]);
        }
        pin(v);
        if constexpr (IMP == 2) {  // median rule: every probability, exp2(s (dot - cc / s))
          e[0] = exp2_fast(__fmul_rn(cur[n][k], kLog2eOver8));
          e[1] = exp2_fast(__fmul_rn(cur[n][k + 1], kLog2eOver8));
          e[2] = exp2_fast(__fmul_rn(cur[n][k + 2], kLog2eOver8));
          e[3] = exp2_fast(__fmul_rn(cur[n][k + 3], kLog2eOver8));
          cur[n][k] = e[0];
          cur[n][k + 1] = e[1];
          cur[n][k + 2] = e[2];
          cur[n][k + 3] = e[3];
        }
      },
      [&](int t, int half) __attribute__((always_inline)) {
        cm[slot][2 * wave + hf][32 * half + r32] = v;
        v = IMP == 1 ? 0.f : -INFINITY;
        if constexpr (IMP == 2) {
          const int key = tile_at(c, t) * kTile + 32 * half + r32;
          if (key < c.n) {
            float* ac = p.acol + ((int64_t)c.b * c.n + key) * p.H * c.n + (int64_t)c.h * c.n;
            auto& s = half == 0 ? s0 : s1;
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                const int q = qw + 32 * m + 8 * g + 4 * hf;
                store_probs4(ac + q, s[m][4 * g], s[m][4 * g + 1], s[m][4 * g + 2], s[m][4 * g + 3], q, c.n);
              }
          }
        }
        if (half == 1) slot = slot == 2 ? 0 : slot + 1;
      },
      [&](int t) __attribute__((always_inline)) {  // the barrier of this iteration follows every wave's tile t - 1
        if (t > 0) combine(t - 1, slot == 0 ? 2 : slot - 1);
      });
  wait_vmcnt<0>();  // the trailing loads have landed before the wave ends
  lds_barrier();
  combine(nvis - 1, slot == 0 ? 2 : slot - 1);
}

// float32 rows of more than 8 key tiles
template <bool BAND>
hipError_t launch_scores_stream(const FwdParams& p, hipStream_t s) {
  const dim3 grid((unsigned)(p.qtiles * p.H * p.B)), blk(kThreads);
  if constexpr (BAND) {  // the mean and median rules are defined for full attention only
    return launch_stage_kernel((k_scores_stream<true, 0>), grid, blk, 0, s, p);
  } else {
    if (p.importance == 1) return launch_stage_kernel((k_scores_stream<false, 1>), grid, blk, 0, s, p);
    if (p.importance == 2) return launch_stage_kernel((k_scores_stream<false, 2>), grid, blk, 0, s, p);
    return launch_stage_kernel((k_scores_stream<false, 0>), grid, blk, 0, s, p);
  }
}

// bfloat16: p.qtiles says how many queries a block takes (score_block_queries)
template <bool BAND>
hipError_t launch_scores_stream32(const FwdParams& p, hipStream_t s) {
  const dim3 grid((unsigned)(p.qtiles * p.H * p.B)), blk(kThreads);
  if constexpr (BAND) {
    return launch_stage_kernel((k_scores_stream32<true, 0, 1>), grid, blk, 0, s, p);
  } else if (p.qtiles == (p.n + 127) / 128) {
    if (p.importance == 1) return launch_stage_kernel((k_scores_stream32<false, 1, 1>), grid, blk, 0, s, p);
    if (p.importance == 2) return launch_stage_kernel((k_scores_stream32<false, 2, 1>), grid, blk, 0, s, p);
    return launch_stage_kernel((k_scores_stream32<false, 0, 1>), grid, blk, 0, s, p);
  } else {
    if (p.qtiles != (p.n + 255) / 256) return hipErrorInvalidValue;
    if (p.importance == 1) return launch_stage_kernel((k_scores_stream32<false, 1, 2>), grid, blk, 0, s, p);
    if (p.importance == 2) return launch_stage_kernel((k_scores_stream32<false, 2, 2>), grid, blk, 0, s, p);
    return launch_stage_kernel((k_scores_stream32<false, 0, 2>), grid, blk, 0, s, p);
  }
}

// The one-sweep score passes with the importance rule as a template parameter (the mean and
// median rules are defined for full attention only).
template <int BF, int NT, bool BAND, bool RS>
hipError_t launch_scores_onesweep(const FwdParams& p, hipStream_t s) {
  const dim3 grid((unsigned)(p.qtiles * p.H * p.B)), blk(kThreads);
  if (!BAND && p.importance == 1) {
    if constexpr (RS) return launch_stage_kernel(k_scores_rs<BF, NT, BAND, 1>, grid, blk, 0, s, p);
    else return launch_stage_kernel(k_scores_res<BF, NT, BAND, 1>, grid, blk, 0, s, p);
  }
  if (!BAND && p.importance == 2) {
    if constexpr (RS) return launch_stage_kernel(k_scores_rs<BF, NT, BAND, 2>, grid, blk, 0, s, p);
    else return launch_stage_kernel(k_scores_res<BF, NT, BAND, 2>, grid, blk, 0, s, p);
  }
  if constexpr (RS) return launch_stage_kernel(k_scores_rs<BF, NT, BAND, 0>, grid, blk, 0, s, p);
  else return launch_stage_kernel(k_scores_res<BF, NT, BAND, 0>, grid, blk, 0, s, p);
}

// Resident variants for padded lengths up to 256 keys (bf16) or 128 keys (fp32), the
// one-sweep streamed variant up to 8 key tiles, the two-sweep streaming variant beyond.
template <bool BAND>
hipError_t launch_scores_band(const FwdParams& p, hipStream_t s) {
  const int nt = (p.n + kTile - 1) / kTile;
  if (p.bf16) {
    if (nt <= 1) return launch_scores_onesweep<1, 1, BAND, false>(p, s);
    else if (nt <= 2) return launch_scores_onesweep<1, 2, BAND, false>(p, s);
    else if (nt <= 4) return launch_scores_onesweep<1, 4, BAND, false>(p, s);
    else if (nt <= 8) return launch_scores_onesweep<1, 8, BAND, true>(p, s);
    else return launch_scores_stream32<BAND>(p, s);
  } else {
    if (nt <= 1) return launch_scores_onesweep<0, 1, BAND, false>(p, s);
    else if (nt <= 2) return launch_scores_onesweep<0, 2, BAND, false>(p, s);
    else if (nt <= 8) return launch_scores_onesweep<0, 8, BAND, true>(p, s);
    else return launch_scores_stream<BAND>(p, s);
  }
}

template <bool BAND>
hipError_t launch_attn_band(const FwdParams& p, hipStream_t s) {
  const dim3 grid((unsigned)(p.qtiles * p.H * p.B)), blk(kThreads);
  const int nt = (p.n + kTile - 1) / kTile;
  if (p.bf16) {
    if (nt <= 1) return launch_stage_kernel((k_attn_res<1, 1, BAND>), grid, blk, 0, s, p);
    else if (nt <= 2) return launch_stage_kernel((k_attn_res<1, 2, BAND>), grid, blk, 0, s, p);
    else if (nt <= 4) return launch_stage_kernel((k_attn_res<1, 4, BAND>), grid, blk, 0, s, p);
    const int64_t q128 = (p.n + 127) / 128;
    if (!BAND && wide_output_blocks(p.n, p.H, p.B))
      return launch_stage_kernel((k_attn_stream32<false, 2>), dim3((unsigned)((q128 + 1) / 2 * p.H * p.B)), blk, 0, s, p);
    // Rows of up to 8 key tiles: the 16x16 kernel where a CU gets five blocks or more (the cause was
    // not isolated; 96 x 448, 4 heads: 28.4 against 29.8 us; 256 x 300: 41.2 against 44.6), below
    // that the 32x32 one, whose blocks take less time each (6 x 512, 4 heads 9.2 against 8.1; 16 x
    // 384, 16 heads 15.8 against 15.2).
    if (!BAND && nt <= 8 && blocks_per_cu(q128 * p.H * p.B) >= 5)
      return launch_stage_kernel((k_attn_stream<1, false, 2>), dim3((unsigned)(q128 * p.H * p.B)), blk, 0, s, p);
    return launch_stage_kernel((k_attn_stream32<BAND, 1>), dim3((unsigned)(q128 * p.H * p.B)), blk, 0, s, p);
  } else {
    if (nt <= 1) return launch_stage_kernel((k_attn_res<0, 1, BAND>), grid, blk, 0, s, p);
    else if (nt <= 2) return launch_stage_kernel((k_attn_res<0, 2, BAND>), grid, blk, 0, s, p);
    // float32, bound by its MFMAs: 128 queries per block, or 64 (half the work each) where the CU
    // with the most blocks then has less (8 x 333 tokens, 12 heads: two blocks per CU against three
    // of half the work, 51 -> 34 us). Blocks of 64, us a call against those of 128, 12 heads: 1 x 200 41.0
    // (50.0), 2 x 640 106.9 (126.2), 4 x 1024 291.6 (314.3), window 256 267.0 (326.0); where the
    // rule keeps 128: 32 x 200 142.2 (140.4), 4 x 512, 16 heads 95.5 (98.5).
    const int64_t b128 = (int64_t)((p.n + 127) / 128) * p.H * p.B, b64 = (int64_t)nt * p.H * p.B;
    if (blocks_per_cu(b64) < 2 * blocks_per_cu(b128))
      return launch_stage_kernel((k_attn_stream<0, BAND, 1>), dim3((unsigned)b64), blk, 0, s, p);
    return launch_stage_kernel((k_attn_stream<0, BAND, 2>), dim3((unsigned)b128), blk, 0, s, p);
  }
}
}  // namespace

hipError_t launch_scores_colmax(const FwdParams& p, hipStream_t s) {
  return p.band_half > 0 ? launch_scores_band<true>(p, s) : launch_scores_band<false>(p, s);
}

hipError_t launch_attn_out(const FwdParams& p, hipStream_t s) {
  return p.band_half > 0 ? launch_attn_band<true>(p, s) : launch_attn_band<false>(p, s);
}

}  // namespace mca
