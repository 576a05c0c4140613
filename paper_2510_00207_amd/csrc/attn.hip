// The multi-head attention of AT_r (Sec. 2.1): per sequence and head,
// A = softmax(Q K^T / sqrt(d)) V with Q, K, V the head's columns of
// I [W^Q | W^K | W^V], then I' = A W^O. The projections run on the grouped
// GEMM as one dense expert; the attention runs in the kernels below, which
// stream K and V tiles through LDS and never store the N x N scores.
//
// Forward (one block: 128 queries of one sequence and head, 4 waves of 32):
// each wave computes S^T = K Q^T for a 64-key tile with
// v_mfma_f32_32x32x16_bf16, so that a lane's accumulator column is one query
// and the online-softmax statistics (running max and sum, base-2 exponents)
// live in the lane pair (l, l + 32) that holds that query's 64 scores. The
// bf16 probabilities P^T are then the second MFMA's column operand straight
// from the registers, and O^T += V^T P^T takes V^T from LDS by transposing
// reads (ds_read_b64_tr_b16). The log-sum-exp of each row is kept for the
// backward.
//
// Backward (no atomics; every sum in a fixed order):
//   dq kernel (blocks of 128 queries, loop over 32-key tiles): recomputes P
//     from S and the log-sum-exp, dP^T = V dO^T, dS = P (dP - delta) with
//     delta = rowsum(dO * O) (computed here and stored for the next kernel),
//     dQ^T += K^T dS^T;
//   dkdv kernel (blocks of 128 keys, loop over 32-query steps): S and dP with
//     the key as the accumulator column, dV^T += dO^T P, dK^T += Q^T dS.
#include <math.h>

#include "common.hpp"

namespace flowmoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16_t;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.69314718055994531f;

struct AttnArgs {
  const bf16_t* qkv;  // T x 3M = [Q | K | V]; head h at columns h * D of each
  const bf16_t* o;    // T x M: the heads' outputs (backward)
  const bf16_t* d_o;  // T x M: their gradient (backward)
  bf16_t* out;        // forward: T x M
  bf16_t* d_qkv;      // backward: T x 3M
  float* lse;         // heads x T: natural log-sum-exp of each row's scores
  float* delta;       // heads x T: rowsum(dO * O) over the head's columns
  int T, M, N, heads, nseq;
  int shared;  // query tiles of a head side by side on one XCD (decode)
  int pair;  // causal grid of one round of resident blocks: pair long and short tiles (decode)
  float c2;  // log2(e) / sqrt(D): a score times c2 is its base-2 exponent
  float rs;  // 1 / sqrt(D)
};

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// the LDS stage of a double-buffered loop as a compile-time constant: the
// loops run their steps in pairs (stage 0, stage 1), so every LDS address of
// a step is a register base plus an immediate offset
template <int S>
struct Stage {
  static constexpr int value = S;
};

__device__ __forceinline__ bf16x8 zero8() { return __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0}); }

__device__ __forceinline__ floatx16 zero16() {
  floatx16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.0f;
  return z;
}

// LDS tiles hold rows of D bf16 (2D bytes); the 16-byte chunk c of row r
// sits at chunk c ^ sw(r). For D = 128 (a row is one pass over the 64 banks)
// sw is one-to-one on any 16 consecutive rows, so a row read (16 lanes on 16
// rows, one chunk each) touches 16 distinct bank groups; sw / 2 takes 4
// distinct values of one parity on 4 aligned rows, so a transposing read
// (4 aligned rows x two adjacent 32-byte column pairs per 32 lanes) does too.
// For D = 64 (two rows per pass) the same holds with the row parity as the
// extra bank bit.
template <int D>
__device__ __forceinline__ int sw(int r) {
  if constexpr (D == 128) return 4 * (r & 3) + ((r >> 2) & 3);
  else return 4 * ((r >> 1) & 1) + 2 * ((r >> 2) & 1) + ((r >> 3) & 1);
}
template <int D>
__device__ __forceinline__ int toff(int r, int c) {
  return r * (2 * D) + ((c ^ sw<D>(r)) << 4);
}

// Two MFMA operand forms are read from these tiles:
//   row operand (d contiguous): lane l supplies row r0 + l % 32 of a 32-row
//     block at d = 16 ks + 8 (l / 32) .. + 7, one 16-byte read of chunk
//     2 ks + l / 32 (row_base, frag_row_x);
//   transposed operand: lane l supplies column cb + l % 32 of the tile at
//     the 8 rows of its k-slots, slot 4 i + j (i = 0, 1; j = 0..3) being row
//     rb + 4 (l / 32) + 8 i + j, as two transposing reads (tr_base,
//     frag_tr_x). Each ds_read_b64_tr_b16 hands lane l' of a 16-lane group
//     element l' % 4 of the 4 values that lane 4 q + l' / 4 addressed, in
//     slot q; lanes aimed at rows r0 + s / 4, columns c0 + 4 (s % 4) give
//     lane l' column c0 + l' at rows r0 .. r0 + 3.

// The swizzle lets a lane's fragment addresses be formed from three per-lane
// bases: a row read of row r0 + lq (r0 a multiple of 32) at k step ks is at
// r0 * 2D + (row_base ^ 32 ks), and a transposing read at rows rb (a
// multiple of 16) and columns cb (a multiple of 32) at
// rb * 2D + (tr_base_i ^ 2 cb) for its two halves i. The loops rebuild the
// XORs in every step from bases they mark as changed (opaque()): the
// compiler would otherwise keep every combination live across the loop and,
// short of registers, spill them and reload one before each LDS read.
template <int D>
__device__ __forceinline__ int row_base(int lq, int h2) {
  return toff<D>(lq, h2);
}
template <int D>
__device__ __forceinline__ int tr_base(int lane, int i) {
  const int G = lane >> 4, sl = lane & 15;
  const int col = (G & 1) * 16 + 4 * (sl & 3);
  const int r = 4 * (G >> 1) + 8 * i + (sl >> 2);
  return toff<D>(r, col >> 3) + ((col & 7) << 1);
}
template <int D>
__device__ __forceinline__ bf16x8 frag_row_x(const char* t, int base, int r0, int ks) {
  return *reinterpret_cast<const bf16x8*>(t + r0 * 2 * D + (base ^ (ks << 5)));
}
template <int D>
__device__ __forceinline__ bf16x8 frag_tr_x(const char* t, int b0, int b1, int rb, int cb) {
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(t + rb * 2 * D + (b0 ^ (2 * cb))));
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(t + rb * 2 * D + (b1 ^ (2 * cb))));
  const short __attribute__((ext_vector_type(8))) s = {lo[0], lo[1], lo[2], lo[3],
                                                       hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, s);
}
__device__ __forceinline__ void opaque(int& a, int& b, int& c) {
  asm volatile("" : "+v"(a), "+v"(b), "+v"(c));
}

// Rows 16 s .. 16 s + 15 of a 32 x 32 accumulator (lane l: column l % 32,
// element 4 J + j = row 8 J + 4 (l / 32) + j) as an MFMA column operand in
// the transposed operand's slot order: slot 4 i + j <- element 8 s + 4 i + j.
__device__ __forceinline__ bf16x8 pfrag(const floatx16& a, int s) {
  bf16x8 r;
#pragma unroll
  for (int t = 0; t < 8; ++t) r[t] = (__bf16)a[8 * s + t];
  return r;
}

__device__ __forceinline__ floatx16 mfma(const bf16x8& a, const bf16x8& b, const floatx16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// store a 32-row block of a transposed accumulator (lane: column = token,
// rows = d) as bf16 row segments dst[8 J + 4 (l / 32) .. + 3] * scale
__device__ __forceinline__ void store_cols(bf16_t* dst, const floatx16& a, int h2, float scale) {
#pragma unroll
  for (int J = 0; J < 4; ++J) {
    uint2 v;
    v.x = pack_bf16x2(a[4 * J] * scale, a[4 * J + 1] * scale);
    v.y = pack_bf16x2(a[4 * J + 2] * scale, a[4 * J + 3] * scale);
    *reinterpret_cast<uint2*>(dst + 8 * J + 4 * h2) = v;
  }
}

// One operand's ROWS-row tiles of a (sequence, head) by LDS-DMA, in the layout
// above: wave w of NW fills 1 KB blocks w, w + NW, ... (64 / CPR rows each), every
// lane fetching the chunk that belongs at its place. Rows at or past N (every
// row of a tile past the last) load zeros without traffic.
template <int D, int ROWS, int NW>
struct TileDma {
  static constexpr int TB = ROWS * D * 2;        // bytes of a tile
  static constexpr int CPR = D / 8, RPB = 64 / CPR;  // chunks a row, rows a block
  static constexpr int NB = TB / 1024, LD = (NB + NW - 1) / NW;  // blocks, loads a wave
  static_assert(NB % NW == 0, "whole loads");
  unsigned lds0, ld2, full;  // this wave's first block in slot 0; bytes of a row step, of a tile
  unsigned off[LD];
  __device__ __forceinline__ TileDma(unsigned lds, int w, int lane, long ld)
      : lds0(lds + w * 1024), ld2((unsigned)(2 * ld)), full((ROWS - 1) * ld2 + 2 * D) {
#pragma unroll
    for (int u = 0; u < LD; ++u) {
      const int r = (w + NW * u) * RPB + lane / CPR, c = (lane % CPR) ^ sw<D>(r);
      off[u] = r * ld2 + 16 * c;
    }
  }
  // the tile whose first row is at g, of which `rows` are there
  __device__ __forceinline__ void load(const bf16_t* g, int rows, int slot) const {
    const unsigned n = rows >= ROWS ? full : rows <= 0 ? 0u : (rows - 1) * ld2 + 2 * D;
    const unsigned long a = reinterpret_cast<unsigned long>(g);
    const u32x4 rs = {(unsigned)a, (unsigned)(a >> 32) & 0xFFFFu, n, 0x00020000u};
    dma16_row<LD, NW * 1024>(rs, lds0 + slot, off);
  }
};

// the maximum and the sum over a lane pair (l, l + 32)
__device__ __forceinline__ float pair_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// block -> (query or key tile, head, sequence). Blocks are dispatched in
// order; u = blockIdx / (heads x sequences) ranks the tiles by their causal
// work, longest first (`rev`: tiles in descending order, the query tiles of
// the forward and of dQ; else ascending, the key tiles of dK/dV). With
// `a.pair` (every block resident at once, two to a CU: the second half of
// the grid lands on the CUs of the first half) the second half runs the
// shortest tiles first, so that a CU's two blocks have complementary work
// (ranks u and nt - 1 - u) instead of ranks u and u + nt / 2.
//
// `shared` (query tiles; shared_order): the tiles of a head one after the other on
// one XCD (blocks go to the 8 XCDs round-robin), so that its K and V are read
// through that L2 once. In the order above they are per blocks apart, and a launch
// whose K and V exceed the caches reads them from HBM for every tile.
__device__ __forceinline__ void decode(const AttnArgs& a, bool rev, bool shared, int& tile, int& hd,
                                       int& sq, int rows) {
  const int per = a.heads * a.nseq, nt = (a.N + rows - 1) / rows;
  if (shared && per % 8 == 0) {
    const int i = blockIdx.x >> 3, rest = i / nt * 8 + (blockIdx.x & 7);
    tile = rev ? nt - 1 - i % nt : i % nt;
    hd = rest % a.heads;
    sq = rest / a.heads;
    return;
  }
  const int u = (int)(blockIdx.x / per), rest = (int)(blockIdx.x % per);
  const int h = (nt + 1) / 2;
  const int r = a.pair && u >= h ? nt - 1 - (u - h) : u;  // rank in work order
  tile = rev ? nt - 1 - r : r;
  hd = rest % a.heads;
  sq = rest / a.heads;
}

// Forward: blocks of 4 waves of 32 queries (8 in some launches of heads of 64), two to
// four to a CU.
//
// The matrix pipes should bound it, but a tile's softmax takes about as many issue
// cycles as its 32 products take matrix cycles, and products that wait for their
// own LDS read or a softmax after them leave both idle (pipes busy 0.39 of the
// cycles). So a step runs one tile ahead: the products S(t + 1) = K Q are issued
// between the exponentials of S(t), the products with V(t) between the maxima of
// S(t + 1), and every LDS read two groups of products before its use. K and V
// tiles come by LDS-DMA into two slots each: step t reads K(t + 1) and V(t), and
// refills K(t)'s and V(t - 1)'s slots. Measured, before -> now: 4 x 4096 tokens, 32
// heads of 128, causal 635 -> 590 us; one sequence of 4096, 16 heads 112 -> 93; 4 x
// 2048, 32 heads, bidirectional 326 -> 297. Blocks of 8 waves (half the staging)
// are 0-4% slower, and 12% on short causal sequences; four slots instead of two,
// raised priority around the V products, and timing copies without the barrier
// or the wait for the loads change 0-2%, without the exponentials 7%, without the
// DMA 17% (less switching): two independent blocks a CU hide what there is.
//
// Heads of 64 have half the products for the same softmax, and room for four waves
// on a SIMD (128 registers) if a step does not run ahead: then the other waves
// hide a wave's softmax, and K(t), V(t) are used in turn. The one-tile-ahead loop
// with two waves a SIMD had made them up to 13 % slower than the loop before it,
// where a launch is several rounds. us of the loop before, ahead, in turn: 32
// sequences of 512, 16 heads, bidirectional 56, 62, 51 (8 waves); 4 x 4096, 24 heads,
// causal 252, 266, 229; 8 x 512 20, 19, 18; 1 x 4096, 8 heads 64, 54, 55.
template <int D, bool CAUSAL, int NW>
__global__ __launch_bounds__(64 * NW, D == 128 ? 2 : 4) void attn_fwd_kernel(AttnArgs a) {
  constexpr bool AHEAD = D == 128;
  constexpr int KS = D / 16, DB = D / 32, QB = 32 * NW;
  using Dma = TileDma<D, 64, NW>;
  constexpr int TB = Dma::TB;
  __shared__ __attribute__((aligned(1024))) char lds[4 * TB];  // K slots 0, 1, then V slots 0, 1
  // the wave index through readfirstlane: the compiler then knows it is
  // wave-uniform, and the branches on a wave's query or key range are
  // scalar branches instead of exec-mask ones (backward 7-10% faster)
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6),
            h2 = lane >> 5, lq = lane & 31;
  int qt, hd, sq;
  decode(a, CAUSAL, a.shared != 0, qt, hd, sq, QB);
  const long tok0 = (long)sq * a.N, ld = 3L * a.M;
  const bf16_t* Qg = a.qkv + tok0 * ld + (long)hd * D;
  const bf16_t* Kg = Qg + a.M;
  const bf16_t* Vg = Qg + 2L * a.M;
  const int q0 = qt * QB, qw = q0 + 32 * w + lq;

  const int kend = CAUSAL ? min(a.N, q0 + QB) : a.N;
  const int nk = (kend + 63) / 64;
  // (causal: a wave whose queries all precede a tile has nothing in it)
  const int nkw = CAUSAL ? min(nk, (q0 + 32 * w + 31) / 64 + 1) : nk;
  const Dma dma(lds_base(lds), w, lane, ld);
  const long kstep = 64 * ld;
  dma.load(Kg, kend, 0);
  dma.load(Vg, kend, 2 * TB);
  if constexpr (AHEAD) dma.load(Kg + kstep, kend - 64, TB);  // (past the last tile: no traffic)

  bf16x8 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qf[ks] = qw < a.N ? *reinterpret_cast<const bf16x8*>(Qg + qw * ld + 16 * ks + 8 * h2) : zero8();
  floatx16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = zero16();
  float m = -INFINITY, l = 0.0f;

  int rbase = row_base<D>(lq, h2), tb0 = tr_base<D>(lane, 0), tb1 = tr_base<D>(lane, 1);
  auto mask = [&](floatx16 (&s)[2], int kb0) {
    if (kb0 + 64 > a.N || (CAUSAL && kb0 + 63 > q0 + 32 * w)) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kb0 + 32 * kb + 8 * (r >> 2) + 4 * h2 + (r & 3);
          if (key >= a.N || (CAUSAL && key > qw)) s[kb][r] = -INFINITY;
        }
    }
  };
  auto row_max = [&](const floatx16 (&s)[2]) {
    float mx = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
    return mx;
  };
  // The reference m of the exponents moves only when a score exceeds it
  // by more than 2^8 (then the sum and the accumulators are rescaled):
  // probabilities up to 256 stay exact in float and in bf16's exponent
  // range, and the final lse = m + log2(l) is the same. Every query sees
  // key 0 in the first tile, so m is finite from then on.
  auto move_ref = [&](float mx) {
    mx = pair_max(mx) * a.c2;
    const bool up = mx > m + 8.0f;
    if (__any(up)) {
      const float mn = up ? mx : m;
      const float al = exp2_fast(m - mn);
      l *= al;
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db] *= al;
      m = mn;
    }
  };

  // The LDS reads of a step in groups of two fragments, each read two groups ahead
  // of its products (a product that waits for its own read waits a whole LDS
  // latency): groups 0 .. KS - 1, both key blocks of K(t + 1) at k step i; then 2 DB
  // groups of V(t), 16 keys by 64 columns each
  constexpr int VG = 2 * DB, NG = KS + VG;
  bf16x8 fr[3][2];
  auto read_group = [&](const char* tk, const char* tv, int i) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (i < KS) fr[i % 3][u] = frag_row_x<D>(tk, rbase, 32 * u, i);
      else if (i < NG)
        fr[i % 3][u] = frag_tr_x<D>(tv, tb0, tb1, 16 * ((i - KS) / (DB / 2)),
                                    32 * (2 * ((i - KS) % (DB / 2)) + u));
    }
  };
  auto mul_k = [&](floatx16 (&s)[2], int i) {
#pragma unroll
    for (int u = 0; u < 2; ++u) s[u] = mfma(fr[i % 3][u], qf[i], i == 0 ? zero16() : s[u]);
  };

  // heads of 64: K(t) and V(t) in slots t % 2; the scores, the softmax and the value
  // products one after the other
  auto step_in_turn = [&](const int t, auto stc) {
    constexpr int st = decltype(stc)::value;
    opaque(rbase, tb0, tb1);
    wait_vm<0>();  // K(t) and V(t): loaded a step ago
    lds_barrier();  // and every wave's reads of the slots refilled now are done
    const char* tk = lds + st * TB;
    const char* tv = lds + (2 + st) * TB;
    const bool live = t < nkw;
    if (live) {
      read_group(tk, tv, 0);
      read_group(tk, tv, 1);
    }
    Kg += kstep;  // K(t + 1), V(t + 1)
    Vg += kstep;
    dma.load(Kg, kend - 64 * (t + 1), (st ^ 1) * TB);
    dma.load(Vg, kend - 64 * (t + 1), (2 + (st ^ 1)) * TB);
    if (!live) return;
    floatx16 sc[2];
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      read_group(tk, tv, i + 2);
      __builtin_amdgcn_sched_barrier(0);
      mul_k(sc, i);
      __builtin_amdgcn_sched_barrier(0);
    }
    mask(sc, 64 * t);
    move_ref(row_max(sc));
    unsigned pw[16];
    float rsum = 0.0f;
#pragma unroll
    for (int q = 0; q < 32; q += 2) {
      const float p0 = exp2_fast(fmaf(sc[q >> 4][q & 15], a.c2, -m));
      const float p1 = exp2_fast(fmaf(sc[q >> 4][(q & 15) + 1], a.c2, -m));
      rsum += p0;
      rsum += p1;
      pw[q >> 1] = pack_bf16x2(p0, p1);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < VG; ++j) {
      read_group(tk, tv, KS + j + 2);
      __builtin_amdgcn_sched_barrier(0);
      const int g = j / (DB / 2);
      const bf16x8 pb = __builtin_bit_cast(bf16x8, u32x4{pw[4 * g], pw[4 * g + 1], pw[4 * g + 2], pw[4 * g + 3]});
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int db = 2 * (j % (DB / 2)) + u;
        o[db] = mfma(fr[(KS + j) % 3][u], pb, o[db]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    l += pair_sum(rsum);
  };

  floatx16 s[2][2];  // [tile parity][32-key block]
  if constexpr (AHEAD) {
    wait_vm<0>();
    lds_barrier();
    read_group(lds, lds, 0);
    read_group(lds, lds, 1);
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      if (i + 2 < KS) read_group(lds, lds, i + 2);
      __builtin_amdgcn_sched_barrier(0);
      mul_k(s[0], i);
    }
    mask(s[0], 0);
    move_ref(row_max(s[0]));
  }

  auto step_ahead = [&](const int t, auto stc) {
    constexpr int st = decltype(stc)::value;
    opaque(rbase, tb0, tb1);
    wait_vm<0>();  // K(t + 1) and V(t): loaded a step ago
    lds_barrier();  // and every wave's reads of the slots refilled now are done
    const char* tk = lds + (st ^ 1) * TB;
    const char* tv = lds + (2 + st) * TB;
    floatx16(&sc)[2] = s[st];
    floatx16(&sn)[2] = s[st ^ 1];
    const bool live = t < nkw, next = t + 1 < nkw;
    if (next) {
      read_group(tk, tv, 0);
      read_group(tk, tv, 1);
    }
    Kg += kstep;  // K(t + 1), V(t + 1)
    Vg += kstep;
    dma.load(Kg + kstep, kend - 64 * (t + 2), st * TB);
    dma.load(Vg, kend - 64 * (t + 1), (2 + (st ^ 1)) * TB);
    if (!live) return;
    unsigned pw[16];  // the 32 probabilities of this lane, bf16 pairs
    // (the sum in key order, then the lane pair's two halves, tile by tile: results do
    // not depend on how the step is scheduled)
    float rsum = 0.0f;
    auto exps = [&](int q0s, int q1s) {  // scores q0s .. q1s - 1: exponentials, sum, bf16
#pragma unroll
      for (int q = q0s; q < q1s; q += 2) {
        const float p0 = exp2_fast(fmaf(sc[q >> 4][q & 15], a.c2, -m));
        const float p1 = exp2_fast(fmaf(sc[q >> 4][(q & 15) + 1], a.c2, -m));
        rsum += p0;
        rsum += p1;
        pw[q >> 1] = pack_bf16x2(p0, p1);
        // (computed here, not where they are used)
        asm volatile("" : "+v"(pw[q >> 1]), "+v"(rsum));
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    if (next) {
      constexpr int CH = 32 / KS;  // scores exponentiated beside a group's two products
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        read_group(tk, tv, i + 2);
        __builtin_amdgcn_sched_barrier(0);
        exps(i * CH, (i + 1) * CH);
        mul_k(sn, i);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x402, 7 * CH / 4, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      mask(sn, (t + 1) * 64);
    } else {
      read_group(tk, tv, KS);
      read_group(tk, tv, KS + 1);
      exps(0, 32);
    }
    __builtin_amdgcn_sched_barrier(0);
    float mx = sn[0][0];
#pragma unroll
    for (int j = 0; j < VG; ++j) {
      read_group(tk, tv, KS + j + 2);
      __builtin_amdgcn_sched_barrier(0);
      const int g = j / (DB / 2);
      const bf16x8 pb = __builtin_bit_cast(bf16x8, u32x4{pw[4 * g], pw[4 * g + 1], pw[4 * g + 2], pw[4 * g + 3]});
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int db = 2 * (j % (DB / 2)) + u;
        o[db] = mfma(fr[(KS + j) % 3][u], pb, o[db]);
      }
      constexpr int CH = 32 / VG;
#pragma unroll
      for (int q = j * CH; q < (j + 1) * CH; ++q) mx = fmaxf(mx, sn[q >> 4][q & 15]);
      asm volatile("" : "+v"(mx));
      __builtin_amdgcn_sched_barrier(0);
    }
    l += pair_sum(rsum);
    if (next) move_ref(mx);
  };
  auto step = [&](const int t, auto stc) {
    if constexpr (AHEAD) step_ahead(t, stc);
    else step_in_turn(t, stc);
  };
  for (int t = 0; t < nk; t += 2) {
    step(t, Stage<0>{});
    if (t + 1 < nk) step(t + 1, Stage<1>{});
  }
  if (qw < a.N) {
    const float inv = 1.0f / l;
    bf16_t* Og = a.out + (tok0 + qw) * a.M + (long)hd * D;
#pragma unroll
    for (int db = 0; db < DB; ++db) store_cols(Og + 32 * db, o[db], h2, inv);
    if (h2 == 0) a.lse[(long)hd * a.T + tok0 + qw] = (m + log2f(l)) * kLn2;
  }
}

// dQ and delta: blocks of 4 waves of 32 queries, two to a CU, over 32-key tiles.
//
// As the forward it runs one tile ahead: S(t + 1) = K Q and dP(t + 1) = V dO are
// issued between the elementwise work of tile t, dQ += K^T dS(t) follows, and each
// LDS read is one (D = 64: two) groups of products ahead of its use. K(t) is read in
// two steps (rows, then transposed), so K has three slots and V two; the block's dO
// rows are read from LDS (registers hold Q). Before -> now: 4 x 4096 tokens, 32 heads
// of 128, causal 970 -> 850 us; one sequence of 4096, 16 heads 171 -> 135; 4 x 1500, 20
// heads of 64, bidirectional 112 -> 102.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void attn_dq_kernel(AttnArgs a) {
  constexpr int KS = D / 16, DB = D / 32, NW = 4, QB = 32 * NW;
  using Dma = TileDma<D, 32, NW>;
  constexpr int TB = Dma::TB, VB = 3 * TB, GB = 5 * TB;  // K slots, V slots, the dO rows
  __shared__ __attribute__((aligned(1024))) char lds[GB + QB * D * 2];
  // the wave index through readfirstlane: the compiler then knows it is
  // wave-uniform, and the branches on a wave's query or key range are
  // scalar branches instead of exec-mask ones (backward 7-10% faster)
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6),
            h2 = lane >> 5, lq = lane & 31;
  int qt, hd, sq;
  decode(a, CAUSAL, a.shared != 0, qt, hd, sq, QB);
  const long tok0 = (long)sq * a.N, ld = 3L * a.M;
  const bf16_t* Qg = a.qkv + tok0 * ld + (long)hd * D;
  const bf16_t* Kg = Qg + a.M;
  const bf16_t* Vg = Qg + 2L * a.M;
  const bf16_t* Gg = a.d_o + tok0 * a.M + (long)hd * D;
  const bf16_t* Og = a.o + tok0 * a.M + (long)hd * D;
  const int q0 = qt * QB, qw = q0 + 32 * w + lq;
  const bool live = qw < a.N;

  const int kend = CAUSAL ? min(a.N, q0 + QB) : a.N;
  const int nk = (kend + 31) / 32;
  // (causal: a wave whose queries all precede a tile has nothing in it)
  const int nkw = CAUSAL ? min(nk, (q0 + 32 * w + 31) / 32 + 1) : nk;
  const long kstep = 32 * ld;
  const Dma dma(lds_base(lds), w, lane, ld);
  {
    const Dma dmag(lds_base(lds), w, lane, a.M);
#pragma unroll
    for (int i = 0; i < NW; ++i)
      dmag.load(Gg + (long)(q0 + 32 * i) * a.M, a.N - q0 - 32 * i, GB + i * TB);
  }
  dma.load(Kg, kend, 0);
  dma.load(Vg, kend, VB);
  dma.load(Kg + kstep, kend - 32, TB);  // (past the last tile: no traffic)
  dma.load(Vg + kstep, kend - 32, VB + TB);
  bf16x8 qf[KS];
  float dl = 0.0f;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    qf[ks] = live ? *reinterpret_cast<const bf16x8*>(Qg + qw * ld + 16 * ks + 8 * h2) : zero8();
    const bf16x8 gv = live ? *reinterpret_cast<const bf16x8*>(Gg + (long)qw * a.M + 16 * ks + 8 * h2) : zero8();
    const bf16x8 ov = live ? *reinterpret_cast<const bf16x8*>(Og + (long)qw * a.M + 16 * ks + 8 * h2) : zero8();
#pragma unroll
    for (int t = 0; t < 8; ++t) dl += (float)gv[t] * (float)ov[t];
  }
  dl += __shfl_xor(dl, 32);
  const long srow = (long)hd * a.T + tok0 + qw;
  if (live && h2 == 0) a.delta[srow] = dl;
  const float l2 = live ? a.lse[srow] * kLog2e : 0.0f;
  floatx16 dq[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) dq[db] = zero16();

  int rbase = row_base<D>(lq, h2), tb0 = tr_base<D>(lane, 0), tb1 = tr_base<D>(lane, 1);
  // read groups: 0 .. KS - 1, the K, V and dO rows at k step i of tile t + 1; then DB
  // groups of tile t's K transposed, 16 keys by 64 columns each
  constexpr int NG = KS + DB;
  constexpr int RS = D == 128 ? 2 : 3;  // groups in registers (128: three spill)
  bf16x8 fr[RS][3];
  auto read_group = [&](const char* tk, const char* tv, const char* tkt, int i) {
    if (i < KS) {
      fr[i % RS][0] = frag_row_x<D>(tk, rbase, 0, i);
      fr[i % RS][1] = frag_row_x<D>(tv, rbase, 0, i);
      fr[i % RS][2] = frag_row_x<D>(lds + GB, rbase, 32 * w, i);
    } else if (i < NG) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
        fr[i % RS][u] = frag_tr_x<D>(tkt, tb0, tb1, 16 * ((i - KS) / (DB / 2)),
                                    32 * (2 * ((i - KS) % (DB / 2)) + u));
    }
  };
  floatx16 s[2], dp[2];  // [tile parity]
  auto mul = [&](floatx16& x, floatx16& y, int i) {
    x = mfma(fr[i % RS][0], qf[i], i == 0 ? zero16() : x);
    y = mfma(fr[i % RS][1], fr[i % RS][2], i == 0 ? zero16() : y);
  };
  auto mask = [&](floatx16& x, int kb0) {
    if (kb0 + 32 > a.N || (CAUSAL && kb0 + 31 > q0 + 32 * w)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = kb0 + 8 * (r >> 2) + 4 * h2 + (r & 3);
        if (key >= a.N || (CAUSAL && key > qw)) x[r] = -INFINITY;
      }
    }
  };

  wait_vm<0>();
  lds_barrier();
  read_group(lds, lds + VB, lds, 0);
  if constexpr (RS > 2) read_group(lds, lds + VB, lds, 1);
#pragma unroll
  for (int i = 0; i < KS; ++i) {
    if (i + RS - 1 < KS) read_group(lds, lds + VB, lds, i + RS - 1);
    __builtin_amdgcn_sched_barrier(0);
    mul(s[0], dp[0], i);
  }
  mask(s[0], 0);

  int k0s = 0;  // tile t's K slot
  auto step = [&](const int t, auto stc) {
    constexpr int st = decltype(stc)::value;
    opaque(rbase, tb0, tb1);
    wait_vm<0>();   // K(t + 1) and V(t + 1)
    lds_barrier();  // and every wave's reads of the slots refilled now are done
    const int k1s = k0s == 2 ? 0 : k0s + 1, k2s = k1s == 2 ? 0 : k1s + 1;
    const char* tk = lds + k1s * TB;
    const char* tv = lds + VB + (st ^ 1) * TB;
    const char* tkt = lds + k0s * TB;
    const bool next = t + 1 < nkw;
    if (next) {
      read_group(tk, tv, tkt, 0);
      if constexpr (RS > 2) read_group(tk, tv, tkt, 1);
    }
    Kg += kstep;  // K(t + 1), V(t + 1)
    Vg += kstep;
    dma.load(Kg + kstep, kend - 32 * (t + 2), k2s * TB);
    dma.load(Vg + kstep, kend - 32 * (t + 2), VB + st * TB);
    k0s = k1s;
    if (t >= nkw) return;
    unsigned pw[8];  // dS^T of this lane, bf16 pairs
    auto elem = [&](int r0, int r1) {
#pragma unroll
      for (int r = r0; r < r1; r += 2) {
        const float d0 = exp2_fast(fmaf(s[st][r], a.c2, -l2)) * (dp[st][r] - dl);
        const float d1 = exp2_fast(fmaf(s[st][r + 1], a.c2, -l2)) * (dp[st][r + 1] - dl);
        pw[r >> 1] = pack_bf16x2(d0, d1);
        asm volatile("" : "+v"(pw[r >> 1]));  // (computed here, not where it is used)
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    if (next) {
      constexpr int CH = 16 / KS;  // scores beside a group's two products
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        read_group(tk, tv, tkt, i + RS - 1);
        __builtin_amdgcn_sched_barrier(0);
        elem(i * CH, (i + 1) * CH);
        mul(s[st ^ 1], dp[st ^ 1], i);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x402, 9 * CH / 4, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      mask(s[st ^ 1], 32 * (t + 1));
    } else {
      read_group(tk, tv, tkt, KS);
      if constexpr (RS > 2) read_group(tk, tv, tkt, KS + 1);
      elem(0, 16);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < DB; ++j) {
      read_group(tk, tv, tkt, KS + j + RS - 1);
      __builtin_amdgcn_sched_barrier(0);
      const int g = j / (DB / 2);
      const bf16x8 pb = __builtin_bit_cast(bf16x8, u32x4{pw[4 * g], pw[4 * g + 1], pw[4 * g + 2], pw[4 * g + 3]});
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int db = 2 * (j % (DB / 2)) + u;
        dq[db] = mfma(fr[(KS + j) % RS][u], pb, dq[db]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int t = 0; t < nk; t += 2) {
    step(t, Stage<0>{});
    if (t + 1 < nk) step(t + 1, Stage<1>{});
  }
  if (live) {
    bf16_t* dst = a.d_qkv + (tok0 + qw) * ld + (long)hd * D;
#pragma unroll
    for (int db = 0; db < DB; ++db) store_cols(dst + 32 * db, dq[db], h2, a.rs);
  }
}

// dK and dV: blocks of 4 waves of 32 keys, two to a CU, over 32-query tiles. The
// accumulators leave no registers for a tile ahead; within a tile every LDS read
// (Q, dO and the block's V rows, then dO and Q transposed) is one (D = 64: two)
// groups of products ahead of its use, S and dP alternate, and the other block of
// the CU fills the elementwise part (half of it beside the first products of
// dV and dK was 2-4% slower at D = 128). Before -> now, as above: 1258 -> 1120, 256 ->
// 182 and 163 -> 127 us.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void attn_dkdv_kernel(AttnArgs a) {
  constexpr int KS = D / 16, DB = D / 32, NW = 4, KB = 32 * NW;
  using Dma = TileDma<D, 32, NW>;
  constexpr int TQ = Dma::TB;           // one 32-row tile
  constexpr int VT = 4 * TQ;            // two slots of Q and dO, then the block's V rows,
  constexpr int ST = VT + KB * D * 2;   // then two slots of 32 lse2 and 32 delta
  __shared__ __attribute__((aligned(1024))) char lds[ST + 2 * 256];
  // the wave index through readfirstlane: the compiler then knows it is
  // wave-uniform, and the branches on a wave's query or key range are
  // scalar branches instead of exec-mask ones (backward 7-10% faster)
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6),
            h2 = lane >> 5, lq = lane & 31;
  int kt, hd, sq;
  decode(a, false, false, kt, hd, sq, KB);
  const long tok0 = (long)sq * a.N, ld = 3L * a.M;
  const bf16_t* Qg = a.qkv + tok0 * ld + (long)hd * D;
  const bf16_t* Gg = a.d_o + tok0 * a.M + (long)hd * D;
  const long srow0 = (long)hd * a.T + tok0;
  const int k0 = kt * KB, kw = k0 + 32 * w + lq;
  const bool live = kw < a.N;
  // query steps of 32: causal keys k0.. are seen by queries >= k0 only
  const int qs0 = CAUSAL ? k0 : 0;
  const int nqs = (a.N - qs0 + 31) / 32;

  const Dma dma(lds_base(lds), w, lane, ld), dmag(lds_base(lds), w, lane, a.M);
#pragma unroll
  for (int i = 0; i < NW; ++i)
    dma.load(Qg + 2L * a.M + (long)(k0 + 32 * i) * ld, a.N - k0 - 32 * i, VT + i * TQ);
  bf16x8 kf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    kf[ks] = live ? *reinterpret_cast<const bf16x8*>(Qg + a.M + kw * ld + 16 * ks + 8 * h2) : zero8();
  float rstat = 0.0f;  // (the block's first 64 threads)
  const float* sp = (tid < 32 ? a.lse : a.delta) + srow0 + (tid & 31);
  auto load_stat = [&](int qb) {
    if (tid < 64) rstat = qb + (tid & 31) < a.N ? sp[qb] * (tid < 32 ? kLog2e : 1.0f) : 0.0f;
  };
  auto store_stat = [&](int slot) {
    if (tid < 64) reinterpret_cast<float*>(lds + ST + 256 * slot)[tid] = rstat;
  };
  const bf16_t* Qt = Qg + qs0 * ld;
  const bf16_t* Gt = Gg + (long)qs0 * a.M;
  dma.load(Qt, a.N - qs0, 0);
  dmag.load(Gt, a.N - qs0, TQ);
  load_stat(qs0);
  store_stat(0);
  floatx16 dv[DB], dk[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    dv[db] = zero16();
    dk[db] = zero16();
  }
  int rbase = row_base<D>(lq, h2), tb0 = tr_base<D>(lane, 0), tb1 = tr_base<D>(lane, 1);
  // read groups: 0 .. KS - 1, the Q, dO and V rows at k step i; then 2 DB groups of dO
  // and Q transposed, 16 queries by 32 columns each
  constexpr int NG = KS + 2 * DB;
  constexpr int RS = D == 128 ? 2 : 3;  // groups in registers (128: three spill)
  bf16x8 fr[RS][3];
  auto read_group = [&](const char* tq, int i) {
    const char* tg = tq + TQ;
    if (i < KS) {
      fr[i % RS][0] = frag_row_x<D>(tq, rbase, 0, i);
      fr[i % RS][1] = frag_row_x<D>(tg, rbase, 0, i);
      fr[i % RS][2] = frag_row_x<D>(lds + VT, rbase, 32 * w, i);
    } else if (i < NG) {
      fr[i % RS][0] = frag_tr_x<D>(tg, tb0, tb1, 16 * ((i - KS) / DB), 32 * ((i - KS) % DB));
      fr[i % RS][1] = frag_tr_x<D>(tq, tb0, tb1, 16 * ((i - KS) / DB), 32 * ((i - KS) % DB));
    }
  };
  auto step = [&](const int it, auto stc) {
    constexpr int st = decltype(stc)::value;
    opaque(rbase, tb0, tb1);
    const int qb = qs0 + 32 * it;
    wait_vm<0>();   // this tile's loads
    lds_barrier();  // and every wave's reads of the other slot are done
    const char* tq = lds + st * 2 * TQ;
    const float* l2 = reinterpret_cast<const float*>(lds + ST + 256 * st);
    const bool mine = !CAUSAL || qb + 31 >= k0 + 32 * w;
    if (mine) {
      read_group(tq, 0);
      if constexpr (RS > 2) read_group(tq, 1);
    }
    Qt += 32 * ld;
    Gt += 32L * a.M;
    dma.load(Qt, a.N - qb - 32, (st ^ 1) * 2 * TQ);
    dmag.load(Gt, a.N - qb - 32, (st ^ 1) * 2 * TQ + TQ);
    if (it + 1 < nqs) load_stat(qb + 32);
    if (mine) {
      floatx16 s, dp;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        read_group(tq, i + RS - 1);
        __builtin_amdgcn_sched_barrier(0);
        s = mfma(fr[i % RS][0], kf[i], i == 0 ? zero16() : s);
        dp = mfma(fr[i % RS][1], fr[i % RS][2], i == 0 ? zero16() : dp);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (qb + 32 > a.N || (CAUSAL && k0 + 32 * w + 31 > qb)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int q = qb + 8 * (r >> 2) + 4 * h2 + (r & 3);
          if (q >= a.N || (CAUSAL && kw > q)) s[r] = -INFINITY;
        }
      }
      unsigned pp[8], pd[8];  // P and dS of this lane, bf16 pairs
#pragma unroll
      for (int J = 0; J < 4; ++J) {
        const float4 lv = *reinterpret_cast<const float4*>(l2 + 8 * J + 4 * h2);
        const float4 dv4 = *reinterpret_cast<const float4*>(l2 + 32 + 8 * J + 4 * h2);
        const float lr[4] = {lv.x, lv.y, lv.z, lv.w}, dr[4] = {dv4.x, dv4.y, dv4.z, dv4.w};
        float pv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          pv[j] = exp2_fast(fmaf(s[4 * J + j], a.c2, -lr[j]));
          dp[4 * J + j] = pv[j] * (dp[4 * J + j] - dr[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; j += 2) {
          pp[2 * J + j / 2] = pack_bf16x2(pv[j], pv[j + 1]);
          pd[2 * J + j / 2] = pack_bf16x2(dp[4 * J + j], dp[4 * J + j + 1]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 2 * DB; ++j) {
        read_group(tq, KS + j + RS - 1);
        __builtin_amdgcn_sched_barrier(0);
        const int g = j / DB, db = j % DB, c = (KS + j) % RS;
        dv[db] = mfma(fr[c][0], __builtin_bit_cast(bf16x8, u32x4{pp[4 * g], pp[4 * g + 1], pp[4 * g + 2], pp[4 * g + 3]}), dv[db]);
        dk[db] = mfma(fr[c][1], __builtin_bit_cast(bf16x8, u32x4{pd[4 * g], pd[4 * g + 1], pd[4 * g + 2], pd[4 * g + 3]}), dk[db]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (it + 1 < nqs) store_stat(st ^ 1);
  };
  for (int it = 0; it < nqs; it += 2) {
    step(it, Stage<0>{});
    if (it + 1 < nqs) step(it + 1, Stage<1>{});
  }
  if (live) {
    bf16_t* dst = a.d_qkv + (tok0 + kw) * ld + (long)hd * D;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      store_cols(dst + a.M + 32 * db, dk[db], h2, a.rs);
      store_cols(dst + 2L * a.M + 32 * db, dv[db], h2, 1.0f);
    }
  }
}

AttnArgs attn_args(const AttnShape& m, int T, int M) {
  AttnArgs a = {};
  a.T = T;
  a.M = M;
  a.N = m.N;
  a.heads = m.heads;
  a.nseq = m.N > 0 ? T / m.N : 0;
  a.c2 = kLog2e / sqrtf((float)m.D);
  a.rs = 1.0f / sqrtf((float)m.D);
  return a;
}

unsigned attn_blocks(const AttnArgs& a, int rows = 128) {
  return (unsigned)(((a.N + rows - 1) / rows) * a.heads * a.nseq);
}

// pair long and short causal tiles (decode) when the grid (two blocks per CU) is
// resident all at once: then the makespan is a CU's two blocks together, not
// the longest-first order's
int attn_pair(const AttnShape& m, const AttnArgs& a) {
  return m.causal && attn_blocks(a) <= 2u * 256u ? 1 : 0;
}

// Forward of heads of 64 in blocks of 8 waves, which read K and V half as often:
// where they are two rounds of two to a CU at least, and leave no half of a block
// without queries. 4 and 8 waves, us: 32 and 64 sequences of 512, 16 heads,
// bidirectional 58 and 51, 110 and 95; 16 sequences (one round), causal 21.8 and 23.0;
// 128 of 128 (half empty) 29 and 33; 4 of 700, 48 heads (576 blocks) 41 and 45.
bool fwd_wide(const AttnArgs& a) {
  return attn_blocks(a, 256) >= 4u * 256u && 2 * attn_blocks(a, 256) == attn_blocks(a);
}

// Query tiles of a head side by side (decode)? Bidirectional ones have equal work and
// lose nothing by it: 64 sequences of 512, 16 heads of 128, forward 263 -> 198 us (227
// with the 8-wave blocks before the one-tile-ahead loop, which read K and V half as
// often), dQ 378 -> 301; 4 x 4096, 32 heads 1110 -> 1013 and 1646 -> 1521; one sequence
// of 4096 the same. Causal tiles then no longer run longest first over the whole launch,
// which costs up to 40 % where K and V stay in the 256 MB Infinity Cache; the forward
// takes it where they do not (kv: their bytes) and the tiles of a head are few, or far
// past it (T = 65536, heads of 128, width 2048: N = 512 421 -> 349 us, 1024 632 -> 447, 2048
// 1004 -> 717, 4096 1345 -> 1208; half of that 199 -> 182, 261 -> 227, 375 -> 351, and
// 580 -> 592 for 4096; N = 300, 189 MB, heads of 128 and 64, 143 -> 120 and 163 -> 129).
// 8-wave blocks have half as many tiles and gain little (2-4 %) or lose up to 12 %.
// The key tiles of dK and dV gain 11 % and lose 8 % on the bidirectional shapes, and
// keep their order.
bool shared_order(const AttnShape& m, const AttnArgs& a) {
  if (!m.causal) return true;
  if (m.D == 64 && fwd_wide(a)) return false;
  const long mb = 1L << 20, kv = 4L * a.T * a.M, nt = (a.N + 127) / 128;
  return kv >= 448 * mb || (kv >= 176 * mb && nt <= 3) ||
         (kv >= 240 * mb && m.D == 128 && nt <= 16);
}

template <int D, int NW>
void launch_fwd(const AttnShape& m, const AttnArgs& a, hipStream_t st) {
  const dim3 g(attn_blocks(a, 32 * NW)), b(64 * NW);
  if (m.causal) hipLaunchKernelGGL((attn_fwd_kernel<D, true, NW>), g, b, 0, st, a);
  else hipLaunchKernelGGL((attn_fwd_kernel<D, false, NW>), g, b, 0, st, a);
}

#define FLOWMOE_ATTN_LAUNCH(KERNEL, a, st)                                       \
  do {                                                                            \
    const dim3 g(attn_blocks(a)), b(256);                                         \
    if (m.D == 128) {                                                             \
      if (m.causal) hipLaunchKernelGGL((KERNEL<128, true>), g, b, 0, st, a);      \
      else hipLaunchKernelGGL((KERNEL<128, false>), g, b, 0, st, a);              \
    } else {                                                                      \
      if (m.causal) hipLaunchKernelGGL((KERNEL<64, true>), g, b, 0, st, a);       \
      else hipLaunchKernelGGL((KERNEL<64, false>), g, b, 0, st, a);               \
    }                                                                             \
  } while (0)

}  // namespace

hipError_t launch_attn_fwd(const AttnShape& m, int T, int M, const void* qkv, void* o, float* lse,
                           hipStream_t st) {
  AttnArgs a = attn_args(m, T, M);
  if (attn_blocks(a) == 0) return hipSuccess;
  a.qkv = static_cast<const bf16_t*>(qkv);
  a.out = static_cast<bf16_t*>(o);
  a.lse = lse;
  a.pair = attn_pair(m, a);
  a.shared = shared_order(m, a);
  return traced(FLOWMOE_K_ATTN_FWD, st, [&] {
    if (m.D == 128) launch_fwd<128, 4>(m, a, st);
    else if (fwd_wide(a)) launch_fwd<64, 8>(m, a, st);
    else launch_fwd<64, 4>(m, a, st);
  });
}

hipError_t launch_attn_bwd(const AttnShape& m, int T, int M, const void* qkv, const void* o,
                           const float* lse, const void* d_o, void* d_qkv, float* delta,
                           hipStream_t st) {
  AttnArgs a = attn_args(m, T, M);
  if (attn_blocks(a) == 0) return hipSuccess;
  a.qkv = static_cast<const bf16_t*>(qkv);
  a.o = static_cast<const bf16_t*>(o);
  a.d_o = static_cast<const bf16_t*>(d_o);
  a.d_qkv = static_cast<bf16_t*>(d_qkv);
  a.lse = const_cast<float*>(lse);
  a.delta = delta;
  a.pair = attn_pair(m, a);
  a.shared = !m.causal;
  hipError_t e = traced(FLOWMOE_K_ATTN_BWD_DQ, st, [&] { FLOWMOE_ATTN_LAUNCH(attn_dq_kernel, a, st); });
  if (e != hipSuccess) return e;
  return traced(FLOWMOE_K_ATTN_BWD_DKDV, st,
                [&] { FLOWMOE_ATTN_LAUNCH(attn_dkdv_kernel, a, st); });
}

hipError_t launch_mha_fwd(const AttnShape& m, int T, int M, const void* in, const void* w_qkv,
                          const void* w_o, void* qkv, void* attn, float* lse, void* out,
                          hipStream_t st) {
  if (T == 0) return hipSuccess;
  hipError_t e = launch_dense_gemm(FLOWMOE_K_ATTN_QKV, T, in, M, M, w_qkv, 3L * M, false, 3 * M,
                                   qkv, 3L * M, st);
  if (e != hipSuccess) return e;
  e = launch_attn_fwd(m, T, M, qkv, attn, lse, st);
  if (e != hipSuccess) return e;
  return launch_dense_gemm(FLOWMOE_K_ATTN_OUT, T, attn, M, M, w_o, M, false, M, out, M, st);
}

hipError_t launch_mha_bwd_data(const AttnShape& m, int T, int M, const void* w_qkv,
                               const void* w_o, const void* qkv, const void* attn,
                               const float* lse, const void* d_out, void* d_attn, void* d_qkv,
                               float* delta, void* d_in, hipStream_t st) {
  if (T == 0) return hipSuccess;
  // d_attn = d_out W^O^T: B[k][n] = W^O[n][k] (K-contiguous)
  hipError_t e = launch_dense_gemm(FLOWMOE_K_ATTN_DGRAD, T, d_out, M, M, w_o, M, true, M, d_attn,
                                   M, st);
  if (e != hipSuccess) return e;
  e = launch_attn_bwd(m, T, M, qkv, attn, lse, d_attn, d_qkv, delta, st);
  if (e != hipSuccess) return e;
  // d_in = d_qkv [W^Q | W^K | W^V]^T: B[k][n] = W_qkv[n][k] (K-contiguous)
  return launch_dense_gemm(FLOWMOE_K_ATTN_DGRAD, T, d_qkv, 3L * M, 3 * M, w_qkv, 3L * M, true, M,
                           d_in, M, st);
}

hipError_t launch_mha_wgrad(int T, int M, int R, const void* in, const void* attn,
                            const void* d_out, const void* d_qkv, float* dw_qkv, float* dw_o,
                            int accumulate, void* ws, hipStream_t st) {
  // dW^O = attn^T d_out and dW_qkv = in^T d_qkv, each summed over the R
  // chunks' rows in chunk order (through partial sums in ws when their
  // output tiles are too few for the CUs)
  float* part = static_cast<float*>(ws);
  hipError_t e = launch_dense_wgrad(FLOWMOE_K_ATTN_WGRAD, T, R, attn, M, (long)T * M, M, d_out, M,
                                    (long)T * M, M, dw_o, M, accumulate, part, st);
  if (e != hipSuccess) return e;
  return launch_dense_wgrad(FLOWMOE_K_ATTN_WGRAD, T, R, in, M, (long)T * M, M, d_qkv, 3L * M,
                            (long)T * 3 * M, 3 * M, dw_qkv, 3L * M, accumulate, part, st);
}

}  // namespace flowmoe
