// Expert FFN (E_r of Sec. 2.1) as grouped GEMMs over the dispatched rows.
//
// Two grouping modes:
//   ROWS  C_e[rows_e x N] = A[rows of e][K] * B_e[K x N]   (forward, dgrad):
//         the M dimension is ragged per expert (counts on the device), the
//         grid covers an upper bound of row tiles and each block finds its
//         expert by a prefix over the per-expert tile counts.
//   KSUM  C_e[Mdim x N]  = sum over rows r of e: A[r][.]^T B[r][.]  (wgrad):
//         the reduction length K = counts[e] is ragged.
//
// bf16 path: v_mfma_f32_32x32x16_bf16 over 256 x 256 tiles or, where those are few, 256 x
// 128 or (row mode) 128 x 128 ones, the operands streamed global -> LDS.
// fp32 path: v_mfma_f32_32x32x2_f32 over 128-, 64- or 32-row x 128-column tiles,
// the same modes and epilogues.
#include <math.h>

#include <algorithm>
#include <atomic>

#include "common.hpp"

namespace flowmoe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

enum { MODE_ROWS = 0, MODE_KSUM = 1 };
constexpr int kCUs = 256;
enum {
  EPI_STORE = 0,       // C0 = acc
  EPI_GELU_FWD = 1,    // C0 = h = acc, C1 = a = gelu(acc)
  EPI_SWIGLU_FWD = 2,  // dual accumulators h1, h3: C0 = [h1 | h3], C1 = silu(h1) h3
  EPI_GELU_BWD = 3,    // C0 = acc * gelu'(aux h)
  EPI_SWIGLU_BWD = 4,  // C0 = [acc h3 silu'(h1) | acc silu(h1)] with aux = [h1 | h3]
  EPI_WGRAD = 5,       // fp32 C0 (cols < nsplit) / C1 (cols >= nsplit), optional +=
  EPI_GATE_DW = 6,     // as EPI_WGRAD (its own instance: the gate's dW_g partials)
  EPI_ADD = 7          // C0 += acc (bf16; aux = C0 itself, prefetched like a pre-activation)
};

struct GemmParams {
  const void* A;
  long lda;
  const void* B0;
  const void* B1;    // second B source: W3 (dual forward) or k >= ksplit (dgrad)
  long ldb;
  long b_estride;    // per-expert stride of B (ROWS mode)
  int ksplit;        // ROWS, K-contiguous B: k >= ksplit reads B1 at k - ksplit
  int Mdim, N, K;    // KSUM: Mdim rows of C; ROWS: K reduction length
  const int32_t* counts;
  const int32_t* offsets;
  int E;
  int padC;          // padded layout: every expert spans C rows (0 = packed)
  int tiles;         // ROWS, bf16: tile shape (FLOWMOE_TILES_*)
  void* C0;
  void* C1;
  long ldc, ldc1;
  long c_estride;    // KSUM: per-expert stride of C
  int nsplit;        // EPI_WGRAD: first column that goes to C1
  const void* aux;   // h (GELU) or [h1 | h3] (SwiGLU), ld = ldaux
  long ldaux;
  int Hh;            // SwiGLU: H (offset of the second half)
  int accumulate;
  // KSUM: the reduction runs over nseg row segments (the chunks of a layer
  // call), in segment order; segment g's rows of expert e are those of
  // counts[g * E + e] and offsets[g * (E + 1) + e] in A + g * a_sstride and
  // B0 + g * b_sstride (elements)
  int nseg;
  long a_sstride, b_sstride;
  // rows of each row buffer (of each segment's): an expert's range
  // [offsets[e], offsets[e] + rows) is cut at it
  long rows_cap;
  // forward epilogues: per-expert float biases added to the data rows' outputs
  // (bias0 to C0's columns: b1 for h / h1, b2 for y; bias1: b3 for the dual
  // forward's h3), bias0[e * bias_estride + column]; null: none
  const float* bias0;
  const float* bias1;
  long bias_estride;
  // streaming kernel, row mode: an expert's light row tiles walked with its
  // heavy ones (1) or after every heavy tile (0)
  int joined;
  // bf16: reduction rows of a non-K-contiguous operand that one buffer descriptor
  // covers (buffer_piece); longer reductions run in pieces of so many
  int piece;
};


// counts and offsets are device data: a range that inconsistent ones would
// take past the row buffers is cut there, not followed
__device__ __forceinline__ int clip_rows(long off, int n, long cap) {
  if (off < 0 || off >= cap || n <= 0) return 0;
  return (int)min((long)n, cap - off);
}

// Expert e's rows in segment g: counts[g * E + e] rows from row
// offsets[g * (E + 1) + e]. A dense launch (counts null: the attention's
// projections) splits the rows_cap rows of every segment into E equal
// parts, part e being rows [e rows_cap / E, (e + 1) rows_cap / E) (E = 1:
// all of them; E > 1: the token splits of a weight gradient).
__device__ __forceinline__ int seg_offset(const GemmParams& p, int g, int e) {
  return p.counts ? p.offsets[g * (p.E + 1) + e] : (int)(p.rows_cap * e / p.E);
}
__device__ __forceinline__ int seg_count(const GemmParams& p, int g, int e) {
  return p.counts ? p.counts[g * p.E + e]
                  : (int)(p.rows_cap * (e + 1) / p.E - p.rows_cap * e / p.E);
}

// ---------------------------------------------------------------------------
// bf16 kernels: tile order, LDS layout, epilogue
// ---------------------------------------------------------------------------
// LDS tile layout: 128-byte rows (64 bf16 of K), 16-byte chunks XOR-swizzled
// by (row / 2) % 8. A ds_read_b128 is serviced 16 lanes per cycle over 64
// banks; the 16 consecutive rows it touches then fall into 16 distinct
// 16-byte bank slots.
__device__ __forceinline__ int lds_off(int row, int chunk) {
  return row * 128 + (((chunk ^ (row >> 1)) & 7) << 4);
}

__device__ __forceinline__ float silu_f(float z) { return z * sigmoid_f(z); }

// Blocks are dispatched round-robin over the 8 XCDs (each with its own L2);
// renumber them so that every XCD works on one contiguous range of tiles.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
  const int q = nblocks >> 3, rem = nblocks & 7;
  const int x = bid & 7, i = bid >> 3;
  return x * q + (x < rem ? x : rem) + i;
}

// Tile of dispatch position P (blocks go to the 8 XCDs round-robin: position
// P runs on XCD P % 8, as its (P / 8)-th block) in an nrows x ncols grid of
// output tiles walked in blocks of (at most) 16 x 16 tiles, row block by row
// block. XCD x takes a sub-block of each block, m tile fastest: split 4 x 2
// (rows (x % 4) r/4 .., columns (x / 4) c/2 ..) when the block's r rows and
// c columns allow it, else 8 x 1 or 1 x 8, else the block is walked m tile
// fastest. A full block's 256 tiles are one round of all 256 CUs: inside an
// XCD the 32 tiles running together share 12 operand panels through its L2,
// and across XCDs every B panel is read by four XCDs and every A panel by
// two at about the same time, so that the Infinity Cache serves the
// repeats instead of HBM (with each XCD on a range of its own, the XCDs
// stream eight different experts' weights at once). Every block starts at a
// multiple of 16, so its positions j have j % 8 == P % 8.
__device__ __forceinline__ void shared_block_tile(int P, int nrows, int ncols, int& mt, int& nt) {
  constexpr int SB = 16;
  const int rb = P / (SB * ncols);
  const int r = min(SB, nrows - rb * SB);   // rows of this row block
  const int Pr = P - rb * SB * ncols;       // position inside the row block
  const int cb = Pr / (r * SB);
  const int c = min(SB, ncols - cb * SB);   // columns of this block
  const int j = Pr - cb * r * SB;           // position inside the r x c block
  const int gr = (r % 4 == 0 && c % 2 == 0) ? 4 : (r % 8 == 0) ? 8 : (c % 8 == 0) ? 1 : 0;
  int lr, lc;
  if (gr != 0) {
    const int gc = 8 / gr, sr = r / gr, sc = c / gc;  // sub-block of sr x sc tiles per XCD
    const int x = j & 7, s = j >> 3;
    lr = (x % gr) * sr + s % sr;
    lc = (x / gr) * sc + s / sr;
  } else {
    lr = j % r;
    lc = j / r;
  }
  mt = rb * SB + lr;
  nt = cb * SB + lc;
}

constexpr int kRowGroup = 4;  // row tiles per group of the row-mode tile order

template <int V>
struct IntC {
  static constexpr int value = V;
};

// inclusive prefix sum of v over the lanes of a wave: DPP moves inside the rows
// of 16 lanes, then the row totals broadcast to the rows after them (six vector
// adds; through ds_bpermute each of six exchanges is an LDS round trip)
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ int wave_incl_scan(int v) {
  v = dpp_add<0x111, 0xF>(v);  // row_shr 1, 2, 4, 8
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  v = dpp_add<0x118, 0xF>(v);
  v = dpp_add<0x142, 0xA>(v);  // row_bcast 15: rows 1 and 3 add the row before
  v = dpp_add<0x143, 0xC>(v);  // row_bcast 31: rows 2 and 3 add the first two
  return v;
}

// Row-mode tile of the streaming kernel for block `bid`. The row tiles fall
// in two classes: heavy ones (at least half a tile of live rows) and light
// ones (an expert's short last tile, or padding only). Every XCD (blocks are
// dispatched round-robin over the 8 XCDs) takes an equal share of each class
// and runs its heavy tiles first, so that the light tiles make up the last,
// partial round on every XCD instead of a full-cost round on some. The heavy
// tiles (the experts' heavy row tiles one after the other x the column
// tiles) are walked in shared 16 x 16 blocks (shared_block_tile); inside the
// light class, consecutive tiles walk kRowGroup row tiles x the column
// tiles, row tiles fastest. Returns false for a block with no tile.
struct LaneRows {  // lane x: expert x's live rows, first row, and rows with the padding
  int c, o, r;
};

template <int BM>
__device__ __forceinline__ bool row_tile_of_block(const GemmParams& p, int ntiles, const LaneRows& lr,
                                                  int bid, int& e, int& mt, int& nt, int& rows_e,
                                                  int& cnt_e, int& off_e) {
  // lane x holds expert x (E <= 64): its count and first row were loaded
  // together (one memory round trip), its tile counts per class are summed over
  // the lanes by a prefix scan, and the block's expert found by a ballot
  // (a walk over the experts in scalar registers cost ~0.15 us per expert)
  const int lane = threadIdx.x & 63;
  const bool live = lane < p.E;
  const int c = lr.c, o = lr.o, r = lr.r;
  const int te = (r + BM - 1) / BM;
  // heavy row tiles of this expert (joined order: all of them)
  const int he = p.joined ? te : min(te, (c + BM / 2) / BM);
  const int le = te - he;                     // light ones
  const int hin = wave_incl_scan(he), lin = wave_incl_scan(le);
  const int HR = __builtin_amdgcn_readlane(hin, 63), LR = __builtin_amdgcn_readlane(lin, 63);
  const int x = bid & 7, i = bid >> 3;
  const int H = HR * ntiles, L = LR * ntiles;
  const int hx = (H >> 3) + (x < (H & 7)), lx = (L >> 3) + (x < (L & 7));
  bool heavy;
  int ml;
  if (i < hx) {
    heavy = true;
    shared_block_tile(i * 8 + x, HR, ntiles, ml, nt);  // (i * 8 + x < H)
  } else if (i < hx + lx) {
    heavy = false;
    const int idx = x * (L >> 3) + min(x, L & 7) + (i - hx);
    const int gsz = kRowGroup * ntiles;
    const int g = idx / gsz, rg = idx - g * gsz;
    const int gm = min(kRowGroup, LR - g * kRowGroup);  // row tiles in this group
    nt = rg / gm;
    ml = g * kRowGroup + (rg - nt * gm);
  } else {
    return false;
  }
  // the expert whose range of class tiles holds ml: the one lane with
  // (inclusive sum - own count) <= ml < inclusive sum
  const int inc = heavy ? hin : lin, own = heavy ? he : le;
  const uint64_t hit = __ballot(live && ml < inc && ml >= inc - own);
  if (hit == 0) return false;
  e = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(hit));
  mt = (heavy ? 0 : __builtin_amdgcn_readlane(he, e)) + ml -
       (__builtin_amdgcn_readlane(inc, e) - __builtin_amdgcn_readlane(own, e));
  rows_e = __builtin_amdgcn_readlane(r, e);
  cnt_e = __builtin_amdgcn_readlane(c, e);
  off_e = __builtin_amdgcn_readlane(o, e);
  return true;
}

// grid of the streaming kernel in row mode: ceil(tiles / 8) + 1 blocks per
// XCD cover any split of the tile bound into the two classes
__host__ __device__ constexpr long row_mode_blocks(long tile_bound) { return 8 * ((tile_bound + 7) / 8 + 1); }

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16_t;
// Epilogue of the bf16 kernel: the accumulators of wave (wm, wn) of the tile,
// acc[i][j][4*g + q] = C[row (i/2)*128 + wm*64 + (i%2)*32 + lane%32]
//                       [col j*128 + wn*32 + 8*g + 4*(lane/32) + q],
// to global memory, 128 rows at a time through LDS (smem: 128 x 128 NB floats,
// 16-byte chunks XOR-swizzled by row): all waves stage, then wave w writes rows
// 16 w .. 16 w + 15 whole, consecutive lanes taking consecutive 16 bytes of a
// row's 512 (bf16) or 1024 (fp32). A wave that stored its own 64 columns wrote
// pieces of 64 or 128 bytes (weight gradients of a skewed layer's 16 experts, M =
// 1024, H = 4096: 69 -> 63 us). nhf: 128-row halves to write.
template <int MODE, int EPI, int BM, int NB>
__device__ __forceinline__ void gemm_epilogue(const GemmParams& p, floatx16 (&acc)[4][NB],
                                              char* smem, int e, int mt, int n0, int row0,
                                              int rows_e, int cnt_e, int wm, int wn, int nhf) {
  constexpr bool DUAL = EPI == EPI_SWIGLU_FWD;
  constexpr int BN = 128 * NB;
  // items of a row: 8 outputs (dual: of each of h1, h3 and a), or 4 fp32 ones
  constexpr int IPR = DUAL ? BN / 16 : MODE == MODE_KSUM ? BN / 4 : BN / 8;
  constexpr int PER = 16 * IPR / 64;  // items a lane and half; all of one column group
  static_assert(64 % IPR == 0, "one column group per lane");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lrow = lane & 31, lcol = 4 * (lane >> 5);
  const int cg = lane % IPR, r_first = wave * 16 + lane / IPR;  // item it: row r_first + it * RSTEP
  constexpr int RSTEP = 64 / IPR;
  float* stage = reinterpret_cast<float*>(smem);
  auto sidx = [&](int r, int c4) { return r * BN + ((c4 ^ (r & 15)) << 2); };
  bf16_t* C0 = static_cast<bf16_t*>(p.C0);
  bf16_t* C1 = static_cast<bf16_t*>(p.C1);
  const bf16_t* aux = static_cast<const bf16_t*>(p.aux);
  const int n = n0 + cg * (MODE == MODE_KSUM ? 4 : 8);
  const bool n_ok = n < p.N;  // (N and nsplit are multiples of 8)
  // forward biases: a lane's 8 (dual: 2 x 8) values, loaded once, before any
  // store (a wait for a load issued after stores would wait for those too)
  constexpr bool BIASED = MODE == MODE_ROWS && (EPI == EPI_STORE || EPI == EPI_GELU_FWD || DUAL);
  float bias0[8], bias1[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) bias0[q] = bias1[q] = 0.f;
  if constexpr (BIASED) {
    if (n_ok) {
      if (p.bias0 != nullptr) load8(p.bias0 + (long)e * p.bias_estride + n, bias0);
      if (p.bias1 != nullptr) load8(p.bias1 + (long)e * p.bias_estride + n, bias1);
    }
  }
#pragma unroll
  for (int hf = 0; hf < 2; ++hf) {
    if (hf >= nhf) break;
    // activation-backward epilogues read the saved pre-activations: all of
    // this half's loads go out before the staging, and none waits behind
    // an output store (one memory round trip per half, not one per item)
    constexpr bool AUXB = MODE == MODE_ROWS &&
                          (EPI == EPI_GELU_BWD || EPI == EPI_SWIGLU_BWD || EPI == EPI_ADD);
    Raw8b hr[AUXB ? PER : 1], h3r[AUXB ? PER : 1];
    if constexpr (AUXB) {
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        const int ti = hf * 128 + r_first + it * RSTEP;
        const bool ok = mt * BM + ti < rows_e && n_ok;
        const long off = ok ? (long)(row0 + ti) * p.ldaux + n : 0;  // (clamped: every load issued)
        hr[it] = raw8_load(aux + off);
        if constexpr (EPI == EPI_SWIGLU_BWD) h3r[it] = raw8_load(aux + off + (ok ? p.Hh : 0));
      }
    }
    if (hf > 0) lds_barrier();  // the first half's rows are read
#pragma unroll
    for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
          const floatx16& a = acc[hf * 2 + i2][j];
          *reinterpret_cast<float4*>(
              stage + sidx(wm * 64 + i2 * 32 + lrow, (j * 128 + wn * 32 + 8 * gq + lcol) >> 2)) =
              make_float4(a[4 * gq], a[4 * gq + 1], a[4 * gq + 2], a[4 * gq + 3]);
        }
    lds_barrier();
    auto read8 = [&](int r, int c8, float v[8]) {
      const float4 lo = *reinterpret_cast<const float4*>(stage + sidx(r, 2 * c8));
      const float4 hi = *reinterpret_cast<const float4*>(stage + sidx(r, 2 * c8 + 1));
      v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w;
      v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
    };
    if constexpr (MODE == MODE_KSUM) {  // fp32 weight gradient, C0 | C1 split at nsplit
      constexpr int PB = PER >= 8 ? 8 : PER;  // items per batch of accumulation loads
      float* D0 = static_cast<float*>(p.C0);
      float* D1 = static_cast<float*>(p.C1);
      float* col = (n < p.nsplit ? D0 + n : D1 + (n - p.nsplit)) + (long)e * p.c_estride;
#pragma unroll
      for (int b0 = 0; b0 < PER; b0 += PB) {
        // accumulation: the batch's old values are all loaded before any
        // store (from clamped addresses), one memory round trip per batch
        float4 old[PB];
        if (p.accumulate) {
#pragma unroll
          for (int i = 0; i < PB; ++i) {
            const int m = mt * BM + hf * 128 + r_first + (b0 + i) * RSTEP;
            old[i] = *reinterpret_cast<const float4*>(m < p.Mdim && n_ok ? col + (long)m * p.ldc : D0);
          }
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
          const int rr = r_first + (b0 + i) * RSTEP, m = mt * BM + hf * 128 + rr;
          if (m >= p.Mdim || !n_ok) continue;
          float4 v = *reinterpret_cast<const float4*>(stage + sidx(rr, cg));
          if (p.accumulate) {
            v.x += old[i].x;
            v.y += old[i].y;
            v.z += old[i].z;
            v.w += old[i].w;
          }
          *reinterpret_cast<float4*>(col + (long)m * p.ldc) = v;
        }
      }
    } else {
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        const int rr = r_first + it * RSTEP, ti = hf * 128 + rr;
        const int li = mt * BM + ti;
        if (li >= rows_e || !n_ok) continue;
        const bool data = li < cnt_e;
        const long g = row0 + ti;
        float v[8];
        read8(rr, cg, v);
        if (!data) {
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] = 0.f;
        }
        if constexpr (BIASED) {
          if (data) {
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] += bias0[q];
          }
        }
        if constexpr (DUAL) {
          float h3[8], a[8];
          read8(rr, IPR + cg, h3);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            h3[q] = data ? h3[q] + bias1[q] : 0.f;
            a[q] = silu_f(v[q]) * h3[q];
          }
          store8(C0 + g * p.ldc + n, v);
          store8(C0 + g * p.ldc + p.Hh + n, h3);
          store8(C1 + g * p.ldc1 + n, a);
        } else if constexpr (EPI == EPI_STORE) {
          store8(C0 + g * p.ldc + n, v);
        } else if constexpr (EPI == EPI_ADD) {
          float o[8];
          raw8_f32(hr[it], o);
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] += o[q];
          store8(C0 + g * p.ldc + n, v);
        } else if constexpr (EPI == EPI_GELU_FWD) {
          float a[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) a[q] = gelu_f(v[q]);
          store8(C0 + g * p.ldc + n, v);
          store8(C1 + g * p.ldc1 + n, a);
        } else if constexpr (EPI == EPI_GELU_BWD) {
          float h[8];
          raw8_f32(hr[it], h);
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] *= gelu_grad_f(h[q]);
          store8(C0 + g * p.ldc + n, v);
        } else if constexpr (EPI == EPI_SWIGLU_BWD) {
          float h1[8], h3[8], d3[8];
          raw8_f32(hr[it], h1);
          raw8_f32(h3r[it], h3);
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const float sg = sigmoid_f(h1[q]);
            d3[q] = v[q] * h1[q] * sg;
            v[q] = v[q] * h3[q] * sg * (1.f + h1[q] * (1.f - sg));
          }
          store8(C0 + g * p.ldc + n, v);
          store8(C0 + g * p.ldc + p.Hh + n, d3);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// bf16 kernel: two wave groups taking turns on the matrix pipes
// ---------------------------------------------------------------------------
// 8 waves, two along M (wm) and four along N (wn), one of each wm on every SIMD.
// A k-tile is 64 deep and held as two 128-row A halves and two (wide: 256 x 256
// tiles) or one (narrow: 256 x 128) 128-column B halves of 16 KB; a wave
// multiplies 64 rows of each A half by 32 columns of each B half, one (A half, B
// half) pair a phase: 8 v_mfma_f32_32x32x16_bf16, 256 cycles of a matrix pipe.
// Phases of wide tile t: (A0, BX), (A0, BY), (A1, BY), (A1, BX), X = t % 2, Y = 1 -
// X, so that the half a phase starts to use was read from LDS one phase before and
// its registers were free by then; of narrow tile t: (A0, B), (A1, B), tile t + 1's
// B in the other of two register sets.
//
// A phase is a memory part (LDS reads of the next phase's half, LDS-DMA loads of
// a half of a later tile, the wait for the half that the next phase reads), a
// barrier, the MFMAs, a barrier. The waves of wm = 1 run one part behind those of
// wm = 0, so on every SIMD one wave's MFMAs run beside the other's memory part,
// and no wave waits for its own reads or loads: the reads have a whole part to
// arrive, the loads six phases (wide; four narrow), 80 KB a block staying in
// flight. A half's LDS is refilled two phases after its read, when the barriers
// between have ordered every wave's reads before it.
//
// The last tile of a reduction (of either part of a split one) may be ragged:
// K-contiguous chunks past its length are masked to zeros.
//
// What it measured, and why 64 deep: 32-deep tiles (a four-stage ring, one
// barrier a tile, reads interleaved with the MFMAs of the same wave) fetched the
// K-contiguous operands in 64-byte pieces of 128-byte lines and kept the pipes
// busy 0.56-0.72 of the cycles; here it is 0.67-0.81 (SwiGLU experts of 16384
// rows at M = 4096, H = 14336: W1|W3 forward 6.68 -> 5.99 ms, W2 forward 3.21 ->
// 2.92, their dgrads 3.82 -> 3.24 and 7.08 -> 6.03, both weight gradients 9.33
// -> 9.04). What is left there is power and the L2 -> LDS stream (64 KB a tile at
// about 26 bytes a cycle): the clock falls to 1.54-1.6 GHz as the pipes get
// busier, and waiting for four more loads, issuing the loads first, or raising
// the MFMAs' wave priority changed nothing (0.0 to 0.5% slower). Narrow tiles
// need 48 KB for half the products; they replaced 4-wave ones of 32-deep tiles,
// two blocks to a CU (16 experts of mostly few rows, N = 1024, K = 4096: 100 -> 73
// us forward, 76 -> 59 dgrad) and a register-staged kernel for reductions that
// are no multiple of 32 (8 experts of 750 rows, N = 1024, K = 2728: 108 -> 58 us;
// K = 5456 in two parts: 183 -> 126).
constexpr int WBK = 64;           // k depth of a tile
constexpr int kHalf = 128 * WBK * 2;  // bytes of a half tile: 128 rows (or columns) x 64 k

// Fragments of a half tile (32 rows or columns from a wave's first one).
// K-contiguous: [128 rows][64 k], 128-byte rows, 16-byte chunk c of row r at
// c ^ ((r / 2) % 8); M/N-contiguous: [64 k][128 columns], 256-byte rows, chunk
// m of k-row k at m ^ (4 (k % 4)), two transposing reads a fragment. A lane's
// address is one base register, an XOR with the k step (K-contiguous) or the
// 32-column block (M/N-contiguous), and an immediate offset.
__device__ __forceinline__ int half_base(bool kc, int r0, int lane) {
  if (kc) return lds_off(r0 + (lane & 31), lane >> 5);
  const int G = lane >> 4, sl = lane & 15;
  const int col = r0 + (G & 1) * 16 + 4 * (sl & 3), kr = (G >> 1) * 8 + (sl >> 2);
  return kr * 256 + (((col >> 3) ^ ((kr & 3) << 2)) << 4) + ((col & 7) << 1);
}
// fragment of 32-row block i (rows r0 + 32 i ..; r0 a multiple of 64 where i > 0) at k step kk
template <bool KC>
__device__ __forceinline__ bf16x8 half_frag(const char* h, int base, int i, int kk) {
  if constexpr (KC) {
    return *reinterpret_cast<const bf16x8*>(h + (base ^ (kk << 5)) + i * 4096);
  } else {
    const char* a = h + (base ^ (i << 6)) + kk * 4096;
    const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)a);
    const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(a + 1024));
    const short __attribute__((ext_vector_type(8))) v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
}

// The same of a quarter tile [64 k][64 columns]: 128-byte rows, chunk m of k-row k at
// m ^ (4 (k / 2 % 2)) (four k-rows of 64 bytes fall into distinct banks).
__device__ __forceinline__ int quarter_base(int r0, int lane) {
  const int G = lane >> 4, sl = lane & 15;
  const int col = r0 + (G & 1) * 16 + 4 * (sl & 3), kr = (G >> 1) * 8 + (sl >> 2);
  return kr * 128 + (((col >> 3) ^ ((kr & 2) << 1)) << 4) + ((col & 7) << 1);
}
__device__ __forceinline__ bf16x8 quarter_frag(const char* q, int base, int kk) {
  const char* a = q + base + kk * 2048;
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)a);
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_t*)(a + 512));
  const short __attribute__((ext_vector_type(8))) v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}

constexpr int kGemmSmem = 9 * kHalf;  // 144 KB

// One tile of the kernels below. BM = 128: low tiles (row mode), light loops only.
// PIECES (row mode): a B of more bytes than a buffer descriptor's range, in pieces.
template <int MODE, bool A_KC, bool B_KC, int EPI, bool NARROW, int BM, bool PIECES = false>
__device__ __forceinline__ void gemm_tile(const GemmParams& p, char* smem, int ntiles, const LaneRows& lr) {
  constexpr int BN = NARROW ? 128 : 256;
  constexpr bool DUAL = EPI == EPI_SWIGLU_FWD;
  // the dual forward pairs 128-column W1 and W3 halves; narrow, the two 64-column
  // quarters of one half
  constexpr bool QUARTERS = DUAL && NARROW;
  static_assert(!QUARTERS || BM == 128, "quarters in the light loops only");
  // k-tiles in LDS (stages), the halves of one (A0, A1, B0 and wide B1) and its bytes
  constexpr int NST = NARROW ? 3 : 2, NB = NARROW ? 1 : 2, STB = (2 + NB) * kHalf;
  constexpr int SMEM = kGemmSmem;
  static_assert(NST * STB <= SMEM, "k-tiles do not fit");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const unsigned lds0 = lds_base(smem);

  // ---- which tile ----
  int e = 0, mt = 0, nt = 0, row0 = 0, rows_e = 0, cnt_e = 0;
  int seg_o = 0, seg_c = 0;  // KSUM: segment ranges, one lane per segment
  if constexpr (MODE == MODE_ROWS) {
    int off_e = 0;
    if (!row_tile_of_block<BM>(p, ntiles, lr, blockIdx.x, e, mt, nt, rows_e, cnt_e, off_e)) return;
    rows_e = clip_rows(off_e, rows_e, p.rows_cap);
    cnt_e = clip_rows(off_e, cnt_e, p.rows_cap);
    row0 = off_e + mt * BM;
  } else {
    const int mtn = (p.Mdim + BM - 1) / BM, ntn = (p.N + BN - 1) / BN;
    e = blockIdx.x / (mtn * ntn);
    shared_block_tile(blockIdx.x - e * (mtn * ntn), mtn, ntn, mt, nt);
    const int g = lane;
    seg_o = g < p.nseg ? seg_offset(p, g, e) : 0;
    seg_c = g < p.nseg ? seg_count(p, g, e) : 0;
    row0 = __builtin_amdgcn_readlane(seg_o, 0);
    cnt_e = clip_rows(row0, __builtin_amdgcn_readlane(seg_c, 0), p.rows_cap);
  }
  constexpr int NCOLS = DUAL ? BN / 2 : BN;
  const int n0 = nt * NCOLS;

  const bf16_t* A = static_cast<const bf16_t*>(p.A);
  const bf16_t* B0 = static_cast<const bf16_t*>(p.B0);
  const bf16_t* B1 = static_cast<const bf16_t*>(p.B1);

  // ---- buffer resources and per-lane source offsets (bytes) ----
  // A wave fills 1 KB blocks wave and wave + 8 of each half: 8 rows of a
  // K-contiguous half, 4 k-rows of an M/N-contiguous one.
  const int kc8 = ((lane & 7) ^ ((4 * (wave & 1) + (lane >> 4)) & 7)) * 8;  // k of a K-contiguous chunk
  const int kc_row = 8 * wave + (lane >> 3);
  const int mnc_k = 4 * wave + (lane >> 4);
  const int mnc_c = ((lane & 15) ^ ((lane >> 4) << 2)) * 8;
  const unsigned aoff = (unsigned)(A_KC ? ((long)kc_row * p.lda + kc8) * 2 : ((long)mnc_k * p.lda + mnc_c) * 2);
  // (quarters: 8 k-rows of 8 chunks a block)
  const unsigned boff = (unsigned)(B_KC ? ((long)kc_row * p.ldb + kc8) * 2
                                   : QUARTERS
                                       ? ((long)kc_row * p.ldb + ((lane & 7) ^ ((lane >> 4 & 1) << 2)) * 8) * 2
                                       : ((long)mnc_k * p.ldb + mnc_c) * 2);
  // byte steps: second block of a half, second half, k-tile
  const unsigned a_blk = (unsigned)((A_KC ? 64 : 32) * p.lda * 2), a_half = (unsigned)(A_KC ? 128 * p.lda * 2 : 256);
  const unsigned b_blk = (unsigned)((B_KC ? 64 : 32) * p.ldb * 2),
                 b_half = (unsigned)(DUAL ? 0 : B_KC ? 128 * p.ldb * 2 : 256);
  const unsigned a_kt = (unsigned)(A_KC ? WBK * 2 : WBK * p.lda * 2);
  const unsigned b_kt = (unsigned)(B_KC ? WBK * 2 : WBK * p.ldb * 2);

  u32x4 ra, rb0, rb1;
  int nk, nk0 = 1 << 30;  // k-tiles, those before the K split
  int k_lim = 0;          // ROWS: reduction length (of the part before the split)
  if constexpr (MODE == MODE_ROWS) {
    ra = make_rsrc(A + (long)row0 * p.lda, (long)(cnt_e - mt * BM) * p.lda * 2);
    k_lim = min(p.K, p.ksplit);
    if constexpr (B_KC) {
      const long valid = (long)min(p.N - n0, BN) * p.ldb * 2;
      rb0 = make_rsrc(B0 + (long)e * p.b_estride + (long)n0 * p.ldb, valid);
      rb1 = B1 != nullptr ? make_rsrc(B1 + (long)e * p.b_estride + (long)n0 * p.ldb, valid) : rb0;
    } else {
      if constexpr (PIECES) k_lim = min(p.K, p.piece);
      const long span = (long)k_lim * p.ldb;
      rb0 = make_rsrc(B0 + (long)e * p.b_estride + n0, (span - n0) * 2);
      rb1 = DUAL ? make_rsrc(B1 + (long)e * p.b_estride + n0, (span - n0) * 2) : rb0;
    }
    nk = (k_lim + WBK - 1) / WBK;
    if (B_KC && p.K > p.ksplit) {
      nk0 = nk;
      nk += (p.K - p.ksplit + WBK - 1) / WBK;
    }
    // a padding-only tile (padded layout) has nothing to reduce: zeros
    if (cnt_e <= mt * BM) nk = 0;
  } else {
    const int m0 = mt * BM, n = min(cnt_e, p.piece);
    ra = make_rsrc(A + (long)row0 * p.lda + m0, ((long)n * p.lda - m0) * 2);
    rb0 = make_rsrc(B0 + (long)row0 * p.ldb + n0, ((long)n * p.ldb - n0) * 2);
    rb1 = rb0;
    nk = (n + WBK - 1) / WBK;
  }
  // KSUM: rows r0 .. r0 + piece - 1 of segment g of the reduction (g >= 1 or r0 > 0)
  auto bind_rows = [&](int g, int r0) {
    row0 = g < 64 ? __builtin_amdgcn_readlane(seg_o, g) : seg_offset(p, g, e);
    cnt_e = clip_rows(row0, g < 64 ? __builtin_amdgcn_readlane(seg_c, g) : seg_count(p, g, e),
                      p.rows_cap);
    const int m0 = mt * BM, n = min(cnt_e - r0, p.piece);
    const long r = (long)row0 + r0;
    ra = make_rsrc(A + g * p.a_sstride + r * p.lda + m0, ((long)n * p.lda - m0) * 2);
    rb0 = make_rsrc(B0 + g * p.b_sstride + r * p.ldb + n0, ((long)n * p.ldb - n0) * 2);
    rb1 = rb0;
    nk = (n + WBK - 1) / WBK;
  };
  // ROWS, M/N-contiguous B: k from kb on (kb > 0, a multiple of the piece)
  auto bind_k = [&](int kb) {
    k_lim = min(p.K - kb, p.piece);
    ra = make_rsrc(A + (long)row0 * p.lda + kb, ((long)(cnt_e - mt * BM) * p.lda - kb) * 2);
    const long b = (long)e * p.b_estride + (long)kb * p.ldb + n0, span = (long)k_lim * p.ldb - n0;
    rb0 = make_rsrc(B0 + b, span * 2);
    rb1 = DUAL ? make_rsrc(B1 + b, span * 2) : rb0;
    nk = (k_lim + WBK - 1) / WBK;
  };
  auto drain = [] {  // every load and LDS read done before the stages are filled again
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  };

  // Loads of half h of tile t's operand A or B. Chunks past the reduction
  // length (and every chunk of a tile past the last) are out of the buffer's
  // range: they load zeros without traffic. The tile's byte offset stays in a
  // scalar register (opaque to the compiler, which would otherwise step a
  // vector register per load along the loop, and spill it).
  auto issue = [&](u32x4 r, unsigned dst, unsigned voff, unsigned so, unsigned blk, bool kc, int lim,
                   bool both = true) {
    unsigned so2 = so + blk;
    asm("" : "+s"(so), "+s"(so2));
    unsigned o = voff + so, o2 = voff + so2;
    if (kc) {
      const bool ok = kc8 < lim;
      o = ok ? o : 0xFFFFFFF0u;
      o2 = ok ? o2 : 0xFFFFFFF0u;
    }
    if (both) {
      const unsigned off[2] = {o, o2};
      dma16_row<2, 8192>(r, dst, off);
    } else {
      const unsigned off[1] = {o};
      dma16_row<1, 0>(r, dst, off);
    }
  };
  auto issue_a_to = [&](int t, int h, unsigned dst, bool both) {
    if constexpr (A_KC) {
      const bool sec = t >= nk0;
      const int k0 = (sec ? t - nk0 : t) * WBK, lim = (sec ? p.K - p.ksplit : k_lim) - k0;
      issue(ra, dst, aoff, (unsigned)((k0 + (sec ? p.ksplit : 0)) * 2) + h * a_half, a_blk, true, lim,
            both);
    } else {
      issue(ra, dst, aoff, (unsigned)t * a_kt + h * a_half, a_blk, false, 0, both);
    }
  };
  auto issue_b_to = [&](int t, int h, unsigned dst) {
    if constexpr (B_KC) {
      const bool sec = t >= nk0;
      const int k0 = (sec ? t - nk0 : t) * WBK, lim = (sec ? p.K - p.ksplit : k_lim) - k0;
      issue(sec ? rb1 : rb0, dst, boff, (unsigned)(k0 * 2) + h * b_half, b_blk, true, lim);
    } else if constexpr (QUARTERS) {
      issue(rb0, dst, boff, (unsigned)t * b_kt, 0, false, 0, false);
      issue(rb1, dst + 8192, boff, (unsigned)t * b_kt, 0, false, 0, false);
    } else {
      issue((DUAL && h) ? rb1 : rb0, dst, boff, (unsigned)t * b_kt + h * b_half, b_blk, false, 0);
    }
  };
  auto issue_a = [&](int t, int h, int stage) {
    issue_a_to(t, h, lds0 + stage * STB + h * kHalf + wave * 1024, true);
  };
  auto issue_b = [&](int t, int h, int stage) {
    issue_b_to(t, h, lds0 + stage * STB + (2 + h) * kHalf + wave * 1024);
  };

  floatx16 acc[4][NB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  auto barrier = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  int abase = half_base(A_KC, wm * 64, lane);
  int bbase = QUARTERS ? (wn >> 1) * 8192 + quarter_base((wn & 1) * 32, lane) : half_base(B_KC, wn * 32, lane);
  auto k_loop = [&](auto nh_c) {
    constexpr int NH = decltype(nh_c)::value;  // live A halves of this wave
    // [half][32-row block][k step]; [half (wide) or tile parity (narrow)][k step]
    bf16x8 af[2][2][4], bfr[2][4];
    // (the bases marked as changed: every XOR of them kept across the loop
    // would cost a register)
    auto read_a = [&](int stage, int h) {
      if (h < NH) {
        asm("" : "+v"(abase));
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            af[h][i][kk] = half_frag<A_KC>(smem + stage * STB + h * kHalf, abase, i, kk);
      }
    };
    auto read_b = [&](int stage, int h, int set) {
      if (NH > 0) {
        asm("" : "+v"(bbase));
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          bfr[set][kk] = half_frag<B_KC>(smem + stage * STB + (2 + h) * kHalf, bbase, 0, kk);
      }
    };
    // one phase: mem (reads, loads, the wait), then A half ha times bfr[set] into column block j
    auto phase = [&](auto&& mem, int ha, int set, int j) {
      mem();
      barrier();
      __builtin_amdgcn_sched_barrier(0);
      if (ha < NH) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[2 * ha + i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                bfr[set][kk], af[ha][i][kk], acc[2 * ha + i][j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      wait_lgkm0();
      barrier();
      __builtin_amdgcn_sched_barrier(0);
    };
    auto wait10 = [] {
      __builtin_amdgcn_sched_barrier(0);
      wait_vm<10>();
    };
    if (nk == 0) return;
    if constexpr (!NARROW) {
      auto tile = [&](int t, auto par_c) {
        constexpr int X = decltype(par_c)::value, Y = 1 - X;  // X: this tile's stage
        phase([&] { read_b(X, Y, Y); issue_a(t + 2, 0, X); wait10(); }, 0, X, X);
        phase([&] { read_a(X, 1); issue_b(t + 2, X, X); wait10(); }, 0, Y, Y);
        phase([&] { read_a(Y, 0); issue_b(t + 2, Y, X); wait10(); }, 1, Y, Y);
        phase([&] { read_b(Y, Y, Y); issue_a(t + 2, 1, X); wait10(); }, 1, X, X);
      };
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        issue_a(t, 0, t);
        issue_b(t, t, t);
        issue_b(t, 1 - t, t);
        issue_a(t, 1, t);
      }
      wait_vm<10>();
      barrier();
      read_a(0, 0);
      read_b(0, 0, 0);
      wait_lgkm0();
      barrier();
      if (wave >= 4) barrier();
      for (int t = 0;; t += 2) {
        tile(t, IntC<0>{});
        if (t + 1 >= nk) break;
        tile(t + 1, IntC<1>{});
        if (t + 2 >= nk) break;
      }
    } else {
      int s0 = 0, s1 = 1, s2 = 2;  // stages of tiles t, t + 1, t + 2
      auto tile = [&](int t, auto par_c) {
        constexpr int X = decltype(par_c)::value;
        phase(
            [&] {
              read_a(s0, 1);
              issue_a(t + 2, 1, s2);
              __builtin_amdgcn_sched_barrier(0);
              wait_vm<8>();
            },
            0, X, 0);
        phase([&] { read_a(s1, 0); read_b(s1, 0, 1 - X); issue_a(t + 3, 0, s0); issue_b(t + 3, 0, s0); wait10(); },
              1, X, 0);
        const int s = s0;
        s0 = s1;
        s1 = s2;
        s2 = s;
      };
      issue_a(0, 0, 0);
      issue_b(0, 0, 0);
      issue_a(0, 1, 0);
      issue_a(1, 0, 1);
      issue_b(1, 0, 1);
      issue_a(1, 1, 1);
      issue_a(2, 0, 2);
      issue_b(2, 0, 2);
      wait_vm<10>();
      barrier();
      read_a(0, 0);
      read_b(0, 0, 0);
      wait_lgkm0();
      barrier();
      if (wave >= 4) barrier();
      for (int t = 0;; t += 2) {
        tile(t, IntC<0>{});
        if (t + 1 >= nk) break;
        tile(t + 1, IntC<1>{});
        if (t + 2 >= nk) break;
      }
    }
    if (wave < 4) barrier();
  };
  // A tile of at most LR live rows: the weights' stream bounds it, so the stages
  // hold LR rows of A and the depth goes to B. One barrier a k-tile; tile t + 1's
  // fragments are read while tile t's are multiplied, and tile t's stage is
  // refilled with tile t + NS. 16 experts of 16 rows, N = 1024, K = 4096: 31 us, 134
  // MB of weights at 4.3 TB/s; the fine layer's second row tiles and the
  // balanced layer's light ones 1-6% of their launches faster than the phases.
  auto light_loop = [&](auto lr_c) {
    constexpr int LR = decltype(lr_c)::value;
    constexpr int AB = LR * WBK * 2, LST = AB + NB * kHalf;  // bytes of A, of a stage
    constexpr int NS = SMEM / LST, LPT = LR / 64 + 2 * NB;   // stages, loads a wave a tile
    const bool act = wm * 64 < LR;  // (64 rows: the waves of wm = 0 multiply)
    bf16x8 af[2][2][4], bfr[2][NB][4];  // [tile parity]
    auto issue_tile = [&](int t, int stage) {
      const unsigned st = lds0 + stage * LST + wave * 1024;
      issue_a_to(t, 0, st, LR == 128);
#pragma unroll
      for (int h = 0; h < NB; ++h) issue_b_to(t, h, st + AB + h * kHalf);
    };
    auto read = [&](int stage, auto set_c) {
      constexpr int set = decltype(set_c)::value;
      if (!act) return;
      asm("" : "+v"(abase), "+v"(bbase));
      const char* sa = smem + stage * LST;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
        for (int i = 0; i < 2; ++i) af[set][i][kk] = half_frag<A_KC>(sa, abase, i, kk);
#pragma unroll
        for (int h = 0; h < NB; ++h) {
          if constexpr (QUARTERS) bfr[set][h][kk] = quarter_frag(sa + AB, bbase, kk);
          else bfr[set][h][kk] = half_frag<B_KC>(sa + AB + h * kHalf, bbase, 0, kk);
        }
      }
    };
    if (nk == 0) return;
#pragma unroll
    for (int t = 0; t < NS; ++t) issue_tile(t, t);
    wait_vm<(NS - 1) * LPT>();
    barrier();
    read(0, IntC<0>{});
    wait_lgkm0();
    int s0 = 0;  // tile t's stage
    auto tile = [&](int t, auto set_c) {
      constexpr int set = decltype(set_c)::value;
      wait_vm<(NS - 2) * LPT>();
      barrier();
      __builtin_amdgcn_sched_barrier(0);
      const int s1 = s0 + 1 == NS ? 0 : s0 + 1;
      issue_tile(t + NS, s0);
      read(s1, IntC<1 - set>{});
      if (act) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int h = 0; h < NB; ++h)
              acc[i][h] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][h][kk], af[set][i][kk],
                                                                  acc[i][h], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      wait_lgkm0();
      s0 = s1;
    };
    for (int t = 0;; t += 2) {
      tile(t, IntC<0>{});
      if (t + 1 >= nk) break;
      tile(t + 1, IntC<1>{});
      if (t + 2 >= nk) break;
    }
  };
  // Weight gradient of an expert of few rows: every k-tile fits a stage, so all
  // are loaded at once and each wave multiplies them with no barrier between.
  auto short_loop = [&] {
    for (int t = 0; t < nk; ++t) {
      issue_a(t, 0, t);
      issue_b(t, 0, t);
      if constexpr (!NARROW) issue_b(t, 1, t);
      issue_a(t, 1, t);
    }
    wait_vm<0>();
    barrier();
    for (int t = 0; t < nk; ++t) {
      const char* st = smem + t * STB;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        bf16x8 bq[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) bq[j] = half_frag<B_KC>(st + (2 + j) * kHalf, bbase, 0, kk);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bf16x8 aq = half_frag<A_KC>(st + (i >> 1) * kHalf, abase, i & 1, kk);
#pragma unroll
          for (int j = 0; j < NB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq[j], aq, acc[i][j], 0, 0, 0);
        }
      }
    }
  };
  if constexpr (MODE == MODE_KSUM) {
    if (p.nseg == 1 && nk <= NST && cnt_e <= p.piece) short_loop();
    else {
      for (int g = 0, r0 = 0;;) {
        k_loop(IntC<2>{});
        r0 += p.piece;
        if (r0 >= cnt_e) {
          r0 = 0;
          if (++g >= p.nseg) break;
        }
        drain();
        bind_rows(g, r0);
      }
    }
  } else if constexpr (PIECES) {
    for (int kb = 0;;) {
      k_loop(IntC<2>{});
      kb += p.piece;
      if (kb >= p.K || nk == 0) break;
      drain();
      bind_k(kb);
    }
  } else {
    // light tiles, else live 64-row halves of this wave (wave-uniform): rows
    // wm * 64 .. and 128 + wm * 64 ..
    const int live = cnt_e - mt * BM;
    if (live <= 64) light_loop(IntC<64>{});
    else if (BM == 128 || live <= 128) light_loop(IntC<128>{});
    else if constexpr (BM > 128) {
      if (live > 128 + wm * 64) k_loop(IntC<2>{});
      else k_loop(IntC<1>{});
    }
  }
  drain();  // before the epilogue reuses the stages
  const int rows_t = MODE == MODE_ROWS ? rows_e - mt * BM : p.Mdim - mt * BM;
  gemm_epilogue<MODE, EPI, BM, NB>(p, acc, smem, e, mt, n0, row0, rows_e, cnt_e, wm, wn,
                                   BM > 128 && rows_t > 128 ? 2 : 1);
}

// Row mode: the tile shape is chosen from the experts' rows. Packed rows are known
// on the device only (a skewed gate fills a fifth of the capacity): there every
// block makes the same choice from the counts, and the host makes it for padded
// ones. The chain of k-tiles sets the time of a launch of few tiles, and a
// smaller tile's k-tile is shorter (0.6, 0.8-1.2 and 1.1-1.6 us for 128 x 128, 256 x
// 128 and 256 x 256): so the smallest shape whose tiles, the experts' partial ones
// included, fit one round of the 256 CUs, else 256 x 256. Against 256 x 128 tiles
// wherever the rows' capacity gives at most 1.25 x 256 wide ones (kernel times, H =
// 4096, M = 1024): T = 8192 top-1 on a heavy-tailed gate, E = 16, W2's forward 72.8
// -> 59.5 us and W1's dgrad 59.4 -> 47.0 (128 x 128); T = 4096, k = 2, E = 8, W1's
// dgrad 97.8 -> 89.0 and W2's forward 100.5 -> 102.3 (about 300 narrow tiles before,
// 150 wide ones now). A launch of several rounds pays 0-2 % for the choice.
constexpr int kTilesShort = -1;  // 128 x 128, beside the FLOWMOE_TILES_* values
__host__ __device__ inline int rows_shape(int t256, int t128, int n128, bool dual) {
  if ((long)t128 * n128 <= kCUs) return kTilesShort;
  return !dual && (long)t256 * n128 <= kCUs ? FLOWMOE_TILES_NARROW : FLOWMOE_TILES_WIDE;
}

template <bool B_KC, int EPI>
__global__ __launch_bounds__(512, 2) void gemm_bf16_rows_kernel(GemmParams p) {
  constexpr bool DUAL = EPI == EPI_SWIGLU_FWD;
  __shared__ __attribute__((aligned(1024))) char smem[kGemmSmem];
  const int lane = threadIdx.x & 63;
  const bool live = lane < p.E;
  LaneRows lr;
  lr.c = live ? seg_count(p, 0, lane) : 0;
  lr.o = live ? seg_offset(p, 0, lane) : 0;
  lr.r = live ? (p.padC ? p.padC : lr.c) : 0;
  const int n128 = (p.N + 127) / 128, n256 = DUAL ? n128 : (p.N + 255) / 256;
  int shape = p.tiles;
  if (shape == FLOWMOE_TILES_AUTO)
    shape = rows_shape(__builtin_amdgcn_readlane(wave_incl_scan((lr.r + 255) / 256), 63),
                       __builtin_amdgcn_readlane(wave_incl_scan((lr.r + 127) / 128), 63), n128, DUAL);
  if (shape == kTilesShort) gemm_tile<MODE_ROWS, true, B_KC, EPI, !DUAL, 128>(p, smem, n128, lr);
  else if (shape == FLOWMOE_TILES_WIDE || DUAL)
    gemm_tile<MODE_ROWS, true, B_KC, EPI, false, 256>(p, smem, n256, lr);
  else if constexpr (!DUAL) gemm_tile<MODE_ROWS, true, B_KC, EPI, true, 256>(p, smem, n128, lr);
}

// The dual forward in tiles of 128 x (64 + 64), for launches of few tiles: a k-tile is
// half the weights of a 128 x (128 + 128) one, so the chain of them is shorter and more
// of it in flight, on twice the CUs. A kernel of its own: beside the other shapes in
// the kernel above it made their loops up to 11 % slower (64 experts of 100 rows, M =
// 2048, H = 1408: 208 -> 233 us).
__global__ __launch_bounds__(512, 2) void gemm_bf16_pair64_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024))) char smem[kGemmSmem];
  const int lane = threadIdx.x & 63;
  const bool live = lane < p.E;
  LaneRows lr;
  lr.c = live ? seg_count(p, 0, lane) : 0;
  lr.o = live ? seg_offset(p, 0, lane) : 0;
  lr.r = live ? (p.padC ? p.padC : lr.c) : 0;
  gemm_tile<MODE_ROWS, true, false, EPI_SWIGLU_FWD, true, 128>(p, smem, (p.N + 63) / 64, lr);
}

// The row mode over a B that exceeds a buffer descriptor's range (an expert's
// weights of 2 GiB and more): 256 x 256 tiles, the reduction in pieces. Apart from
// the kernel above, whose loops a piece loop around them makes spill (300 vector
// registers).
template <int EPI>
__global__ __launch_bounds__(512, 2) void gemm_bf16_rows_pieces_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024))) char smem[kGemmSmem];
  const int lane = threadIdx.x & 63;
  const bool live = lane < p.E;
  LaneRows lr;
  lr.c = live ? seg_count(p, 0, lane) : 0;
  lr.o = live ? seg_offset(p, 0, lane) : 0;
  lr.r = live ? (p.padC ? p.padC : lr.c) : 0;
  constexpr int NC = EPI == EPI_SWIGLU_FWD ? 128 : 256;
  gemm_tile<MODE_ROWS, true, false, EPI, false, 256, true>(p, smem, (p.N + NC - 1) / NC, lr);
}

template <int EPI, bool NARROW>
__global__ __launch_bounds__(512, 2) void gemm_bf16_ksum_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024))) char smem[kGemmSmem];
  gemm_tile<MODE_KSUM, false, false, EPI, NARROW, 256>(p, smem, 0, LaneRows{});
}

// ---------------------------------------------------------------------------
// fp32 kernel: v_mfma_f32_32x32x2_f32
// ---------------------------------------------------------------------------
// Tiles of BM = 32 FM rows x 128 columns, 4 waves side by side along the columns:
// every wave holds all BM rows of its 32 columns (and, DUAL, the same 32 columns
// of W3), so that a ragged tile's dead 32-row blocks are skipped by all four
// alike. 16-deep k-tiles, double-buffered through registers into LDS.
//
// The matrix pipes bound it (64 cycles an instruction, 157 TFLOP/s): an
// instruction needs one A and one B value a lane, so LDS and memory are nearly
// idle. A step of the k order takes k and k + 4 (a lane's half-wave takes k % 8
// in 0..3 or 4..7), so that a K-contiguous operand is read 16 bytes a lane for
// four instructions. One launch of the fused SwiGLU forward replaces two GEMMs
// and an activation pass. Measured against the 64 x 64 FMA tiles it replaced
// (fp32 layer of T = 4096, M = 512, H = 1024, E = 32, k = 2, one launch each):
// forward 291 and 278 -> 126 and 117 us, dgrads 396 and 353 -> 123 and 118, weight
// gradients 207 -> 119: 68-73 TFLOP/s, with the experts' 256 +- 16 rows and the
// last partial round of blocks taking most of the rest.
constexpr int FK = 16;         // k depth of a tile
constexpr int FPK = FK + 4;    // LDS pitch of a K-contiguous row (floats): 16 rows, 16 bank groups
constexpr int FPB = 128 + 8;   // pitch of a k-row of B: rows k and k + 4 on other halves of the banks

typedef float floatx4 __attribute__((ext_vector_type(4)));

template <int MODE, bool B_KC, int EPI, int FM>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmParams p) {
  constexpr bool DUAL = EPI == EPI_SWIGLU_FWD;
  constexpr int NB = DUAL ? 2 : 1;
  constexpr int BM = 32 * FM, BN = 128;
  constexpr bool A_KC = MODE == MODE_ROWS;
  constexpr int FPA = A_KC ? FPK : BM + 8;               // pitch of A's rows / k-rows
  constexpr int ASZ = A_KC ? BM * FPK : FK * FPA;        // floats of an A tile
  constexpr int BSZ = B_KC ? BN * FPK : FK * FPB;
  constexpr int ACH = BM * FK / 4, BCH = BN * FK / 4;    // 16-byte chunks of a tile
  constexpr int AL = (ACH + 255) / 256, BL = BCH / 256;  // chunks a thread
  __shared__ __attribute__((aligned(16))) float smem[2][ASZ + NB * BSZ];
  const int tid = threadIdx.x, lane = tid & 63, h2 = lane >> 5, lr = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  int e = 0, mt = 0, nt = 0, row0 = 0, rows_e = 0, cnt_e = 0;
  const int ntn = (p.N + BN - 1) / BN;
  if constexpr (MODE == MODE_ROWS) {
    // column tiles fastest; lane x holds expert x (as row_tile_of_block)
    const int vb = xcd_remap(blockIdx.x, gridDim.x);
    nt = vb % ntn;
    const int ml = vb / ntn;
    const bool live = lane < p.E;
    const int c = live ? seg_count(p, 0, lane) : 0;
    const int o = live ? seg_offset(p, 0, lane) : 0;
    const int r = live ? (p.padC ? p.padC : c) : 0;
    const int te = (r + BM - 1) / BM;
    const int inc = wave_incl_scan(te);
    const uint64_t hit = __ballot(live && ml < inc && ml >= inc - te);
    if (hit == 0) return;
    e = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(hit));
    mt = ml - (__builtin_amdgcn_readlane(inc, e) - __builtin_amdgcn_readlane(te, e));
    const int off = __builtin_amdgcn_readlane(o, e);
    rows_e = clip_rows(off, __builtin_amdgcn_readlane(r, e), p.rows_cap);
    cnt_e = clip_rows(off, __builtin_amdgcn_readlane(c, e), p.rows_cap);
    row0 = off + mt * BM;
  } else {
    const int mtn = (p.Mdim + BM - 1) / BM;
    const int vb = xcd_remap(blockIdx.x, gridDim.x);
    e = vb / (mtn * ntn);
    const int rem = vb - e * (mtn * ntn);
    mt = rem / ntn;
    nt = rem - mt * ntn;
  }
  const int n0 = nt * BN;
  // live 32-row blocks (weight gradients: of the Mdim rows)
  const int live_rows = MODE == MODE_ROWS ? cnt_e - mt * BM : p.Mdim - mt * BM;
  const int nf = min(FM, (max(0, live_rows) + 31) / 32);

  floatx16 acc[FM][NB];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][b][r] = 0.f;

  const int nseg = MODE == MODE_KSUM ? p.nseg : 1;
  for (int g = 0; g < nseg; ++g) {
    const float* A = static_cast<const float*>(p.A);
    const float* B0 = static_cast<const float*>(p.B0);
    const float* B1 = static_cast<const float*>(p.B1);
    int Kred = p.K;
    if constexpr (MODE == MODE_KSUM) {
      row0 = seg_offset(p, g, e);
      Kred = clip_rows(row0, seg_count(p, g, e), p.rows_cap);
      A += g * p.a_sstride + (long)row0 * p.lda + mt * BM;
      B0 += g * p.b_sstride + (long)row0 * p.ldb + n0;
    } else {
      A += (long)row0 * p.lda;
      B0 += (long)e * p.b_estride + (B_KC ? (long)n0 * p.ldb : n0);
      if (B1 != nullptr) B1 += (long)e * p.b_estride + (B_KC ? (long)n0 * p.ldb : n0);
      if (nf == 0) Kred = 0;  // a padding-only tile: zeros
    }
    const int nk = (Kred + FK - 1) / FK;

    floatx4 ra[AL], rb[NB][BL];
    auto load = [&](int k0) {
#pragma unroll
      for (int u = 0; u < AL; ++u) {
        const int q = tid + 256 * u;
        ra[u] = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (A_KC) {
          const int r = q / (FK / 4), k = k0 + 4 * (q % (FK / 4));
          if (q < ACH && r < live_rows && k < Kred)
            ra[u] = *reinterpret_cast<const floatx4*>(A + (long)r * p.lda + k);
        } else {
          const int k = k0 + q / (BM / 4), m = 4 * (q % (BM / 4));
          if (q < ACH && k < Kred && m < live_rows)
            ra[u] = *reinterpret_cast<const floatx4*>(A + (long)k * p.lda + m);
        }
      }
#pragma unroll
      for (int u = 0; u < BL; ++u) {
        const int q = tid + 256 * u;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          rb[b][u] = floatx4{0.f, 0.f, 0.f, 0.f};
          if constexpr (B_KC) {
            const int n = q / (FK / 4), k = k0 + 4 * (q % (FK / 4));
            if (n0 + n < p.N && k < Kred)
              rb[b][u] = *reinterpret_cast<const floatx4*>(
                  k < p.ksplit ? B0 + (long)n * p.ldb + k : B1 + (long)n * p.ldb + (k - p.ksplit));
          } else {
            const int k = k0 + q / (BN / 4), n = 4 * (q % (BN / 4));
            if (n0 + n < p.N && k < Kred)
              rb[b][u] = *reinterpret_cast<const floatx4*>((DUAL && b ? B1 : B0) + (long)k * p.ldb + n);
          }
        }
      }
    };
    auto store = [&](float* sm) {
#pragma unroll
      for (int u = 0; u < AL; ++u) {
        const int q = tid + 256 * u;
        if (ACH % 256 == 0 || q < ACH)
          *reinterpret_cast<floatx4*>(sm + (A_KC ? (q / (FK / 4)) * FPA + 4 * (q % (FK / 4))
                                                 : (q / (BM / 4)) * FPA + 4 * (q % (BM / 4)))) = ra[u];
      }
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int u = 0; u < BL; ++u) {
          const int q = tid + 256 * u;
          *reinterpret_cast<floatx4*>(sm + ASZ + b * BSZ +
                                      (B_KC ? (q / (FK / 4)) * FPK + 4 * (q % (FK / 4))
                                            : (q / (BN / 4)) * FPB + 4 * (q % (BN / 4)))) = rb[b][u];
        }
    };
    if (nk > 0) {
      load(0);
      if (g > 0) __syncthreads();  // the last segment's reads are done
      store(smem[0]);
      __syncthreads();
    }
    for (int kt = 0; kt < nk; ++kt) {
      if (kt + 1 < nk) load((kt + 1) * FK);
      const float* sa = smem[kt & 1];
      const float* sb = sa + ASZ;
#pragma unroll
      for (int k8 = 0; k8 < FK; k8 += 8) {
        const int kh = k8 + 4 * h2;  // this half-wave's four k
        floatx4 bv[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const float* s = sb + b * BSZ;
          if constexpr (B_KC) {
            bv[b] = *reinterpret_cast<const floatx4*>(s + (w * 32 + lr) * FPK + kh);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) bv[b][q] = s[(kh + q) * FPB + w * 32 + lr];
          }
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          if (i >= nf) break;
          floatx4 av;
          if constexpr (A_KC) {
            av = *reinterpret_cast<const floatx4*>(sa + (i * 32 + lr) * FPA + kh);
          } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) av[q] = sa[(kh + q) * FPA + i * 32 + lr];
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int b = 0; b < NB; ++b)
              acc[i][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[q], bv[b][q], acc[i][b], 0, 0, 0);
        }
      }
      if (kt + 1 < nk) store(smem[(kt + 1) & 1]);
      __syncthreads();
    }
  }

  // ---- epilogue: acc[i][b][r] is row 32 i + 8 (r / 4) + 4 h2 + r % 4, column n0 + 32 w + lr
  float* C0 = static_cast<float*>(p.C0);
  float* C1 = static_cast<float*>(p.C1);
  const float* aux = static_cast<const float*>(p.aux);
  const int n = n0 + w * 32 + lr;
  if (n >= p.N) return;
  float bias0 = 0.f, bias1 = 0.f;
  if constexpr (MODE == MODE_ROWS && (EPI == EPI_STORE || EPI == EPI_GELU_FWD || DUAL)) {
    if (p.bias0 != nullptr) bias0 = p.bias0[(long)e * p.bias_estride + n];
    if (DUAL && p.bias1 != nullptr) bias1 = p.bias1[(long)e * p.bias_estride + n];
  }
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    // a block's loads go out before its stores
    float h1[16], h3[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int ti = 32 * i + 8 * (r >> 2) + 4 * h2 + (r & 3);
      h1[r] = h3[r] = 0.f;
      if constexpr (MODE == MODE_ROWS) {
        if constexpr (EPI == EPI_GELU_BWD || EPI == EPI_SWIGLU_BWD) {
          if (mt * BM + ti < rows_e) {
            const float* a = aux + (long)(row0 + ti) * p.ldaux + n;
            h1[r] = *a;
            if constexpr (EPI == EPI_SWIGLU_BWD) h3[r] = a[p.Hh];
          }
        }
      } else if (p.accumulate) {
        const int m = mt * BM + ti;
        if (m < p.Mdim)
          h1[r] = n < p.nsplit ? C0[(long)e * p.c_estride + (long)m * p.ldc + n]
                               : C1[(long)e * p.c_estride + (long)m * p.ldc + (n - p.nsplit)];
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int ti = 32 * i + 8 * (r >> 2) + 4 * h2 + (r & 3);
      float v = acc[i][0][r];
      if constexpr (MODE == MODE_ROWS) {
        const int li = mt * BM + ti;
        if (li >= rows_e) continue;
        const bool data = li < cnt_e;
        v = data ? v + bias0 : 0.f;
        const long g = row0 + ti;
        if constexpr (EPI == EPI_STORE) {
          C0[g * p.ldc + n] = v;
        } else if constexpr (EPI == EPI_GELU_FWD) {
          C0[g * p.ldc + n] = v;
          C1[g * p.ldc1 + n] = gelu_f(v);
        } else if constexpr (DUAL) {
          const float v3 = data ? acc[i][NB - 1][r] + bias1 : 0.f;
          C0[g * p.ldc + n] = v;
          C0[g * p.ldc + p.Hh + n] = v3;
          C1[g * p.ldc1 + n] = silu_f(v) * v3;
        } else if constexpr (EPI == EPI_GELU_BWD) {
          C0[g * p.ldc + n] = v * gelu_grad_f(h1[r]);
        } else if constexpr (EPI == EPI_SWIGLU_BWD) {
          const float sg = sigmoid_f(h1[r]);
          C0[g * p.ldc + n] = v * h3[r] * sg * (1.f + h1[r] * (1.f - sg));
          C0[g * p.ldc + p.Hh + n] = v * h1[r] * sg;
        }
      } else {
        const int m = mt * BM + ti;
        if (m >= p.Mdim) continue;
        float* dst = (n < p.nsplit) ? C0 + (long)e * p.c_estride + (long)m * p.ldc + n
                                    : C1 + (long)e * p.c_estride + (long)m * p.ldc + (n - p.nsplit);
        *dst = p.accumulate ? h1[r] + v : v;
      }
    }
  }
}

// C (+)= the S partial sums of P (S x n4 float4), added in split order
__global__ __launch_bounds__(256) void sum_splits_kernel(const float4* __restrict__ P, int S,
                                                         long n4, float4* __restrict__ C,
                                                         int accumulate) {
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n4; i += (long)gridDim.x * 256) {
    float4 a = accumulate ? C[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int s = 0; s < S; ++s) {
      const float4 v = P[s * n4 + i];
      a.x += v.x;
      a.y += v.y;
      a.z += v.z;
      a.w += v.w;
    }
    C[i] = a;
  }
}

// Bias gradients of the experts: per-expert column sums,
// out[e][c] (+)= sum over expert e's rows r of src[r][c], over nseg row
// segments (the chunks of a layer call: segment g's rows of expert e are
// counts[g * E + e] rows from offsets[g * (E + 1) + e] of src + g * seg_stride)
// in segment order; columns at or past nsplit go to out1[e][c - nsplit]
// (SwiGLU's dH3 half), a null output is skipped. Memory bounds it (src is read
// once), so the grid is made of narrow blocks: 64 columns of one expert, 8 lanes
// of 8 columns by 32 row lanes, row lane w summing the rows w, w + 32, ... in
// order (four in flight), then the 32 sums added in a fixed order. Blocks of
// 512 columns and 4 row lanes had left most of the CUs idle (8 experts of 750
// rows, 1024 and 5456 columns: 64 -> 32 us for the two; 32 fp32 experts of 256 rows,
// 512 and 1024 columns: 26 -> 18 us).
template <typename TE>
__global__ __launch_bounds__(256) void bias_grad_kernel(
    const TE* __restrict__ src, long ld, long seg_stride, const int32_t* __restrict__ counts,
    const int32_t* __restrict__ offsets, int E, int nseg, long rows_cap, int ncols, int nsplit,
    float* __restrict__ out0, float* __restrict__ out1, int accumulate) {
  constexpr int RL = 32;
  __shared__ float part[RL][64], sum4[4][64];
  const int tid = threadIdx.x, cl = tid & 7, w = tid >> 3;
  const int e = blockIdx.y;
  const int c0 = blockIdx.x * 64 + cl * 8;  // ncols is a multiple of 8
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto add = [&](const auto& raw) {
    float v[8];
    raw8_f32(raw, v);
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] += v[q];
  };
  if (c0 < ncols) {
    for (int g = 0; g < nseg; ++g) {
      const long off = offsets[g * (E + 1) + e];
      const int n = clip_rows(off, counts[g * E + e], rows_cap);
      const TE* base = src + g * seg_stride + off * ld + c0;
      int r = w;
      for (; r + 3 * RL < n; r += 4 * RL) {
        const auto a0 = raw8_load(base + (long)r * ld);
        const auto a1 = raw8_load(base + (long)(r + RL) * ld);
        const auto a2 = raw8_load(base + (long)(r + 2 * RL) * ld);
        const auto a3 = raw8_load(base + (long)(r + 3 * RL) * ld);
        add(a0);
        add(a1);
        add(a2);
        add(a3);
      }
      for (; r < n; r += RL) add(raw8_load(base + (long)r * ld));
    }
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) part[w][cl * 8 + q] = acc[q];
  __syncthreads();
  const int col = tid & 63, g4 = tid >> 6;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < RL / 4; ++i) s += part[g4 * (RL / 4) + i][col];
  sum4[g4][col] = s;
  __syncthreads();
  const int c = blockIdx.x * 64 + col;
  if (tid < 64 && c < ncols) {
    float* dst = c < nsplit ? out0 : out1;
    if (dst == nullptr) return;
    dst += c < nsplit ? (long)e * nsplit + c : (long)e * (ncols - nsplit) + (c - nsplit);
    const float v = ((sum4[0][col] + sum4[1][col]) + sum4[2][col]) + sum4[3][col];
    *dst = accumulate ? *dst + v : v;
  }
}

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------
int rows_tiles_bound(const Shape& s, int bm) {
  if (s.layout == FLOWMOE_PADDED) return s.E * ((s.C + bm - 1) / bm);
  return (int)((s.rows + bm - 1) / bm) + s.E;
}

GemmParams base_params(const Shape& s, const int32_t* counts, const int32_t* offsets) {
  GemmParams p = {};
  p.counts = counts;
  p.offsets = offsets;
  p.E = s.E;
  p.padC = (s.layout == FLOWMOE_PADDED) ? s.C : 0;
  p.ksplit = 1 << 30;
  p.nsplit = 1 << 30;
  p.Hh = s.H;
  p.nseg = 1;
  p.rows_cap = s.rows;
  return p;
}

// Reduction rows of `ld` bf16 that a buffer descriptor's range (2^31 - 1 bytes)
// covers, in whole k-tiles.
int buffer_piece(long ld) { return (int)std::max<long>(WBK, 0x7FFFFFFFL / (2 * ld) / WBK * WBK); }

std::atomic<int> g_tiles{FLOWMOE_TILES_AUTO};
std::atomic<int> g_tile_order{FLOWMOE_TILE_ORDER_AUTO};

template <bool B_KC, int EPI>
hipError_t run_rows(int kind, const Shape& s, GemmParams p, hipStream_t st) {
  constexpr bool DUAL = EPI == EPI_SWIGLU_FWD;
  if (s.rows == 0 || p.N == 0) return hipSuccess;
  p.piece = buffer_piece(p.ldb);
  const bool pieces = !B_KC && p.K > p.piece;
  p.tiles = DUAL ? (g_tiles.load(std::memory_order_relaxed) == FLOWMOE_TILES_AUTO ? FLOWMOE_TILES_AUTO
                                                                                  : FLOWMOE_TILES_WIDE)
                 : g_tiles.load(std::memory_order_relaxed);
  if (pieces) p.tiles = FLOWMOE_TILES_WIDE;
  // the grid covers the wide tiles, or the narrow ones if asked for; the smaller
  // shapes the kernel chooses have at most one round of tiles
  const int ncols = DUAL || p.tiles == FLOWMOE_TILES_NARROW ? 128 : 256;
  const long tiles = (long)rows_tiles_bound(s, 256) * ((p.N + ncols - 1) / ncols);
  const long blocks = row_mode_blocks(std::max(tiles, p.tiles == FLOWMOE_TILES_AUTO ? (long)kCUs : 0L));
  if (p.tiles == FLOWMOE_TILES_AUTO && s.layout == FLOWMOE_PADDED)
    p.tiles = rows_shape(rows_tiles_bound(s, 256), rows_tiles_bound(s, 128), (p.N + 127) / 128, DUAL);
  // joined tile order: the experts' weights stream from HBM (more than the
  // Infinity Cache holds) and each expert spans few row tiles, so a light
  // tile run after all heavy ones would read its weight panels from HBM
  // again; with many row tiles per expert, or weights that stay cached,
  // running the light tiles last packs the rounds better (measured: fine
  // layer 7.63 -> 7.26 ms per step joined, balanced 0.68 -> 0.74 and large
  // 32.2 -> 32.7 ms)
  const double wbytes = 2.0 * s.E * (double)p.K * p.N * (DUAL ? 2 : 1);
  const int order = g_tile_order.load(std::memory_order_relaxed);
  p.joined = order == FLOWMOE_TILE_ORDER_JOINED ||
             (order == FLOWMOE_TILE_ORDER_AUTO && wbytes > 256.0 * 1024 * 1024 &&
              s.rows <= 2048L * s.E);
  if constexpr (DUAL) {
    // Tiles of 128 x (64 + 64) where all of them run at once, by the rows' bound and
    // the experts' capacity (the grid covers the first, whatever the counts are). us
    // of 128 x (128 + 128) and of these, experts x rows, M, H: 8 x 93, 4928, 320 (40
    // tiles) 91 and 44; 1 x 1000, 4096, 1024 (128) 78 and 40; 1 x 64, 4096, 14336
    // (224) 118 and 103; 8 x 128, 4096, 2048 (256) 143 and 114. In two rounds they
    // gain nothing: 16 x 250, 1024, 704 (352) 31.3 and 31.2; 8 x 128, 1024, 2816
    // (352) 39 and 40; 8 x 100, 4096, 3000 (376) 157 and 163; 8 x 128, 4096, 4096
    // (512) 163 and 189.
    const long n64 = (p.N + 63) / 64, bound = rows_tiles_bound(s, 128);
    const long tiles64 = std::min(bound, (long)s.E * ((s.C + 127) / 128)) * n64;
    if (g_tiles.load(std::memory_order_relaxed) == FLOWMOE_TILES_AUTO && !pieces && tiles64 <= kCUs)
      return traced(kind, st, [&] {
        hipLaunchKernelGGL(gemm_bf16_pair64_kernel, dim3((unsigned)row_mode_blocks(bound * n64)), dim3(512), 0,
                           st, p);
      });
  }
  return traced(kind, st, [&] {
    if constexpr (!B_KC)
      if (pieces) {
        hipLaunchKernelGGL(gemm_bf16_rows_pieces_kernel<EPI>, dim3((unsigned)blocks), dim3(512), 0, st, p);
        return;
      }
    hipLaunchKernelGGL((gemm_bf16_rows_kernel<B_KC, EPI>), dim3((unsigned)blocks), dim3(512), 0, st, p);
  });
}

template <int EPI, bool NARROW>
hipError_t launch_ksum(int kind, const Shape& s, GemmParams p, hipStream_t st) {
  constexpr int BN = NARROW ? 128 : 256;
  p.piece = buffer_piece(std::max(p.lda, p.ldb));
  const long blocks = (long)s.E * ((p.Mdim + 255) / 256) * ((p.N + BN - 1) / BN);
  if (blocks == 0) return hipSuccess;
  return traced(kind, st, [&] {
    hipLaunchKernelGGL((gemm_bf16_ksum_kernel<EPI, NARROW>), dim3((unsigned)blocks), dim3(512), 0, st, p);
  });
}

// Weight gradients: 256 x 128 tiles where they run as one round of the CUs, else 256
// x 256 (a round of wide tiles is shorter than two of narrow ones). Measured, wide
// and narrow, experts of 1024 rows: 256 narrow tiles (8 experts of 1024 x 1024) 32.0
// and 28.7 us, 240 (20 of 1024 x 384) 36.4 and 31.8; 288 (4 of 1536 x 1536) 33 and 42,
// 320 (2 of 2560 x 2048) 32 and 42, 336 (3 of 1792 x 2048) 33 and 42. Under the line
// narrow tiles lose where an expert has few of them, each read again by the next (32
// of 512 x 512: 33 and 39 at 1024 rows, equal at 256, 16.5 and 15.0 at 100).
template <int EPI>
hipError_t run_ksum(int kind, const Shape& s, const GemmParams& p, hipStream_t st) {
  if (p.nseg < 1) return hipErrorInvalidValue;  // (a launcher bug)
  const long narrow = (long)s.E * ((p.Mdim + 255) / 256) * ((p.N + 127) / 128);
  const int tiles = g_tiles.load(std::memory_order_relaxed);
  if (tiles == FLOWMOE_TILES_NARROW || (tiles == FLOWMOE_TILES_AUTO && narrow <= kCUs))
    return launch_ksum<EPI, true>(kind, s, p, st);
  return launch_ksum<EPI, false>(kind, s, p, st);
}

template <int MODE, bool B_KC, int EPI, int FM>
hipError_t launch_f32(int kind, const Shape& s, GemmParams p, hipStream_t st) {
  constexpr int BM = 32 * FM;
  const long rt = (MODE == MODE_ROWS) ? rows_tiles_bound(s, BM) : (long)s.E * ((p.Mdim + BM - 1) / BM);
  const long blocks = rt * ((p.N + 127) / 128);
  if (blocks == 0) return hipSuccess;
  return traced(kind, st, [&] {
    hipLaunchKernelGGL((gemm_f32_kernel<MODE, B_KC, EPI, FM>), dim3((unsigned)blocks), dim3(256), 0,
                       st, p);
  });
}

// Rows a tile: 128, or 64 or 32 where taller tiles would be too few to even out
// over the 256 CUs (several blocks share one). Row mode: below 2048 tiles (8192
// rows of 32 experts at N = 512: 32 rows 116 us, 64 rows 146, 128 rows 155; the
// fused SwiGLU forward of 8 experts at N = 2048, K = 1024: 64 rows 645, 128 rows
// 800, its two accumulator sets leaving one wave a SIMD, so 64 rows at most).
// Weight gradients have full tiles only: below 512 (E = 8, 2048 x 1024: 128 rows
// 335 us, 64 rows 396; E = 32, 1024 x 512: 120 and 121).
template <int MODE, bool B_KC, int EPI>
hipError_t run_f32(int kind, const Shape& s, GemmParams p, hipStream_t st) {
  if (MODE == MODE_KSUM && p.nseg < 1) return hipErrorInvalidValue;  // (a launcher bug)
  if (s.rows == 0 && MODE == MODE_ROWS) return hipSuccess;
  const long rows = MODE == MODE_ROWS ? s.rows : (long)s.E * p.Mdim;
  const long nt = (p.N + 127) / 128, least = MODE == MODE_ROWS ? 2048 : 512;
  if constexpr (EPI != EPI_SWIGLU_FWD)
    if ((rows + 127) / 128 * nt >= least) return launch_f32<MODE, B_KC, EPI, 4>(kind, s, p, st);
  if ((rows + 63) / 64 * nt >= least) return launch_f32<MODE, B_KC, EPI, 2>(kind, s, p, st);
  return launch_f32<MODE, B_KC, EPI, 1>(kind, s, p, st);
}

#define FLOWMOE_TRY(x)                 \
  do {                                 \
    hipError_t err_ = (x);             \
    if (err_ != hipSuccess) return err_; \
  } while (0)

}  // namespace

void set_gemm_tiles(int tiles) { g_tiles.store(tiles, std::memory_order_relaxed); }
void set_tile_order(int order) { g_tile_order.store(order, std::memory_order_relaxed); }

hipError_t launch_gate_dw_gemm(const void* x, int T, int M, const void* d, int N,
                               const int32_t* counts, const int32_t* offsets, int S, float* P,
                               hipStream_t st) {
  Shape s2 = {};
  s2.E = S;
  GemmParams p = {};
  p.counts = counts;
  p.offsets = offsets;
  p.E = S;
  p.A = x;
  p.lda = M;
  p.B0 = d;
  p.ldb = N;
  p.Mdim = M;
  p.N = N;
  p.C0 = P;
  p.C1 = P;
  p.ldc = N;
  p.c_estride = (long)M * N;
  p.nsplit = 1 << 30;
  p.ksplit = 1 << 30;
  p.nseg = 1;
  p.rows_cap = T;
  // 256 x 128 tiles whatever the grid: N is at most 128 (the logit gradients' high
  // and low halves), so half of a wide tile would be outside the output (T = 16384,
  // M = 4096: E = 8 38.8 -> 32.8 us, E = 64 50.7 -> 45.6; T = 4096, M = 1024, E = 8 13.8 ->
  // 10.6)
  return launch_ksum<EPI_GATE_DW, true>(FLOWMOE_K_GATE_BWD_DW, s2, p, st);
}

hipError_t launch_gate_dx_gemm(const void* dlhl, int T, int K, const void* wstack, int M,
                               const int32_t* counts, const int32_t* offsets, int S, void* dx,
                               bool add, hipStream_t st) {
  Shape s2 = {};
  s2.T = T;
  s2.E = S;
  s2.rows = T;
  s2.layout = FLOWMOE_PACKED;
  GemmParams p = {};
  p.counts = counts;
  p.offsets = offsets;
  p.E = S;
  p.A = dlhl;
  p.lda = K;
  p.K = K;
  p.B0 = wstack;  // B[k][n] = wstack[k][n] for every token split (b_estride 0)
  p.ldb = M;
  p.N = M;
  p.C0 = dx;
  p.ldc = M;
  p.aux = dx;     // (EPI_ADD: the values added to)
  p.ldaux = M;
  p.ksplit = 1 << 30;
  p.nsplit = 1 << 30;
  p.nseg = 1;
  p.rows_cap = T;
  if (add)
    return run_rows<false, EPI_ADD>(FLOWMOE_K_GATE_BWD_TOKEN, s2, p, st);
  return run_rows<false, EPI_STORE>(FLOWMOE_K_GATE_BWD_TOKEN, s2, p, st);
}

hipError_t launch_dense_gemm(int kind, long rows, const void* A, long lda, int K, const void* B,
                             long ldb, bool b_kc, int N, void* C, long ldc, hipStream_t st) {
  if (rows == 0 || N == 0) return hipSuccess;
  Shape s2 = {};
  s2.T = (int)rows;
  s2.E = 1;
  s2.rows = rows;
  s2.layout = FLOWMOE_PACKED;
  GemmParams p = {};
  p.E = 1;  // (counts null: one expert of rows_cap rows)
  p.A = A;
  p.lda = lda;
  p.K = K;
  p.B0 = B;
  p.ldb = ldb;
  p.N = N;
  p.C0 = C;
  p.ldc = ldc;
  p.ksplit = 1 << 30;
  p.nsplit = 1 << 30;
  p.nseg = 1;
  p.rows_cap = rows;
  if (b_kc) return run_rows<true, EPI_STORE>(kind, s2, p, st);
  return run_rows<false, EPI_STORE>(kind, s2, p, st);
}

int dense_wgrad_splits(int Mdim, int N, long rows) {
  const long tiles = (long)((Mdim + 255) / 256) * ((N + 255) / 256);
  const long s = std::min<long>(8, (kCUs + tiles - 1) / tiles);
  return (int)std::max<long>(1, std::min<long>(s, rows / 512));
}

size_t mha_wgrad_ws_bytes(int M) {
  const long big = 1L << 40;  // (any number of rows)
  const int s3 = dense_wgrad_splits(M, 3 * M, big), s1 = dense_wgrad_splits(M, M, big);
  const size_t b3 = s3 > 1 ? (size_t)s3 * M * 3 * M * 4 : 0, b1 = s1 > 1 ? (size_t)s1 * M * M * 4 : 0;
  return align256(std::max(b3, b1));
}

hipError_t launch_dense_wgrad(int kind, long rows, int nseg, const void* A, long lda,
                              long a_sstride, int Mdim, const void* B, long ldb, long b_sstride,
                              int N, float* C, long ldc, int accumulate, float* part,
                              hipStream_t st) {
  // few output tiles for the CUs: the rows of every segment are split S ways
  // into partial sums in `part` (S x Mdim x N), which a reduction adds in
  // split order (deterministic)
  const int S = part ? dense_wgrad_splits(Mdim, N, rows * nseg) : 1;
  Shape s2 = {};
  s2.T = (int)rows;
  s2.E = S;
  s2.rows = rows;
  s2.layout = FLOWMOE_PACKED;
  GemmParams p = {};
  p.E = S;
  p.A = A;
  p.lda = lda;
  p.Mdim = Mdim;
  p.B0 = B;
  p.ldb = ldb;
  p.N = N;
  p.C0 = S > 1 ? part : C;
  p.C1 = p.C0;
  p.ldc = S > 1 ? N : ldc;
  p.c_estride = (long)Mdim * N;
  p.ksplit = 1 << 30;
  p.nsplit = 1 << 30;
  p.accumulate = S > 1 ? 0 : accumulate;
  p.nseg = nseg;
  p.a_sstride = a_sstride;
  p.b_sstride = b_sstride;
  p.rows_cap = rows;
  FLOWMOE_TRY((run_ksum<EPI_WGRAD>(kind, s2, p, st)));
  if (S == 1) return hipSuccess;
  const long n4 = (long)Mdim * N / 4;  // (ldc == N here)
  return traced(kind, st, [&] {
    hipLaunchKernelGGL(sum_splits_kernel, dim3((unsigned)std::min<long>(2048, (n4 + 255) / 256)),
                       dim3(256), 0, st, reinterpret_cast<const float4*>(part), S, n4,
                       reinterpret_cast<float4*>(C), accumulate);
  });
}

size_t ffn_bwd_ws_bytes(const Shape& s) {
  const int hw = (s.act == FLOWMOE_SWIGLU) ? 2 * s.H : s.H;
  return align256((size_t)s.rows * hw * esize(s.dtype));
}

hipError_t launch_expert_ffn(const Shape& s, const void* x_disp, const int32_t* counts,
                             const int32_t* offsets, const void* w1, const void* w3,
                             const void* w2, const float* b1, const float* b3, const float* b2,
                             void* h_save, void* a_save, void* y_disp, hipStream_t st) {
  if (s.rows == 0) return hipSuccess;
  const bool swiglu = s.act == FLOWMOE_SWIGLU;
  const int H = s.H, M = s.M;
  // layer 1: h = X W1 (and h3 = X W3)
  GemmParams p = base_params(s, counts, offsets);
  p.A = x_disp;
  p.lda = M;
  p.K = M;
  p.N = H;
  p.B0 = w1;
  p.B1 = w3;
  p.ldb = H;
  p.b_estride = (long)M * H;
  p.C0 = h_save;
  p.C1 = a_save;
  p.ldc = swiglu ? 2L * H : H;
  p.ldc1 = H;
  p.bias0 = b1;
  p.bias1 = swiglu ? b3 : nullptr;
  p.bias_estride = H;
  if (s.dtype == FLOWMOE_BF16) {
    if (swiglu)
      FLOWMOE_TRY((run_rows<false, EPI_SWIGLU_FWD>(FLOWMOE_K_FFN1, s, p, st)));
    else
      FLOWMOE_TRY((run_rows<false, EPI_GELU_FWD>(FLOWMOE_K_FFN1, s, p, st)));
  } else {
    if (swiglu) {
      FLOWMOE_TRY((run_f32<MODE_ROWS, false, EPI_SWIGLU_FWD>(FLOWMOE_K_FFN1, s, p, st)));
    } else {
      FLOWMOE_TRY((run_f32<MODE_ROWS, false, EPI_GELU_FWD>(FLOWMOE_K_FFN1, s, p, st)));
    }
  }
  // layer 2: y = a W2
  GemmParams q = base_params(s, counts, offsets);
  q.A = a_save;
  q.lda = H;
  q.K = H;
  q.N = M;
  q.B0 = w2;
  q.ldb = M;
  q.b_estride = (long)H * M;
  q.C0 = y_disp;
  q.ldc = M;
  q.bias0 = b2;
  q.bias_estride = M;
  if (s.dtype == FLOWMOE_BF16)
    return run_rows<false, EPI_STORE>(FLOWMOE_K_FFN2, s, q, st);
  return run_f32<MODE_ROWS, false, EPI_STORE>(FLOWMOE_K_FFN2, s, q, st);
}

hipError_t launch_expert_ffn_dgrad(const Shape& s, const void* dy_disp, const void* h_save,
                                   const int32_t* counts, const int32_t* offsets, const void* w1,
                                   const void* w3, const void* w2, void* dh, void* dx_disp,
                                   hipStream_t st) {
  if (s.rows == 0) return hipSuccess;
  const bool swiglu = s.act == FLOWMOE_SWIGLU;
  const bool bf = s.dtype == FLOWMOE_BF16;
  const int H = s.H, M = s.M;
  const int HW = swiglu ? 2 * H : H;
  // 1. dA = dY W2^T, through the activation -> dH (rows x HW); an element's
  // pre-activation is read by the lane that then writes its gradient, so dh
  // may be h_save itself
  {
    GemmParams p = base_params(s, counts, offsets);
    p.A = dy_disp;
    p.lda = M;
    p.K = M;
    p.N = H;
    p.B0 = w2;  // B[k=m][n=h] = W2[e][h][m]: K-contiguous
    p.ldb = M;
    p.b_estride = (long)H * M;
    p.C0 = dh;
    p.ldc = HW;
    p.aux = h_save;
    p.ldaux = HW;
    if (bf) {
      if (swiglu)
        FLOWMOE_TRY((run_rows<true, EPI_SWIGLU_BWD>(FLOWMOE_K_DGRAD1, s, p, st)));
      else
        FLOWMOE_TRY((run_rows<true, EPI_GELU_BWD>(FLOWMOE_K_DGRAD1, s, p, st)));
    } else {
      if (swiglu)
        FLOWMOE_TRY((run_f32<MODE_ROWS, true, EPI_SWIGLU_BWD>(FLOWMOE_K_DGRAD1, s, p, st)));
      else
        FLOWMOE_TRY((run_f32<MODE_ROWS, true, EPI_GELU_BWD>(FLOWMOE_K_DGRAD1, s, p, st)));
    }
  }
  // 2. dX = dH1 W1^T (+ dH3 W3^T)
  {
    GemmParams p = base_params(s, counts, offsets);
    p.A = dh;
    p.lda = HW;
    p.K = HW;
    p.N = M;
    p.B0 = w1;  // B[k=h][n=m] = W1[e][m][h]: K-contiguous
    p.B1 = swiglu ? w3 : nullptr;
    p.ksplit = swiglu ? H : (1 << 30);
    p.ldb = H;
    p.b_estride = (long)M * H;
    p.C0 = dx_disp;
    p.ldc = M;
    if (bf)
      FLOWMOE_TRY((run_rows<true, EPI_STORE>(FLOWMOE_K_DGRAD2, s, p, st)));
    else
      FLOWMOE_TRY((run_f32<MODE_ROWS, true, EPI_STORE>(FLOWMOE_K_DGRAD2, s, p, st)));
  }
  return hipSuccess;
}

hipError_t launch_expert_bias_grad(const Shape& s, int R, const void* dy_disp, const void* dh,
                                   const int32_t* counts, const int32_t* offsets, float* db1,
                                   float* db3, float* db2, int accumulate, hipStream_t st) {
  const bool swiglu = s.act == FLOWMOE_SWIGLU;
  const int H = s.H, M = s.M, HW = swiglu ? 2 * H : H;
  const long rows = s.rows;
  auto run = [&](const void* src, int ld, int ncols, int nsplit, float* o0, float* o1) {
    return traced(FLOWMOE_K_BIAS_GRAD, st, [&] {
      const dim3 grid((unsigned)((ncols + 63) / 64), (unsigned)s.E);
      if (s.dtype == FLOWMOE_BF16)
        hipLaunchKernelGGL(bias_grad_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)src,
                           (long)ld, rows * ld, counts, offsets, s.E, R, rows, ncols, nsplit, o0, o1,
                           accumulate);
      else
        hipLaunchKernelGGL(bias_grad_kernel<float>, grid, dim3(256), 0, st, (const float*)src,
                           (long)ld, rows * ld, counts, offsets, s.E, R, rows, ncols, nsplit, o0, o1,
                           accumulate);
    });
  };
  if (db2 != nullptr) FLOWMOE_TRY(run(dy_disp, M, M, M, db2, nullptr));
  if (db1 != nullptr || (swiglu && db3 != nullptr))
    FLOWMOE_TRY(run(dh, HW, HW, H, db1, swiglu ? db3 : nullptr));
  return hipSuccess;
}

hipError_t launch_expert_ffn_wgrad(const Shape& s, int R, const void* dy_disp, const void* x_disp,
                                   const void* a_save, const void* dh, const int32_t* counts,
                                   const int32_t* offsets, float* dw1, float* dw3, float* dw2,
                                   float* db1, float* db3, float* db2, int accumulate,
                                   hipStream_t st) {
  const bool swiglu = s.act == FLOWMOE_SWIGLU;
  const bool bf = s.dtype == FLOWMOE_BF16;
  const int H = s.H, M = s.M;
  const int HW = swiglu ? 2 * H : H;
  const long rows = s.rows;
  // 1. dW2 = sum over chunks of A^T dY  (H x M per expert)
  {
    GemmParams p = base_params(s, counts, offsets);
    p.A = a_save;
    p.lda = H;
    p.Mdim = H;
    p.B0 = dy_disp;
    p.ldb = M;
    p.N = M;
    p.C0 = dw2;
    p.ldc = M;
    p.c_estride = (long)H * M;
    p.accumulate = accumulate;
    p.nseg = R;
    p.a_sstride = rows * H;
    p.b_sstride = rows * M;
    if (bf)
      FLOWMOE_TRY((run_ksum<EPI_WGRAD>(FLOWMOE_K_WGRAD2, s, p, st)));
    else
      FLOWMOE_TRY((run_f32<MODE_KSUM, false, EPI_WGRAD>(FLOWMOE_K_WGRAD2, s, p, st)));
  }
  // 2. [dW1 | dW3] = sum over chunks of X^T [dH1 | dH3]  (M x H per expert, each)
  {
    GemmParams p = base_params(s, counts, offsets);
    p.A = x_disp;
    p.lda = M;
    p.Mdim = M;
    p.B0 = dh;
    p.ldb = HW;
    p.N = HW;
    p.C0 = dw1;
    p.C1 = dw3;
    p.nsplit = H;
    p.ldc = H;
    p.c_estride = (long)M * H;
    p.accumulate = accumulate;
    p.nseg = R;
    p.a_sstride = rows * M;
    p.b_sstride = rows * HW;
    if (bf)
      FLOWMOE_TRY((run_ksum<EPI_WGRAD>(FLOWMOE_K_WGRAD1, s, p, st)));
    else
      FLOWMOE_TRY((run_f32<MODE_KSUM, false, EPI_WGRAD>(FLOWMOE_K_WGRAD1, s, p, st)));
  }
  // 3. the biases' gradients: column sums of dY and dH over each expert's rows
  return launch_expert_bias_grad(s, R, dy_disp, dh, counts, offsets, db1, db3, db2, accumulate,
                                 st);
}

hipError_t launch_expert_ffn_bwd(const Shape& s, const void* dy_disp, const void* x_disp,
                                 const void* h_save, const void* a_save, const int32_t* counts,
                                 const int32_t* offsets, const void* w1, const void* w3,
                                 const void* w2, void* dx_disp, float* dw1, float* dw3,
                                 float* dw2, float* db1, float* db3, float* db2, int accumulate,
                                 void* ws, hipStream_t st) {
  // dH in the workspace (h_save is left as it is)
  FLOWMOE_TRY(launch_expert_ffn_dgrad(s, dy_disp, h_save, counts, offsets, w1, w3, w2, ws, dx_disp,
                                      st));
  return launch_expert_ffn_wgrad(s, 1, dy_disp, x_disp, a_save, ws, counts, offsets, dw1, dw3, dw2,
                                 db1, db3, db2, accumulate, st);
}

}  // namespace flowmoe
