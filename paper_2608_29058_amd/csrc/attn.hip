// Causal dense and pattern-sparse attention prefill for gfx950 (bf16 MFMA, fp32 softmax).
//
// Computes, for each unit (query head, rows [s0, s1)), O_i = sum_{j in S_i} softmax(l_i.)_j v_j
// over the kept key set S_i of the unit's pattern (Sec. 2.1: masked logits are minus
// infinity, rows renormalise on their kept set).  The sets are token-exact:
//   dense      S_i = {j <= i}
//   A-shape    S_i = {j <= i : j < sink or j > i - window}
//   block      S_i = {j <= i : j / 64 in Sel(i / 64)}
//   vert-slash S_i = {j in V, j <= i} u {i - t : t in D, t <= i}
//
// Work decomposition: one workgroup = one 128-row query tile of one unit, 4 waves of 32
// rows each; two workgroups share a CU (<= 256 VGPRs, 64 KB LDS each), so one's softmax
// overlaps the other's matrix work.  Dense and vertical-slash items whose launch would leave
// the GPU idle are split along their keys, and a second kernel merges the pieces' partial
// results; fp32 inputs that a call reads often enough are first rounded to bf16 copies when the
// workspace has room for them.
// Keys stream through two LDS buffers in tiles of 64
// (contiguous keys, or gathered vertical columns for vertical-slash): the next tile is
// copied global -> LDS directly (global_load_lds_dwordx4, no registers) while the current
// one is computed, with one barrier per tile.  K and V tiles are row-major with an XOR
// swizzle of the 16-byte chunks.  Per wave and key tile:
//   S^T[64 keys x 32 rows] = K_tile (A operand) x Q^T (B operand, registers)
// with v_mfma_f32_32x32x16_bf16, so each lane holds one query row and 32 of its keys:
// row max / row sum are in-lane plus one exchange with the other lane half.  Then
//   O^T[d x 32 rows] += V^T (A operand, read transposed with ds_read_b64_tr_b16) x P^T
// (B operand: the probabilities straight from the S^T accumulators, packed to bf16).
// Online softmax in the exp2 domain (logit * scale * log2 e), fp32 statistics; the running
// max is raised only when it grows by more than 2^8, so the O rescale is rare.
// Block-sparse: the workgroup's two 64-row query blocks walk the union of their block
// lists from the diagonal block down; each pair of waves computes only the blocks its own
// query block selected.  The two blocks are the same rows of two heads that read one
// key/value head when both heads' units are block-sparse (their selections overlap far more
// than two consecutive blocks of one head do), else consecutive blocks of one head.
// Vertical-slash takes its diagonal-band tiles from the diagonal down as well, then the
// gathered columns.  (Items that start together share their blocks near the diagonal; taken
// first, those are still in L2 when the neighbours reach them.)
#include <algorithm>
#include <cstring>
#include <map>
#include <tuple>
#include <type_traits>
#include <vector>

#include "common.h"

namespace rs {

enum { P_DENSE = 0, P_ASHAPE = 1, P_VS = 2, P_BS = 3 };

struct AttnArgs {
  const void *q, *k, *v;
  long long sq_h, sq_t, sk_h, sk_t, sv_h, sv_t;
  bf16 *o;
  long long so_h, so_t;
  float *lse;
  int n, group;
  float c, scale;
  const DevUnit *units;
  const int *order;   // items; with queues, queue q's at order[qoff[q] .. qoff[q] + qsize[q])
  const int *qsize;   // [4][8] items per family and key/value bucket (device), or NULL: one item per workgroup
  const int *qoff;    // [4][8]
  int *qcount;        // [4][8] items taken per queue (device counters, start at 0)
  const bf16 *vt;  // V^T layout of rs_transpose_v (used by the VT instantiations)
  int npad;
  const int *vs_vsorted, *vs_dsorted, *vs_count;
  const uint32_t *vs_vbits, *vs_dbits;
  int nv_max, ns_max, nwords, ncand_vs;
  const int *bs_sorted, *bs_count;
  int k_max, nb, ncand_bs;
  AttnParts parts;  // partial results of split items (dense and vertical-slash)
};

// A work list in kernel arguments: up to kDirectUnits units with the same rows and item height, sorted by
// key/value bucket, whose items follow from the workgroup's index, so that the launch needs no
// list in memory and no copy of one (4-5 us of the stream and the host's sorting before every
// launch).  nu = 0: items and units come from the lists in AttnArgs.
// Items are dealt to the non-empty buckets in turn, and a bucket that has run out drops out: position
// x of the grid lies in the segment k with pos[k] <= x < pos[k + 1], where na[k] buckets (4-bit
// numbers in act[k]) take turns from their item first[k] on.
constexpr int kDirectUnits = 64;

// Workgroup b runs on XCD b % 8 (round-robin dispatch), so a fixed bucket per XCD gives the query heads
// of one key/value head one L2, but also ties an XCD's work to its bucket's.  Vertical-slash heads
// keep very different numbers of tiles (and block-sparse mates unite to different numbers), so the
// XCD with the heaviest bucket ran alone at the end.  The buckets therefore move on by one XCD after a
// stay of kRotate items per XCD that a bucket has (with na buckets left each has 8 / na): long
// enough for the items that share tiles, short enough for an even mix.  What it gives depends on how
// uneven the heads are.  Attention calls with fixed buckets -> rotation:
//   one key/value head diffuse (vertical, sink or local the others), 32/8 heads: vertical-slash (1000, 512)
//   n = 16384 2.09 -> 1.31 ms, (1000, 6096) n = 32768 8.75 -> 7.13 ms, block-sparse n = 131072 (100 blocks)
//   21.0 -> 15.5 ms; 28/4 heads: 1.75 -> 1.38, 7.29 -> 6.47, 17.9 -> 15.2 ms;
//   even heads, 32/8: 1.07 -> 1.00, 6.73 -> 6.50, 14.2 -> 14.1 ms; 28/4: 0.86 -> 0.86, 5.55 -> 5.47, 13.0 ->
//   13.1 ms; 8/2 heads: 0.30 -> 0.29, 1.52 -> 1.56, 3.44 -> 3.47 ms (within 2% either way over inputs).
// Stays of kRotate items whatever the number of buckets were 2 to 7% slower than fixed buckets for even
// heads at 2 and 4 key/value heads.  At 8, other stays: vertical-slash n = 32768 every item 3.62, 16 items
// 2.65, 64 items 2.77 ms; block-sparse n = 32768 16 items 3.25, 64 items 3.20 ms.  Dense and A-shape
// heads weigh the same.
template <int PAT>
constexpr int kRotate = PAT == P_VS ? 16 : PAT == P_BS ? 64 : 0;

struct AttnDirect {
  AttnArgs a;
  int nu, tiles, nsplit, nseg;
  int bstart[9];  // first unit of each bucket
  int pos[9], first[8], na[8];
  uint32_t act[8];
  DevUnit u[kDirectUnits];
};
static_assert(sizeof(AttnDirect) <= 4096, "kernel arguments");

constexpr int kMaxTiles = kMaxN / 64;  // key tiles of the longest supported sequence
constexpr int kMaxGather = 2048;       // vertical columns gathered per query tile

// XOR swizzle of the 16-byte chunk index of LDS row r.  With d = 128 a 256-byte row spans all
// 64 LDS banks; rows 0-15 then give K fragment reads (16 rows, one chunk column per 16
// lanes) and transposed V reads (4 rows x 4 adjacent chunks per 32 lanes) distinct banks.
// With d = 64 (128-byte rows) a 3-bit swizzle over 8 rows does the same.
template <int D>
__device__ __forceinline__ int swz(int r) {
  if constexpr (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  else return ((r & 3) << 1) | ((r >> 2) & 1);
}

typedef short v4i16 __attribute__((ext_vector_type(4)));

// Barrier after which every wave's direct-to-LDS copies (global_load_lds, counted by
// vmcnt) and LDS accesses are complete.  The explicit vmcnt wait is required: the
// compiler's LDS release fence does not always wait for the LDS DMA.
__device__ __forceinline__ void lds_fence_barrier() {
  // vmcnt(0) through the builtin, which the compiler's wait insertion knows about (it then
  // treats every earlier load as complete, instead of waiting for them again later)
  __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Vertical-slash bitmap words of one wave's rows and one 64-key tile.  A wave's 32 rows start
// at a multiple of 32, as the tile's keys do, so the diagonals i - j of its rows lie in the same
// three words for every lane: d[k] = word wt - 2 + k, wt = (first row - first key) / 32.
struct MaskWords {
  uint32_t d[3];
  uint32_t v[2];  // the tile's column bits
};
typedef uint32_t u32x3_a4 __attribute__((ext_vector_type(3), aligned(4)));
typedef uint32_t u32x2_a4 __attribute__((ext_vector_type(2), aligned(4)));

// Per-tile description produced ahead of its use (the next tile is issued while the
// current one is computed).
struct TileRef {
  int key0;  // first key of a contiguous tile, or -(1 + gather offset)
  int tag;   // bit 0: rows of waves 0-1 use it, bit 1: rows of waves 2-3 (block-sparse)
  int hm;    // 32-key halves of the tile that are copied and may be kept (bit 0: keys 0-31)
  MaskWords mw;  // vertical-slash: the tile's bitmap words (prefetched)
};

// bit 2m of the result: either of bits 2m, 2m + 1 of w (64-key tile m of a word of 32-key halves)
__device__ __forceinline__ uint32_t tile_bits(uint32_t w) { return (w | (w >> 1)) & 0x55555555u; }

// LDS words of a pattern beside its tile buffers: bitmaps, gathered columns, scan.
template <int PAT>
struct AttnLds {
  static constexpr int kX = PAT == P_VS ? kMaxTiles / 16 : PAT == P_BS ? 2 * (kMaxTiles / 32 + 1) : 1;
  static constexpr int kG = PAT == P_VS ? kMaxGather : 1, kScan = PAT == P_VS ? 4 : 1;
};
// The LDS of a kernel.  K and V tiles are double-buffered separately (K runs one tile ahead of V),
// row-major and swizzled.  Distinct arrays, declared by the kernel and seen as such once attn_item is
// inlined, and a parity known at compile time let the compiler see that a copy in flight never
// overlaps the tiles, bitmaps and columns being read.
#define RS_ATTN_LDS(D, NX, NG, NS)                                                              \
  __shared__ __align__(16) bf16 sK0[64 * (D)], sK1[64 * (D)], sV0[64 * (D)], sV1[64 * (D)];     \
  __shared__ uint32_t sX[NX];                                                                   \
  __shared__ int sG[NG], sScan[NS]

// One work item: piece `item >> 12 & 15` of query tile `item & 0xfff` of unit U.
// VT: V is read from the transposed copy (tiles of D rows x 64 keys), else from V itself.
// sK0..sV1: the tile buffers; sX, sG, sScan: the pattern's LDS (AttnLds), all owned by the kernel.
template <int D, int PAT, typename InT, bool VT, bool kLayer, typename Args>
__device__ __forceinline__ void attn_item(const Args &a, const DevUnit U, const int item, bf16 *sK0, bf16 *sK1, bf16 *sV0,
                                          bf16 *sV1, uint32_t *sX, int *sG, int *sScan) {
  constexpr int NW = 4, NT = 256, BM = 128;
  constexpr int KS = D / 16;             // k-steps of the QK^T contraction
  constexpr int DB = D / 32;             // 32-row blocks of O^T
  constexpr int CPR = D / 8;             // 16-byte chunks per K/V row
  constexpr int RPI = 64 / CPR;          // rows covered by one wave-wide 16-byte load
  constexpr int LPT = 64 / RPI / NW;     // loads per thread per K (or V) tile
  constexpr int TE = 64 * D;             // elements of one K or V tile
  static_assert(LPT % 2 == 0 && LPT <= 4 && LPT * NW * RPI == 64, "K/V copies: two halves of LPT / 2 loads");
  // fragment reads in flight ahead of the products (K for QK^T, V for P V).  Vertical-slash
  // keeps two for V (three: the same time within 0.5%); four for K instead of two took the
  // routed 128K layer from 23.1 to 22.5 ms (its launch 7.0 -> 6.4 ms).
  constexpr int KPF = 4;
  constexpr int VPF = PAT == P_VS ? 2 : 3;
  // the products of the tile-skipping families sit under a branch, where the compiler puts
  // each K read right before its product unless the order is forced (scheduling groups)
  constexpr bool kForceOrder = PAT == P_VS || PAT == P_BS;

  // opaque: what the set-up and the epilogue derive from it is computed again for every item
  // instead of being kept in registers across a persistent workgroup's item loop, where
  // vertical-slash (19 spilled registers) ran 9.0 instead of 6.2 ms on a routed 128K layer, and the
  // layer kernel spilled 40 (9 now).  Dense alone has the registers and is 0.5% faster without.
  int tid = threadIdx.x;
  if constexpr (PAT == P_VS || PAT == P_BS || kLayer) asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;

  const int qt = item & 0xfff;
  // pieces along the keys (dense and vertical-slash): this item takes the tiles of piece `piece`
  constexpr bool kSplit = PAT == P_DENSE || PAT == P_VS;
  [[maybe_unused]] const int piece = (item >> 12) & 15;
  [[maybe_unused]] int npiece = kSplit ? U.nsplit : 1;
  // pieces of this item's `nt` tiles: a short list takes fewer, and the workgroups beyond them have
  // nothing to do (false)
  [[maybe_unused]] auto take_piece = [&](int nt) -> bool {
    npiece = min(npiece, max(1, (nt + U.ptiles - 1) / U.ptiles));
    if (piece == 0 && threadIdx.x == 0) a.parts.n[U.pbase + qt * U.nsplit] = npiece;
    return piece < npiece;
  };
  const int head = U.head, s0 = U.s0, s1 = U.s1;
  const int kvh = head / a.group;
  // A block-sparse unit with a mate runs 64-row items: waves 0-1 take its rows of query block
  // qt, waves 2-3 the same rows of the mate head (same key/value head, so the key blocks the
  // two selections share are copied once); otherwise an item is a 128-row query tile.
  const bool paired = PAT == P_BS && U.mate > 0;
  const int IM = paired ? 64 : BM;  // rows of an item
  const int base = (s0 / IM + qt) * IM;
  const int r_lo = max(s0, base), r_hi = min(s1, base + IM);  // valid rows [r_lo, r_hi)
  const int wbase = base + 32 * (paired ? (wave & 1) : wave);
  const int whead = paired && wave >= 2 ? U.mate - 1 : head;  // this wave's query head
  const int w_lo = max(r_lo, wbase), w_hi = min(r_hi, wbase + 32) - 1;
  const bool wave_active = w_lo <= w_hi;
  const int my_row = wbase + l32;
  const int last_tile = (r_hi - 1) >> 6;

  const InT *Qp = (const InT *)a.q + (long long)whead * a.sq_h;
  const InT *Kp = (const InT *)a.k + (long long)kvh * a.sk_h;
  const InT *Vp = (const InT *)a.v + (long long)kvh * a.sv_h;

  // ---- tile enumeration state ----------------------------------------------------------
  int ntiles = 0;
  int st0 = 0, st1 = 0;  // pattern cursors
  [[maybe_unused]] int st_raw = 0;  // vertical-slash: the cursor's bitmap word (both halves of each tile)
  // block-sparse: key blocks selected by query block bq (sBA) and bq + 1 (sBB) as bitmaps;
  // words for key blocks 0 .. bq + 1, where bq + 1 reaches kMaxTiles for the last 64-row item
  // of a sequence of the maximum length
  [[maybe_unused]] uint32_t *sBA = sX, *sBB = sX + kMaxTiles / 32 + 1;
  const uint32_t *vbits = nullptr, *dbits = nullptr;
  int n_contig = 0, n_gather = 0;
  [[maybe_unused]] int g_first = 0, n_gtiles = 0;  // vertical-slash: gathered tiles of this item's piece
  [[maybe_unused]] int t_first = 0;                // dense: first tile of this item's piece
  // vertical-slash: sTB, one bit per 32-key half of the key range the block's diagonals touch
  // (a 64-key tile is in the list when either of its halves is, and only those halves are
  // copied); sG, the gathered vertical columns.
  [[maybe_unused]] uint32_t *sTB = sX;

  if constexpr (PAT == P_VS) {
    const long long vsrow = (long long)U.slot * a.ncand_vs + U.cl;
    const int *vsorted = a.vs_vsorted + vsrow * a.nv_max;
    const int *dsorted = a.vs_dsorted + vsrow * a.ns_max;
    // counts are read within [0, nv_max] / [0, ns_max]: a malformed set never reads past its row
    const int nvc = min(max(a.vs_count[vsrow * 2 + 0], 0), a.nv_max);
    const int ndc = min(max(a.vs_count[vsrow * 2 + 1], 0), a.ns_max);
    vbits = a.vs_vbits + vsrow * a.nwords;
    dbits = a.vs_dbits + vsrow * a.nwords;
    const int nwt = ((2 * last_tile + 1) >> 5) + 1;
    for (int w = tid; w < nwt; w += NT) sTB[w] = 0u;
    __syncthreads();
    // diagonal t covers keys [r_lo - t, r_hi - 1 - t] of this tile's rows
    for (int x = tid; x < ndc; x += NT) {
      const int t = dsorted[x];
      if (t < 0 || t > r_hi - 1) continue;
      const int lo = max(0, r_lo - t) >> 5, hi = (r_hi - 1 - t) >> 5;
      for (int kh = lo; kh <= hi; ++kh) atomicOr(&sTB[kh >> 5], 1u << (kh & 31));
    }
    __syncthreads();
    // tiles per bitmap word, a word per lane (every wave sums the same words, no barrier)
    for (int w0 = 0; w0 < nwt; w0 += 64) {
      int cnt = w0 + lane < nwt ? __builtin_popcount(tile_bits(sTB[w0 + lane])) : 0;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
      n_contig += cnt;
    }
    n_contig = __builtin_amdgcn_readfirstlane(n_contig);
    // vertical columns outside the diagonal tiles are gathered, ascending
    int total = 0;
    for (int x0 = 0; x0 < nvc; x0 += NT) {
      const int x = x0 + tid;
      const int j = (x < nvc) ? vsorted[x] : 0x7fffffff;
      bool f = false;
      if (x < nvc && j >= 0 && j <= r_hi - 1) {
        const int kh = j >> 5;
        f = !((sTB[kh >> 5] >> (kh & 31)) & 1u);
      }
      const uint64_t bal = __ballot(f);
      const int before = __popcll(bal & ((1ull << lane) - 1ull));
      if (lane == 0) sScan[wave] = __popcll(bal);
      __syncthreads();
      int woff = total, blk = 0;
      for (int w = 0; w < NW; ++w) {
        if (w < wave) woff += sScan[w];
        blk += sScan[w];
      }
      if (f && woff + before < kMaxGather) sG[woff + before] = j;
      total += blk;
      __syncthreads();
      if (x0 + NT <= nvc && vsorted[x0 + NT - 1] > r_hi - 1) break;  // sorted: rest is beyond
    }
    n_gather = min(total, kMaxGather);
    __syncthreads();
    // contiguous tiles are taken from the diagonal down (descending keys)
    st0 = nwt - 1;                                                            // bitmap word of the next contiguous tile
    int skip = 0;                                                             // tiles before this item's piece
    if (npiece > 1) {
      // the list (contiguous tiles, then gathered ones) in pieces of equal length
      const int nt = n_contig + ((n_gather + 63) >> 6);
      if (!take_piece(nt)) return;
      const int lo = (int)((long long)nt * piece / npiece), hi = (int)((long long)nt * (piece + 1) / npiece);
      skip = min(lo, n_contig);
      g_first = max(lo - n_contig, 0);
      n_gtiles = max(hi - n_contig, 0) - g_first;
      n_contig = min(hi, n_contig) - skip;
      // cursor to the first tile of the piece: 64 words at a time, tiles above each word by a scan
      int wtop = nwt - 1;
      while (n_contig > 0) {
        const int w = wtop - lane;
        const int cnt = w >= 0 ? __builtin_popcount(tile_bits(sTB[w])) : 0;
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int y = __shfl_up(incl, o);
          if (lane >= o) incl += y;
        }
        const int all = __builtin_amdgcn_readlane(incl, 63);
        if (all > skip) {  // the lane whose word holds tile number `skip`
          const uint64_t m = __ballot(incl > skip);
          const int l = __builtin_ctzll(m);
          st0 = wtop - l;
          skip -= __builtin_amdgcn_readlane(incl - cnt, l);
          break;
        }
        skip -= all;
        wtop -= 64;
      }
    } else {
      n_gtiles = (n_gather + 63) >> 6;
    }
    st_raw = __builtin_amdgcn_readfirstlane((int)sTB[st0]);
    st1 = (int)tile_bits((uint32_t)st_raw);                                   // remaining tiles (even bits)
    if (n_contig > 0)
      for (; skip > 0; --skip) st1 &= ~(1u << (31 - __builtin_clz((uint32_t)st1)));
  } else if constexpr (PAT == P_DENSE) {
    const int nt = last_tile + 1;
    if (npiece > 1 && !take_piece(nt)) return;
    t_first = nt * piece / npiece;
    ntiles = nt * (piece + 1) / npiece - t_first;
  } else if constexpr (PAT == P_ASHAPE) {
    const int ns = min((U.sink + 63) >> 6, last_tile + 1);
    const int wlo = max(0, r_lo - U.window + 1) >> 6;
    st0 = ns;
    st1 = max(wlo, ns);
    ntiles = ns + max(0, last_tile - st1 + 1);
  } else {  // P_BS: query blocks bq = base/64 (waves 0-1) and bq + 1 (waves 2-3), or block bq
    // of this head (waves 0-1) and of the mate head (waves 2-3)
    // the two sorted selections are loaded in parallel into key-block bitmaps; the tiles are
    // their union, walked from the highest key block down (a tile's tag says which selection
    // holds it)
    const int bq = base >> 6;
    const long long brow = ((long long)head * a.ncand_bs + U.cl) * a.nb + bq;
    const long long brow2 = paired ? ((long long)(U.mate - 1) * a.ncand_bs + U.mate_cl) * a.nb + bq : brow + 1;
    // counts within [0, k_max]; entries outside key blocks [0, bq + 1] (pads, malformed sets)
    // are skipped, so the bitmaps are never written out of range
    const int na = r_lo < base + 64 ? min(max(a.bs_count[brow], 0), a.k_max) : 0;
    const int nb2 = (paired || (r_hi > base + 64 && bq + 1 < a.nb)) ? min(max(a.bs_count[brow2], 0), a.k_max) : 0;
    const int nwb = ((bq + 1) >> 5) + 1;  // words holding key blocks 0 .. bq + 1
    for (int w = tid; w < nwb; w += NT) {
      sBA[w] = 0u;
      sBB[w] = 0u;
    }
    __syncthreads();
    for (int x = tid; x < na + nb2; x += NT) {
      const int v = x < na ? a.bs_sorted[brow * a.k_max + x] : a.bs_sorted[brow2 * a.k_max + x - na];
      if (v < 0 || v > bq + 1) continue;
      atomicOr(x < na ? &sBA[v >> 5] : &sBB[v >> 5], 1u << (v & 31));
    }
    __syncthreads();
    int cnt = 0;  // every wave sums the same words (no further barrier)
    for (int w = lane; w < nwb; w += 64) cnt += __builtin_popcount(sBA[w] | sBB[w]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
    ntiles = cnt;
    // the union is walked from the diagonal block down (descending key blocks)
    st0 = nwb - 1;                                                      // bitmap word of the next tile
    st1 = __builtin_amdgcn_readfirstlane((int)(sBA[st0] | sBB[st0]));  // remaining blocks of that word
  }

  // next tile in order (t increases by one per call; g_next counts the gathered tiles, a phase
  // of their own after the contiguous ones)
  int t_next = t_first;
  [[maybe_unused]] int g_next = g_first;
  // zero in a vector register the compiler cannot see through: the mask words are the same for
  // every lane, but a scalar load in flight would turn every LDS wait into a full drain
  [[maybe_unused]] int vzero = 0;
  if constexpr (PAT == P_VS) asm volatile("" : "+v"(vzero));
  auto next_tile = [&](auto gathered) -> TileRef {
    if constexpr (PAT == P_DENSE) {
      return TileRef{(t_next++) * 64, 3, 3, {}};
    } else if constexpr (PAT == P_ASHAPE) {
      const int t = t_next++;
      return TileRef{(t < st0 ? t : st1 + (t - st0)) * 64, 3, 3, {}};
    } else if constexpr (PAT == P_BS) {
      // the words are the same for every lane: kept in scalar registers
      while (st1 == 0) {
        --st0;
        st1 = __builtin_amdgcn_readfirstlane((int)(sBA[st0] | sBB[st0]));
      }
      const int bit = 31 - __builtin_clz((uint32_t)st1);
      st1 &= ~(1u << bit);
      const int wa = __builtin_amdgcn_readfirstlane((int)sBA[st0]), wb = __builtin_amdgcn_readfirstlane((int)sBB[st0]);
      const int tag = ((wa >> bit) & 1) | (((wb >> bit) & 1) << 1);
      return TileRef{(st0 * 32 + bit) * 64, tag, 3, {}};
    } else if constexpr (decltype(gathered)::value) {
      return TileRef{-(1 + 64 * g_next++), 3, 3, {}};
    } else {
      // the bitmap word is the same for every lane: kept in scalar registers
      while (st1 == 0) {
        st_raw = __builtin_amdgcn_readfirstlane((int)sTB[--st0]);
        st1 = (int)tile_bits((uint32_t)st_raw);
      }
      const int bit = 31 - __builtin_clz((uint32_t)st1);
      st1 &= ~(1u << bit);
      const int key0 = (st0 * 16 + (bit >> 1)) * 64;
      TileRef tr{key0, 3, (st_raw >> bit) & 3, {}};
      // bitmap words of the element mask, fetched with the tile so that their latency hides
      // behind the previous tile's compute; words before the bitmap (keys after a row) are 0
      if (wave_active) {
        const int wt = (wbase >> 5) - (key0 >> 5), wv = key0 >> 5;
        if (wt >= 2) {  // every key of the tile lies before the wave's rows, and so inside both bitmaps
          const u32x3_a4 d = *(const u32x3_a4 *)(dbits + (wt - 2) + vzero);
          const u32x2_a4 v = *(const u32x2_a4 *)(vbits + wv + vzero);
          tr.mw = MaskWords{{d[0], d[1], d[2]}, {v[0], v[1]}};
        } else {
#pragma unroll
          for (int k = 0; k < 3; ++k) tr.mw.d[k] = wt - 2 + k >= 0 ? dbits[wt - 2 + k + vzero] : 0u;
#pragma unroll
          for (int k = 0; k < 2; ++k) tr.mw.v[k] = wv + k < a.nwords ? vbits[wv + k + vzero] : 0u;
        }
      }
      return tr;
    }
  };

  // ---- Q fragment in registers (B operand of QK^T) ---------------------------------------
  u32x4 qf[KS];
  {
    const bool ok = wave_active && my_row < a.n;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qf[ks] = u32x4{0u, 0u, 0u, 0u};
      if (ok) qf[ks] = load8<InT>(Qp + (long long)my_row * a.sq_t + 16 * ks + 8 * hh);
    }
  }

  // ---- tile loads: global -> LDS (direct for bf16, through registers for fp32) ----------
  auto key_of_row = [&](auto gathered, int key0, int row) -> int {
    if constexpr (decltype(gathered)::value) {
      const int g = -key0 - 1 + row;
      return sG[g < n_gather ? g : -key0 - 1];
    }
    return min(key0 + row, a.n - 1);
  };
  // bf16 tiles are copied with buffer loads whose per-lane byte offset is the same for every
  // tile (row within the tile and swizzled chunk); the tile's first key enters as a scalar
  // offset.  One head's K (V) rows span less than 4 GiB (checked by the host).
  const int lrow0 = wave * RPI + lane / CPR;          // tile row of load 0; load i adds i*NW*RPI
  const int lchunk = (lane % CPR) ^ swz<D>(lrow0);    // swz sees only row & 15: same for all i
  const uint32_t bK = (uint32_t)(a.sk_t * sizeof(InT)), bV = (uint32_t)(a.sv_t * sizeof(InT));
  [[maybe_unused]] const __amdgpu_buffer_rsrc_t rK = __builtin_amdgcn_make_buffer_rsrc(
      (void *)Kp, (short)0, (int)((uint32_t)(a.n - 1) * bK + D * sizeof(InT)), 0x00020000);
  [[maybe_unused]] const __amdgpu_buffer_rsrc_t rV = __builtin_amdgcn_make_buffer_rsrc(
      (void *)Vp, (short)0, (int)((uint32_t)(a.n - 1) * bV + D * sizeof(InT)), 0x00020000);
  [[maybe_unused]] const uint32_t voK = (uint32_t)lrow0 * bK + 16u * (uint32_t)lchunk;
  [[maybe_unused]] const uint32_t voV = (uint32_t)lrow0 * bV + 16u * (uint32_t)lchunk;
  // V^T tile: D rows (dims) of 64 keys (128 bytes); a wave instruction copies 8 rows, lane l
  // landing at row l / 8, chunk l % 8, which holds global chunk (l % 8) ^ ((row / 2) % 8) (the
  // read-side swizzle).  Rows of load i are 8 (i NW + wave) + l / 8, so the swizzle is the same
  // for every i.
  const uint32_t bVT = (uint32_t)a.npad * 2u;
  [[maybe_unused]] const __amdgpu_buffer_rsrc_t rVT = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(a.vt + (long long)kvh * D * a.npad), (short)0, (int)((uint32_t)D * bVT), 0x00020000);
  [[maybe_unused]] const uint32_t voVT =
      (uint32_t)(8 * wave + lane / 8) * bVT + 16u * (uint32_t)((lane % 8) ^ ((4 * (wave & 1) + (lane >> 4)) & 7));
  // one K or V tile (64 key rows) into dst
  auto issue = [&](auto gathered, bf16 *dst, int key0, bool isV, int hm) {
    constexpr bool kG = decltype(gathered)::value;
    if constexpr (VT) {
      if (isV) {
        constexpr int LPV = D / 8 / NW;  // 8-row groups per wave
        static_assert(LPV == LPT && NW % 2 == 0, "V^T tile: same load count as a row tile");
        bf16 *dw = dst + wave * 8 * 64;
#pragma unroll
        for (int i = 0; i < LPV; ++i)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rVT, (__attribute__((address_space(3))) void *)(dw + i * NW * 8 * 64),
                                                   16, voVT, (uint32_t)key0 * 2u + (uint32_t)(i * NW * 8) * bVT, 0, 0);
        return;
      }
    }
    const InT *src = isV ? Vp : Kp;
    const long long st = isV ? a.sv_t : a.sk_t;
    if constexpr (sizeof(InT) == 2) {
      const __amdgpu_buffer_rsrc_t rs = isV ? rV : rK;
      const uint32_t b = isV ? bV : bK, vo = isV ? voV : voK;
      bf16 *dw = dst + wave * RPI * D;
      // load i copies tile rows [i NW RPI, (i + 1) NW RPI), inside 32-row half (i NW RPI) / 32
      // loads [h LPT / 2, (h + 1) LPT / 2) fill 32-key half h (one test of hm per half)
      if (!kG && key0 + 64 <= a.n) {  // contiguous rows: offsets are scalar
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (!((hm >> h) & 1)) continue;
#pragma unroll
          for (int i = h * LPT / 2; i < (h + 1) * LPT / 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(dw + i * NW * RPI * D),
                                                     16, vo, (uint32_t)(key0 + i * NW * RPI) * b, 0, 0);
        }
      } else {  // gathered rows, or the last tile (rows clamped to the sequence)
        uint32_t jr[4];  // (LPT <= 4) every row index first: one LDS round trip for a gathered tile
#pragma unroll
        for (int i = 0; i < LPT; ++i) jr[i] = (uint32_t)key_of_row(gathered, key0, lrow0 + i * NW * RPI);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (!((hm >> h) & 1)) continue;
#pragma unroll
          for (int i = h * LPT / 2; i < (h + 1) * LPT / 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(dw + i * NW * RPI * D),
                                                     16, jr[i] * b + 16u * (uint32_t)lchunk, 0, 0, 0);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < LPT; ++i) {
        if (!((hm >> ((i * NW * RPI) >> 5)) & 1)) continue;
        const int row_base = (i * NW + wave) * RPI;
        const int row = row_base + lane / CPR;
        const int cc = (lane % CPR) ^ swz<D>(row);
        const int j = key_of_row(gathered, key0, row);
        *(u32x4 *)(dst + row_base * D + 8 * lane) = load8<InT>(src + (long long)j * st + 8 * cc);
      }
    }
  };

  // ---- per-lane LDS fragment offsets -----------------------------------------------------
  const int kswz = swz<D>(l32);                 // K rows 32 mb + l32
  const int g16 = lane >> 4, i16 = lane & 15;
  const int esrc = i16 >> 2, qv = i16 & 3;   // transposed V read: source row / dd quad
  const int vrow = 4 * hh + esrc;            // + 32 mb + 16 s + 8 half
  // swz<D>(vrow + 8 half + 16 s + 32 mb) depends on the half only
  const int vsw0 = swz<D>(vrow), vsw1 = swz<D>(vrow + 8);
  int voff[DB], voff1[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    const int dd0 = 32 * db + 16 * (g16 & 1) + 4 * qv;
    voff[db] = vrow * D + (((dd0 >> 3) ^ vsw0) << 3) + (dd0 & 7);
    voff1[db] = (vrow + 8) * D + (((dd0 >> 3) ^ vsw1) << 3) + (dd0 & 7);
  }

  f32x16 oacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c = a.c;
  const int my_rows_tag = wave < 2 ? 1 : 2;
  const bf16x2 ones = {(bf16)1.f, (bf16)1.f};

  // Dense and A-shape compute every tile of the list for every wave (a tile outside a
  // wave's rows is fully masked), so that the softmax of one tile and the products of the
  // next form one branch-free block the scheduler interleaves.
  constexpr bool kOverlap = PAT == P_DENSE || PAT == P_ASHAPE;

  // ---- per-tile plan of this wave: participation, mask need, active 32-key halves ---------
  struct Plan {
    bool on, need_mask, do0, do1;
    uint32_t m0, m1;  // vertical-slash contiguous tile: this lane's kept keys of each half (after half shift)
    int g0, g_cnt;    // vertical-slash gathered tile: first column slot, column count
  };
  [[maybe_unused]] const uint32_t dsh = 31u - (uint32_t)(my_row & 31);
  auto plan_of = [&](auto gathered, const TileRef &tr, bool valid) -> Plan {
    Plan p{false, true, true, true, 0u, 0u, 0, 0};
    if (!valid) return p;
    const int key0 = tr.key0;
    if constexpr (kOverlap) {
      p.on = true;
      if constexpr (PAT == P_ASHAPE)
        p.need_mask = !(key0 + 63 <= w_lo && (key0 + 63 < U.sink || key0 > w_hi - U.window));
      else
        p.need_mask = key0 + 63 > w_lo;
      return p;
    }
    if (!wave_active || !(tr.tag & my_rows_tag)) return p;
    if constexpr (PAT == P_VS) {
      if constexpr (decltype(gathered)::value) {
        p.g0 = -key0 - 1;
        p.g_cnt = min(64, n_gather - p.g0);
        p.on = sG[p.g0] <= w_hi;
        p.do1 = p.g_cnt > 32;
        // columns are ascending: the last one before every row of the wave, every slot used
        p.need_mask = p.g_cnt < 64 || sG[p.g0 + p.g_cnt - 1] > w_lo;
      } else if (key0 <= w_hi) {
        // the lane's kept keys are known before any product: a 32-key half no row of the
        // wave keeps skips both of its products.  Diagonals i - j: the reversed words, shifted
        // so that bit 0 of the first is diagonal i - key0; keys after the row read zero words.
        const uint32_t r0 = __builtin_bitreverse32(tr.mw.d[2]), r1 = __builtin_bitreverse32(tr.mw.d[1]),
                       r2 = __builtin_bitreverse32(tr.mw.d[0]);
        uint32_t lo = __builtin_amdgcn_alignbit(r1, r0, dsh) | tr.mw.v[0];
        uint32_t hi = __builtin_amdgcn_alignbit(r2, r1, dsh) | tr.mw.v[1];
        if (key0 + 64 > wbase) {  // columns after the row
          const uint64_t pm = prefix_mask(my_row - key0 + 1);
          lo &= (uint32_t)pm;
          hi &= (uint32_t)(pm >> 32);
        }
        if (!(tr.hm & 1)) lo = 0u;  // halves that were not copied (their columns are gathered)
        if (!(tr.hm & 2)) hi = 0u;
        p.m0 = lo >> (4 * hh);
        p.m1 = hi >> (4 * hh);
        p.do0 = __ballot((p.m0 & 0x0f0f0f0fu) != 0u) != 0ull;
        p.do1 = __ballot((p.m1 & 0x0f0f0f0fu) != 0u) != 0ull;
        p.on = p.do0 || p.do1;
      }
    } else {  // block-sparse
      p.on = key0 <= w_hi;
      p.need_mask = key0 + 63 > w_lo;
    }
    return p;
  };

  // ---- S^T[64 keys x 32 rows] = K_tile x Q^T ---------------------------------------------
  auto qk = [&](f32x16 (&s)[2], const bf16 *sKt, const Plan &p) {
    if constexpr (PAT != P_VS) {
      // fragment f: 32-key block mb = f % 2, k-step ks = f / 2 (the two accumulators
      // alternate); reads run KPF fragments ahead of their products
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[mb][r] = 0.f;
      auto kread = [&](int f) -> u32x4 {
        return *(const u32x4 *)&sKt[(32 * (f & 1) + l32) * D + (((2 * (f >> 1) + hh) ^ kswz) << 3)];
      };
      u32x4 kb[KPF];
#pragma unroll
      for (int f = 0; f < KPF; ++f) kb[f] = kread(f);
#pragma unroll
      for (int f = 0; f < 2 * KS; ++f) {
        s[f & 1] = mfma32(kb[f % KPF], qf[f >> 1], s[f & 1]);
        if (f + KPF < 2 * KS) kb[f % KPF] = kread(f + KPF);
      }
      if constexpr (kForceOrder) {
        __builtin_amdgcn_sched_group_barrier(0x100, KPF, 0);
#pragma unroll
        for (int f = 0; f < 2 * KS - KPF; ++f) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, KPF, 0);
      }
      return;
    }
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      const bool dm = mb ? p.do1 : p.do0;
      if (!dm) continue;  // the mask drops every element of the half, whatever it holds
#pragma unroll
      for (int r = 0; r < 16; ++r) s[mb][r] = 0.f;
      auto kread = [&](int ks) -> u32x4 {
        return *(const u32x4 *)&sKt[(32 * mb + l32) * D + (((2 * ks + hh) ^ kswz) << 3)];
      };
      u32x4 kb[KPF];
#pragma unroll
      for (int ks = 0; ks < KPF; ++ks) kb[ks] = kread(ks);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s[mb] = mfma32(kb[ks % KPF], qf[ks], s[mb]);
        if (ks + KPF < KS) kb[ks % KPF] = kread(ks + KPF);
      }
      if constexpr (kForceOrder) {
        __builtin_amdgcn_sched_group_barrier(0x100, KPF, 0);
#pragma unroll
        for (int ks = 0; ks < KS - KPF; ++ks) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, KPF, 0);
      }
    }
  };

  // ---- masks: this lane's keys are bits 0-3 of every byte of M (after the half shift); a
  // kept key keeps its logit, a dropped one (or a skipped half) becomes -inf ---------------
  auto apply_mask = [&](auto gathered, f32x16 (&s)[2], const TileRef &tr, const Plan &p) -> bool {
    const int key0 = tr.key0, i = my_row;
    uint64_t M;
    if constexpr (PAT == P_VS) {
      if constexpr (decltype(gathered)::value) {
        int lo = 0, hi = p.g_cnt;
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (sG[p.g0 + mid] <= i) lo = mid + 1;
          else hi = mid;
        }
        M = prefix_mask(lo) >> (4 * hh);
      } else {
        M = (uint64_t)p.m0 | ((uint64_t)p.m1 << 32);
      }
    } else if constexpr (PAT == P_ASHAPE) {
      const uint64_t keep = prefix_mask(U.sink - key0) | ~prefix_mask(i - U.window + 1 - key0);
      M = (keep & prefix_mask(i - key0 + 1)) >> (4 * hh);
    } else {
      M = prefix_mask(i - key0 + 1) >> (4 * hh);
    }
    const uint32_t Mw[2] = {(uint32_t)M, (uint32_t)(M >> 32)};
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)Mw[mb], 8 * (r >> 2) + (r & 3), 1);
        // the element goes through a scalar: bit_cast of a vector element in place reads
        // element 0 with this compiler
        const float x = s[mb][r];
        s[mb][r] = __builtin_bit_cast(float, (keep & __builtin_bit_cast(uint32_t, x)) | (~keep & 0xff800000u));
      }
    return (M & 0x0F0F0F0F0F0F0F0Full) != 0ull;
  };

  // ---- online softmax in the exp2 domain with a lazily raised running max ------------------
  // P is formed against the current m_run; only if some lane's probability sum exceeds 2^8
  // (so every probability stays <= 2^8 otherwise), or a row sees its first kept key, is the
  // exact tile max taken, m_run raised, O rescaled and P formed again.  Row sums are taken
  // over the bf16-rounded probabilities that also multiply V.
  u32x4 pb[2][2];
  auto form_p = [&](const f32x16 (&s)[2], float nmc) -> float {
    float ps = 0.f;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(s[mb][8 * h + 2 * w], c, nmc));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(s[mb][8 * h + 2 * w + 1], c, nmc));
          const bf16x2 pk = cvt_bf16x2(p0, p1);
          pb[mb][h][w] = __builtin_bit_cast(uint32_t, pk);
          ps = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, ps, false);
        }
    return ps;
  };

  // ---- O^T[d x 32 rows] += V^T x P^T (V read transposed from its row-major tile, or, with
  // VT, 8 consecutive keys of a V^T row per lane: the tile's keys are stored in the order in
  // which the S^T accumulator hands them to P) ----------------------------------------------
  [[maybe_unused]] const int vts = (l32 >> 1) & 7;
  auto pv = [&](const bf16 *sVt, const Plan &p) {
    if constexpr (VT) {
      // fragment f: 16-key group g = f / DB (g = 2 mb + h), 32-dim block db = f % DB, so that
      // consecutive products accumulate into different blocks; reads run PF fragments ahead
      constexpr int NF = 4 * DB, PF = 4;
      auto vread = [&](int f) -> u32x4 {
        const int g = f / DB, db = f % DB;
        return *(const u32x4 *)(sVt + (32 * db + l32) * 64 + (((2 * g + hh) ^ vts) << 3));
      };
      u32x4 vb[PF];
#pragma unroll
      for (int f = 0; f < PF; ++f) vb[f] = vread(f);
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const int g = f / DB, db = f % DB;
        oacc[db] = mfma32(vb[f % PF], pb[g >> 1][g & 1], oacc[db]);
        if (f + PF < NF) vb[f % PF] = vread(f + PF);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, PF, 0);
#pragma unroll
      for (int f = 0; f < NF - PF; ++f) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, PF, 0);
      return;
    }
    // per 32-key half mb (skipped by vertical-slash when no row of the wave keeps a key of
    // it): fragment f = (h, db) = (f / DB, f % DB), consecutive products into different
    // blocks, reads VPF fragments ahead
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      if constexpr (PAT == P_VS)
        if (!(mb ? p.do1 : p.do0)) continue;
      auto vread = [&](int f) -> u32x4 {
        const int h = f / DB, db = f % DB;
        const bf16 *vp = sVt + voff[db] + (32 * mb + 16 * h) * D;
        const bf16 *vq = sVt + voff1[db] + (32 * mb + 16 * h) * D;
        const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16 *)(vp));
        const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16 *)(vq));
        const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
        return u32x4{l2[0], l2[1], h2[0], h2[1]};
      };
      u32x4 vb[VPF];
#pragma unroll
      for (int f = 0; f < VPF; ++f) vb[f] = vread(f);
#pragma unroll
      for (int f = 0; f < 2 * DB; ++f) {
        oacc[f % DB] = mfma32(vb[f % VPF], pb[mb][f / DB], oacc[f % DB]);
        if (f + VPF < 2 * DB) vb[f % VPF] = vread(f + VPF);
      }
      if constexpr (kForceOrder) {  // two transposing reads per fragment
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * VPF, 0);
#pragma unroll
        for (int f = 0; f < 2 * DB - VPF; ++f) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, VPF, 0);
      }
    }
  };

  // ---- one pipeline step: tile t's softmax and P V, tile t+1's products -------------------
  // On entry sc holds S^T of tile t; K of tile t+1 (in kn) and V of tile t (in vc) are resident
  // after the barrier.  The step copies K of tile t+2 into kc (released by tile t's products)
  // and V of tile t+1 into vn (released by tile t-1's P V).
  TileRef Tc{0, 0, 3, {}}, Tn = Tc;
  Plan Pc{}, Pn{};
  auto step = [&](auto gathered, int t, const int nt, f32x16 (&sc)[2], f32x16 (&sn)[2], bf16 *kc, bf16 *kn, bf16 *vc,
                  bf16 *vn) {
    // the next tile is taken after the barrier: the barrier waits for every load in flight,
    // and the vertical-slash mask words that next_tile fetches are only needed a step later
    lds_fence_barrier();
    TileRef T2{0, 0, 3, {}};
    if (t + 2 < nt) T2 = next_tile(gathered);
    if (t + 2 < nt) issue(gathered, kc, T2.key0, false, T2.hm);
    if (t + 1 < nt) issue(gathered, vn, Tn.key0, true, Tn.hm);
    Pn = plan_of(gathered, Tn, t + 1 < nt);
    bool has_key = true;
    if (kOverlap || Pc.on)
      if (Pc.need_mask) has_key = apply_mask(gathered, sc, Tc, Pc);
    if (kOverlap || Pc.on) {
      float psum = form_p(sc, (m_run == -INFINITY) ? 0.f : -m_run * c);
      const uint64_t want = __ballot(!(psum <= 256.f) || (m_run == -INFINITY && has_key));
      if (want != 0ull) {
        float mx = -INFINITY;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[mb][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        // both lanes of a row take the same decision
        if (((want >> l32) | (want >> (l32 + 32))) & 1ull) {
          const float m_new = fmaxf(m_run, mx);
          if (m_new > m_run) {
            const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c);  // 0 for m_run = -inf
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
              for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
            m_run = m_new;
          }
        }
        psum = form_p(sc, (m_run == -INFINITY) ? 0.f : -m_run * c);
      }
      l_run += psum;
      pv(vc, Pc);
    }
    // tile t+1's products come after tile t's P V, not before its softmax: the two S tiles are
    // then never live together, which leaves registers for fragment read-ahead (1-2% for dense
    // and for block-sparse with mates; A-shape 8K 32/8 heads 179 -> 174 us, 64K 1577 -> 1571)
    if (Pn.on) qk(sn, kn, Pn);
    Tc = Tn;
    Tn = T2;
    Pc = Pn;
  };

  // ---- main loop ---------------------------------------------------------------------------
  f32x16 sA[2], sB[2];
  if constexpr (PAT == P_VS) {  // skipped halves are masked without being computed
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sA[mb][r] = sB[mb][r] = 0.f;
  }
  auto run_tiles = [&](auto gathered, const int nt) {
    if (nt <= 0) return;
    Tc = next_tile(gathered);
    issue(gathered, sK0, Tc.key0, false, Tc.hm);
    issue(gathered, sV0, Tc.key0, true, Tc.hm);
    if (nt > 1) {
      Tn = next_tile(gathered);
      issue(gathered, sK1, Tn.key0, false, Tn.hm);
    }
    lds_fence_barrier();
    Pc = plan_of(gathered, Tc, true);
    if (kOverlap || Pc.on) qk(sA, sK0, Pc);
    for (int t = 0; t < nt; t += 2) {
      step(gathered, t, nt, sA, sB, sK0, sK1, sV0, sV1);
      if (t + 1 >= nt) break;
      step(gathered, t + 1, nt, sB, sA, sK1, sK0, sV1, sV0);
    }
  };
  if constexpr (PAT == P_VS) {
    // contiguous tiles, then gathered ones, each with a loop of its own: neither carries the
    // other's addressing or masks
    run_tiles(std::false_type{}, n_contig);
    if (n_contig > 0 && n_gtiles > 0) lds_fence_barrier();  // every wave is done with the tile buffers
    run_tiles(std::true_type{}, n_gtiles);
  } else {
    run_tiles(std::false_type{}, ntiles);
  }

  // ---- epilogue --------------------------------------------------------------------------
  if (!wave_active) return;
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  const int i = my_row;
  if constexpr (kSplit) {
    if (__builtin_expect(npiece > 1, 0)) {
      // this piece's unnormalised O, running max and sum; attn_merge_kernel finishes the rows
      if (i < r_lo || i >= r_hi) return;
      const int slot0 = U.pbase + qt * U.nsplit;
      const long long at = (long long)(slot0 + piece) * BM + (i - base);
      float *po = a.parts.o + at * D;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int ii = 0; ii < 4; ++ii)
          *(f32x4 *)(po + 32 * db + 8 * ii + 4 * hh) =
              f32x4{oacc[db][4 * ii], oacc[db][4 * ii + 1], oacc[db][4 * ii + 2], oacc[db][4 * ii + 3]};
      if (hh == 0) {
        float *pm = a.parts.ml + at * 2;
        pm[0] = m_run;
        pm[1] = l_tot;
      }
      return;
    }
  }
  if (i < r_lo || i >= r_hi) return;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  bf16 *op = a.o + (long long)whead * a.so_h + (long long)i * a.so_t;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) {
      u32x2 w;
      w[0] = pack_bf16x2(oacc[db][4 * ii + 0] * inv, oacc[db][4 * ii + 1] * inv);
      w[1] = pack_bf16x2(oacc[db][4 * ii + 2] * inv, oacc[db][4 * ii + 3] * inv);
      *(u32x2 *)(op + 32 * db + 8 * ii + 4 * hh) = w;
    }
  if (a.lse && hh == 0)
    a.lse[(long long)whead * a.n + i] = l_tot > 0.f ? m_run * a.scale + logf(l_tot) : -INFINITY;
}

// attn_fwd_kernel: one item per workgroup, from the kernel arguments or the list in memory.
template <int D, int PAT, typename InT, bool VT>
__global__ void __launch_bounds__(256, 2) attn_fwd_kernel(const AttnDirect p) {
  RS_ATTN_LDS(D, AttnLds<PAT>::kX, AttnLds<PAT>::kG, AttnLds<PAT>::kScan);
  int item;
  DevUnit U;
  if (p.nu > 0) {
    const int x = (int)blockIdx.x;
    int k = 0;
    while (k + 1 < p.nseg && x >= p.pos[k + 1]) ++k;
    const int rem = x - p.pos[k], turn = rem / p.na[k];
    int j = rem - turn * p.na[k];
    if constexpr (kRotate<PAT> > 0) j = (j + turn / (kRotate<PAT> * 8 / p.na[k])) % p.na[k];
    const int b = __builtin_amdgcn_readfirstlane((int)(p.act[k] >> (4 * j)) & 7);
    const int i = p.first[k] + turn;  // item i of bucket b
    // longest query tiles first, then the bucket's units, then the pieces of an item
    const int u0 = p.bstart[b], per = (p.bstart[b + 1] - u0) * p.nsplit;
    const int q = i / per, r = i - q * per, u = r / p.nsplit;
    item = ((r - u * p.nsplit) << 12) | (p.tiles - 1 - q);
    U = p.u[__builtin_amdgcn_readfirstlane(u0 + u)];
  } else {
    item = p.a.order[blockIdx.x];
    U = p.a.units[item >> 16];
  }
  // (the merge of the two sources counts as varying over the lanes: back to scalar registers)
  item = __builtin_amdgcn_readfirstlane(item);
  int w[sizeof(DevUnit) / 4];
  __builtin_memcpy(w, &U, sizeof(U));
#pragma unroll
  for (size_t k = 0; k < sizeof(DevUnit) / 4; ++k) w[k] = __builtin_amdgcn_readfirstlane(w[k]);
  __builtin_memcpy(&U, w, sizeof(U));
  attn_item<D, PAT, InT, VT, false>(p.a, U, item, sK0, sK1, sV0, sV1, sX, sG, sScan);
}

// The persistent kernels take items from queues: family f's queue of key/value bucket b holds the
// qsize[8 f + b] items at order[qoff[8 f + b]] (longest first) and a counter of items taken,
// which starts at 0 (the planner writes it) and is only ever incremented, so an empty queue stays
// empty and every workgroup reaches the exit.  Workgroup x (on XCD x % 8 under round-robin
// dispatch) takes bucket x % 8 first, then the others.
template <int D, int PAT, typename InT, bool VT, bool kLayer>
__device__ __forceinline__ void drain_family(const AttnArgs &a, int *sItem, bf16 *sK0, bf16 *sK1, bf16 *sV0,
                                             bf16 *sV1, uint32_t *sX, int *sG, int *sScan) {
  constexpr int f = PAT == P_DENSE ? RS_DENSE : PAT == P_ASHAPE ? RS_ASHAPE : PAT == P_VS ? RS_VSLASH : RS_BSPARSE;
  for (;;) {
    __syncthreads();  // the previous item is done with the tile buffers and sItem
    if (threadIdx.x == 0) {
      int got = -1;
      for (int k = 0; k < 8 && got < 0; ++k) {
        const int q = 8 * f + (((int)blockIdx.x + k) & 7), n = a.qsize[q];
        if (__hip_atomic_load(&a.qcount[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= n) continue;
        const int r = atomicAdd(&a.qcount[q], 1);
        if (r < n) got = a.order[a.qoff[q] + r];
      }
      *sItem = got;
    }
    __syncthreads();
    const int it = *sItem;
    if (it < 0) break;
    if constexpr (kLayer) {
      // the arguments are read again for every item through a pointer the compiler cannot see
      // through: kept in scalar registers across four item loops, 99 of them spilled (routed layers
      // 1-1.5% faster this way; a kernel of one family has fewer, and dense alone loses 1-2%)
      typedef const __attribute__((address_space(4))) AttnArgs CArgs;
      CArgs *pa = (CArgs *)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(pa));
      attn_item<D, PAT, InT, VT, true>(*pa, pa->units[it >> 16], it, sK0, sK1, sV0, sV1, sX, sG, sScan);
    } else {
      attn_item<D, PAT, InT, VT, false>(a, a.units[it >> 16], it, sK0, sK1, sV0, sV1, sX, sG, sScan);
    }
  }
}

// One family's items.
template <int D, int PAT, typename InT, bool VT>
__global__ void __launch_bounds__(256, 2) attn_fwd_queue_kernel(const AttnArgs a) {
  RS_ATTN_LDS(D, AttnLds<PAT>::kX, AttnLds<PAT>::kG, AttnLds<PAT>::kScan);
  __shared__ int sItem;
  drain_family<D, PAT, InT, VT, false>(a, &sItem, sK0, sK1, sV0, sV1, sX, sG, sScan);
}

// Every family's items in one launch, dense first (its items are the longest): a family's last items
// run beside the next family's instead of leaving the chip to a launch's tail.  A routed layer of a
// short prompt has few dense fallback items, each a long chain of tiles: 8K tokens 672 -> 602 us,
// 30K 2895 -> 2853 us, 128K 22.84 -> 22.49 ms.
template <int D, typename InT, bool VT>
__global__ void __launch_bounds__(256, 2) attn_fwd_layer_kernel(const AttnArgs a) {
  RS_ATTN_LDS(D, AttnLds<P_BS>::kX > AttnLds<P_VS>::kX ? AttnLds<P_BS>::kX : AttnLds<P_VS>::kX, AttnLds<P_VS>::kG,
              AttnLds<P_VS>::kScan);
  __shared__ int sItem;
  drain_family<D, P_DENSE, InT, VT, true>(a, &sItem, sK0, sK1, sV0, sV1, sX, sG, sScan);
  drain_family<D, P_VS, InT, false, true>(a, &sItem, sK0, sK1, sV0, sV1, sX, sG, sScan);
  drain_family<D, P_BS, InT, VT, true>(a, &sItem, sK0, sK1, sV0, sV1, sX, sG, sScan);
  drain_family<D, P_ASHAPE, InT, VT, true>(a, &sItem, sK0, sK1, sV0, sV1, sX, sG, sScan);
}

// ---- fp32 inputs -----------------------------------------------------------------------------
// The attention kernels copy bf16 tiles straight into LDS; fp32 tiles go through registers, and the
// load, its wait and the rounding then sit in front of every tile step.  Where a call reads its inputs
// often enough, they are rounded once instead, as load8 does it (the results are the same bits): the
// query rows of the heads that the units name, and their key/value heads up to the last key that a
// unit sees.  One 8-element chunk per thread, d / 8 threads per row; grid (row blocks, heads), or one
// row of workgroups that look their head up where the heads' rows are uneven (the search costs 1 us of
// 13 for 48 heads).  Bound by memory: 302 MB read and written in 44 us (6.9 TB/s) for
// 32/8 heads of 8192 tokens, d = 128.
constexpr int kCvtHeads = 192;  // heads of one launch (more: several launches)
struct CvtArray {                  // Q, K or V
  const float *src;
  bf16 *dst;             // of head 0, token 0 (inside the copy for the heads and rows below only)
  long long sh, st, dh;  // element strides: heads and tokens of the input, heads of the copy
};
struct CvtHead {
  int which, row0, rows, start;  // 4 * head + array, its rows, its first workgroup
};
struct CvtArgs {
  CvtArray x[3];
  int d, lgc, nheads, blocks;  // lgc: log2 of 8-element chunks per row
  CvtHead head[kCvtHeads];
};
static_assert(sizeof(CvtArgs) <= 4096, "kernel arguments");
__global__ void __launch_bounds__(256) attn_cvt_kernel(const CvtArgs a) {
  int lo = blockIdx.y, b = blockIdx.x;
  if (gridDim.y == 1) {
    int hi = a.nheads - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (a.head[mid].start <= b) lo = mid;
      else hi = mid - 1;
    }
    b -= a.head[lo].start;
  }
  const CvtHead e = a.head[lo];
  const CvtArray X = a.x[e.which & 3];
  const int h = e.which >> 2, x = b * 256 + (int)threadIdx.x, r = x >> a.lgc, c = x & ((1 << a.lgc) - 1);
  if (r >= e.rows) return;
  const long long row = e.row0 + r;
  *(u32x4 *)(X.dst + h * X.dh + row * a.d + 8 * c) = load8<float>(X.src + h * X.sh + row * X.st + 8 * c);
}

// What a conversion for these units covers.
struct CvtPlan {
  int h0 = 0, h1 = 0, g0 = 0, g1 = 0;  // the copies hold query heads [h0, h1), key/value heads [g0, g1)
  int q0 = 0, q1 = 0, k1 = 0;          // ... rows [q0, q1), keys [0, k1)
  std::vector<int> qa, qb, kb;         // rows [qa, qb) of query head h, keys [0, kb) of key/value head g
  long long read = 0;                  // elements converted, V apart
  long long read_v = 0;
};
static CvtPlan cvt_plan(const rs_qkv *qkv, const rs_unit *units, int32_t nunits) {
  CvtPlan p;
  const int group = qkv->hq / qkv->hkv, n = qkv->n;
  p.qa.assign(qkv->hq, n);
  p.qb.assign(qkv->hq, 0);
  p.kb.assign(qkv->hkv, 0);
  p.h0 = qkv->hq;
  p.g0 = qkv->hkv;
  p.q0 = n;
  for (int i = 0; i < nunits; ++i) {
    const rs_unit &u = units[i];
    if (u.head < 0 || u.head >= qkv->hq || u.s0 < 0 || u.s1 <= u.s0 || u.s1 > n) continue;  // a size query's
    const int g = u.head / group;
    // whole query tiles of 128 rows and key tiles of 64
    p.qa[u.head] = std::min(p.qa[u.head], u.s0 / 128 * 128);
    p.qb[u.head] = std::max(p.qb[u.head], std::min(n, (u.s1 + 127) / 128 * 128));
    p.kb[g] = std::max(p.kb[g], std::min(n, (u.s1 + 63) / 64 * 64));
    p.h0 = std::min(p.h0, u.head);
    p.h1 = std::max(p.h1, u.head + 1);
    p.g0 = std::min(p.g0, g);
    p.g1 = std::max(p.g1, g + 1);
  }
  for (int h = p.h0; h < p.h1; ++h) {
    p.q0 = std::min(p.q0, p.qa[h]);
    p.q1 = std::max(p.q1, p.qb[h]);
    p.read += (long long)std::max(0, p.qb[h] - p.qa[h]) * qkv->d;
  }
  for (int g = p.g0; g < p.g1; ++g) {
    p.k1 = std::max(p.k1, p.kb[g]);
    p.read += (long long)p.kb[g] * qkv->d;
    p.read_v += (long long)p.kb[g] * qkv->d;
  }
  return p;
}

static size_t cvt_plan_bytes(const rs_qkv *qkv, const CvtPlan &p, bool v) {
  if (p.h1 <= p.h0) return 0;
  Arena ar(nullptr, 0);
  ar.take<bf16>((size_t)(p.h1 - p.h0) * (p.q1 - p.q0) * qkv->d);
  ar.take<bf16>((size_t)(p.g1 - p.g0) * p.k1 * qkv->d);
  if (v) ar.take<bf16>((size_t)(p.g1 - p.g0) * p.k1 * qkv->d);
  return ar.off + 256;
}

// Time in us that bf16 copies save a call of these units, on average over the candidates (ncand = 0: the
// most that any candidate can save): what a tile step saves in a chain of them, times the steps of the
// launch's longest item, and with the chip full, times all steps over the 512 workgroups that it holds.
// Both, and the costs below, were fitted to the times of 740 calls with and without the conversion (every
// family, 1 to 64 heads, 300 to 8192 tokens, whole prompts and chunks): over them the rule is 0.2% slower
// than the better choice each time, converting always 3.4% and never 24%.  fp32 tiles at d = 128 cost
// most where their lists are gathered or uneven (vertical-slash).  A vertical-slash list is known on
// the device only: one tile per diagonal is assumed (apart from each other diagonals touch three, side by
// side a 64th).  Examples: one head's first 2048 tokens of 131072, 32/8 heads: 65 us with fp32 tiles, 55 us
// with copies of what it reads (381 us with copies of everything); A-shape, 2048 rows x 32 heads at 64K:
// 76 us with fp32 tiles (chosen), 221 us with copies; dense, 32/8 heads at 8K: 722 and 557 us.
constexpr double kCvtFull[4][2] = {{0.16, 0.37}, {0.26, 0.72}, {0.63, 1.74}, {0.19, 1.10}};   // [family][d = 128]
constexpr double kCvtChain[4][2] = {{0.45, 0.59}, {0.38, 0.59}, {0.45, 1.50}, {0.26, 1.13}};
static double cvt_saves(const rs_qkv *qkv, const rs_unit *units, int32_t nunits, const rs_candidate *grid,
                        int32_t ncand) {
  double sum = 0.0;
  for (int c = 0; c < std::max(ncand, 1); ++c) {
    const int fam = ncand > 0 ? grid[c].fam : RS_VSLASH, a = ncand > 0 ? grid[c].a : 0, b = ncand > 0 ? grid[c].b : 0;
    double all = 0.0, longest = 0.0;  // tile steps
    for (int i = 0; i < nunits; ++i) {
      const rs_unit &u = units[i];
      if (u.head < 0 || u.head >= qkv->hq || u.s0 < 0 || u.s1 <= u.s0 || u.s1 > qkv->n) continue;
      const double full = (u.s1 + 63) / 64, mean = (u.s0 / 64 + full + 1) / 2;  // key tiles before the last row; on average
      double most = full;
      SplitRule sp{1, 1};
      if (ncand > 0) {
        if (fam == RS_ASHAPE) most = std::min(full, (a + 63) / 64 + (b + 63) / 64 + 2.0);
        if (fam == RS_VSLASH) most = std::min(full, a / 64 + b + 2.0);
        if (fam == RS_BSPARSE) most = std::min(full, 1.5 * a);  // of two query blocks
        sp = attn_split(qkv->hq, qkv->d, qkv->n, u.s0, u.s1, fam);
      }
      all += std::min(mean, most) * ((u.s1 - 1) / 128 - u.s0 / 128 + 1);
      longest = std::max(longest, most / std::max(1, std::min(sp.nsplit, (int)most / sp.ptiles)));
    }
    const double us = kCvtFull[fam][qkv->d == 128] * all / 512 + kCvtChain[fam][qkv->d == 128] * longest;
    // with V^T only K goes through registers (dense, 32/8 heads at 8K: 100 us saved instead of 170)
    sum += ncand > 0 && qkv->vt && fam != RS_VSLASH ? 0.6 * us : us;
  }
  return sum / std::max(ncand, 1);
}

// ... and what the conversion takes: its launch, and 6 bytes an element at 8.1 TB/s.
static double cvt_costs(const CvtPlan &p, bool v) { return 3.4 + (p.read + (v ? p.read_v : 0)) * 6.0 / 8.1e6; }

size_t attn_cvt_bytes(const rs_qkv *qkv, const rs_unit *units, int32_t nunits) {
  if (!qkv || qkv->dtype != RS_F32 || nunits <= 0 || qkv->hkv < 1 || qkv->hq < qkv->hkv || qkv->n < 1) return 0;
  const CvtPlan p = cvt_plan(qkv, units, nunits);
  return cvt_saves(qkv, units, nunits, nullptr, 0) > cvt_costs(p, !qkv->vt) ? cvt_plan_bytes(qkv, p, true) : 0;
}

rs_status attn_cvt_launch(const rs_qkv *qkv, const rs_unit *units, int32_t nunits, const rs_candidate *grid,
                          int32_t ncand, void *ws, size_t room, rs_qkv *out, hipStream_t st) {
  *out = *qkv;
  if (qkv->dtype != RS_F32 || !ws || ((uintptr_t)ws & 15)) return RS_OK;
  bool v = !qkv->vt;  // vertical-slash items gather rows of V itself
  for (int c = 0; c < ncand; ++c) v = v || grid[c].fam == RS_VSLASH;
  const CvtPlan p = cvt_plan(qkv, units, nunits);
  if (cvt_plan_bytes(qkv, p, v) > room || cvt_saves(qkv, units, nunits, grid, ncand) <= cvt_costs(p, v)) return RS_OK;
  const int d = qkv->d;
  const long long rows = p.q1 - p.q0;
  Arena ar(ws, room);
  bf16 *q = ar.take<bf16>((size_t)(p.h1 - p.h0) * rows * d);
  bf16 *k = ar.take<bf16>((size_t)(p.g1 - p.g0) * p.k1 * d);
  bf16 *vv = v ? ar.take<bf16>((size_t)(p.g1 - p.g0) * p.k1 * d) : k;  // else V is not read
  const long long dq = rows * d, dk = (long long)p.k1 * d;
  CvtArgs a;
  a.x[0] = CvtArray{(const float *)qkv->q, q - p.h0 * dq - (long long)p.q0 * d, qkv->sq_h, qkv->sq_t, dq};
  a.x[1] = CvtArray{(const float *)qkv->k, k - p.g0 * dk, qkv->sk_h, qkv->sk_t, dk};
  a.x[2] = CvtArray{(const float *)qkv->v, vv - p.g0 * dk, qkv->sv_h, qkv->sv_t, dk};
  a.d = d;
  a.lgc = d == 128 ? 4 : 3;
  a.nheads = a.blocks = 0;
  const int rpw = 256 >> a.lgc;  // rows of a workgroup
  int per = 0;                   // workgroups of the longest head
  auto flush = [&]() -> rs_status {
    if (a.nheads == 0) return RS_OK;
    const bool even = (long long)per * a.nheads * 4 <= (long long)a.blocks * 5;
    hipLaunchKernelGGL(attn_cvt_kernel, even ? dim3(per, a.nheads) : dim3(a.blocks), dim3(256), 0, st, a);
    RS_HIP(hipGetLastError());
    a.nheads = a.blocks = per = 0;
    return RS_OK;
  };
  auto add = [&](int head, int which, int row0, int n) -> rs_status {
    if (n <= 0) return RS_OK;
    a.head[a.nheads++] = CvtHead{4 * head + which, row0, n, a.blocks};
    a.blocks += (n + rpw - 1) / rpw;
    per = std::max(per, (n + rpw - 1) / rpw);
    return a.nheads == kCvtHeads ? flush() : RS_OK;
  };
  rs_status s = RS_OK;
  for (int h = p.h0; h < p.h1 && s == RS_OK; ++h) s = add(h, 0, p.qa[h], p.qb[h] - p.qa[h]);
  for (int w = 1; w <= (v ? 2 : 1); ++w)
    for (int g = p.g0; g < p.g1 && s == RS_OK; ++g) s = add(g, w, 0, p.kb[g]);
  if (s == RS_OK) s = flush();
  if (s != RS_OK) return s;
  out->dtype = RS_BF16;
  out->q = a.x[0].dst;
  out->k = a.x[1].dst;
  out->v = a.x[2].dst;
  out->sq_h = dq;
  out->sk_h = out->sv_h = dk;
  out->sq_t = out->sk_t = out->sv_t = d;
  return RS_OK;
}

// ---- merge of split items ------------------------------------------------------------------
// grid (items, 8), 256 threads: 16 rows of an item per workgroup, 16 threads per row.  Piece p of
// a row holds O_p relative to its own running max m_p: with M the largest and w_p = exp(m_p - M),
// O = sum w_p O_p / sum w_p l_p, in piece order (a fixed order: the result is deterministic).  A
// piece that kept no key of the row has l_p = 0 and m_p = -inf.  Bound by reading the pieces.
// Its units in kernel arguments, as AttnDirect holds them (tiles = 0: units and items in memory).
struct MergeDirect {
  int tiles, nsplit, s0, s1;
  int head[kDirectUnits];
};
template <int D>
__global__ void __launch_bounds__(256) attn_merge_kernel(const DevUnit *units, const AttnParts parts,
                                                         const MergeDirect m, bf16 *o, long long so_h, long long so_t,
                                                         float *lse, int n, float c, float scale) {
  constexpr int EPT = D / 16, BM = 128;  // elements per thread, rows of an item
  int slot0, qt, head, s0, s1;
  if (m.tiles > 0) {
    const int u = (int)blockIdx.x / m.tiles;
    qt = (int)blockIdx.x - u * m.tiles;
    slot0 = (int)blockIdx.x * m.nsplit;
    head = m.head[u];
    s0 = m.s0;
    s1 = m.s1;
  } else {
    const int item = parts.items[blockIdx.x];
    if (item < 0) return;
    const DevUnit U = units[item >> 16];
    qt = item & 0xfff;
    slot0 = U.pbase + qt * U.nsplit;
    head = U.head;
    s0 = U.s0;
    s1 = U.s1;
  }
  const int np = parts.n[slot0];
  if (np <= 1) return;  // the item's one workgroup wrote the rows itself
  const int base = (s0 / BM + qt) * BM;
  const int r = blockIdx.y * 16 + (threadIdx.x >> 4), i = base + r, x = threadIdx.x & 15;
  if (i < s0 || i >= s1) return;
  const float *ml = parts.ml + ((long long)slot0 * BM + r) * 2;
  float M = -INFINITY;
  for (int p = 0; p < np; ++p) M = fmaxf(M, ml[(long long)p * BM * 2]);
  float acc[EPT], L = 0.f;
#pragma unroll
  for (int e = 0; e < EPT; ++e) acc[e] = 0.f;
  const float *po = parts.o + ((long long)slot0 * BM + r) * D + EPT * x;
  for (int p = 0; p < np; ++p) {
    const float l = ml[(long long)p * BM * 2 + 1];
    const float w = l > 0.f ? __builtin_amdgcn_exp2f((ml[(long long)p * BM * 2] - M) * c) : 0.f;
    L += w * l;
#pragma unroll
    for (int e = 0; e < EPT; e += 4) {
      const f32x4 v = *(const f32x4 *)(po + (long long)p * BM * D + e);
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[e + k] += w * v[k];
    }
  }
  const float inv = L > 0.f ? 1.f / L : 0.f;
  bf16 *op = o + (long long)head * so_h + (long long)i * so_t + EPT * x;
#pragma unroll
  for (int e = 0; e < EPT; e += 4)
    *(u32x2 *)(op + e) = u32x2{pack_bf16x2(acc[e] * inv, acc[e + 1] * inv), pack_bf16x2(acc[e + 2] * inv, acc[e + 3] * inv)};
  if (lse && x == 0) lse[(long long)head * n + i] = L > 0.f ? M * scale + logf(L) : -INFINITY;
}

size_t attn_parts_bytes(int d, size_t slots) {
  if (slots == 0) return 0;
  Arena ar(nullptr, 0);
  ar.take<float>(slots * 128 * d);
  ar.take<float>(slots * 128 * 2);
  ar.take<int>(slots);
  ar.take<int>(slots);
  return ar.off + 256;
}

AttnParts attn_parts_at(void *p, int d, size_t slots) {
  Arena ar(p, ~size_t(0));
  AttnParts a;
  a.o = ar.take<float>(slots * 128 * d);
  a.ml = ar.take<float>(slots * 128 * 2);
  a.n = ar.take<int>(slots);
  a.items = ar.take<int>(slots);
  return a;
}

static rs_status merge_launch(const rs_qkv *qkv, float scale, const DevUnit *d_units, const AttnParts &parts,
                              const MergeDirect &m, int blocks, void *o, int64_t so_h, int64_t so_t, float *lse,
                              hipStream_t st) {
  const dim3 grid(blocks, 8);
  if (qkv->d == 128)
    hipLaunchKernelGGL(attn_merge_kernel<128>, grid, dim3(256), 0, st, d_units, parts, m, (bf16 *)o, (long long)so_h,
                       (long long)so_t, lse, qkv->n, scale * kLog2e, scale);
  else
    hipLaunchKernelGGL(attn_merge_kernel<64>, grid, dim3(256), 0, st, d_units, parts, m, (bf16 *)o, (long long)so_h,
                       (long long)so_t, lse, qkv->n, scale * kLog2e, scale);
  RS_HIP(hipGetLastError());
  return RS_OK;
}

rs_status attn_merge_launch(const rs_qkv *qkv, float scale, const DevUnit *d_units, const AttnParts &parts,
                            int nitems, void *o, int64_t so_h, int64_t so_t, float *lse, hipStream_t st) {
  return merge_launch(qkv, scale, d_units, parts, MergeDirect{}, nitems, o, so_h, so_t, lse, st);
}

// ---- V^T: [hkv][d][npad] bf16, keys permuted within groups of 16 ---------------------------
// Position j of a 16-key group holds key perm[j]: in the P V product a lane of half hh supplies
// the keys {4 hh .. 4 hh + 3, 8 + 4 hh .. 8 + 4 hh + 3} of each group of 16 (the order in which
// the S^T accumulator hands them to P), which are then 8 consecutive positions.
__device__ __forceinline__ int vt_perm(int j) { return (j & 3) | ((j & 4) << 1) | ((j & 8) >> 1); }

// grid (npad / 64, hkv), 256 threads: 64 keys of one key/value head through LDS
template <int D, typename InT>
__global__ void __launch_bounds__(256) transpose_v_kernel(const InT *v, long long sv_h, long long sv_t, int n,
                                                          int npad, bf16 *vt) {
  constexpr int LD = D + 8;
  __shared__ __align__(16) bf16 sT[64][LD];
  const int k0 = blockIdx.x * 64, g = blockIdx.y, tid = threadIdx.x;
  const InT *vp = v + (long long)g * sv_h;
  // 64 rows x D, 8 elements per 16-byte chunk of the bf16 tile
  for (int x = tid; x < 64 * (D / 8); x += 256) {
    const int r = x / (D / 8), c = x % (D / 8), key = k0 + r;
    u32x4 w = {0u, 0u, 0u, 0u};
    if (key < n) w = load8<InT>(vp + (long long)key * sv_t + 8 * c);
    *(u32x4 *)&sT[r][8 * c] = w;
  }
  __syncthreads();
  bf16 *out = vt + (long long)g * D * npad + k0;
  for (int x = tid; x < D * 8; x += 256) {
    const int dd = x / 8, c = x % 8;  // row dd of V^T, positions 8c .. 8c + 7 of the 64 keys
    bf16 e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int p = 8 * c + j;
      e[j] = sT[(p & ~15) + vt_perm(p & 15)][dd];
    }
    *(u32x4 *)(out + (long long)dd * npad + 8 * c) = __builtin_bit_cast(u32x4, e);
  }
}

size_t vt_bytes(const rs_qkv *qkv) {
  const long long npad = ((long long)qkv->n + 63) / 64 * 64;
  return (size_t)qkv->hkv * qkv->d * npad * sizeof(bf16);
}

rs_status transpose_v_launch(const rs_qkv *qkv, void *vt, hipStream_t st) {
  const int npad = (qkv->n + 63) / 64 * 64;
  const dim3 grid(npad / 64, qkv->hkv);
  if (qkv->d == 128) {
    if (qkv->dtype == RS_BF16)
      hipLaunchKernelGGL((transpose_v_kernel<128, bf16>), grid, dim3(256), 0, st, (const bf16 *)qkv->v,
                         (long long)qkv->sv_h, (long long)qkv->sv_t, qkv->n, npad, (bf16 *)vt);
    else
      hipLaunchKernelGGL((transpose_v_kernel<128, float>), grid, dim3(256), 0, st, (const float *)qkv->v,
                         (long long)qkv->sv_h, (long long)qkv->sv_t, qkv->n, npad, (bf16 *)vt);
  } else {
    if (qkv->dtype == RS_BF16)
      hipLaunchKernelGGL((transpose_v_kernel<64, bf16>), grid, dim3(256), 0, st, (const bf16 *)qkv->v,
                         (long long)qkv->sv_h, (long long)qkv->sv_t, qkv->n, npad, (bf16 *)vt);
    else
      hipLaunchKernelGGL((transpose_v_kernel<64, float>), grid, dim3(256), 0, st, (const float *)qkv->v,
                         (long long)qkv->sv_h, (long long)qkv->sv_t, qkv->n, npad, (bf16 *)vt);
  }
  RS_HIP(hipGetLastError());
  return RS_OK;
}

// ---- host side ---------------------------------------------------------------------------

static int family_bm(int) { return 128; }

static int tiles_of(const rs_unit &u, int bm) { return (u.s1 - 1) / bm - u.s0 / bm + 1; }

// Bytes of a launch's work list, without partial results: [DevUnit x nunits][items]
// (a unit with a mate has at most twice its 128-row tiles in 64-row blocks, and its mate none)
static size_t attn_list_bytes(int32_t nunits, size_t items) {
  Arena ar(nullptr, 0);
  ar.take<DevUnit>((size_t)nunits);
  ar.take<int>(items);
  return ar.off + 256;  // (rounded down to 256 bytes: at or past the list's end)
}

size_t attn_ws_bytes(const rs_qkv *qkv, const rs_unit *units, int32_t nunits) {
  size_t items = 0, slots = 0;
  for (int i = 0; i < nunits; ++i) {
    const rs_unit &u = units[i];
    const int s = qkv && u.s0 >= 0 && u.s1 > u.s0 && qkv->hq > 0 ? attn_split_slots(qkv->hq, qkv->d, qkv->n, u.s0, u.s1) : 0;
    items += std::max<size_t>((size_t)tiles_of(u, 128), (size_t)s);
    slots += (size_t)s;
  }
  return attn_list_bytes(nunits, items) + attn_parts_bytes(qkv ? qkv->d : 0, slots) +
         attn_cvt_bytes(qkv, units, nunits);
}

// Block-sparse mates: a unit of an even head takes along the unit of the next head with the
// same rows when both heads read the same key/value head (their items then run the two
// heads' selections of one 64-row query block side by side).  mate[u]: the unit taken along
// by u, -2 for a unit taken along, -1 otherwise.
static void pair_units(const rs_unit *units, int nunits, int group, std::vector<int> &mate) {
  mate.assign(nunits, -1);
  std::map<std::tuple<int, int, int>, int> at;  // (head, s0, s1) -> first unit
  for (int u = 0; u < nunits; ++u) at.emplace(std::make_tuple(units[u].head, units[u].s0, units[u].s1), u);
  for (int u = 0; u < nunits; ++u) {
    const int h = units[u].head;
    if ((h & 1) || mate[u] != -1 || (h + 1) / group != h / group) continue;
    const auto it = at.find(std::make_tuple(h + 1, units[u].s0, units[u].s1));
    if (it == at.end() || mate[it->second] != -1) continue;
    mate[u] = it->second;
    mate[it->second] = -2;
  }
}

// Build the dispatch order: items bucketed by key/value head (round-robin workgroup
// dispatch places workgroup b on XCD b % 8, so the query heads sharing one K/V stream
// share one XCD's L2), longest query tiles first within a bucket.  Items of a unit with a
// mate are 64-row query blocks, others bm-row query tiles (bm = 128); units taken along by a
// mate have none.  Pieces of a split item follow one another.  rotate: kRotate of the pattern, applied
// as attn_fwd_kernel does.
static void build_order(const rs_unit *units, int nunits, int group, int bm, int rotate, const std::vector<int> &mate,
                        const std::vector<SplitRule> &split, std::vector<int> &order) {
  std::vector<std::vector<std::pair<int, int>>> buckets(8);  // (-first row / 64, item)
  for (int u = 0; u < nunits; ++u) {
    if (mate[u] == -2) continue;
    const int im = mate[u] >= 0 ? 64 : bm;
    const int t0 = units[u].s0 / im, nt = tiles_of(units[u], im);
    const int b = (units[u].head / group) & 7;
    for (int t = 0; t < nt; ++t)
      for (int p = 0; p < split[u].nsplit; ++p)
        buckets[b].push_back({-((t0 + t) * (im / 64)), (u << 16) | (p << 12) | t});
  }
  size_t mx = 0;
  for (auto &b : buckets) {
    std::stable_sort(b.begin(), b.end(),
                     [](const std::pair<int, int> &x, const std::pair<int, int> &y) { return x.first < y.first; });
    mx = std::max(mx, b.size());
  }
  order.clear();
  size_t first = 0;  // item from which the buckets now left take turns
  int left = 0;
  for (size_t i = 0; i < mx; ++i) {
    int act[8], na = 0;
    for (int b = 0; b < 8; ++b)
      if (i < buckets[b].size()) act[na++] = b;
    if (na != left) {
      left = na;
      first = i;
    }
    for (int j = 0; j < na; ++j) order.push_back(buckets[act[(j + (rotate ? (i - first) / (rotate * 8 / na) : 0)) % na]][i].second);
  }
}

template <int D, int PAT, typename InT, bool VT>
static void launch_one(const AttnDirect &p, int nblocks, hipStream_t st) {
  if (p.a.qsize)
    hipLaunchKernelGGL((attn_fwd_queue_kernel<D, PAT, InT, VT>), dim3(nblocks), dim3(256), 0, st, p.a);
  else
    hipLaunchKernelGGL((attn_fwd_kernel<D, PAT, InT, VT>), dim3(nblocks), dim3(256), 0, st, p);
}

template <int D, int PAT>
static hipError_t launch_pat(int dtype, const AttnDirect &p, int nblocks, hipStream_t st) {
  if constexpr (PAT != P_VS) {  // vertical-slash gathers V rows: it keeps the row-major V
    if (p.a.vt) {
      if (dtype == RS_BF16) launch_one<D, PAT, bf16, true>(p, nblocks, st);
      else launch_one<D, PAT, float, true>(p, nblocks, st);
      return hipGetLastError();
    }
  }
  if (dtype == RS_BF16) launch_one<D, PAT, bf16, false>(p, nblocks, st);
  else launch_one<D, PAT, float, false>(p, nblocks, st);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_layer(int dtype, const AttnArgs &a, int nblocks, hipStream_t st) {
  if (a.vt) {
    if (dtype == RS_BF16)
      hipLaunchKernelGGL((attn_fwd_layer_kernel<D, bf16, true>), dim3(nblocks), dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL((attn_fwd_layer_kernel<D, float, true>), dim3(nblocks), dim3(256), 0, st, a);
  } else {
    if (dtype == RS_BF16)
      hipLaunchKernelGGL((attn_fwd_layer_kernel<D, bf16, false>), dim3(nblocks), dim3(256), 0, st, a);
    else
      hipLaunchKernelGGL((attn_fwd_layer_kernel<D, float, false>), dim3(nblocks), dim3(256), 0, st, a);
  }
  return hipGetLastError();
}

template <int D>
static hipError_t launch_d(int fam, int dtype, const AttnDirect &p, int nblocks, hipStream_t st) {
  switch (fam) {
    case RS_DENSE: return launch_pat<D, P_DENSE>(dtype, p, nblocks, st);
    case RS_ASHAPE: return launch_pat<D, P_ASHAPE>(dtype, p, nblocks, st);
    case RS_VSLASH: return launch_pat<D, P_VS>(dtype, p, nblocks, st);
    default: return launch_pat<D, P_BS>(dtype, p, nblocks, st);
  }
}

static AttnArgs attn_args(const rs_qkv *qkv, float scale, int fam, const rs_index_set *idx, const AttnParts &parts,
                          void *o, int64_t so_h, int64_t so_t, float *lse) {
  AttnArgs a{};
  a.q = qkv->q; a.k = qkv->k; a.v = qkv->v;
  a.sq_h = qkv->sq_h; a.sq_t = qkv->sq_t; a.sk_h = qkv->sk_h; a.sk_t = qkv->sk_t;
  a.sv_h = qkv->sv_h; a.sv_t = qkv->sv_t;
  a.o = (bf16 *)o; a.so_h = so_h; a.so_t = so_t; a.lse = lse;
  a.n = qkv->n; a.group = qkv->hq / qkv->hkv; a.scale = scale; a.c = scale * kLog2e;
  a.parts = parts;
  a.vt = (const bf16 *)qkv->vt; a.npad = (qkv->n + 63) / 64 * 64;
  if (idx && (fam == RS_VSLASH || fam < 0)) {
    a.vs_vsorted = idx->vs_vsorted; a.vs_dsorted = idx->vs_dsorted; a.vs_count = idx->vs_count;
    a.vs_vbits = idx->vs_vbits; a.vs_dbits = idx->vs_dbits;
    a.nv_max = idx->nv_max; a.ns_max = idx->ns_max; a.nwords = idx->nwords; a.ncand_vs = idx->ncand_vs;
  }
  if (idx && (fam == RS_BSPARSE || fam < 0)) {
    a.bs_sorted = idx->bs_sorted; a.bs_count = idx->bs_count;
    a.k_max = idx->k_max; a.nb = idx->nb; a.ncand_bs = idx->ncand_bs;
  }
  return a;
}

// The persistent launch of a family (fam < 0: of every family) over the device planner's queues:
// `nblocks` workgroups drain them.
rs_status attn_launch_queues(const rs_qkv *qkv, float scale, int fam, const rs_index_set *idx,
                             const DevUnit *d_units, const int *d_order, const AttnQueues &queues, int nblocks,
                             const AttnParts &parts, void *o, int64_t so_h, int64_t so_t, float *lse, hipStream_t st) {
  if (nblocks <= 0) return RS_OK;
  AttnDirect p{};
  p.a = attn_args(qkv, scale, fam, idx, parts, o, so_h, so_t, lse);
  p.a.units = d_units; p.a.order = d_order;
  p.a.qsize = queues.size; p.a.qoff = queues.off; p.a.qcount = queues.count;
  hipError_t e;
  if (fam < 0)
    e = qkv->d == 128 ? launch_layer<128>(qkv->dtype, p.a, nblocks, st) : launch_layer<64>(qkv->dtype, p.a, nblocks, st);
  else
    e = qkv->d == 128 ? launch_d<128>(fam, qkv->dtype, p, nblocks, st) : launch_d<64>(fam, qkv->dtype, p, nblocks, st);
  if (e != hipSuccess) return hip_check(e, "attention kernel launch");
  return RS_OK;
}

// Fills p's list of units for units of the same rows that all have mates or all have none
// (taken-along ones apart); false when the list does not fit.  `mate` as pair_units gives it.
static bool direct_list(const rs_unit *units, int nunits, int group, const std::vector<int> &mate,
                        const std::vector<DevUnit> &du, AttnDirect &p) {
  int cnt[8] = {0, 0, 0, 0, 0, 0, 0, 0}, nu = 0, lead = -1;
  for (int u = 0; u < nunits; ++u) {
    if (mate[u] == -2) continue;
    if (lead < 0) lead = u;
    if (units[u].s0 != units[lead].s0 || units[u].s1 != units[lead].s1 || (mate[u] >= 0) != (mate[lead] >= 0) ||
        ++nu > kDirectUnits)
      return false;
    ++cnt[(units[u].head / group) & 7];
  }
  if (lead < 0) return false;
  p.nu = nu;
  p.tiles = tiles_of(units[lead], mate[lead] >= 0 ? 64 : 128);
  p.nsplit = du[lead].nsplit;
  int fill[8];
  for (int b = 0; b < 8; ++b) {
    fill[b] = p.bstart[b];
    p.bstart[b + 1] = p.bstart[b] + cnt[b];
  }
  for (int u = 0; u < nunits; ++u)
    if (mate[u] != -2) {
      const int at = fill[(units[u].head / group) & 7]++;
      p.u[at] = du[u];
      p.u[at].pbase = at * p.tiles * p.nsplit;
    }
  // segments of the grid: buckets in turn until the shortest of those left runs out
  const int per = p.tiles * p.nsplit;  // items per unit
  int done = 0, pos = 0;
  for (;;) {
    int na = 0, mn = 0;
    uint32_t act = 0;
    for (int b = 0; b < 8; ++b)
      if (cnt[b] * per > done) {
        act |= (uint32_t)b << (4 * na++);
        mn = mn == 0 ? cnt[b] * per : std::min(mn, cnt[b] * per);
      }
    if (na == 0) break;
    p.pos[p.nseg] = pos;
    p.first[p.nseg] = done;
    p.na[p.nseg] = na;
    p.act[p.nseg++] = act;
    pos += (mn - done) * na;
    done = mn;
  }
  p.pos[p.nseg] = pos;
  return true;
}

// Shared entry of the dense and sparse calls (arguments validated by the caller).
rs_status attn_launch(const rs_qkv *qkv, float scale, const rs_unit *units, int32_t nunits,
                      int fam, const rs_candidate *cand, int cand_local,
                      const rs_index_set *idx, void *o, int64_t so_h, int64_t so_t, float *lse,
                      void *ws, size_t ws_bytes, hipStream_t st) {
  if (nunits == 0) return RS_OK;
  const int bm = family_bm(fam);
  const int group = qkv->hq / qkv->hkv;
  std::vector<int> mate(nunits, -1), order;
  if (fam == RS_BSPARSE) pair_units(units, nunits, group, mate);
  // items split along the keys, where the workspace holds their partial results too
  std::vector<SplitRule> split(nunits, SplitRule{1, 1});
  size_t slots = 0, items = 0;
  for (int u = 0; u < nunits; ++u) {
    if (mate[u] == -2) continue;
    split[u] = attn_split(qkv->hq, qkv->d, qkv->n, units[u].s0, units[u].s1, fam);
    const size_t nt = (size_t)tiles_of(units[u], mate[u] >= 0 ? 64 : bm);
    if (split[u].nsplit > 1) slots += nt * split[u].nsplit;
    items += nt * split[u].nsplit;
  }
  size_t lbytes = attn_list_bytes(nunits, items);
  if (slots > 0 && (!ws || ((uintptr_t)ws & 15) || ws_bytes < lbytes + attn_parts_bytes(qkv->d, slots))) {
    for (int u = 0; u < nunits; ++u)
      if (split[u].nsplit > 1) items -= (size_t)tiles_of(units[u], bm) * (split[u].nsplit - 1);
    slots = 0;
    std::fill(split.begin(), split.end(), SplitRule{1, 1});
    lbytes = attn_list_bytes(nunits, items);
  }
  if (!ws || ws_bytes < lbytes)
    return fail(RS_ERR_WORKSPACE, "attention workspace too small: need " + std::to_string(lbytes) +
                                      " bytes, got " + std::to_string(ws_bytes));
  AttnParts parts{};
  char *at = (char *)ws + lbytes / 256 * 256;  // past the list's end
  if (slots > 0) parts = attn_parts_at(at, qkv->d, slots);
  at += attn_parts_bytes(qkv->d, slots) / 256 * 256;
  const size_t used = (size_t)(at - (char *)ws);
  const rs_candidate own = cand ? *cand : rs_candidate{RS_DENSE, 0, 0, 0};
  rs_qkv conv;
  rs_status rc = attn_cvt_launch(qkv, units, nunits, &own, 1, at, ws_bytes > used ? ws_bytes - used : 0, &conv, st);
  if (rc != RS_OK) return rc;
  qkv = &conv;
  std::vector<DevUnit> du(nunits);
  int pbase = 0;
  for (int u = 0; u < nunits; ++u) {
    du[u] = DevUnit{units[u].head, units[u].s0, units[u].s1, cand_local, units[u].slot,
                    fam == RS_ASHAPE ? cand->a : 0, fam == RS_ASHAPE ? cand->b : 0,
                    mate[u] >= 0 ? units[mate[u]].head + 1 : 0, cand_local, split[u].nsplit, split[u].ptiles, pbase};
    if (split[u].nsplit > 1) pbase += tiles_of(units[u], bm) * split[u].nsplit;
  }
  AttnDirect p{};
  p.a = attn_args(qkv, scale, fam, idx, parts, o, so_h, so_t, lse);
  MergeDirect md{};
  int nmerge = 0;  // items that may have pieces
  DevUnit *d_units = nullptr;
  if (direct_list(units, nunits, group, mate, du, p)) {
    md = MergeDirect{p.tiles, p.nsplit, p.u[0].s0, p.u[0].s1, {}};
    for (int u = 0; u < p.nu; ++u) md.head[u] = p.u[u].head;
    nmerge = p.nu * p.tiles;
  } else {
    // the list in the workspace: [DevUnit x nunits][order], and the split items
    p.nu = 0;
    const int rotate = fam == RS_VSLASH ? kRotate<P_VS> : fam == RS_BSPARSE ? kRotate<P_BS> : 0;
    build_order(units, nunits, group, bm, rotate, mate, split, order);
    Arena ar(ws, ws_bytes);
    d_units = ar.take<DevUnit>((size_t)nunits);
    int *d_order = ar.take<int>(order.size());
    const size_t off_order = (char *)d_order - (char *)ws;
    std::vector<char> stage(off_order + order.size() * sizeof(int));
    memcpy(stage.data(), du.data(), du.size() * sizeof(DevUnit));
    memcpy(stage.data() + off_order, order.data(), order.size() * sizeof(int));
    RS_HIP(hipMemcpyAsync(ws, stage.data(), stage.size(), hipMemcpyHostToDevice, st));
    if (slots > 0) {
      std::vector<int> h_items;
      for (int u = 0; u < nunits; ++u)
        if (split[u].nsplit > 1)
          for (int t = 0; t < tiles_of(units[u], bm); ++t) h_items.push_back((u << 16) | t);
      nmerge = (int)h_items.size();
      RS_HIP(hipMemcpyAsync(parts.items, h_items.data(), h_items.size() * sizeof(int), hipMemcpyHostToDevice, st));
    }
    p.a.units = d_units;
    p.a.order = d_order;
  }
  const hipError_t e = qkv->d == 128 ? launch_d<128>(fam, qkv->dtype, p, (int)items, st)
                                     : launch_d<64>(fam, qkv->dtype, p, (int)items, st);
  if (e != hipSuccess) return hip_check(e, "attention kernel launch");
  if (slots > 0)
    return merge_launch(qkv, scale, d_units, parts, md, nmerge, o, so_h, so_t, lse, st);
  return RS_OK;
}

}  // namespace rs
