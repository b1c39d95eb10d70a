// Causal attention under the <CL>/<CR> span-exclusion mask (prefill).
// Section 1 (tokens after a <CR> do not attend to the tokens its span
// encloses) and Section 3.1 (<CL> attends only to itself; normal tokens attend
// to earlier <CR> and normal tokens).
//
// With vu[] as in sckv.h, row i may attend to column j iff
//   j <= i <= vu[j]  and  (vu[i] != i or j == i).
//
// plan kernel: for every (sequence, 128-row query block [I, I+128)) the list
//   of key columns j < I+128 with vu[j] >= I, i.e. the columns at least one
//   row of the block may see, in ascending order, packed as
//   j | min(vu[j]-I, 255) << 24.  Columns hidden from the whole block (closed
//   spans, <CL>s before the block) are not in the list and are never read.
//   It then summarises each 64-entry tile of the list (first and last token,
//   smallest rank, valid entries), so the main kernel stages a tile without
//   reductions of its own.
// main kernel: one workgroup per (sequence, head, query block), 4 waves of 32
//   query rows.  Key/value rows named by the list are gathered 64 at a time
//   into LDS (double buffered for bf16); S^T = K Q^T and O^T += V^T P^T run
//   on 32x32 MFMA tiles (bf16 inputs, fp32 accumulation; fp32 inputs use the
//   fp32 MFMA), with an online softmax per query held in the lane that owns
//   the query's column.  Element masks are applied only on tiles that are
//   not entirely visible to a wave; a tile entirely in a wave's future is
//   skipped.  A <CL> row's output is its own value row (it sees only itself),
//   written directly in the epilogue.
//
// Cached variant (block-wise prompt processing, Section 3 "Manipulating
// Key-Value Memory": enclosed tokens are freed block by block when a prompt
// does not fit): the queries are a block of the prompt, tokens tok0 .. tok0+nq-1,
// and the keys are the rows of a cache, row r holding token tok[r] (rows of
// earlier blocks that survived compaction, then the block's own rows from
// row0).  The plan lists cache rows instead of columns, with the same
// visibility rule applied to their tokens; the kernel gathers by row and
// masks by token.
#include <math.h>

#include <cmath>
#include <type_traits>

#include "sckv_common.h"

namespace sckv {

// waves per workgroup, 32 query rows each (six and eight waves, sharing each
// staged tile among more rows, measured 20-45% slower than four)
constexpr int PF_WAVES = 4;
constexpr int PF_BQ = 32 * PF_WAVES;
constexpr int PF_BK = 64;
// a block's list has room for at least two tiles (its first two are loaded early)
static_assert(PF_BQ >= 2 * PF_BK, "list of at least two tiles");
constexpr int PF_THREADS = 64 * PF_WAVES;
// (sequence, head) slices whose query blocks are ordered together,
// heaviest first (a dispatch simulation over the two prompt shapes puts
// groups of 8 within 3-6% of an ideal balance, against 9-18% for one slice)
constexpr int PF_GROUP = 8;
// Groups of four waves per workgroup (bf16), each with every NS-th key tile:
// a launch of fewer workgroups than the chip holds leaves its SIMDs one wave
// each, whose tiles follow one another.  The groups take the room of the
// workgroups that are not there (d = 80: three, d = 64: four fit a CU; two
// groups of d = 64 fit it twice).  Measured, one group and so (us a layer, 32
// heads unless stated): 777 tokens 19.7 and 16.5 (d = 80, three), 18.4 and
// 15.1 (d = 64, two; four 15.5), 8 heads of 2048 tokens (d = 64) 28.1 and 19.8
// (four; two 21.6), 1500 tokens (384 workgroups, d = 64) 23.0 and 18.8 (two).
// With more workgroups each waits for a whole CU: 1024 of d = 64 36.2 and 38.1
// (two), 512 of d = 80 17.8 and 22.1 (4 sequences of 512 tokens, three).
constexpr int PF_ONE_PER_CU = 256, PF_TWO_PER_CU = 512;
// A short list has no tiles to share, and larger workgroups start and merge
// slower.  The host knows the prompt's tokens (or the cache's rows), of which
// the spans may free most.  One group and so, nothing / half / 80% freed:
//   d = 80: 40 tokens 5.8 and 8.0 (three), 128 7.7 / 8.1 / 8.2 and 9.3 / 10.1 /
//     10.1; 2 sequences of 256 10.2 / 10.8 / 9.7 and 11.4 / 11.8 / 10.9, of 512
//     15.3 / 12.4 / 11.0 and 13.8 / 12.4 / 12.0
//   d = 64, up to one workgroup per CU: 40 tokens 5.5 and 6.4 (two); 4 sequences
//     of 192 8.3 / 8.3 / 8.6 and 8.7 / 8.7 / 9.0, of 256 10.4 / 10.7 / 9.9 and
//     9.9 / 10.2 / 10.3
//   d = 64, beyond: 16 sequences of 40 tokens 6.0 and 8.1, 4 of 320 12.0 / 12.0 /
//     11.1 and 13.1 / 12.9 / 12.1, of 512 18.3 / 15.5 / 13.1 and 17.9 / 15.8 /
//     14.1
constexpr int PF_SHARE_80 = 512, PF_SHARE_64 = 256, PF_SHARE_64_TWO = 512;
// Over a cache a block sees the freed rows' room too, and blocks of one
// workgroup a slice are all as long: beyond one workgroup per CU nothing is left
// for groups to even out.  Half freed unless stated:
//   d = 80: 128 single tokens over 513 rows 10.4 and 11.0, over 769 12.8 and 12.6
//   d = 64, up to one workgroup per CU (40% freed): 32 blocks of 64 tokens over 320
//     rows 8.1 and 8.6, of 300 over 300 10.2 and 10.4, of 128 over 384 11.7 and 11.2
//   d = 64, beyond: 512 single tokens over 513 rows 10.9 and 12.8, over 1501 21.3
//     and 23.4, blocks of 64 over 576 16.1 and 17.9, over 1564 27.3 and 28.1; 128
//     blocks of 512 (four workgroups each) over 712 19.5 and 20.4, over 1024 23.7
//     and 22.6, over 3012 46.0 and 41.3
constexpr int PF_CACHED_80 = 640, PF_CACHED_64 = 384, PF_CACHED_64_TWO = 896;
constexpr int PF_LONG = 1409;  // tokens or rows from which four groups have tiles enough
// Few slices are long ones, whose heaviest blocks outlast the rest of the
// launch: with at most eight, up to 512 workgroups of d = 80 take three groups
// too (8 heads of 8192 tokens, half freed, 87.7 and 69.5; 80% freed 42.7 and
// 39.7; 8 of 5120 53.4 and 36.3; 4 of 16384 166 and 120; but 8 of 12288 139
// and 144, and ten heads of 6144, 80% freed, 33.4 and 34.5), up to 768 of
// d = 64 two (8 of 9216 96.0 and 73.2; 8 of 12288 130 and 110, 80% freed 60.0
// and 56.6; but 8 of 16384, 80% freed, 84.6 and 85.3).  Not over a cache,
// where a launch's blocks all see as much (blocks of 512 tokens 1171 and 1286
// a prompt).
constexpr int PF_FEW_SLICES = 8, PF_THREE_PER_CU = 768;
static int prefill_groups(int d, int n_work, int keys, int slices, bool cached) {
  const bool few = !cached && slices <= PF_FEW_SLICES;
  if (d == 80)
    return keys >= (cached ? PF_CACHED_80 : PF_SHARE_80) &&
                   n_work <= (few ? PF_TWO_PER_CU : PF_ONE_PER_CU) ? 3 : 1;
  if (n_work <= PF_ONE_PER_CU)
    return keys >= PF_LONG ? 4 : keys >= (cached ? PF_CACHED_64 : PF_SHARE_64) ? 2 : 1;
  if (cached && n_work == slices) return 1;
  return keys >= (cached ? PF_CACHED_64_TWO : PF_SHARE_64_TWO) &&
                 n_work <= (few ? PF_THREE_PER_CU : PF_TWO_PER_CU) ? 2 : 1;
}
constexpr uint32_t PF_NONE = 0x00ffffffu;  // list entry of a padding column
constexpr float PF_LOG2E = 1.4426950408889634f;
// The running maximum of a query row is only moved (and the accumulators
// rescaled) when a tile's maximum exceeds it by more than this many powers of
// two; until then probabilities are taken relative to the older, smaller
// maximum, which is exact and keeps them below 2^PF_RESCALE.
constexpr float PF_RESCALE = 8.f;

// Cached variant's arguments (unused by the plain prefill).
struct PfCached {
  const int32_t* row0;   // [b] cache row of the block's first query token
  const int32_t* tok;    // [b][L_cap] token held by each cache row
  uint32_t* rows;        // plan output: cache row of each list entry
  int32_t tok0;          // token of the block's first query
  int32_t L_cap;
  int32_t* status;       // nullable: SCKV_STATUS_CAP for a block that does not fit
};

// Summary of one 64-entry tile of a list, written by the plan kernel: first
// and last listed token, smallest rank byte | valid entries << 8, and the row
// a padding slot of the tile repeats (the last valid entry's row).
struct TileSum {
  int32_t jmin, jmax, vr_n, pad_row;
};

// Plain: columns j < min(I+128, L) with token j.  Cached: cache rows
// r < row0 + min(I_loc+128, nq) with token tok[r], where I_loc is the query
// block's first local row and I = tok0 + I_loc its first token.
template <bool CACHED>
__global__ __launch_bounds__(256) void prefill_plan_kernel(const int32_t* __restrict__ vu,
                                                           int32_t L_meta, int32_t L, int32_t n_qt,
                                                           int32_t L_pad,
                                                           uint32_t* __restrict__ list,
                                                           int32_t* __restrict__ count,
                                                           TileSum* __restrict__ info,
                                                           PfCached cc) {
  const int qt = blockIdx.x;
  const int s = blockIdx.y;
  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int I_loc = qt * PF_BQ;
  int I = I_loc, jend = min(I_loc + PF_BQ, L);
  if constexpr (CACHED) {
    I = cc.tok0 + I_loc;
    const int r0 = cc.row0[s];
    const bool fits = r0 >= 0 && (int64_t)r0 + L <= cc.L_cap;
    jend = fits ? r0 + min(I_loc + PF_BQ, L) : 0;
  }
  const int32_t* v = vu + (int64_t)s * L_meta;
  uint32_t* out = list + ((int64_t)s * n_qt + qt) * L_pad;
  // PLAN_U columns a thread in flight together: the rounds follow one another
  // and each costs a round trip to memory and two barriers (prompts of 4096
  // tokens, 16 sequences: 18.2 us with one column a thread, 10.9 us with four)
  constexpr int PLAN_U = 4;
  __shared__ int cnt[PLAN_U * 4];  // listed columns of (pass u, wave w) at [4u + w]
  int carry = 0;
  for (int base = 0; base < jend; base += 256 * PLAN_U) {
    bool ok[PLAN_U];
    uint32_t e[PLAN_U];
    int tok[PLAN_U], x[PLAN_U];
    uint64_t m[PLAN_U];
#pragma unroll
    for (int u = 0; u < PLAN_U; ++u) {
      // the column's token: the row itself, or the token a cache row holds
      // (a row whose token lies outside [0, L_meta) is never listed)
      const int j = base + u * 256 + tid;
      ok[u] = j < jend;
      tok[u] = CACHED ? (ok[u] ? cc.tok[(int64_t)s * cc.L_cap + j] : 0) : j;
    }
#pragma unroll
    for (int u = 0; u < PLAN_U; ++u) {
      if (CACHED) ok[u] = ok[u] && tok[u] >= 0 && tok[u] < L_meta;
      x[u] = ok[u] ? v[tok[u]] : 0;
    }
#pragma unroll
    for (int u = 0; u < PLAN_U; ++u) {
      ok[u] = ok[u] && x[u] >= I;
      const int64_t rel = (int64_t)x[u] - I;
      e[u] = (uint32_t)tok[u] | ((uint32_t)(rel > 255 ? 255 : rel) << 24);
      m[u] = __ballot(ok[u]);
      if ((tid & 63) == 0) cnt[4 * u + wave] = __popcll(m[u]);
    }
    __syncthreads();
    int sum = carry;
#pragma unroll
    for (int u = 0; u < PLAN_U; ++u) {
      int off = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (w == wave) off = sum;
        sum += cnt[4 * u + w];
      }
      if (ok[u]) {
        out[off + mask_rank(m[u])] = e[u];
        if constexpr (CACHED)
          cc.rows[((int64_t)s * n_qt + qt) * L_pad + off + mask_rank(m[u])] = base + u * 256 + tid;
      }
    }
    carry = sum;
    __syncthreads();
  }
  if (tid == 0) count[(int64_t)s * n_qt + qt] = carry;

  // tile summaries: wave w takes tiles w, w+4, ... of the list just written
  // (the barrier that ended the last round orders those writes before these
  // reads), two at a time
  const int lane = tid & 63;
  const uint32_t* rws = CACHED ? cc.rows + ((int64_t)s * n_qt + qt) * L_pad : nullptr;
  TileSum* sum = info + ((int64_t)s * n_qt + qt) * (L_pad / 64);
  for (int t0 = wave; t0 * 64 < carry; t0 += 8) {
    uint32_t e[2];
    int row[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int at = (t0 + 4 * i) * 64 + lane;
      e[i] = at < carry ? out[at] : PF_NONE;
      row[i] = CACHED && at < carry ? (int)rws[at] : 0;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int t = t0 + 4 * i;
      if (t * 64 >= carry) break;
      const int nvalid = min(64, carry - t * 64);
      const int vr = (int)-wave_max(-(float)(lane < nvalid ? (int)(e[i] >> 24) : 255));
      const int jmin = __builtin_amdgcn_readlane((int)(e[i] & 0x00ffffffu), 0);
      const int jmax = __builtin_amdgcn_readlane((int)(e[i] & 0x00ffffffu), nvalid - 1);
      const int pad = CACHED ? __builtin_amdgcn_readlane(row[i], nvalid - 1) : jmax;
      if (lane == 0) sum[t] = TileSum{jmin, jmax, vr | (nvalid << 8), pad};
    }
  }
}

// ---------------------------------------------------------------------------
// tile geometry per element type
// ---------------------------------------------------------------------------
template <typename T, int D> struct PfCfg;

template <int D> struct PfCfg<uint16_t, D> {
  static constexpr int NBUF = 2;
  static constexpr int DP = (D + 31) / 32 * 32;     // value columns padded to whole 32-row MFMA blocks
  static constexpr int KP = D + 8;                  // K tile: [64][KP] bf16 (one 16-byte pad slot)
  // V tile: [64][VP] bf16, row-major like K; the PV operand is read with the
  // transposing LDS read.  With a ones row (D = 80) the pitch is 192 bytes,
  // which puts the four rows one transposing read touches in disjoint groups
  // of 16 banks.  At D = 64 the rows are unpadded (128 bytes) and the
  // 16-byte pieces of a row are swizzled instead: logical piece p of row r
  // sits in slot p ^ (4 * bit 1 of r), which spreads the rows of one
  // transposing read over the banks the same way in two thirds of the space.
  static constexpr bool VSWZ = (D == 64);
  static constexpr int VP = VSWZ ? D : 96;
  static constexpr int NB = D == 64 ? 1 : 2;        // 32-key blocks per softmax step
  static_assert(DP <= VP, "value tile pitch");
  static constexpr int E = 8;                       // elements per 16-byte slot
  static constexpr int KSTEPS = D / 16;
};

template <int D> struct PfCfg<float, D> {
  static constexpr int NBUF = 1;
  static constexpr bool VSWZ = false;
  static constexpr int NB = 2;
  static constexpr int DP = (D + 31) / 32 * 32;
  static constexpr int KP = D + 4;                  // K tile: [64][KP] f32
  static constexpr int VP = DP + 8;                 // V tile: [64][VP] f32 (row-major)
  static constexpr int E = 4;
  static constexpr int KSTEPS = D / 2;
};

// Row slots of a staged tile.  Rows are copied global -> LDS by the
// direct-to-LDS load (16 bytes per lane, lane i of an instruction writes
// slot base+i), so a tile is a whole number of 1 KiB blocks of 64 slots.
template <typename T, int D>
struct PfTile {
  using C = PfCfg<T, D>;
  static constexpr int PPR = D / C::E;                         // data slots per row
  static constexpr int KSLOT = C::KP * (int)sizeof(T) / 16;    // slots per K row
  static constexpr int VSLOT = C::VP * (int)sizeof(T) / 16;    // slots per V row
  static_assert(C::KP * sizeof(T) % 16 == 0 && C::VP * sizeof(T) % 16 == 0, "slot pitch");
  static constexpr int KBYTES = PF_BK * KSLOT * 16;            // == KSLOT KiB
  static constexpr int VBYTES = PF_BK * VSLOT * 16;
};

struct TileInfo {
  int jmin, jmax, vrmin, nvalid;
};

// maximum of x over lanes l and l^32: one lane swap between the two
// 32-lane halves of the wave (v_permlane32_swap leaves each lane holding
// the pair's two values, one in each result)
__device__ __forceinline__ float max_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

constexpr int PF_ER = 4;  // ring of list entries: tile kt+2 is fetched while kt is computed

typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Work order.  Workgroup x is dispatched to XCD x mod 8.  Each XCD takes
// nbh / 8 of the (sequence, head) slices whole, in groups of PF_GROUP that
// share its L2.  Inside a group the blocks go heaviest first: every slice's
// last query block (the most visible keys), then every slice's block before
// it, and so on, so that the light blocks fill the end of the launch instead
// of one slice's heavy block running alone there.  The nbh mod 8 slices left
// over come first, their blocks dealt over all XCDs, heaviest first.  (One
// contiguous range of blocks per XCD, in groups of 8 slices whatever their
// number, gave half the XCDs the heavy half of each group below 64 slices:
// 32 slices of 16384 tokens at d = 64 took 822 us, and 665 us in this order;
// 256 and 512 slices, whose groups fell whole to one XCD, take the same.)
__device__ __forceinline__ void work_item(int x, int nbh, int n_qt, int* bh, int* qt) {
  const int per = nbh >> 3, rem = nbh & 7;
  const int first = rem * n_qt;
  if (x < first) {
    *bh = 8 * per + x % rem;
    *qt = n_qt - 1 - x / rem;
    return;
  }
  const int y = x - first;
  const int xcd = y & 7, idx = y >> 3;
  const int grp = idx / (PF_GROUP * n_qt);
  const int gsz = min(PF_GROUP, per - grp * PF_GROUP);
  const int in_grp = idx - grp * PF_GROUP * n_qt;
  *bh = xcd * per + grp * PF_GROUP + in_grp % gsz;
  *qt = n_qt - 1 - in_grp / gsz;
}

// ---------------------------------------------------------------------------
// main kernel
// ---------------------------------------------------------------------------
// NS > 1 (bf16): NS groups of four waves share the workgroup's query rows and
// take every NS-th tile each, with tile buffers of their own; their partial
// outputs are merged through LDS at the end.
template <typename T, int D, bool CACHED, int NS = 1>
__device__ __forceinline__ void prefill_attn_body(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, T* __restrict__ o,
    int32_t H, int32_t L, int64_t qs, int64_t kvs, int64_t os, float c2,
    const int32_t* __restrict__ vu, int32_t L_meta, const uint32_t* __restrict__ list,
    const int32_t* __restrict__ count, const TileSum* __restrict__ info, int32_t n_qt,
    int32_t L_pad, int32_t n_work, PfCached cc) {
  using C = PfCfg<T, D>;
  using TL = PfTile<T, D>;
  constexpr bool BF = sizeof(T) == 2;
  constexpr int NDB = C::DP / 32;                           // output d blocks

  // Separate objects per buffer: the compiler then knows that a
  // direct-to-LDS load into one buffer does not feed reads of the other.
  // With several groups the buffers of a group are found at run time: the
  // copies are then written in assembly, out of the compiler's sight (dma_rows).
  static_assert(NS == 1 || (BF && C::NBUF == 2), "groups are for bf16");
  constexpr int TILEB = TL::KBYTES + TL::VBYTES;
  __shared__ __align__(1024) char kbuf0_s[NS == 1 ? TL::KBYTES : 1];
  __shared__ __align__(1024) char vbuf0_s[NS == 1 ? TL::VBYTES : 1];
  __shared__ __align__(1024) char kbuf1_s[NS != 1 ? 1 : C::NBUF == 2 ? TL::KBYTES : 1024];
  __shared__ __align__(1024) char vbuf1_s[NS != 1 ? 1 : C::NBUF == 2 ? TL::VBYTES : 1024];
  __shared__ __align__(1024) char tiles[NS == 1 ? 1 : NS * 2 * TILEB];
  // per entry its token and, in the second row, how many tokens after it still
  // see it: row i sees it iff i - token, taken as unsigned, is at most that
  __shared__ int32_t ent_rings[NS][PF_ER][2][PF_BK];
  __shared__ int32_t row_rings[NS][PF_ER][PF_BK];  // bare row index per entry
  __shared__ TileInfo info_rings[NS][PF_ER];

  int bh, qt;
  work_item(blockIdx.x, n_work / n_qt, n_qt, &bh, &qt);
  const int s = bh / H;
  // query rows are local (0 .. L-1); their tokens start at tok0 (cached) or 0
  const int tok0 = CACHED ? cc.tok0 : 0;
  const int I_loc = qt * PF_BQ;
  const int I = tok0 + I_loc;

  // thread, wave and group; all but the group count within the group
  const int grp = NS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / PF_THREADS);
  const int tid = (int)threadIdx.x - grp * PF_THREADS;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const int l32 = lane & 31;
  const int g = lane >> 5;
  char* const kbuf0 = NS == 1 ? kbuf0_s : tiles + grp * 2 * TILEB;
  char* const vbuf0 = NS == 1 ? vbuf0_s : tiles + grp * 2 * TILEB + TL::KBYTES;
  char* const kbuf1 = NS == 1 ? kbuf1_s : tiles + grp * 2 * TILEB + TILEB;
  char* const vbuf1 = NS == 1 ? vbuf1_s : tiles + grp * 2 * TILEB + TILEB + TL::KBYTES;
  auto& ent_ring = ent_rings[grp];
  auto& row_ring = row_rings[grp];
  auto& info_ring = info_rings[grp];
  const int Iw_loc = I_loc + wave * 32;
  const int Iw = I + wave * 32;
  const int qrow = Iw_loc + l32;  // local query row
  const int qtok = Iw + l32;      // its token
  const bool wave_live = Iw_loc < L;

  const T* qb = q + (int64_t)bh * qs;
  const T* kb = k + (int64_t)bh * kvs;
  const T* vb = v + (int64_t)bh * kvs;
  const uint32_t* ents = list + ((int64_t)s * n_qt + qt) * L_pad;
  const uint32_t* rws = CACHED ? cc.rows + ((int64_t)s * n_qt + qt) * L_pad : nullptr;
  const TileSum* tsum = info + ((int64_t)s * n_qt + qt) * (L_pad / 64);
  int own_row0 = 0;  // cache row of local query row 0
  if constexpr (CACHED) {
    own_row0 = cc.row0[s];
    if (own_row0 < 0 || (int64_t)own_row0 + L > cc.L_cap) {
      // the block's rows are not in the cache: NaN outputs, nothing read
      if (cc.status && threadIdx.x == 0 && qt == 0 && (bh % H) == 0) atomicOr(cc.status, SCKV_STATUS_CAP);
      if (grp == 0 && wave_live && qrow < L) {
        T* orow = o + (int64_t)bh * os + (int64_t)qrow * D;
        for (int e = g; e < D; e += 2) {
          if constexpr (sizeof(T) == 2) orow[e] = (T)0x7fc0;
          else orow[e] = NAN;
        }
      }
      return;
    }
  }
  // clamped into the list, so that a workspace holding no valid plan (a
  // caller's mistake with the planned entry point) reads nothing outside it
  const int n_vis = min(max(count[(int64_t)s * n_qt + qt], 0), L_pad);
  const int nt_all = (n_vis + PF_BK - 1) / PF_BK;
  // the group's tiles: its tile kt is the list's tile NS * kt + grp
  const int nt = NS == 1 ? nt_all : (nt_all - grp + NS - 1) / NS;

  // Padding value rows/columns are written once and never again.  For bf16
  // with padding, V^T row D is all ones, so the PV MFMA also produces each
  // query's probability sum (O^T row D) and no separate row sum is needed.
  constexpr bool ONES_SUM = BF && (C::DP != D);
  // Without padding (bf16, D = 64) the sums come from a 16x16x32 MFMA of the
  // probabilities against a 0/1 matrix: lane L's A operand is all ones when
  // bit 2 of L equals bit 4 of L, so D[4*(L/16) + j][L%16] adds the two
  // lanes that hold query L%32's probabilities (lanes q and q + 32 of the
  // 32x32x16 B operand), and every lane receives its own query's sum.
  constexpr bool MFMA_SUM = BF && !ONES_SUM;
  if constexpr (C::DP != D) {
    for (int b = 0; b < C::NBUF; ++b) {
      char* vbuf = b == 0 ? vbuf0 : vbuf1;
      if constexpr (BF) {
        uint16_t* vs = reinterpret_cast<uint16_t*>(vbuf);
        for (int i = tid; i < PF_BK * (C::DP - D); i += PF_THREADS) {
          const int c = D + i % (C::DP - D);
          vs[(i / (C::DP - D)) * C::VP + c] = (c == D) ? (uint16_t)0x3f80 : (uint16_t)0;
        }
      } else {
        float* vs = reinterpret_cast<float*>(vbuf);
        for (int i = tid; i < PF_BK * (C::DP - D); i += PF_THREADS)
          vs[(i / (C::DP - D)) * C::VP + D + i % (C::DP - D)] = 0.f;
      }
    }
  }

  // Q^T operand, held for the whole kernel
  using QReg = typename std::conditional<BF, bf16x8, float>::type;
  QReg qreg[C::KSTEPS];
#pragma unroll
  for (int kk = 0; kk < C::KSTEPS; ++kk) {
    if constexpr (BF) {
      u32x4 w = qrow < L ? ld16(qb + (int64_t)qrow * D + kk * 16 + g * 8) : u32x4{0, 0, 0, 0};
      qreg[kk] = __builtin_bit_cast(bf16x8, w);
    } else {
      qreg[kk] = qrow < L ? qb[(int64_t)qrow * D + 2 * kk + g] : 0.f;
    }
  }

  // A <CL> row's output is its own value row, copied before the loop: after it
  // nothing hides the two dependent loads.  Behind the first tile's copies they
  // wait for all of them, which short lists show (2048 heads of 128 tokens, 60%
  // freed: 40.1 us so and 36.0 ahead of them at d = 80, 33.9 and 31.4 at d = 64).
  //   d = 80: here.
  //   d = 64, short of registers: a slice's only block while its first entries
  //     are on their way, others behind the copies (256 heads of 777 tokens 33.8
  //     so, 34.5 ahead of them; 8 x 32 of 1024 46.5 and 48.1).
  //   groups of waves (over a cache at d = 64 they would spill) and fp32 (256 heads
  //     of 512 tokens, 40% freed, d = 64: 104.0, and 109.9 here): behind the copies.
  constexpr bool CL_HERE = NS == 1 && BF && D == 80;
  const bool cl_late = NS > 1 || !BF || (D == 64 && n_qt > 1);
  bool is_cl = false;
  auto mark_cl = [&]() { is_cl = qrow < L && vu[(int64_t)s * L_meta + qtok] == qtok; };
  auto copy_cl = [&]() {
    if (!is_cl || grp > 0) return;
    T* const orow = o + (int64_t)bh * os + (int64_t)qrow * D;
    const T* vrow = vb + (int64_t)(own_row0 + qrow) * D;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int d0 = db * 32 + 8 * jj + 4 * g;
        if (d0 >= D) continue;
        if constexpr (BF) *reinterpret_cast<u32x2*>(orow + d0) = *reinterpret_cast<const u32x2*>(vrow + d0);
        else st16(orow + d0, ld16(vrow + d0));
      }
  };
  if (!cl_late) mark_cl();
  if constexpr (CL_HERE) copy_cl();

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
  // the running maximum as the steps use it: negated (0 while there is none),
  // and the value from which a step moves it
  float m_neg = 0.f, m_next = -INFINITY, l_run = 0.f;
  f32x4 lacc = {0.f, 0.f, 0.f, 0.f};

  // ---- staging: list entries run two tiles ahead through an LDS ring; the
  // key/value rows of tile kt+1 go global -> LDS by direct loads addressed
  // from the ring while tile kt is multiplied ----
  // a tile's list entries (wave 0's lanes), their cache rows (cached) and the
  // plan's summary of the tile, between their load and their ring slot
  struct Staged {
    uint32_t e;
    int r;
    TileSum s;
  };
  Staged stg = {PF_NONE, 0, {0, 0, 0, 0}};
  auto list_tile = [&](int kt) { return NS == 1 ? kt : NS * kt + grp; };
  auto nvalid_of = [&](int kt) { return min(PF_BK, n_vis - list_tile(kt) * PF_BK); };
  // The loads do not depend on the list's length (the list has room for at
  // least two tiles, and later ones are clamped into it), so the first tiles'
  // loads need not wait for the count; the length masks them when stored.
  auto load_entries = [&](int kt, Staged& st) {
    const int lt = NS == 1 ? kt : min(list_tile(kt), L_pad / PF_BK - 1);
    if (tid < PF_BK) {
      st.e = ents[lt * PF_BK + tid];
      if constexpr (CACHED) st.r = (int)rws[lt * PF_BK + tid];
    }
    if (wave == 0) st.s = tsum[lt];
  };
  // wave 0 writes the ring slot of tile kt from the entries and the plan's
  // summary of the tile
  auto store_entries = [&](int kt, const Staged& st) {
    const bool in = lane < nvalid_of(kt);
    const uint32_t ereg = in ? st.e : PF_NONE;
    const int rreg = in ? st.r : 0;
    const TileSum sreg = st.s;
    const int slot = kt % PF_ER;
    if (wave == 0) {
      const int vr_n = __builtin_amdgcn_readfirstlane(sreg.vr_n);
      const int nvalid = NS == 1 ? vr_n >> 8 : min(vr_n >> 8, nvalid_of(kt));
      const int tok = (int)(ereg & 0x00ffffffu);
      ent_ring[slot][0][lane] = tok;
      // ranks of 255 stand for any larger one; the block's rows end before
      ent_ring[slot][1][lane] = in ? max(I + (int)(ereg >> 24) - tok, 0) : 0;
      // a padding row of the tile repeats the last valid row (its score is
      // masked, so any finite row will do)
      const int row = CACHED ? rreg : tok;
      row_ring[slot][lane] = lane < nvalid ? row : __builtin_amdgcn_readfirstlane(sreg.pad_row);
      if (lane == 0) {
        TileInfo ti;
        ti.jmin = sreg.jmin;
        ti.jmax = sreg.jmax;
        ti.vrmin = vr_n & 255;
        ti.nvalid = nvalid;
        info_ring[slot] = ti;
      }
    }
  };
  // K and V of tile kt into kdst/vdst: slot sl = r*NSLOT + sg of a matrix
  // holds elements [sg*E, sg*E+E) of row r; pad slots are not written (they
  // keep their initial contents).  All row indices are read from the ring
  // first, then the copies are issued.  The indices come from row_ring, which
  // holds them bare: no masking of the packed entry happens on this path.
  constexpr int KRND = (TL::KSLOT + PF_WAVES - 1) / PF_WAVES;
  constexpr int VRND = (TL::VSLOT + PF_WAVES - 1) / PF_WAVES;
  // Copies go through buffer loads with an LDS destination: a 32-bit byte
  // offset per lane against a descriptor of the slice's rows (at most 32768),
  // the LDS block address in scalar registers.  The descriptor ends with the
  // last row, not with the stride to the next slice: behind the last slice's
  // rows the buffer may end, and what is read past the descriptor (the last
  // row's pad slot, rows of a plan made for a longer prompt) is zero instead.
  // Each lane's tile row and piece offset per round are fixed for the kernel
  // and computed once here.
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int slice_bytes = (CACHED ? cc.L_cap : L) * D * (int)sizeof(T);
  const __amdgpu_buffer_rsrc_t krs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(kb), 0, slice_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(vb), 0, slice_bytes, 0x00020000);
  constexpr int ROWB = D * (int)sizeof(T);
  // Over a cache at D = 64 the registers don't suffice for all of them (the one
  // spilled was reloaded in the middle of a step's copies, behind a wait for
  // every copy before it): wave 0, which alone copies a key block in the last
  // round, works that round's piece offset out from its row (5 x 32 blocks of
  // 512 tokens over 1500 rows 50.7 -> 49.0 us, 8 x 32 over 600 29.1 -> 28.3).
  constexpr bool LATE_K = CACHED && BF && D == 64 && NS == 1;
  static_assert(!LATE_K || TL::KSLOT % PF_WAVES == 1, "the last round is wave 0's");
  int k_row[KRND], k_off[KRND], v_row[VRND], v_off[VRND];
#pragma unroll
  for (int rnd = 0; rnd < KRND; ++rnd) {
    const int sl = (rnd * PF_WAVES + wave) * 64 + lane;
    const int sg = sl % TL::KSLOT;
    k_row[rnd] = min(sl / TL::KSLOT, PF_BK - 1);
    // a key row's pad slot is never read, so it is copied too (the first 16
    // bytes of the next row): no lane of a copy is masked off
    k_off[rnd] = sg * 16;
  }
#pragma unroll
  for (int rnd = 0; rnd < VRND; ++rnd) {
    if constexpr (C::VSWZ) {
      // a round moves a whole number of rows, by a multiple of 4: the later
      // rounds' rows and pieces follow from the first's (registers saved)
      static_assert(PF_THREADS % TL::VSLOT == 0 && PF_THREADS / TL::VSLOT % 4 == 0, "whole rows a round");
      if (rnd > 0) {
        v_row[rnd] = v_row[0] + rnd * (PF_THREADS / TL::VSLOT);
        v_off[rnd] = v_off[0];
        continue;
      }
    }
    const int sl = (rnd * PF_WAVES + wave) * 64 + lane;
    const int sg = sl % TL::VSLOT;
    v_row[rnd] = min(sl / TL::VSLOT, PF_BK - 1);
    int vpiece = sg;  // the logical piece slot sg holds
    if constexpr (BF) {
      if constexpr (C::VSWZ) vpiece = sg ^ (((v_row[rnd] >> 1) & 1) << 2);
    }
    // the value tile's pad slots hold the ones row and zeros (D = 80) and
    // must not be overwritten; without them (D = 64) every slot is data
    v_off[rnd] = sg < TL::PPR ? vpiece * 16 : -1;
  }
  // A copy in assembly has no register results; wait_vmem and the step's
  // barrier order it.  (Through the builtin, the compiler makes every LDS read
  // wait for every copy where it cannot tell the buffers apart.)  The compiler
  // sees no memory instruction here, so the five wait states between a vector
  // instruction's write of a scalar register (the descriptor's) and its use by
  // the copy are kept in the asm, whatever stands before it.
  typedef uint32_t rsrc_t __attribute__((ext_vector_type(4)));
  auto rsrc_words = [&](const void* base) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    return rsrc_t{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                  (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) & 0xffffu,
                  (uint32_t)__builtin_amdgcn_readfirstlane(slice_bytes), 0x00020000u};
  };
  const rsrc_t krw = rsrc_words(kb), vrw = rsrc_words(vb);
  auto copy_rows = [&](const __amdgpu_buffer_rsrc_t& rs, const rsrc_t& rw, char* dst, int off) {
    if constexpr (NS == 1) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)dst, 16, off, 0, 0, 0);
    } else {
      const uint32_t lds = (uint32_t)__builtin_amdgcn_readfirstlane(
          (int)(uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)dst);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(lds), "v"(off), "s"(rw) : "m0", "memory");
    }
  };
  auto dma_rows = [&](int kt, char* kdst, char* vdst) {
    const int32_t* rows = row_ring[kt % PF_ER];
    int kj[KRND], vj[VRND];
#pragma unroll
    for (int rnd = 0; rnd < KRND; ++rnd) kj[rnd] = rows[k_row[rnd]];
#pragma unroll
    for (int rnd = 0; rnd < VRND; ++rnd) vj[rnd] = rows[v_row[rnd]];
#pragma unroll
    for (int rnd = 0; rnd < KRND; ++rnd) {
      const int blk = rnd * PF_WAVES + wave_s;
      if (blk < TL::KSLOT) {
        int off = k_off[rnd];
        if constexpr (LATE_K) {
          if (rnd == KRND - 1) {
            int lane_k = lane, row_k = k_row[rnd];
            asm volatile("" : "+v"(lane_k), "+v"(row_k));  // not ahead of the loop
            off = (rnd * PF_THREADS + lane_k - row_k * TL::KSLOT) * 16;
          }
        }
        copy_rows(krs, krw, kdst + blk * 1024, kj[rnd] * ROWB + off);
      }
    }
#pragma unroll
    for (int rnd = 0; rnd < VRND; ++rnd) {
      const int blk = rnd * PF_WAVES + wave_s;
      if (blk < TL::VSLOT && (TL::VSLOT == TL::PPR || v_off[rnd] >= 0))
        copy_rows(vrs, vrw, vdst + blk * 1024, vj[rnd] * ROWB + v_off[rnd]);
    }
  };

  // Transposing-read addresses of the V^T operand, per 32-column block db
  // of the value tile: within each group of 16 lanes, lane j points at
  // V[kbase + j/4][dbase + 4*(j%4)]; the read hands lane i the four keys
  // kbase..kbase+3 of column dbase + i.  Offsets in elements from the tile
  // start; a step t of 16 keys adds (16 t) rows, its upper 8 keys 8 rows.
  int v_lane_off[NDB];
  {
    const int G = lane >> 4, j16 = lane & 15;
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      const int col = 32 * db + 16 * (G & 1) + 4 * (j16 & 3);
      const int row = 4 * g + (j16 >> 2);  // bit 1 of the row is bit 1 of j16 >> 2
      if constexpr (BF && C::VSWZ)
        v_lane_off[db] = row * C::VP + (((col >> 3) ^ (((row >> 1) & 1) << 2)) << 3) + (col & 7);
      else
        v_lane_off[db] = row * C::VP + col;
    }
  }

  // summary of the tile being computed, read from the ring one step early
  // so that the step starts with its key reads
  TileInfo tcur;
  // Neither unit is full: vector issue is the busier one (SQ counters over a
  // launch: vector instructions active 66% of the clocks and matrix cores busy
  // 50% at 16384 tokens, d = 64; 50 and 41% at 16 x 4096, d = 80), and a wave's
  // dependent steps, which three or four waves a SIMD cover in part, take the
  // rest.  Instructions shorten that chain too: the running maximum is kept in
  // the form its users take, and an element mask is one unsigned compare of a
  // difference (3 vector instructions an element instead of 4 and a scalar
  // one).  2-4% of a layer at either head size (16 x 4096 tokens, d = 80: 1011
  // -> 988 us; 8 x 2048, d = 64: 120.4 -> 117.5), bit for bit.
  // A 64-key tile is weighed in softmax steps of NB 32-key blocks: scores
  // of the step, its online softmax, its share of the value product.  At
  // D = 64 a step is one block (32 keys), so only half a tile's scores and
  // probabilities are live at a time and four waves fit per SIMD; at D = 80
  // a step is the whole tile (measured faster there, at three waves either
  // way).
  constexpr int NB = C::NB;
  // With `peak`, the step's scores of the tile in tcur only give the running
  // maximum of the rows that have none yet, from the list's first tile.
  auto compute = [&](int kt, const char* kcur, const char* vcur, auto peak) {
    const TileInfo ti = tcur;
    const int32_t* tent = peak ? ent_rings[0][0][0] : ent_ring[kt % PF_ER][0];
    if (wave_live && ti.jmin <= Iw + 31) {
      const bool full = ti.nvalid == PF_BK && ti.jmax <= Iw && ti.vrmin >= Iw + 31 - I;
      // With one 32-key block per step, the second block is skipped where
      // no row of this wave can see any of it: it lies past the list's end,
      // or (the list being in token order) its first token is later than the
      // wave's last row.
      bool skip2 = false;
      if constexpr (NB == 1) {
        if (!full) {
          const int j32 = __builtin_amdgcn_readfirstlane(tent[32]);
          skip2 = ti.nvalid <= 32 || j32 > Iw + 31;
        }
      }
#pragma unroll
      for (int st = 0; st < 2 / NB; ++st) {
        if (st == 1 && skip2) break;
        // ---- S^T = K Q^T for the step's key blocks, key step outer so that
        // consecutive matrix instructions write different accumulators ----
        f32x16 sacc[NB];
#pragma unroll
        for (int kb = 0; kb < NB; ++kb)
#pragma unroll
          for (int i = 0; i < 16; ++i) sacc[kb][i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < C::KSTEPS; ++kk) {
#pragma unroll
          for (int kb = 0; kb < NB; ++kb) {
            const int kb2 = st * NB + kb;
            if constexpr (BF) {
              const char* krow = kcur + ((kb2 * 32 + l32) * C::KP + g * 8 + kk * 16) * 2;
              const bf16x8 a = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(krow));
              sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[kk], sacc[kb], 0, 0, 0);
            } else {
              const float* krow = reinterpret_cast<const float*>(kcur) + (kb2 * 32 + l32) * C::KP + g;
              sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(krow[2 * kk], qreg[kk], sacc[kb], 0, 0, 0);
            }
          }
        }
        // ---- element mask on tiles not entirely visible to this wave ----
        if (!full) {
          // the lane's token and key offset are worked out here again: held
          // across the tile loop they cost registers that it needs
          int lane_m = threadIdx.x & 63;
          asm volatile("" : "+v"(lane_m));
          const int tok_m = Iw + (lane_m & 31), g_m = lane_m >> 5;
#pragma unroll
          for (int kb = 0; kb < NB; ++kb)
#pragma unroll
            for (int vv = 0; vv < 16; ++vv) {
              const int key = (st * NB + kb) * 32 + 8 * (vv >> 2) + 4 * g_m + (vv & 3);
              const bool vis = (uint32_t)(tok_m - tent[key]) <= (uint32_t)tent[PF_BK + key];
              sacc[kb][vv] = vis ? sacc[kb][vv] : -INFINITY;
            }
        }
        // ---- online softmax (log2 units), lazy rescaling ----
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < NB; ++kb)
#pragma unroll
          for (int vv = 0; vv < 16; ++vv) mx = fmaxf(mx, sacc[kb][vv]);
        mx = max_across_halves(mx) * c2;
        if constexpr (peak) {
          if (m_next == -INFINITY && mx > -INFINITY) {
            m_neg = -mx;
            m_next = mx + PF_RESCALE;
          }
          if (__ballot(m_next == -INFINITY) == 0) break;
          continue;
        }
        const bool grow = mx > m_next;
        if (__ballot(grow) != 0) {
          // without an old maximum 0
          const float alpha = !grow ? 1.f : m_next == -INFINITY ? 0.f : fast_exp2(-m_neg - mx);
          if (grow) {
            m_neg = -mx;
            m_next = mx + PF_RESCALE;
          }
          if constexpr (MFMA_SUM) lacc *= alpha;
          else l_run *= alpha;
#pragma unroll
          for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
        }
        float rs = 0.f;
#pragma unroll
        for (int kb = 0; kb < NB; ++kb)
#pragma unroll
          for (int vv = 0; vv < 16; ++vv) {
            const float p = fast_exp2(fmaf(sacc[kb][vv], c2, m_neg));
            sacc[kb][vv] = p;
            if constexpr (!ONES_SUM && !MFMA_SUM) rs += p;
          }
        if constexpr (!ONES_SUM && !MFMA_SUM) l_run += rs;
        // ---- O^T += V^T P^T over the step's keys, 16 at a time ----
        if constexpr (BF) {
          bf16x8 pb[2 * NB];
#pragma unroll
          for (int tt = 0; tt < 2 * NB; ++tt) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              w[i] = pack_bf16x2(sacc[tt >> 1][8 * (tt & 1) + 2 * i], sacc[tt >> 1][8 * (tt & 1) + 2 * i + 1]);
            pb[tt] = __builtin_bit_cast(bf16x8, w);
          }
          if constexpr (MFMA_SUM) {
            const int ln = threadIdx.x & 63;
            const uint32_t one = (((ln >> 2) ^ (ln >> 4)) & 1) ? 0u : 0x3f803f80u;
            const bf16x8 ones_a = __builtin_bit_cast(bf16x8, u32x4{one, one, one, one});
#pragma unroll
            for (int tt = 0; tt < 2 * NB; ++tt)
              lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones_a, pb[tt], lacc, 0, 0, 0);
          }
          const uint16_t* vs = reinterpret_cast<const uint16_t*>(vcur);
#pragma unroll
          for (int tt = 0; tt < 2 * NB; ++tt) {
            const int t = 2 * NB * st + tt;
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
              const s16x4 lo = lds_read_tr16(vs + v_lane_off[db] + (16 * t) * C::VP);
              const s16x4 hi = lds_read_tr16(vs + v_lane_off[db] + (16 * t + 8) * C::VP);
              const s16x8 vw = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
              oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vw),
                                                                 pb[tt], oacc[db], 0, 0, 0);
            }
          }
        } else {
          const float* vs = reinterpret_cast<const float*>(vcur);
#pragma unroll
          for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int kb = 0; kb < NB; ++kb)
#pragma unroll
              for (int vv = 0; vv < 16; ++vv) {
                const int key = (st * NB + kb) * 32 + 8 * (vv >> 2) + 4 * g + (vv & 3);
                oacc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vs[key * C::VP + db * 32 + l32],
                                                                sacc[kb][vv], oacc[db], 0, 0, 0);
              }
        }
      }
    }
  };

  // one tile: rows of kt+1 start moving, kt is multiplied, everything is
  // waited for, the ring advances
  auto iteration = [&](int kt, const char* kc, const char* vc, char* kn, char* vn) {
    if constexpr (C::NBUF == 2) {
      if (kt + 1 < nt) dma_rows(kt + 1, kn, vn);
    }
    if (kt + 2 < nt) load_entries(kt + 2, stg);
    if (NS == 1 || kt < nt) compute(kt, kc, vc, std::false_type{});
    if (kt + 1 < nt) tcur = info_ring[(kt + 1) % PF_ER];
    if constexpr (C::NBUF == 1) {
      __syncthreads();
      if (kt + 1 < nt) dma_rows(kt + 1, kn, vn);
    }
    wait_vmem();
    if (kt + 2 < nt) store_entries(kt + 2, stg);
    __syncthreads();
  };

  // tiles 0 and 1 staged with one round trip: both loads (issued without
  // waiting for the list's length) before either store
  {
    Staged st1 = {PF_NONE, 0, {0, 0, 0, 0}};
    load_entries(0, stg);
    load_entries(1, st1);
    if (NS == 1 || nt > 0) store_entries(0, stg);
    if (nt > 1) store_entries(1, st1);
  }
  if (!CL_HERE && !cl_late) copy_cl();
  __syncthreads();
  if (NS == 1 || nt > 0) dma_rows(0, kbuf0, vbuf0);
  if (cl_late) {
    mark_cl();
    copy_cl();
  }

  wait_vmem();
  __syncthreads();
  // The other groups start from the running maximum that the first group (and
  // a launch of one group) takes from the list's first tile: probabilities are
  // rounded to bf16 relative to the running maximum, and with one of its own
  // each group rounded them otherwise than a launch of one group (outputs
  // 1.2e-3 apart, as far as either is from 64 bits; 1e-5 so).  It costs them
  // that tile's scores (d = 80: 777 tokens 16.2 -> 16.5 us, 300 tokens 9.3 ->
  // 9.6; d = 64: 777 tokens 15.2 either way).  The first group's tile stays
  // until the barrier that ends the first step.
  if constexpr (NS > 1) {
    if (grp > 0 && nt > 0) {
      tcur = info_rings[0][0];
      compute(0, tiles, nullptr, std::true_type{});
    }
  }
  tcur = info_ring[0];

  // every group takes as many steps as the first, which has the most tiles
  // (the barriers are the workgroup's)
  const int steps = NS == 1 ? nt : (nt_all + NS - 1) / NS;
  for (int kt = 0; kt < steps; kt += 2) {
    if constexpr (C::NBUF == 2) {
      iteration(kt, kbuf0, vbuf0, kbuf1, vbuf1);
      if (kt + 1 < steps) iteration(kt + 1, kbuf1, vbuf1, kbuf0, vbuf0);
    } else {
      iteration(kt, kbuf0, vbuf0, kbuf0, vbuf0);
      if (kt + 1 < nt) iteration(kt + 1, kbuf0, vbuf0, kbuf0, vbuf0);
    }
  }

  // ---- the groups' outputs to the first group: a wave's accumulators go
  // through LDS (the tile buffers are free) register by register ----
  if constexpr (NS > 1) {
    constexpr int NR = 16 * NDB + 2;  // accumulators, running maximum, sum
    static_assert((NS - 1) * PF_WAVES * NR * 256 <= (int)sizeof(tiles), "room for the partials");
    auto slot = [&](int gi) {
      return reinterpret_cast<float*>(tiles) + ((gi - 1) * PF_WAVES + wave) * NR * 64 + lane;
    };
    const float m_run = m_next == -INFINITY ? -INFINITY : -m_neg;
    if (grp > 0) {
      float* w = slot(grp);
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) w[(db * 16 + i) * 64] = oacc[db][i];
      w[16 * NDB * 64] = m_run;
      w[(16 * NDB + 1) * 64] = lacc[0];
    }
    __syncthreads();
    if (grp > 0) return;
    float mg[NS], mx = m_run;
#pragma unroll
    for (int gi = 1; gi < NS; ++gi) {
      mg[gi] = slot(gi)[16 * NDB * 64];
      mx = fmaxf(mx, mg[gi]);
    }
    // a group without a visible tile for the row has weight 0 (and zeros)
    const float f0 = fast_exp2(m_run - mx);
    lacc[0] *= f0;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[db][i] *= f0;
#pragma unroll
    for (int gi = 1; gi < NS; ++gi) {
      const float f = fast_exp2(mg[gi] - mx);
      const float* w = slot(gi);
      lacc[0] = fmaf(w[(16 * NDB + 1) * 64], f, lacc[0]);
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = fmaf(w[(db * 16 + i) * 64], f, oacc[db][i]);
    }
  }

  // ---- epilogue: normalise and write (<CL> rows were written at the start) ----
  if (!wave_live) return;
  float l_tot;
  if constexpr (ONES_SUM) {
    // O^T row D sits in d-block D/32, accumulator 8*((D%32)/8) of lane group 0
    static_assert((D % 32) % 8 == 0, "ones row must start a group of 8 rows");
    l_tot = __shfl(oacc[D / 32][4 * ((D % 32) / 8)], l32, 64);
  } else if constexpr (MFMA_SUM) {
    l_tot = lacc[0];
  } else {
    l_tot = l_run + __shfl_xor(l_run, 32, 64);
  }
  if (qrow >= L || is_cl) return;
  const float inv = 1.f / l_tot;
  // The output row's address is recomputed here from an opaque copy of the
  // lane index rather than kept from the start of the kernel: holding it
  // (and the lane's column offset) across the tile loop costs registers the
  // loop needs.
  int lane_e = threadIdx.x & 63;
  asm volatile("" : "+v"(lane_e));
  T* const orow_e = o + (int64_t)bh * os + (int64_t)(Iw_loc + (lane_e & 31)) * D + 4 * (lane_e >> 5);
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int d0 = db * 32 + 8 * jj;
      if (d0 >= D) continue;  // D and d0 are multiples of 8
      if constexpr (BF) {
        u32x2 w;
        w[0] = pack_bf16x2(oacc[db][4 * jj] * inv, oacc[db][4 * jj + 1] * inv);
        w[1] = pack_bf16x2(oacc[db][4 * jj + 2] * inv, oacc[db][4 * jj + 3] * inv);
        *reinterpret_cast<u32x2*>(orow_e + d0) = w;
      } else {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = __float_as_uint(oacc[db][4 * jj + i] * inv);
        st16(orow_e + d0, w);
      }
    }
}

// bf16 runs at four waves per SIMD at D = 64 (at most 128 registers; 36.9 KB
// of LDS per workgroup, so four workgroups share a CU) and at three at D = 80
// (at most 168 registers; 49 KB of LDS), each measured faster than one wave
// fewer; the fp32 variant (small parity cases) is not capped.
template <int D, bool CACHED, int NS>
__global__ __launch_bounds__(PF_THREADS * NS) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 3))) void prefill_attn_kernel_bf16(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    uint16_t* __restrict__ o, int32_t H, int32_t L, int64_t qs, int64_t kvs, int64_t os, float c2,
    const int32_t* __restrict__ vu, int32_t L_meta, const uint32_t* __restrict__ list,
    const int32_t* __restrict__ count, const TileSum* __restrict__ info, int32_t n_qt,
    int32_t L_pad, int32_t n_work, PfCached cc) {
  prefill_attn_body<uint16_t, D, CACHED, NS>(q, k, v, o, H, L, qs, kvs, os, c2, vu, L_meta, list,
                                         count, info, n_qt, L_pad, n_work, cc);
}

template <int D, bool CACHED>
__global__ __launch_bounds__(PF_THREADS) void prefill_attn_kernel_f32(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ o, int32_t H, int32_t L, int64_t qs, int64_t kvs, int64_t os, float c2,
    const int32_t* __restrict__ vu, int32_t L_meta, const uint32_t* __restrict__ list,
    const int32_t* __restrict__ count, const TileSum* __restrict__ info, int32_t n_qt,
    int32_t L_pad, int32_t n_work, PfCached cc) {
  prefill_attn_body<float, D, CACHED>(q, k, v, o, H, L, qs, kvs, os, c2, vu, L_meta, list, count,
                                      info, n_qt, L_pad, n_work, cc);
}

// ---------------------------------------------------------------------------
// fp32, few workgroups: the keys split over the waves
// ---------------------------------------------------------------------------
// The fp32 matrix instruction takes 64 clocks for 2 of the head's elements, so
// a wave is bound by its own products (128 of them a 64-key tile) and a short
// prompt's few workgroups by a few CUs.  Here a workgroup has 32 query rows
// instead of 128, and its four waves take 32 keys each of a 128-key tile; the
// waves' partial outputs are merged through LDS.  It stages every tile four
// times as often for the same rows, so it is for launches that leave CUs idle
// (4 heads of 256 tokens, d = 64: 29.5 us with 128 rows a workgroup, 16.0 us so).
// A CU holds two such workgroups at d = 64, one at d = 80 (73 and 98 KB of LDS).
// The line is at one round of them, further for long prompts or caches, whose
// light blocks leave room, and nearer for short blocks over few keys; it is drawn
// where neither nothing freed nor 60% is slower.  us with 128 rows a workgroup and
// so, nothing freed and 60%:
//   d = 64: 128 heads of 128 tokens (512 workgroups) 18.9 / 19.5 and 18.2 / 19.1,
//     64 of 256 28.9 / 29.5 and 20.6 / 21.2; of 65 tokens 96 (288) 16.2 / 16.6 and
//     13.7 / 14.8, 128 (384) 16.3 / 16.8 and 17.1 / 18.1; 192 blocks of 64 over 320
//     rows (384) 33.3 / 22.4 and 30.6 / 24.6; beyond one round 16 of 1500 (752) 126 /
//     63.1 and 74.0 / 55.8, 16 of 2048 (1024) 169 / 85.1 and 121 / 79.0, but 32 of 700
//     (704) 60.9 / 39.8 and 44.9 / 41.3, 32 of 1000 (1024) 88.1 / 49.6 and 74.7 / 54.1
//   d = 80: 64 heads of 128 tokens (256 workgroups) 22.7 / 23.3 and 14.6 / 15.9; 32 of
//     512 (512) 61.2 / 43.2 and 42.5 / 39.2, but 48 of 300 (480) 38.7 / 30.4 and 36.9 /
//     34.1; 64 blocks of 256 over 512 rows (512) 62.1 / 43.4 and 51.8 / 43.5, but 192 of
//     64 over 320 (384) 43.7 / 28.5 and 47.8 / 38.9; 16 of 1200 (608) 127 / 68.8 and
//     93.6 / 64.8, 8 of 3000 (752) 309 / 139 and 229 / 122, but 16 of 1500 (752) 163 /
//     80.0 and 129 / 82.6
// With one tile of keys there is nothing to split (8 heads of 40 tokens, d = 80:
// 12.2 and 14.8).
static bool prefill_f32_split(int d, int n_split, int rows, int keys, bool cached) {
  if (keys <= PF_BK) return false;
  if (d == 64) {
    if (rows < PF_BQ && keys < 512) return n_split <= 320;
    return n_split <= (cached || keys < 1200 ? 512 : keys < 2048 ? 768 : 1024);
  }
  if (keys < (cached ? 512 : 400)) return n_split <= 256;
  return n_split <= (cached || keys < 1200 ? 512 : keys < 2048 ? 640 : 768);
}
template <int D, bool CACHED>
__device__ __forceinline__ void prefill_f32_split_body(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ o, int32_t H, int32_t L, int64_t qs, int64_t kvs, int64_t os, float c2,
    const int32_t* __restrict__ vu, int32_t L_meta, const uint32_t* __restrict__ list,
    const int32_t* __restrict__ count, int32_t n_pq, int32_t L_pad, int32_t n_work, PfCached cc) {
  using C = PfCfg<float, D>;
  using TL = PfTile<float, D>;
  constexpr int NDB = C::DP / 32, KS = C::KSTEPS, BK = 2 * PF_BK;
  __shared__ __align__(1024) char kbuf[2 * TL::KBYTES];
  __shared__ __align__(1024) char vbuf[2 * TL::VBYTES];
  __shared__ int32_t rows[BK], toks[BK], lens[BK];

  int bh, qt;
  const int n_qt = (L + 31) / 32;
  work_item(blockIdx.x, n_work / n_qt, n_qt, &bh, &qt);
  const int s = bh / H;
  const int tok0 = CACHED ? cc.tok0 : 0;
  const int64_t pblk = (int64_t)s * n_pq + qt / PF_WAVES;  // the plan's block
  const int I = tok0 + qt / PF_WAVES * PF_BQ;              // its first token
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int l32 = lane & 31;
  const int g = lane >> 5;
  const int Iw = tok0 + qt * 32;
  const int qrow = qt * 32 + l32;  // local query row
  const int qtok = Iw + l32;       // its token

  const float* qb = q + (int64_t)bh * qs;
  const float* kb = k + (int64_t)bh * kvs;
  const float* vb = v + (int64_t)bh * kvs;
  float* const orow = o + (int64_t)bh * os + (int64_t)qrow * D;
  const uint32_t* ents = list + pblk * L_pad;
  const uint32_t* rws = CACHED ? cc.rows + pblk * L_pad : nullptr;
  int own_row0 = 0;
  if constexpr (CACHED) {
    own_row0 = cc.row0[s];
    if (own_row0 < 0 || (int64_t)own_row0 + L > cc.L_cap) {
      // the block's rows are not in the cache: NaN outputs, nothing read
      if (cc.status && tid == 0 && qt == 0 && (bh % H) == 0) atomicOr(cc.status, SCKV_STATUS_CAP);
      if (wave == 0 && qrow < L)
        for (int e = g; e < D; e += 2) orow[e] = NAN;
      return;
    }
  }
  const int n_vis = min(max(count[pblk], 0), L_pad);  // clamped, as in prefill_attn_body

  // the padding value columns are zero once and for all
  if constexpr (C::DP != D) {
    float* vs = reinterpret_cast<float*>(vbuf);
    for (int i = tid; i < BK * (C::DP - D); i += 256)
      vs[(i / (C::DP - D)) * C::VP + D + i % (C::DP - D)] = 0.f;
  }
  float qreg[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) qreg[kk] = qrow < L ? qb[(int64_t)qrow * D + 2 * kk + g] : 0.f;

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  const int slice_bytes = (CACHED ? cc.L_cap : L) * D * 4;  // the slice's rows, as in prefill_attn_body
  const __amdgpu_buffer_rsrc_t krs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(kb), 0, slice_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(vb), 0, slice_bytes, 0x00020000);
  // entry `tid` of the tile that starts at list entry e0 (threads below BK)
  uint32_t e = PF_NONE;
  int r = 0;
  auto load_entry = [&](int e0) {
    const int at = min(e0 + tid, n_vis - 1);  // past the end the last entry again
    if (tid < BK && at >= 0) {
      e = ents[at];
      r = CACHED ? (int)rws[at] : (int)(e & 0x00ffffffu);
    }
  };
  load_entry(0);
  for (int e0 = 0; e0 < n_vis; e0 += BK) {
    if (tid < BK) {
      const bool in = e0 + tid < n_vis;
      const int t = (int)(e & 0x00ffffffu);
      rows[tid] = r;  // a padding row repeats the last row; its score is masked
      toks[tid] = in ? t : (int)PF_NONE;
      lens[tid] = in ? max(I + (int)(e >> 24) - t, 0) : 0;
    }
    __syncthreads();
    for (int blk = wave; blk < 2 * TL::KSLOT; blk += 4) {
      const int sl = blk * 64 + lane;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(krs, (lds_ptr_t)(kbuf + blk * 1024), 16,
                                               rows[sl / TL::KSLOT] * (D * 4) + sl % TL::KSLOT * 16,
                                               0, 0, 0);
    }
    for (int blk = wave; blk < 2 * TL::VSLOT; blk += 4) {
      const int sl = blk * 64 + lane;
      if (sl % TL::VSLOT < TL::PPR)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vrs, (lds_ptr_t)(vbuf + blk * 1024), 16,
                                                 rows[sl / TL::VSLOT] * (D * 4) + sl % TL::VSLOT * 16,
                                                 0, 0, 0);
    }
    load_entry(e0 + BK);
    wait_vmem();
    __syncthreads();
    // the list is in token order: a wave whose first key is later than the
    // workgroup's last row has nothing to do
    const int key0 = 32 * wave;
    if (toks[key0] <= Iw + 31) {
      f32x16 sacc;
#pragma unroll
      for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
      const float* krow = reinterpret_cast<const float*>(kbuf) + (key0 + l32) * C::KP + g;
#pragma unroll
      for (int kk = 0; kk < KS; ++kk)
        sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(krow[2 * kk], qreg[kk], sacc, 0, 0, 0);
      float mx = -INFINITY;
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) {
        const int key = key0 + 8 * (vv >> 2) + 4 * g + (vv & 3);
        const bool vis = (uint32_t)(qtok - toks[key]) <= (uint32_t)lens[key];
        sacc[vv] = vis ? sacc[vv] : -INFINITY;
        mx = fmaxf(mx, sacc[vv]);
      }
      mx = max_across_halves(mx) * c2;
      const bool grow = mx > m_run + PF_RESCALE;
      if (__ballot(grow) != 0) {
        // whole maxima: rescaling, here and in the merge, is by powers of two
        // and adds no rounding to that of one wave's sums
        const float m_new = ceilf(mx);
        const float alpha = grow ? fast_exp2(m_run - m_new) : 1.f;  // m_run == -inf gives 0
        if (grow) m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
      }
      const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
#pragma unroll
      for (int vv = 0; vv < 16; ++vv) {
        sacc[vv] = fast_exp2(fmaf(sacc[vv], c2, -m_use));
        l_run += sacc[vv];
      }
      const float* vs = reinterpret_cast<const float*>(vbuf);
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int vv = 0; vv < 16; ++vv) {
          const int key = key0 + 8 * (vv >> 2) + 4 * g + (vv & 3);
          oacc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vs[key * C::VP + db * 32 + l32], sacc[vv],
                                                          oacc[db], 0, 0, 0);
        }
    }
    __syncthreads();
  }

  // merge: the waves' accumulators, maxima and sums to wave 0, register by register
  l_run += __shfl_xor(l_run, 32, 64);
  constexpr int NR = 16 * NDB + 2;
  static_assert(3 * NR * 256 <= (int)sizeof(kbuf), "room for the partials");
  float* const part = reinterpret_cast<float*>(kbuf) + lane;
  if (wave > 0) {
    float* w = part + (wave - 1) * NR * 64;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) w[(db * 16 + i) * 64] = oacc[db][i];
    w[16 * NDB * 64] = m_run;
    w[(16 * NDB + 1) * 64] = l_run;
  }
  __syncthreads();
  if (wave > 0 || qrow >= L) return;
  if (vu[(int64_t)s * L_meta + qtok] == qtok) {  // a <CL> row's output is its own value row
    const float* vrow = vb + (int64_t)(own_row0 + qrow) * D;
    for (int d0 = 4 * g; d0 < D; d0 += 8) st16(orow + d0, ld16(vrow + d0));
    return;
  }
  float m_all = m_run;
#pragma unroll
  for (int w = 0; w < 3; ++w) m_all = fmaxf(m_all, part[(w * NR + 16 * NDB) * 64]);
  // a wave without a visible key for the row has weight 0 (and zeros)
  float f = fast_exp2(m_run - m_all);
  l_run *= f;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) oacc[db][i] *= f;
#pragma unroll
  for (int w = 0; w < 3; ++w) {
    const float* x = part + w * NR * 64;
    f = fast_exp2(x[16 * NDB * 64] - m_all);
    l_run = fmaf(x[(16 * NDB + 1) * 64], f, l_run);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) oacc[db][i] = fmaf(x[(db * 16 + i) * 64], f, oacc[db][i]);
  }
  const float inv = 1.f / l_run;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int d0 = db * 32 + 8 * jj;
      if (d0 >= D) continue;
      u32x4 w;
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = __float_as_uint(oacc[db][4 * jj + i] * inv);
      st16(orow + d0 + 4 * g, w);
    }
}

template <int D, bool CACHED>
__global__ __launch_bounds__(256) void prefill_f32_split_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ o, int32_t H, int32_t L, int64_t qs, int64_t kvs, int64_t os, float c2,
    const int32_t* __restrict__ vu, int32_t L_meta, const uint32_t* __restrict__ list,
    const int32_t* __restrict__ count, int32_t n_pq, int32_t L_pad, int32_t n_work, PfCached cc) {
  prefill_f32_split_body<D, CACHED>(q, k, v, o, H, L, qs, kvs, os, c2, vu, L_meta, list, count,
                                    n_pq, L_pad, n_work, cc);
}

template <typename T, int D, bool CACHED>
static int launch_prefill(const void* q, const void* k, const void* v, void* o, int32_t b,
                          int32_t H, int32_t L, int64_t qs, int64_t kvs, int64_t os, float scale,
                          const int32_t* vu, int32_t L_meta, uint32_t* list, int32_t* count,
                          TileSum* info, int32_t n_qt, int32_t L_pad, PfCached cc, bool plan,
                          hipStream_t stream) {
  if (plan) {
    prefill_plan_kernel<CACHED><<<dim3(n_qt, b), 256, 0, stream>>>(vu, L_meta, L, n_qt, L_pad,
                                                                   list, count, info, cc);
    int rc = hip_check(hipGetLastError(), "span_masked_prefill_attn: plan launch");
    if (rc) return rc;
  }
  const int n_work = b * H * n_qt;
  if constexpr (sizeof(T) == 2) {
    const int groups = prefill_groups(D, n_work, CACHED ? cc.L_cap : L, b * H, CACHED);
    auto kernel = prefill_attn_kernel_bf16<D, CACHED, 1>;
    if constexpr (D == 64) {
      if (groups == 2) kernel = prefill_attn_kernel_bf16<D, CACHED, 2>;
      if (groups == 4) kernel = prefill_attn_kernel_bf16<D, CACHED, 4>;
    } else {
      if (groups == 3) kernel = prefill_attn_kernel_bf16<D, CACHED, 3>;
    }
    kernel<<<n_work, PF_THREADS * groups, 0, stream>>>(
        static_cast<const T*>(q), static_cast<const T*>(k), static_cast<const T*>(v),
        static_cast<T*>(o), H, L, qs, kvs, os, scale * PF_LOG2E, vu, L_meta, list, count, info,
        n_qt, L_pad, n_work, cc);
  } else {
    const int64_t n_split = (int64_t)b * H * ((L + 31) / 32);  // at most four times n_work
    if (n_work <= PF_ONE_PER_CU &&
        prefill_f32_split(D, (int)n_split, L, CACHED ? cc.L_cap : L, CACHED))
      prefill_f32_split_kernel<D, CACHED><<<(int)n_split, 256, 0, stream>>>(
          static_cast<const T*>(q), static_cast<const T*>(k), static_cast<const T*>(v),
          static_cast<T*>(o), H, L, qs, kvs, os, scale * PF_LOG2E, vu, L_meta, list, count, n_qt,
          L_pad, (int)n_split, cc);
    else
      prefill_attn_kernel_f32<D, CACHED><<<n_work, PF_THREADS, 0, stream>>>(
          static_cast<const T*>(q), static_cast<const T*>(k), static_cast<const T*>(v),
          static_cast<T*>(o), H, L, qs, kvs, os, scale * PF_LOG2E, vu, L_meta, list, count, info,
          n_qt, L_pad, n_work, cc);
  }
  return hip_check(hipGetLastError(), "span_masked_prefill_attn: launch");
}

template <bool CACHED>
static int dispatch_prefill(const void* q, const void* k, const void* v, void* o, int32_t b,
                            int32_t H, int32_t L, int32_t d_head, sckv_dtype dt, int64_t qs,
                            int64_t kvs, int64_t os, float scale, const int32_t* vu,
                            int32_t L_meta, uint32_t* list, int32_t* cnt, TileSum* info,
                            int32_t n_qt, int32_t L_pad, PfCached cc, bool plan,
                            hipStream_t stream) {
  if (dt == SCKV_BF16)
    return d_head == 64 ? launch_prefill<uint16_t, 64, CACHED>(q, k, v, o, b, H, L, qs, kvs, os, scale, vu, L_meta, list, cnt, info, n_qt, L_pad, cc, plan, stream)
                        : launch_prefill<uint16_t, 80, CACHED>(q, k, v, o, b, H, L, qs, kvs, os, scale, vu, L_meta, list, cnt, info, n_qt, L_pad, cc, plan, stream);
  return d_head == 64 ? launch_prefill<float, 64, CACHED>(q, k, v, o, b, H, L, qs, kvs, os, scale, vu, L_meta, list, cnt, info, n_qt, L_pad, cc, plan, stream)
                      : launch_prefill<float, 80, CACHED>(q, k, v, o, b, H, L, qs, kvs, os, scale, vu, L_meta, list, cnt, info, n_qt, L_pad, cc, plan, stream);
}

static void plan_geometry(int32_t L, int32_t* n_qt, int32_t* L_pad) {
  *n_qt = (L + PF_BQ - 1) / PF_BQ;
  *L_pad = *n_qt * PF_BQ;
}

// cached: a query block lists at most row0 + nq <= L_cap rows
static void plan_geometry_cached(int32_t nq, int32_t L_cap, int32_t* n_qt, int32_t* L_pad) {
  *n_qt = (nq + PF_BQ - 1) / PF_BQ;
  *L_pad = (L_cap + PF_BQ - 1) / PF_BQ * PF_BQ;
}

}  // namespace sckv

using namespace sckv;

extern "C" size_t sckv_prefill_workspace_bytes(int32_t b, int32_t L) {
  if (b <= 0 || L <= 0) return 0;
  int32_t n_qt, L_pad;
  plan_geometry(L, &n_qt, &L_pad);
  const size_t list = (size_t)b * n_qt * L_pad * sizeof(uint32_t);
  const size_t sums = (size_t)b * n_qt * (L_pad / 64) * sizeof(TileSum);
  const size_t cnt = ((size_t)b * n_qt * sizeof(int32_t) + 255) / 256 * 256;
  return list + sums + cnt;
}

// workspace of the plain prefill: list entries | tile summaries | counts
struct PlainPlan {
  uint32_t* list;
  TileSum* sums;
  int32_t* cnt;
  int32_t n_qt, L_pad;
};
static PlainPlan plain_plan(void* ws, int32_t b, int32_t L) {
  PlainPlan p;
  plan_geometry(L, &p.n_qt, &p.L_pad);
  const size_t list_bytes = (size_t)b * p.n_qt * p.L_pad * sizeof(uint32_t);
  const size_t sum_bytes = (size_t)b * p.n_qt * (p.L_pad / 64) * sizeof(TileSum);
  p.list = static_cast<uint32_t*>(ws);
  p.sums = reinterpret_cast<TileSum*>(static_cast<char*>(ws) + list_bytes);
  p.cnt = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + list_bytes + sum_bytes);
  return p;
}

// checks shared by the plan-only call and the attention calls
static int check_plan_args(const char* W, const int32_t* vu, int32_t b, int32_t L, int32_t L_meta,
                           const void* ws, size_t ws_bytes) {
  if (!vu || !ws) return fail(SCKV_EINVAL, std::string(W) + ": null pointer");
  if (b <= 0 || L <= 0) return fail(SCKV_EINVAL, std::string(W) + ": sizes must be positive");
  if (L > 32768) return fail(SCKV_EUNSUP, std::string(W) + ": L above 32768");
  if (L_meta < L) return fail(SCKV_EINVAL, std::string(W) + ": L_meta < L");
  if (!aligned16(ws)) return fail(SCKV_EINVAL, std::string(W) + ": workspace must be 16-byte aligned");
  if (ws_bytes < sckv_prefill_workspace_bytes(b, L))
    return fail(SCKV_EINVAL, std::string(W) + ": workspace too small");
  return SCKV_OK;
}

static int prefill_entry(const char* W, bool plan, const void* q, const void* k, const void* v,
                         void* o, int32_t b, int32_t H, int32_t L, int32_t d_head,
                         int64_t q_stride_bh, int64_t kv_stride_bh, int64_t o_stride_bh,
                         sckv_dtype dt, float scale, const int32_t* vu, int32_t L_meta, void* ws,
                         size_t ws_bytes, hipStream_t stream) {
  clear_error();
  if (!q || !k || !v || !o) return fail(SCKV_EINVAL, std::string(W) + ": null pointer");
  int rc = check_plan_args(W, vu, b, L, L_meta, ws, ws_bytes);
  if (rc) return rc;
  if (!valid_dtype(dt)) return fail(SCKV_EINVAL, std::string(W) + ": unknown dtype");
  if (!supported_d(d_head)) return fail(SCKV_EUNSUP, std::string(W) + ": d_head must be 64 or 80");
  if (H <= 0) return fail(SCKV_EINVAL, std::string(W) + ": sizes must be positive");
  const int64_t rowlen = (int64_t)L * d_head;
  if (q_stride_bh < rowlen || kv_stride_bh < rowlen || o_stride_bh < rowlen)
    return fail(SCKV_EINVAL, std::string(W) + ": slice stride smaller than L*d_head");
  const int eb = elem_bytes(dt);
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) ||
      (q_stride_bh * eb) % 16 || (kv_stride_bh * eb) % 16 || (o_stride_bh * eb) % 16)
    return fail(SCKV_EINVAL, std::string(W) + ": buffers and strides must be 16-byte aligned");
  if (!(scale > 0.f) || std::isinf(scale)) return fail(SCKV_EINVAL, std::string(W) + ": scale must be finite and > 0");
  const PlainPlan p = plain_plan(ws, b, L);
  if ((int64_t)b * H * p.n_qt > 0x7fffffff) return fail(SCKV_EUNSUP, std::string(W) + ": grid too large");
  return dispatch_prefill<false>(q, k, v, o, b, H, L, d_head, dt, q_stride_bh, kv_stride_bh,
                                 o_stride_bh, scale, vu, L_meta, p.list, p.cnt, p.sums, p.n_qt,
                                 p.L_pad, PfCached{}, plan, stream);
}

extern "C" int span_masked_prefill_attn(const void* q, const void* k, const void* v, void* o,
                                        int32_t b, int32_t H, int32_t L, int32_t d_head,
                                        int64_t q_stride_bh, int64_t kv_stride_bh,
                                        int64_t o_stride_bh, sckv_dtype dt, float scale,
                                        const int32_t* vu, int32_t L_meta, void* ws,
                                        size_t ws_bytes, hipStream_t stream) {
  return prefill_entry("span_masked_prefill_attn", true, q, k, v, o, b, H, L, d_head, q_stride_bh,
                       kv_stride_bh, o_stride_bh, dt, scale, vu, L_meta, ws, ws_bytes, stream);
}

extern "C" int sckv_prefill_plan(const int32_t* vu, int32_t L_meta, int32_t b, int32_t L,
                                 void* ws, size_t ws_bytes, hipStream_t stream) {
  clear_error();
  const char* W = "sckv_prefill_plan";
  int rc = check_plan_args(W, vu, b, L, L_meta, ws, ws_bytes);
  if (rc) return rc;
  const PlainPlan p = plain_plan(ws, b, L);
  prefill_plan_kernel<false><<<dim3(p.n_qt, b), 256, 0, stream>>>(vu, L_meta, L, p.n_qt, p.L_pad,
                                                                  p.list, p.cnt, p.sums,
                                                                  PfCached{});
  return hip_check(hipGetLastError(), "sckv_prefill_plan: launch");
}

extern "C" int span_masked_prefill_attn_planned(const void* q, const void* k, const void* v,
                                                void* o, int32_t b, int32_t H, int32_t L,
                                                int32_t d_head, int64_t q_stride_bh,
                                                int64_t kv_stride_bh, int64_t o_stride_bh,
                                                sckv_dtype dt, float scale, const int32_t* vu,
                                                int32_t L_meta, void* ws, size_t ws_bytes,
                                                hipStream_t stream) {
  return prefill_entry("span_masked_prefill_attn_planned", false, q, k, v, o, b, H, L, d_head,
                       q_stride_bh, kv_stride_bh, o_stride_bh, dt, scale, vu, L_meta, ws,
                       ws_bytes, stream);
}

extern "C" size_t sckv_prefill_cached_workspace_bytes(int32_t b, int32_t nq, int32_t L_cap) {
  if (b <= 0 || nq <= 0 || L_cap <= 0) return 0;
  int32_t n_qt, L_pad;
  plan_geometry_cached(nq, L_cap, &n_qt, &L_pad);
  const size_t list = (size_t)b * n_qt * L_pad * sizeof(uint32_t);  // entries, then rows
  const size_t sums = (size_t)b * n_qt * (L_pad / 64) * sizeof(TileSum);
  const size_t cnt = ((size_t)b * n_qt * sizeof(int32_t) + 255) / 256 * 256;
  return 2 * list + sums + cnt;
}

// workspace of the cached prefill: list entries | their cache rows | tile
// summaries | counts
struct CachedPlan {
  uint32_t* list;
  TileSum* sums;
  int32_t* cnt;
  PfCached cc;
  int32_t n_qt, L_pad;
};
static CachedPlan cached_plan(void* ws, int32_t b, int32_t nq, int32_t L_cap, int32_t tok0,
                              const int32_t* row0, const int32_t* tok_idx, int32_t* status) {
  CachedPlan p;
  plan_geometry_cached(nq, L_cap, &p.n_qt, &p.L_pad);
  const size_t list_bytes = (size_t)b * p.n_qt * p.L_pad * sizeof(uint32_t);
  const size_t sum_bytes = (size_t)b * p.n_qt * (p.L_pad / 64) * sizeof(TileSum);
  char* base = static_cast<char*>(ws);
  p.list = reinterpret_cast<uint32_t*>(base);
  p.cc.rows = reinterpret_cast<uint32_t*>(base + list_bytes);
  p.sums = reinterpret_cast<TileSum*>(base + 2 * list_bytes);
  p.cnt = reinterpret_cast<int32_t*>(base + 2 * list_bytes + sum_bytes);
  p.cc.row0 = row0;
  p.cc.tok = tok_idx;
  p.cc.tok0 = tok0;
  p.cc.L_cap = L_cap;
  p.cc.status = status;
  return p;
}

// checks shared by the cached plan-only call and the cached attention calls
static int check_cached_plan_args(const char* W, const int32_t* vu, int32_t L_meta, int32_t tok0,
                                  const int32_t* row0, const int32_t* tok_idx, int32_t L_cap,
                                  int32_t b, int32_t nq, const void* ws, size_t ws_bytes) {
  if (!vu || !row0 || !tok_idx || !ws) return fail(SCKV_EINVAL, std::string(W) + ": null pointer");
  if (b <= 0 || nq <= 0 || L_cap <= 0)
    return fail(SCKV_EINVAL, std::string(W) + ": sizes must be positive");
  if (L_cap > 32768 || nq > L_cap) return fail(SCKV_EUNSUP, std::string(W) + ": nq <= L_cap <= 32768 required");
  // list entries hold a token in 24 bits; 0xffffff marks padding
  if (L_meta <= 0 || L_meta >= (int32_t)PF_NONE)
    return fail(SCKV_EUNSUP, std::string(W) + ": L_meta must be in (0, 2^24 - 1)");
  if (tok0 < 0 || (int64_t)tok0 + nq > L_meta)
    return fail(SCKV_EINVAL, std::string(W) + ": query tokens [tok0, tok0+nq) exceed L_meta");
  if (!aligned16(ws)) return fail(SCKV_EINVAL, std::string(W) + ": workspace must be 16-byte aligned");
  if (ws_bytes < sckv_prefill_cached_workspace_bytes(b, nq, L_cap))
    return fail(SCKV_EINVAL, std::string(W) + ": workspace too small");
  return SCKV_OK;
}

static int cached_entry(const char* W, bool plan, const void* q, const void* k_cache,
                        const void* v_cache, void* o, int32_t b, int32_t H, int32_t nq,
                        int32_t d_head, int64_t q_stride_bh, int64_t kv_stride_bh,
                        int64_t o_stride_bh, sckv_dtype dt, float scale, const int32_t* vu,
                        int32_t L_meta, int32_t tok0, const int32_t* row0, const int32_t* tok_idx,
                        int32_t L_cap, void* ws, size_t ws_bytes, int32_t* status,
                        hipStream_t stream) {
  clear_error();
  if (!q || !k_cache || !v_cache || !o) return fail(SCKV_EINVAL, std::string(W) + ": null pointer");
  int rc = check_cached_plan_args(W, vu, L_meta, tok0, row0, tok_idx, L_cap, b, nq, ws, ws_bytes);
  if (rc) return rc;
  if (!valid_dtype(dt)) return fail(SCKV_EINVAL, std::string(W) + ": unknown dtype");
  if (!supported_d(d_head)) return fail(SCKV_EUNSUP, std::string(W) + ": d_head must be 64 or 80");
  if (H <= 0) return fail(SCKV_EINVAL, std::string(W) + ": sizes must be positive");
  if (q_stride_bh < (int64_t)nq * d_head || o_stride_bh < (int64_t)nq * d_head ||
      kv_stride_bh < (int64_t)L_cap * d_head)
    return fail(SCKV_EINVAL, std::string(W) + ": slice stride too small");
  const int eb = elem_bytes(dt);
  if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(o) ||
      (q_stride_bh * eb) % 16 || (kv_stride_bh * eb) % 16 || (o_stride_bh * eb) % 16)
    return fail(SCKV_EINVAL, std::string(W) + ": buffers and strides must be 16-byte aligned");
  if (!(scale > 0.f) || std::isinf(scale)) return fail(SCKV_EINVAL, std::string(W) + ": scale must be finite and > 0");
  const CachedPlan p = cached_plan(ws, b, nq, L_cap, tok0, row0, tok_idx, status);
  if ((int64_t)b * H * p.n_qt > 0x7fffffff) return fail(SCKV_EUNSUP, std::string(W) + ": grid too large");
  return dispatch_prefill<true>(q, k_cache, v_cache, o, b, H, nq, d_head, dt, q_stride_bh,
                                kv_stride_bh, o_stride_bh, scale, vu, L_meta, p.list, p.cnt,
                                p.sums, p.n_qt, p.L_pad, p.cc, plan, stream);
}

extern "C" int span_masked_prefill_attn_cached(
    const void* q, const void* k_cache, const void* v_cache, void* o, int32_t b, int32_t H,
    int32_t nq, int32_t d_head, int64_t q_stride_bh, int64_t kv_stride_bh, int64_t o_stride_bh,
    sckv_dtype dt, float scale, const int32_t* vu, int32_t L_meta, int32_t tok0,
    const int32_t* row0, const int32_t* tok_idx, int32_t L_cap, void* ws, size_t ws_bytes,
    int32_t* status, hipStream_t stream) {
  return cached_entry("span_masked_prefill_attn_cached", true, q, k_cache, v_cache, o, b, H, nq,
                      d_head, q_stride_bh, kv_stride_bh, o_stride_bh, dt, scale, vu, L_meta, tok0,
                      row0, tok_idx, L_cap, ws, ws_bytes, status, stream);
}

extern "C" int sckv_prefill_cached_plan(const int32_t* vu, int32_t L_meta, int32_t tok0,
                                        const int32_t* row0, const int32_t* tok_idx,
                                        int32_t L_cap, int32_t b, int32_t nq, void* ws,
                                        size_t ws_bytes, hipStream_t stream) {
  clear_error();
  const char* W = "sckv_prefill_cached_plan";
  int rc = check_cached_plan_args(W, vu, L_meta, tok0, row0, tok_idx, L_cap, b, nq, ws, ws_bytes);
  if (rc) return rc;
  const CachedPlan p = cached_plan(ws, b, nq, L_cap, tok0, row0, tok_idx, nullptr);
  prefill_plan_kernel<true><<<dim3(p.n_qt, b), 256, 0, stream>>>(vu, L_meta, nq, p.n_qt, p.L_pad,
                                                                 p.list, p.cnt, p.sums, p.cc);
  return hip_check(hipGetLastError(), "sckv_prefill_cached_plan: launch");
}

extern "C" int span_masked_prefill_attn_cached_planned(
    const void* q, const void* k_cache, const void* v_cache, void* o, int32_t b, int32_t H,
    int32_t nq, int32_t d_head, int64_t q_stride_bh, int64_t kv_stride_bh, int64_t o_stride_bh,
    sckv_dtype dt, float scale, const int32_t* vu, int32_t L_meta, int32_t tok0,
    const int32_t* row0, const int32_t* tok_idx, int32_t L_cap, void* ws, size_t ws_bytes,
    int32_t* status, hipStream_t stream) {
  return cached_entry("span_masked_prefill_attn_cached_planned", false, q, k_cache, v_cache, o, b,
                      H, nq, d_head, q_stride_bh, kv_stride_bh, o_stride_bh, dt, scale, vu,
                      L_meta, tok0, row0, tok_idx, L_cap, ws, ws_bytes, status, stream);
}
