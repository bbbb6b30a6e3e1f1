// Multi-token queries (prefill chunks) over the paged KV cache, for gfx950.
//
// Rollout runs prefill over the prompt tokens before it decodes them (Sec. 3,
// rollout); the prefill cost model (App. A.1.2) charges its attention with a term
// quadratic in the prompt length, so unlike decode this operation is a dense
// contraction and runs on the matrix cores.  Sequence b brings n_b query rows (its
// last n_b cached tokens, K/V already in the cache); row i attends causally to
// positions 0 .. seq_lens[b] - n_b + i.
//
// Work.  The query rows of one (sequence, KV head) are its n_b * G (token, query
// head) pairs, token-major, so every K/V row read serves all G heads sharing that
// KV head.  A workgroup takes 128 of them: each of its 4 waves owns one 32-row
// MFMA tile.  Workgroups are numbered heaviest first over the whole call (the row
// blocks that attend to the most keys are dispatched first), so the slots of the
// GPU fill longest-job-first.  Calls of few row blocks may take 32 rows to a workgroup
// instead, its waves sharing the keys (see use_split).
//
// Keys.  The workgroup walks its causal key range in blocks of 32 keys (two
// pages).  Each wave brings one page of K or V of every block (page ids come
// through the scalar cache one block before that): bf16 pages at d = 128 by
// buffer-load DMA straight into LDS, two blocks ahead; other caches through
// registers one block ahead (fp8 converted exactly to bf16 on the way).  Per block:
//   S^T[key][row] = K Q^T    v_mfma_f32_32x32x16_bf16, K from LDS, Q in registers;
//   online softmax per row (lanes l and l^32 hold one row), with the reference
//   maximum moved only when a score exceeds it by more than 2^8;
//   O^T[d][row] += V^T P^T   the score registers are the P^T operand as they are;
//                            V^T comes from the row-major V block through the
//                            LDS transpose read (ds_read_b64_tr_b16).
// The causal mask is evaluated only on blocks that reach a row's limit.  fp8 K
// scales multiply the scores and V scales multiply P, per page.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "rlda_device.h"
#include "rlda_params.h"

namespace rlda {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

#ifndef RLDA_MQ_KPAD
#define RLDA_MQ_KPAD 16                       // LDS row padding of the K block (bytes)
#endif
#ifndef RLDA_MQ_VPAD
#define RLDA_MQ_VPAD 32                       // ... of the V block
#endif
constexpr int kTile = 32;                     // rows (and keys) of one MFMA tile
constexpr int kNT = kMultiTiles;              // 32-row tiles per wave
constexpr int kKH = kMultiKeyTiles;           // 32-key score tiles per key block
constexpr int kKeys = kTile * kKH;            // keys per block (2 kKH pages)

#ifndef RLDA_MQ_WAVES_D64
#define RLDA_MQ_WAVES_D64 4                   // waves per SIMD at d = 64 (about 100 registers)
#endif
#ifndef RLDA_MQ_PREFETCH
#define RLDA_MQ_PREFETCH 1                    // blocks loaded ahead into registers (register staging)
#endif
#ifndef RLDA_MQ_DMA
#define RLDA_MQ_DMA 1                         // bf16, d = 128: pages go to LDS by buffer-load DMA
#endif

// Workgroup barrier for the DMA path: wait until at most N vector-memory
// operations of this wave are outstanding (the DMAs of the newest block) and its
// LDS operations are done, then s_barrier.  __syncthreads would wait for every
// outstanding DMA (its release fence counts them as stores).  The asm's memory
// clobber keeps the compiler from moving memory accesses across it.
template <int N>
__device__ __forceinline__ void dma_barrier() {
  static_assert(N >= 0 && N < 16, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
static_assert(kTile * kNT * kWaves == kMultiRows, "a workgroup's rows are its waves' tiles");

// SMALL: calls of few row blocks, which may take 32 rows to a workgroup and deal the keys
// to its waves (chosen on the device, see "How few row blocks are cut").
template <int D, bool FP8, bool SMALL>
struct MqShape {
  static constexpr int KS = D / 16;           // 32x32x16 k-steps of K Q^T
  static constexpr int DT = D / 32;           // 32-wide output tiles of O^T
  static constexpr int EB = FP8 ? 1 : 2;      // bytes per cached element
  // bf16 pages at d = 128 are copied to LDS by the buffer-load DMA (no registers,
  // no LDS writes by the waves) into unpadded rows whose 16-byte chunks are
  // permuted per row (see chunk_pos); other caches, and waves that split the keys, are
  // staged through registers (fp8 is converted on the way) into padded rows.
  static constexpr bool DMA = !FP8 && D == 128 && RLDA_MQ_DMA;
  static constexpr int NBUF = SMALL ? kWaves : DMA ? 3 : 2;    // LDS block buffers
  // Waves per SIMD (register budget 512 / waves).  With the V operands read after
  // the softmax, three fit (168 registers): the DMA path without staging registers,
  // the register path with one block of staging in flight.  At d = 64 the state is
  // about 100 registers, and four fit.
#ifdef RLDA_MQ_WAVES
  static constexpr int WAVES = SMALL ? 2 : RLDA_MQ_WAVES;
#else
  static constexpr int WAVES = SMALL ? 2 : kNT == 1 ? (D == 64 ? RLDA_MQ_WAVES_D64 : 3) : 1;
#endif
  static constexpr int krs(bool dma) { return dma ? 2 * D : 2 * D + RLDA_MQ_KPAD; }   // LDS row stride of the K block (bytes)
  static constexpr int vrs(bool dma) { return dma ? 2 * D : 2 * D + RLDA_MQ_VPAD; }   // ... of the V block
  static constexpr bool kPadded = SMALL || !DMA;   // register-staged blocks occur
  static constexpr int KRS = krs(!kPadded), VRS = vrs(!kPadded);
  static constexpr int CPR = D * EB / 16;     // 16-byte chunks per cached row
  static constexpr int LPL = kPage * CPR / 64; // 16-byte loads per lane to stage one page
};

// How few row blocks are cut.  128 rows to a workgroup leave most of the chip idle on
// calls of few rows, each workgroup walking its keys one block after another; with 32
// rows and the keys dealt to its waves there are four times the workgroups, each a
// quarter as long, for staging and merging the waves' states.  Two fit a CU.  us a call,
// 128 rows against 32 with the keys split, by 32-row items and longest sequence:
//   up to two a CU:   8 heads, 4 x 64 rows over 18.5k keys    416 / 215
//                     40/8 fp8, 8 x 64 rows over 5.5k         175 / 86
//                     12/2 bf16 d 128, 178 rows               12.6 / 11.1
//                     16/16 d 64, prompts of up to 137        10.3 / 9.3
//                     8/1 fp8, 38 keys                        8.8 / 9.5
//   up to four a CU:  12/2, 3 prompts of up to 1432           38.9 / 35.3
//                     8/1, 7 chunks of 512, up to 1800        49.1 / 46.6
//                     12/2, 26 chunks of 64, up to 265        15.2 / 18.5
//                     40/8, 12 prompts of up to 53            10.7 / 17.6
// (above four the grid is not built for it).
__device__ __forceinline__ bool use_split(int items32, int keys, int cus) {
  return keys >= (items32 <= 2 * cus ? 96 : 640);
}

// Max / sum of a value with the one 32 lanes away (the other half of a score
// row), both halves getting the result: v_permlane32_swap of x with itself leaves
// the lower halves of x in one result and the upper halves in the other.
__device__ __forceinline__ float pair_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ bf16x4 lds_tr_read(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(__attribute__((address_space(3))) char*)p);
}

template <int D, bool FP8, bool SMALL>
__global__ __attribute__((amdgpu_flat_work_group_size(kThreads, kThreads),
                          amdgpu_waves_per_eu(MqShape<D, FP8, SMALL>::WAVES, MqShape<D, FP8, SMALL>::WAVES)))
void multi_query_kernel(const Params p) {
  using S = MqShape<D, FP8, SMALL>;
  // Block buffers: block kb is computed from one while the next blocks are written to
  // the others; waves that split the keys have one each.
  __shared__ __align__(16) char s_k[S::NBUF][kKeys * S::KRS];
  __shared__ __align__(16) char s_v[S::NBUF][kKeys * S::VRS];
  __shared__ float s_scale[S::NBUF][4 * kKH];   // fp8: K scales of the block's pages, then V's
  __shared__ int32_t s_bad[S::NBUF][2 * kKH];   // page of the block not in the pool (contributes nothing)
  __shared__ int32_t s_scan[kWaves], s_emax[kWaves], s_sum32[kWaves];
  __shared__ int16_t s_qh[kMaxQHeads];
  // Batches above 64, per sequence: {L - n_b (position of query token 0), n_b} (n_b 0
  // when its offsets are inconsistent), and its ordering key.
  extern __shared__ int2 s_sq[];   // [batch], then s_key [batch]

  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int batch = p.batch, Hkv = p.num_kv_heads, G = p.group, Hq = p.num_q_heads;
  const int cap = p.max_pages * kPage;
  int32_t* s_key = (int32_t*)(s_sq + batch);

  // 1. Rows of every sequence and the number of row blocks (identical in every wave).
  //    Inconsistent offsets give a sequence no rows; they, and lengths out of range or
  //    shorter than the rows, raise the flag.  Lane l holds sequence l: up to 64
  //    sequences every wave reads for itself, without a barrier; above that they meet
  //    in LDS.  An item's search, below, costs every workgroup the same again, so the
  //    reductions go through DPP and the search takes three points a step: with LDS
  //    shuffles and a binary search over all lengths the call on one or two short
  //    sequences took 9.2 to 11.5 us, and 7.1 to 8.8 so; whole prompts (32 x 512 tokens,
  //    12/2 heads) 58.2 and 53.5 us; chunks of long sequences 1420 and 1390 us.
  int2 sq0 = make_int2(0, 0);   // the sequence of this lane: {L - n_b, n_b}
  int key0 = -1;                // its ordering key (below)
  int nitems = 0, emax = 0;     // row blocks; the most keys any sequence's rows see
  bool split = false;           // SMALL: 32 rows to a workgroup, its waves split the keys
  int rshift = kMultiRowsLog2;  // log2 of a row block's rows
  {
    int sum = 0, sum32 = 0, bad = 0, lmax = 0;   // 128-row blocks, 32-row blocks
    const bool many = batch > 64;
    for (int b = many ? tid : lane; b < batch; b += kThreads) {
      const int q0 = p.q_start[b], q1 = p.q_start[b + 1];
      const bool ok = q0 >= 0 && q1 >= q0 && q1 <= p.total_q;
      const int n = ok ? q1 - q0 : 0;   // n G < 2^24: q is addressed with 31-bit offsets
      int L = p.seq_lens[b];
      if (!ok || L < 0 || L > cap || n > L) bad = 1;
      L = min(max(L, 0), cap);
      sq0 = make_int2(L - n, n);
      if (many) s_sq[b] = sq0;
      sum += (n * G + kMultiRows - 1) / kMultiRows;
      if (SMALL) sum32 += (n * G + kTile - 1) / kTile;
      if (n > 0) lmax = max(lmax, L);
    }
    if (__builtin_amdgcn_ballot_w64(bad) != 0 && blockIdx.x == 0 && lane == 0) atomicOr(p.flags, kFlagBadLen);
    sum = __builtin_amdgcn_readlane(wave_scan(sum), 63);
    lmax = __builtin_amdgcn_readlane(wave_scan_max(lmax), 63);
    if (SMALL) sum32 = __builtin_amdgcn_readlane(wave_scan(sum32), 63);
    for (int e = tid; e < Hq; e += kThreads) s_qh[e] = p.q_head[e];
    // Ordering key of each sequence's row blocks.  A sequence whose rows see at most an
    // eighth of the largest job's keys apart is dispatched as a group (its row blocks
    // then read its pages together): its key count L; -1: each row block is ordered by
    // its own key count.
    auto key_of = [&](int2 sq) { return sq.y > 0 && 8 * (int64_t)sq.y <= emax ? max(0, sq.x + sq.y) : -1; };
    if (!many) {
      nitems = sum;
      emax = lmax;
      key0 = key_of(sq0);
      lds_barrier();   // s_qh
    } else {
      if (lane == 0) {
        s_scan[wave] = sum;
        s_emax[wave] = lmax;
        if (SMALL) s_sum32[wave] = sum32;
      }
      lds_barrier();
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        nitems += s_scan[w];
        emax = max(emax, s_emax[w]);
      }
      emax = uni(emax);
      if (SMALL) sum32 = s_sum32[0] + s_sum32[1] + s_sum32[2] + s_sum32[3];
      for (int b = tid; b < batch; b += kThreads) s_key[b] = key_of(s_sq[b]);
      lds_barrier();
      sq0 = s_sq[lane];
      key0 = s_key[lane];
    }
    if constexpr (SMALL) {
      split = use_split(sum32 * Hkv, emax, p.nranges);
      if (split) {
        rshift = 5;
        nitems = sum32;
      }
    }
  }
  auto blocks_of = [&](int rows) { return (rows + (1 << rshift) - 1) >> rshift; };
  const int64_t items = (int64_t)nitems * Hkv;
  if (blockIdx.x == 0 && tid == 0 && items > (int64_t)gridDim.x) atomicOr(p.flags, kFlagBadLen);

  // 2. The (sequence b, row block rb, KV head g) items of this workgroup.  Row block
  //    rb of sequence b covers rows [128 rb, r1), r1 = min(128 (rb + 1), n_b G), and
  //    reads the keys below E = max(0, L - n_b + (r1 - 1) / G + 1), its cost.
  //    Placement: workgroups are dispatched round-robin over the 8 XCDs (block u on
  //    XCD u % 8), and the row blocks of one (sequence, KV head) read the same pages,
  //    so they are kept on one XCD, whose L2 then serves the repeats:
  //      Hkv a multiple of 8: XCD x takes KV heads (x + b) % 8, + 8, ... of every
  //                           sequence b;
  //      Hkv = 4:             XCD x takes KV head (x + b) % 4 of the sequences b of
  //                           class x / 4, the two classes balanced by work (rank by
  //                           estimated keys, snake order; batches above 64: b mod 2),
  //                           the grid holding 8 blocks per (sequence, row block) so
  //                           that either class fits;
  //      otherwise:           one set over the whole grid, no placement.
  //    Within its set each XCD dispatches heaviest first (keys descending; ties by
  //    sequence, then last row block first, then KV head), so the slots of the XCD
  //    fill longest-job-first.  The row blocks of a sequence whose rows span at most
  //    an eighth of the largest job's keys all take the sequence's key count L: they
  //    run together and read the sequence's pages side by side, once from HBM; block t of the XCD takes item t of its set (blocks
  //    past the set's end return).  Item t is found by a search on the key count, three
  //    points a step: with C(x) the items having at least x keys (a closed form per
  //    sequence, summed across the wave), its key count x* is the largest x with C(x) > t.
  //    Every wave finds it (no barrier).
  const int u = blockIdx.x, xcd = u & 7;
  const bool by_head = Hkv % 8 == 0, by_class = Hkv == 4;
  const int ncls = by_class ? 8 / Hkv : 1, my_cls = by_class ? xcd / Hkv : 0;
  const int hx = by_head ? Hkv / 8 : (by_class ? 1 : Hkv);   // KV heads per (b, rb) in the set
  const int t_first = (by_head || by_class) ? u >> 3 : u;
  bool mine = true;   // batches of at most 64: this lane's sequence is in the set
  if (by_class && batch <= 64) {
    // Class of each sequence: its rank by estimated keys (descending, ties by sequence;
    // the keys compare as integers, being positive floats), the ranks dealt out in
    // snake order 0, 1, .., K-1, K-1, .., 0.
    const int nrb = blocks_of(sq0.y * G);
    const int key = __float_as_int((float)nrb * ((float)max(sq0.x, 0) + 0.5f * (float)sq0.y + 1.f));
    int rank = 0;
    for (int j = 0; j < batch; ++j) {
      const int kj = __builtin_amdgcn_readlane(key, j);
      rank += kj > key || (kj == key && j < lane);
    }
    const int rr = rank % (2 * ncls);
    mine = (rr < ncls ? rr : 2 * ncls - 1 - rr) == my_cls;
  }
  // Row blocks of sequence `sq` with at least x >= 1 keys (E is non-decreasing in rb).
  auto at_least = [&](int2 sq, int key, int x) -> int {
    const int nrb = blocks_of(sq.y * G);
    if (key >= 0) return key >= x ? nrb : 0;   // dispatched as a group
    if (x - 1 <= sq.x) return nrb;             // E >= x iff (r1 - 1) / G >= k
    const uint32_t k = (uint32_t)(x - 1) - (uint32_t)sq.x;
    return k < (uint32_t)sq.y ? nrb - (int)((uint32_t)G * k >> rshift) : 0;   // ... iff r1 > G k
  };
  // f({L - n, n}, key) of each of the set's sequences that this lane holds (the first 64
  // in registers), and a lane's count summed over the wave.
  auto in_set = [&](int b) { return b < batch && (by_class && batch > 64 ? b % ncls == my_cls : mine); };
  auto each = [&](auto f) {
    if (in_set(lane)) f(sq0, key0);
    for (int b = lane + 64; b < batch; b += 64)
      if (in_set(b)) f(s_sq[b], s_key[b]);
  };
  auto total = [&](int c) { return __builtin_amdgcn_readlane(wave_scan(c), 63); };
  int set_items = 0;
  each([&](int2 sq, int) { set_items += blocks_of(sq.y * G); });
  set_items = total(set_items) * hx;

  if (t_first >= set_items) return;
  const int v = t_first / hx, hsub = t_first - v * hx;
  int b = 0, rb = 0;
  {
    int lo = 0, hi = emax + 1, chi = 0;   // C(lo) > v >= C(hi) = chi
    while (hi - lo > 1) {
      // Three points strictly between where there is room (else some coincide).
      const int d = hi - lo, x2 = lo + (d >> 1), x1 = lo + max(d >> 2, 1), x3 = min(x2 + max(d >> 2, 1), hi - 1);
      int c1 = 0, c2 = 0, c3 = 0;
      each([&](int2 sq, int key) {
        c1 += at_least(sq, key, x1);
        c2 += at_least(sq, key, x2);
        c3 += at_least(sq, key, x3);
      });
      c1 = total(c1);
      c2 = total(c2);
      c3 = total(c3);
      if (c3 > v) {
        lo = x3;
      } else {
        hi = x3;
        chi = c3;
        if (c2 > v) {
          lo = x2;
        } else {
          hi = x2;
          chi = c2;
          if (c1 > v) {
            lo = x1;
          } else {
            hi = x1;
            chi = c1;
          }
        }
      }
    }
    // Among the items with exactly lo keys, the (v - chi)-th in sequence order.
    int j = v - chi, found = 0;
    for (int b0 = 0; b0 < batch && !found; b0 += 64) {
      const int bb = b0 + lane;
      int c1 = 0, c2 = 0, nrb = 0;
      if (in_set(bb)) {
        const int2 sq = b0 ? s_sq[bb] : sq0;
        const int key = b0 ? s_key[bb] : key0;
        nrb = blocks_of(sq.y * G);
        c1 = lo > 0 ? at_least(sq, key, lo) : nrb;
        c2 = at_least(sq, key, lo + 1);
      }
      const int eq = c1 - c2, incl = wave_scan(eq);
      const uint64_t hit = __builtin_amdgcn_ballot_w64(j >= incl - eq && j < incl);
      if (hit) {
        const int src = __builtin_ctzll(hit);
        b = __builtin_amdgcn_readlane(bb, src);
        rb = __builtin_amdgcn_readlane(nrb - c2 - 1, src) - (j - __builtin_amdgcn_readlane(incl - eq, src));
        found = 1;
      } else {
        j -= __builtin_amdgcn_readlane(incl, 63);
      }
    }
    b = uni(b);
    rb = uni(rb);
  }
  // The KV head: rotated by the sequence, so that every XCD serves every head (the
  // head fixes the page tiles' offset, and with it their HBM channels).
  const int g = by_head ? ((xcd + b) & 7) + 8 * hsub : (by_class ? (xcd + b) % Hkv : hsub);
  const int q0 = p.q_start[b];
  const int2 sqb = batch > 64 ? make_int2(uni(s_sq[b].x), uni(s_sq[b].y))
                              : make_int2(__builtin_amdgcn_readlane(sq0.x, b), __builtin_amdgcn_readlane(sq0.y, b));
  const int n = sqb.y;
  const int L = sqb.x + n;
  const int rows = n * G;
  const int r0 = rb << rshift, r1 = min(r0 + (1 << rshift), rows);
  const int base_pos = L - n;                                   // position of query token 0
  const int E = max(0, base_pos + (r1 - 1) / G + 1);            // keys the workgroup reads
  const int nkb = (E + kKeys - 1) / kKeys;
  const int wr0 = r0 + (split ? 0 : kTile * kNT * wave), wr1 = min(wr0 + kTile * kNT, r1);
  const int Ew = wr0 < wr1 ? max(0, base_pos + (wr1 - 1) / G + 1) : 0;       // keys this wave needs
  const int Ew_full = wr0 < wr1 ? max(0, base_pos + wr0 / G + 1) : 0;       // ... visible to all its rows

  // This lane's query rows, one per tile: lanes i and i + 32 share row wr0 + 32 t + i.
  const int i = lane & 31, hh = lane >> 5;
  bool live[kNT];
  int qi[kNT], head[kNT], lim[kNT];
#pragma unroll
  for (int t = 0; t < kNT; ++t) {
    const int row = wr0 + kTile * t + i;
    live[t] = row < wr1;
    qi[t] = live[t] ? row / G : 0;
    head[t] = live[t] ? s_qh[g * G + (row - qi[t] * G)] : 0;
    lim[t] = live[t] ? base_pos + qi[t] + 1 : 0;               // keys [0, lim) are visible
  }

  // Q operands (B of K Q^T): lane 32h + i holds its row's elements [16s + 8h, 16s + 8h + 8).
  bf16x8 qop[kNT][S::KS];
  {
    const __amdgpu_buffer_rsrc_t rq = make_rsrc_uni(p.q, (uint32_t)p.total_q * (uint32_t)Hq * D * 2u);
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      const int off = live[t] ? ((q0 + qi[t]) * Hq + head[t]) * D * 2 : kPastRange;
#pragma unroll
      for (int s = 0; s < S::KS; ++s)
        qop[t][s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rq, off + 16 * (2 * s + hh), 0, 0));
    }
  }

  // Staging: wave w brings pages (w & 1) + 2h, h < kKH, of each block's K (w < 2)
  // or V (w >= 2).
  const int which = wave >> 1, pgw = wave & 1;
  // Register sets of the blocks in flight: block kb is loaded into set kb % PD
  // PD blocks before it is computed (global latency is several blocks' work).
  constexpr int PD = RLDA_MQ_PREFETCH;
  struct Staged {   // one page of K or V in flight
    u32x4 r[S::LPL];
    float scale;
    int bad;
  };
  // Page ids come through the scalar cache (the block table is read-only here),
  // one block ahead of the loads that use them; the index is clamped into the row
  // so the load is always in bounds (pages past the keys are not used).
  typedef const __attribute__((address_space(4))) int32_t bt_elem;
  bt_elem* bt_row = (bt_elem*)(const void*)(p.block_table + (int64_t)b * p.max_pages);
  const int32_t* bt_vec = p.block_table + (int64_t)b * p.max_pages;
  auto page_index = [&](int kb, int h) { return 2 * kKH * kb + pgw + 2 * h; };
  auto page_id = [&](int j) -> int { return bt_row[min(j, p.max_pages - 1)]; };
  auto page_ids = [&](int kb, int* pid) {
#pragma unroll
    for (int h = 0; h < kKH; ++h) pid[h] = page_id(page_index(kb, h));
  };
  // Page j of the sequence, K or V, into registers and from there to page `slot` of
  // block buffer `buf`.
  auto page_load = [&](Staged& st, int is_v, int j, int pid) {
    int tok = min(max(E - j * kPage, 0), kPage);
    st.bad = 0;
    if (tok > 0) {
      if ((unsigned)pid >= (unsigned)p.num_pages) {
        if (lane == 0) atomicOr(p.flags, kFlagBadPage);
        tok = 0;
        st.bad = 1;
      }
    }
    const int64_t po = tok > 0 ? (int64_t)pid * p.stride_page + (int64_t)g * p.stride_head : 0;
    const uint32_t nrec = tok > 0 ? (uint32_t)((tok - 1) * p.stride_slot + D * S::EB) : 0u;
    const __amdgpu_buffer_rsrc_t r = make_rsrc_uni((const char*)(is_v ? p.v : p.k) + po, nrec);
#pragma unroll
    for (int k = 0; k < S::LPL; ++k) {
      const int ci = lane + 64 * k, rr = ci / S::CPR, c = ci % S::CPR;
      st.r[k] = __builtin_amdgcn_raw_buffer_load_b128(r, rr * p.stride_slot + 16 * c, 0, 0);
    }
    if constexpr (FP8) st.scale = tok > 0 ? (is_v ? p.v_scale : p.k_scale)[(int64_t)pid * Hkv + g] : 0.f;
  };
  auto page_write = [&](const Staged& st, int is_v, int buf, int slot) {
    char* dst = is_v ? s_v[buf] : s_k[buf];
    const int RS = is_v ? S::vrs(false) : S::krs(false);
#pragma unroll
    for (int k = 0; k < S::LPL; ++k) {
      const int ci = lane + 64 * k, rr = ci / S::CPR, c = ci % S::CPR;
      char* rowp = dst + (kPage * slot + rr) * RS;
      if constexpr (!FP8) {
        *(u32x4*)(rowp + 16 * c) = st.r[k];
      } else {   // 16 E4M3 values -> 16 bf16 (exact)
        uint32_t w[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (kFp8Direct) {
            w[2 * e] = fp8x2_to_bf16x2(st.r[k][e], false);
            w[2 * e + 1] = fp8x2_to_bf16x2(st.r[k][e], true);
          } else {
            const f32x2 a = fp8x2_to_f32(st.r[k][e], false), bb = fp8x2_to_f32(st.r[k][e], true);
            w[2 * e] = pack_bf16(a[0], a[1]);
            w[2 * e + 1] = pack_bf16(bb[0], bb[1]);
          }
        }
        *(u32x4*)(rowp + 32 * c) = u32x4{w[0], w[1], w[2], w[3]};
        *(u32x4*)(rowp + 32 * c + 16) = u32x4{w[4], w[5], w[6], w[7]};
      }
    }
    if (lane == 0) {
      if constexpr (FP8) s_scale[buf][2 * kKH * is_v + slot] = st.scale;
      if (!is_v) s_bad[buf][slot] = st.bad;
    }
  };
  Staged stg[PD][kKH];
  auto stage_load = [&](int kb, int set, const int* pid) {
#pragma unroll
    for (int h = 0; h < kKH; ++h) page_load(stg[set][h], which, page_index(kb, h), pid[h]);
  };
  auto stage_write = [&](int set, int buf) {
#pragma unroll
    for (int h = 0; h < kKH; ++h) page_write(stg[set][h], which, buf, pgw + 2 * h);
  };

  // DMA path: 16-byte chunk c of row r (the row's slot in its page) sits at chunk
  // position c ^ (r & 15) in K rows and c ^ 4 (r & 3) in V rows, so that the
  // score operand reads (16 rows, one chunk) and the transpose reads (4 rows, 4
  // chunks, two 16-lane groups) each touch all 64 banks once.  Lane l of the k-th
  // DMA of a page fills slot 64k + l of the page, row (64k + l) / 16, position
  // (64k + l) % 16, so it fetches the chunk that belongs there.
  auto chunk_pos = [](bool v_rows, int r, int c) { return c ^ (v_rows ? 4 * (r & 3) : (r & 15)); };
  int bad_pages = 0;   // DMA path: the flag is raised after the loop (no atomics between the DMAs)
  auto dma_issue = [&](int kb, int buf, const int* pid) {
    char* dst = which ? s_v[buf] : s_k[buf];
#pragma unroll
    for (int h = 0; h < kKH; ++h) {
      const int j = page_index(kb, h);
      int tok = min(max(E - j * kPage, 0), kPage);
      int badp = 0;
      if (tok > 0 && (unsigned)pid[h] >= (unsigned)p.num_pages) {
        tok = 0;
        badp = 1;
      }
      bad_pages |= badp;
      const int64_t po = tok > 0 ? (int64_t)pid[h] * p.stride_page + (int64_t)g * p.stride_head : 0;
      const uint32_t nrec = tok > 0 ? (uint32_t)((tok - 1) * p.stride_slot + D * S::EB) : 0u;
      const __amdgpu_buffer_rsrc_t r = make_rsrc_uni((const char*)(which ? p.v : p.k) + po, nrec);
      char* page_base = dst + kPage * (pgw + 2 * h) * S::krs(true);
#pragma unroll
      for (int k = 0; k < S::LPL; ++k) {
        const int sl = 64 * k + lane, rr = sl / S::CPR, c = chunk_pos(which != 0, rr, sl % S::CPR);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            r, (__attribute__((address_space(3))) void*)(page_base + 1024 * k), 16, rr * p.stride_slot + 16 * c, 0, 0, 0);
      }
      if (which == 0 && lane == 0) s_bad[buf][pgw + 2 * h] = badp;
    }
  };

  f32x16 acc[kNT][S::DT];
  float m[kNT], l[kNT];
#pragma unroll
  for (int t = 0; t < kNT; ++t) {
#pragma unroll
    for (int c = 0; c < S::DT; ++c) acc[t][c] = f32x16{};
    m[t] = neg_inf();
    l[t] = 0.f;
  }

  // P^T operands of the current block per tile: key tile kh, key step kk.
  bf16x8 pb[kNT][kKH][2];
  // Online softmax of tile t on block kb: updates (m, l), rescales the tile's
  // accumulators when m moves and leaves the block's P^T operands in pb[t].
  auto softmax = [&](int t, int kb, int buf, const f32x16* sc) {
    // Lane 32h + i holds S^T[key 32kh + 8(j/4) + 4h + j%4][row i] of key tile kh,
    // j < 16: page 2kh for j < 8, 2kh + 1 above.
    float km[2 * kKH], vm[2 * kKH];
    int bad = 0;
#pragma unroll
    for (int q = 0; q < 2 * kKH; ++q) {
      km[q] = FP8 ? p.scale_log2 * s_scale[buf][q] : p.scale_log2;
      vm[q] = FP8 ? s_scale[buf][2 * kKH + q] : 1.f;
      bad |= s_bad[buf][q];
    }
    // bf16: one positive factor for the whole block, so the maximum is taken on the
    // raw scores and the factor enters the exponent's fma; fp8: per-page factors.
    float sv[kKH][16];
#pragma unroll
    for (int kh = 0; kh < kKH; ++kh)
#pragma unroll
      for (int j = 0; j < 16; ++j) sv[kh][j] = FP8 ? sc[kh][j] * km[2 * kh + (j >> 3)] : sc[kh][j];
    if ((kb + 1) * kKeys > Ew_full || bad) {
#pragma unroll
      for (int kh = 0; kh < kKH; ++kh)
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int key = kb * kKeys + kTile * kh + 8 * (j >> 2) + 4 * hh + (j & 3);
          if (key >= lim[t] || s_bad[buf][2 * kh + (j >> 3)]) sv[kh][j] = neg_inf();
        }
    }
    float mx = neg_inf();
#pragma unroll
    for (int kh = 0; kh < kKH; ++kh) {
#pragma unroll
      for (int j = 0; j < 16; j += 2) mx = fmaxf(fmaxf(mx, sv[kh][j]), sv[kh][j + 1]);
    }
    mx = pair_max(mx);
    if constexpr (!FP8) mx *= km[0];
    // Lazy rescale: the reference maximum moves only when a score exceeds it by
    // more than 2^kRescaleLog2 (always when it is still -inf and a score is not).
    // A row whose keys are all masked so far keeps m = -inf and alpha = 1.
    const bool up = mx > m[t] + kRescaleLog2;
    if (__builtin_amdgcn_ballot_w64(up) != 0) {
      const float alpha = up ? __builtin_amdgcn_exp2f(m[t] - mx) : 1.f;
      l[t] *= alpha;
      m[t] = up ? mx : m[t];
#pragma unroll
      for (int c = 0; c < S::DT; ++c) acc[t][c] *= alpha;
    }
    const float mu = (m[t] == neg_inf()) ? 0.f : m[t];
    const float fk = FP8 ? 1.f : km[0];
#pragma unroll
    for (int kh = 0; kh < kKH; ++kh) {
      float pr[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        pr[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[kh][j], fk, -mu));
        l[t] += pr[j];
      }
      // P^T operand of key step kk: K position 8h + e is key 16kk + 8(e/4) + 4h + e%4
      // of the key tile.
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const float v = vm[2 * kh + kk];
        const u32x4 w = {pack_bf16(pr[8 * kk] * v, pr[8 * kk + 1] * v), pack_bf16(pr[8 * kk + 2] * v, pr[8 * kk + 3] * v),
                         pack_bf16(pr[8 * kk + 4] * v, pr[8 * kk + 5] * v), pack_bf16(pr[8 * kk + 6] * v, pr[8 * kk + 7] * v)};
        pb[t][kh][kk] = __builtin_bit_cast(bf16x8, w);
      }
    }
  };
  // Operand reads.  K rows of block buffer `buf` for S^T = K Q^T: lane 32h + i
  // reads key i, elements [16s + 8h, 16s + 8h + 8).  V^T operands: the transpose read gives lane (16-lane group q, index c) the 4 keys
  // k0 .. k0+3 of column d = 16 (q & 1) + c of a 32-column tile, when lane c' of the
  // group addresses key k0 + c'/4, columns 4 (c' % 4) .. +3; operand kk*DT + t is
  // key step kk, column tile t.
  auto read_k = [&](auto dma, bf16x8* ka, int buf, int kh) {
    constexpr bool kDma = decltype(dma)::value;
    const int R = kTile * kh + i;
    const char* kl = s_k[buf] + R * S::krs(kDma);
#pragma unroll
    for (int s = 0; s < S::KS; ++s) {
      const int c = 2 * s + hh;
      ka[s] = *(const bf16x8*)(kl + 16 * (kDma ? chunk_pos(false, R, c) : c));
    }
  };
  const int lr = (lane & 15) >> 2, lc = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  auto read_v = [&](auto dma, bf16x8* va, int buf, int kh) {
    constexpr bool kDma = decltype(dma)::value;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const int R = kTile * kh + 16 * kk + 4 * hh + lr;   // and R + 8: the same R & 3
      const char* vr = s_v[buf] + R * S::vrs(kDma);
#pragma unroll
      for (int t = 0; t < S::DT; ++t) {
        // column 32t + lc: chunk (32t + lc) / 8, byte 2 ((32t + lc) % 8) = 8 (lane & 1) in it
        const int c = 4 * t + (lc >> 3);
        const int off = kDma ? 16 * chunk_pos(true, R, c) + 8 * (lane & 1) : 2 * (32 * t + lc);
        const bf16x4 x0 = lds_tr_read(vr + off);
        const bf16x4 x1 = lds_tr_read(vr + 8 * S::vrs(kDma) + off);
        va[kk * S::DT + t] = bf16x8{x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
      }
    }
  };
  static_assert(S::KS == 2 * S::DT, "as many V^T operands as score k-steps");

  // Block kb in LDS buffer buf: scores, softmax, P V, for the wave's row tiles.
  auto compute_block = [&](auto dma, int kb, int buf) {   // dma: the block's layout
    if (kb * kKeys < Ew) {
      // Each K and V operand read serves every row tile of the wave.
      f32x16 sc[kNT][kKH];
      bf16x8 va[kKH][S::KS];
#pragma unroll
      for (int kh = 0; kh < kKH; ++kh) {
        bf16x8 ka[S::KS];
        read_k(dma, ka, buf, kh);
#pragma unroll
        for (int t = 0; t < kNT; ++t) sc[t][kh] = f32x16{};
#pragma unroll
        for (int s = 0; s < S::KS; ++s)
#pragma unroll
          for (int t = 0; t < kNT; ++t)
            sc[t][kh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s], qop[t][s], sc[t][kh], 0, 0, 0);
      }
#pragma unroll
      for (int t = 0; t < kNT; ++t) softmax(t, kb, buf, sc[t]);
#pragma unroll
      for (int kh = 0; kh < kKH; ++kh) read_v(dma, va[kh], buf, kh);
#pragma unroll
      for (int kh = 0; kh < kKH; ++kh)
#pragma unroll
        for (int s = 0; s < S::KS; ++s)
#pragma unroll
          for (int t = 0; t < kNT; ++t)
            acc[t][s % S::DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[kh][s], pb[t][kh][s / S::DT],
                                                                        acc[t][s % S::DT], 0, 0, 0);
    }
  };

  // 3. Key blocks.
  if (SMALL && split) {
    // Wave w computes blocks w, w + 4, .. of the workgroup's one row tile, each staged
    // through registers into the wave's own buffer: no barrier.  The next block's pages
    // are loaded while a block is computed.
    static_assert(!SMALL || kMultiSplits, "one row tile, two pages a block");
    // Page ids come 32 blocks of the wave at a time: lane 2k + h, page h of its k-th.
    Staged sk[2], sv[2];
    int ids = 0;
    auto load = [&](int k) {   // the wave's k-th block; past the keys the loads read nothing
      const int kb = wave + kWaves * k;
      if ((k & 31) == 0) ids = bt_vec[min(2 * (kb + kWaves * (lane >> 1)) + (lane & 1), p.max_pages - 1)];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int pid = __builtin_amdgcn_readlane(ids, 2 * (k & 31) + h);
        page_load(sk[h], 0, 2 * kb + h, pid);
        page_load(sv[h], 1, 2 * kb + h, pid);
      }
    };
    load(0);
    for (int k = 0; wave + kWaves * k < nkb; ++k) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        page_write(sk[h], 0, wave, h);
        page_write(sv[h], 1, wave, h);
      }
      // A wave's LDS operations complete in order; the compiler keeps theirs.
      asm volatile("" ::: "memory");
      load(k + 1);
      compute_block(std::false_type{}, wave + kWaves * k, wave);
      asm volatile("" ::: "memory");
    }
    // The waves' states meet in LDS, weighted by their maxima: thread (row, chunk of
    // D / 8 outputs).  The block buffers are done with.
    constexpr int RSF = D + 4, DPT = D / 8;
    static_assert(!SMALL || (2 * kTile * RSF * 4 <= (int)sizeof s_k && 2 * kTile * RSF * 4 <= (int)sizeof s_v),
                  "two waves' states fit each block buffer");
    auto part = [&](int w) { return (float*)(w < 2 ? s_k[0] : s_v[0]) + (w & 1) * kTile * RSF; };
    __shared__ float2 s_ml[kWaves][kTile];
    const float lt = pair_sum(l[0]);
    lds_barrier();
    if (wave < nkb) {
#pragma unroll
      for (int c = 0; c < S::DT; ++c)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          *(f32x4*)&part(wave)[i * RSF + 32 * c + 8 * jj + 4 * hh] =
              f32x4{acc[0][c][4 * jj], acc[0][c][4 * jj + 1], acc[0][c][4 * jj + 2], acc[0][c][4 * jj + 3]};
    }
    if (hh == 0) s_ml[wave][i] = make_float2(m[0], lt);
    lds_barrier();
    const int row = tid >> 3, d0 = (tid & 7) * DPT;
    if (r0 + row >= r1) return;
    float M = neg_inf(), Ls = 0.f, o[DPT];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, s_ml[w][row].x);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float aw = s_ml[w][row].x == neg_inf() ? 0.f : __builtin_amdgcn_exp2f(s_ml[w][row].x - M);
      Ls += aw * s_ml[w][row].y;
    }
#pragma unroll
    for (int e = 0; e < DPT; ++e) o[e] = 0.f;
    for (int w = 0; w < min(kWaves, nkb); ++w) {   // the others have no state in LDS
      const float aw = s_ml[w][row].x == neg_inf() ? 0.f : __builtin_amdgcn_exp2f(s_ml[w][row].x - M);
#pragma unroll
      for (int c = 0; c < DPT; c += 4) {
        const f32x4 v = *(const f32x4*)&part(w)[row * RSF + d0 + c];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[c + e] += aw * v[e];
      }
    }
    const float inv = Ls > 0.f ? 1.f / Ls : 0.f;
    const int rq = (r0 + row) / G;
    const int64_t ob = ((int64_t)(q0 + rq) * Hq + s_qh[g * G + (r0 + row - rq * G)]) * D + d0;
#pragma unroll
    for (int c = 0; c < DPT; c += 4) {
      if (p.out_bf16)
        *(u32x2*)((uint16_t*)p.out + ob + c) = u32x2{pack_bf16(o[c] * inv, o[c + 1] * inv), pack_bf16(o[c + 2] * inv, o[c + 3] * inv)};
      else
        *(f32x4*)((float*)p.out + ob + c) = f32x4{o[c] * inv, o[c + 1] * inv, o[c + 2] * inv, o[c + 3] * inv};
    }
    return;
  }
  if constexpr (S::DMA) {
    // Iteration kb starts the DMA of block kb + 2 into buffer (kb + 2) % 3 (read
    // last in iteration kb - 1), computes block kb, then waits until only block
    // kb + 2's DMAs are outstanding (block kb + 1 has landed) before the barrier.
    // Past the keys the DMAs read nothing, so every iteration issues the same count.
    constexpr int kDmaPerBlock = S::LPL * kKH;
    {
      int pid[kKH];
      page_ids(0, pid);
      dma_issue(0, 0, pid);
      page_ids(1, pid);
      dma_issue(1, 1, pid);
    }
    int pid_next[kKH];
    page_ids(2, pid_next);
    dma_barrier<kDmaPerBlock>();
    for (int kb0 = 0; kb0 < nkb; kb0 += 3) {
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const int kb = kb0 + u;
        if (kb < nkb) {
          dma_issue(kb + 2, (u + 2) % 3, pid_next);
          compute_block(std::true_type{}, kb, u);
          page_ids(kb + 3, pid_next);
          dma_barrier<kDmaPerBlock>();
        }
      }
    }
    if (bad_pages && lane == 0) atomicOr(p.flags, kFlagBadPage);
  } else {
    // Blocks 0 .. PD-1 are loaded before the loop, block 0 is written to LDS, and
    // iteration kb loads block kb + PD (past the wave's keys nothing is read, but
    // the loads are issued so that every iteration has the same loads in flight),
    // computes block kb and writes block kb + 1 to the other buffer.  The loop is
    // unrolled PD times so that each register set is fixed.
    {
      int pid[kKH];
#pragma unroll
      for (int u = 0; u < PD; ++u) {
        page_ids(u, pid);
        stage_load(u, u, pid);
      }
    }
    int pid_next[kKH];
    page_ids(PD, pid_next);
    stage_write(0, 0);
    __syncthreads();
    for (int kb0 = 0; kb0 < nkb; kb0 += PD) {
#pragma unroll
      for (int u = 0; u < PD; ++u) {
        const int kb = kb0 + u;
        if (kb < nkb) {
          const int buf = kb & 1;
          stage_load(kb + PD, u, pid_next);
          compute_block(std::false_type{}, kb, buf);
          if (kb + 1 < nkb) stage_write((u + 1) % PD, buf ^ 1);
          // The next page ids are read here: a scalar load shares its completion
          // counter with the LDS reads, so issued earlier it would hold up the
          // first MFMA's operand wait; here the barrier's wait covers it.
          page_ids(kb + PD + 1, pid_next);
          __syncthreads();
        }
      }
    }
  }

  // 4. Normalise and write: lane 32h + i holds O^T[d = 32c + 8jj + 4h + 0..3][its row].
#pragma unroll
  for (int t = 0; t < kNT; ++t) {
    const float lt = pair_sum(l[t]);
    if (!live[t]) continue;
    const float inv = lt > 0.f ? 1.f / lt : 0.f;
    const int64_t ob = ((int64_t)(q0 + qi[t]) * Hq + head[t]) * D;
#pragma unroll
    for (int c = 0; c < S::DT; ++c)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const int d = 32 * c + 8 * jj + 4 * hh;
        const float o0 = acc[t][c][4 * jj] * inv, o1 = acc[t][c][4 * jj + 1] * inv;
        const float o2 = acc[t][c][4 * jj + 2] * inv, o3 = acc[t][c][4 * jj + 3] * inv;
        if (p.out_bf16)
          *(u32x2*)((uint16_t*)p.out + ob + d) = u32x2{pack_bf16(o0, o1), pack_bf16(o2, o3)};
        else
          *(f32x4*)((float*)p.out + ob + d) = f32x4{o0, o1, o2, o3};
      }
  }
}

template <int D, bool FP8, bool SMALL>
int launch_multi_t(const Params& p, int grid, void* stream, void* ev_begin, void* ev_end) {
  hipStream_t st = (hipStream_t)stream;
  if (ev_begin && hipEventRecord((hipEvent_t)ev_begin, st) != hipSuccess) return -1;
  const size_t lds = p.batch > 64 ? (sizeof(int2) + sizeof(int32_t)) * (size_t)p.batch : 0;
  hipLaunchKernelGGL((multi_query_kernel<D, FP8, SMALL>), dim3(grid), dim3(kThreads), lds, st, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return (int)e;
  if (ev_end && hipEventRecord((hipEvent_t)ev_end, st) != hipSuccess) return -1;
  return 0;
}

}  // namespace

int launch_multi(KvKind kind, int head_dim, bool small, const Params& p, int grid, void* stream, void* ev_begin,
                 void* ev_end) {
  if (kind != KvKind::BF16 && kind != KvKind::FP8) return -1;
  constexpr bool S = kMultiSplits;
  auto* const launch = kind == KvKind::BF16
                           ? (head_dim == 128 ? (small ? launch_multi_t<128, false, S> : launch_multi_t<128, false, false>)
                                              : (small ? launch_multi_t<64, false, S> : launch_multi_t<64, false, false>))
                           : (head_dim == 128 ? (small ? launch_multi_t<128, true, S> : launch_multi_t<128, true, false>)
                                              : (small ? launch_multi_t<64, true, S> : launch_multi_t<64, true, false>));
  return launch(p, grid, stream, ev_begin, ev_end);
}

}  // namespace rlda
