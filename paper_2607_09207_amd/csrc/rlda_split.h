// How a decode call's flattened (sequence, KV head, page) list is cut over the
// workgroups: the kernel's rule, in plain C++ so that it can be compiled for the host
// as well (where square root and reciprocal are the exact ones).
#pragma once
#include "rlda_params.h"

#if defined(__HIP__)
#define RLDA_HD __host__ __device__ __forceinline__
#else
#define RLDA_HD inline
#endif

namespace rlda {

RLDA_HD float split_rcp(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf(x);
#else
  return 1.f / x;
#endif
}
RLDA_HD float split_sqrt(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_sqrtf(x);
#else
  return __builtin_sqrtf(x);
#endif
}

// The calls that the lines below tell apart: plain ones by the size of their pages (half:
// at most 4 KiB of K and V per page and KV head, two workgroups per CU), and the ones
// that stream whole segments through the general loop (several query tokens, packed
// groups, the launch after a prompt pass).
enum SplitForm { kSplitFullPages, kSplitHalfPages128, kSplitHalfPages64, kSplitGeneral };

struct Split {
  bool whole;   // each workgroup takes one whole segment
  int shares;   // ... otherwise: equal-cost shares
};

// calibrate.work_split mirrors it for plain calls.
//   Whole segments: each workgroup takes one segment.  That skips the share search and
// the hand-off of cut pieces (store, count, read back), about 5 us together, and its
// waves stream (nbmax - fair) / 4 pages more than under equal shares of `fair` pages,
// 0.4 to 0.6 us each while so few of them run.  us a call on batches of equal lengths,
// equal shares against whole segments, 16 / 32 / 64 / 112 pages:
//   28/4 bf16 d 128, B = 4:   13.2 / 13.9 / 14.6 / 15.4   against  8.1 / 9.7 / 15.8 / 26.7
//                    B = 16:  11.2 / 12.4 / 14.3 / 17.5            8.2 / 10.3 / 17.7 / 28.7
//                    B = 32:  12.3 / 14.3 / 18.7 / 25.9            8.4 / 11.7 / 19.7 / 31.5
//   40/8 fp8 d 128,  B = 4:   14.2 / 14.5 / 14.9 / 15.5            7.4 / 9.5 / 14.3 / 21.5
//                    B = 32:  12.9 / 15.1 / 20.0 / 27.5            7.7 / 10.0 / 15.0 / 22.4
//   64/8 bf16 d 64,  B = 16:  10.9 / 12.3 / 14.4 / 17.7            6.5 / 8.2 / 12.2 / 18.3
// (28/4, B = 60, 200 pages: 68.6 against 62.3).  `over` is where the two meet, in pages
// over an equal share, by segments per workgroup: with one workgroup per CU whole
// segments leave CUs idle that could read, with two (half-size pages) they don't until
// half the workgroups are gone.  Multi-token, packed and prompt-state runs stream whole
// segments through the general loop, which is slower a page.
//   Equal shares hold at least 4 pages (one a wave), and so many that the largest
// segment falls into at most 16 pieces, one batch of its final merge (17, where lengths
// differ and it begins inside a share); of segments above 300 pages at least
// sqrt(1.25 nbmax), where pages and pieces cost alike (a share's page 0.15 us, a piece
// 0.19 us).  us a call at d 128, one sequence of 64 / 112 / 188 pages: 8/1 heads bf16
// 14.4 / - / 16.5 with nbmax / 16 - 1 (18 to 22 pieces) and 13.1 / - / 15.0 so; 12/2 fp8
// - / 15.1 / - and - / 13.3 / - (12/2 bf16 in 256 shares 31.4).  Where that bound holds the shares are a multiple of the segments, so that equal
// segments are cut alike.
//   W workgroups (inv_ranges = 1 / W, or 0: the caller fixed the share count), nseg
// segments costing `cost` together, the largest of nb_max pages.
RLDA_HD Split split_of(SplitForm form, int W, float inv_ranges, int nseg, int cost, int nb_max) {
  if (!(inv_ranges > 0.f)) return {false, W};
  const float nb = (float)nb_max, fair = (float)cost * inv_ranges, segs = (float)nseg * inv_ranges;
  const float over = form == kSplitGeneral     ? __builtin_fmaxf(40.f - 48.f * segs, 20.f)
                     : form == kSplitFullPages ? __builtin_fmaxf(54.f - 72.f * segs, 26.f)
                                               : (form == kSplitHalfPages64 ? 78.f : 57.f) + __builtin_fmaxf(80.f * segs - 20.f, 0.f);
  Split s = {nseg <= W && nb - fair <= over, W};
  const float least = __builtin_fmaxf(__builtin_fminf(0.0625f * (nb + (float)kStartCost), split_sqrt(1.25f * nb)), 4.f);
  if (fair < least) {
    const float n = (float)nseg * __builtin_ceilf((float)cost * split_rcp((float)nseg * least));
    s.shares = n < (float)W ? (int)n : W;
  }
  return s;
}

// Share (or segment) of block b of the grid, of the n in use, -1: none.  Workgroups are
// dispatched round-robin over the 8 XCDs (block b runs on XCD b % 8); each gets a
// contiguous run of the n, so neighbouring work (the sequences of a GRPO group reading the
// same prompt pages, the pieces of one split segment) shares one L2, and as many as the
// others or one more, however few they are.  (Numbered over the whole grid, the 29 shares
// of one segment of 1024 pages were all on one XCD.  us a call then and so, fp8 d 128:
// 12/2 heads, one sequence of 400 pages 20.3 / 17.8, two of up to 1000 26.0 / 22.3; 28/4,
// one of 1024 25.6 / 21.6; bf16 22.5 / 21.3 for 8/1, one of 1024, but 16.2 / 16.5 for 188.)
RLDA_HD int share_of_block(int b, int n) {
  const int x = b & 7, r = n & 7;
  return b < n ? x * (n >> 3) + (x < r ? x : r) + (b >> 3) : -1;
}

}  // namespace rlda
