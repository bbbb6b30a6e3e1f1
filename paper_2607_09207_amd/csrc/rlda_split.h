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
// the hand-off of cut pieces (store, count, read back), 3 to 5 us together, and its waves
// stream (nbmax - fair) / 4 pages more than under equal shares of `fair` pages, 0.4 to
// 0.6 us each while so few of them run.  us a call on batches of equal lengths, equal
// shares against whole segments, 16 / 32 / 64 / 112 / 160 pages:
//   28/4 bf16 d 128, B = 4:   11.8 / 12.8 / 14.7 / 15.5 / 16.2   against   8.0 / 9.9 / 14.7 / 21.8 / 31.2
//                    B = 16:  11.2 / 12.1 / 13.9 / 16.7 / 20.3             8.1 / 10.2 / 17.6 / 27.9 / 38.5
//                    B = 32:  12.0 / 13.6 / 18.1 / 25.4 / 32.9             8.2 / 11.6 / 19.4 / 31.1 / 42.4
//                    B = 60:  15.1 / 19.1 / 28.4 / 42.2 / 55.6             8.9 / 13.0 / 22.5 / 36.7 / 50.7
//   40/8 fp8 d 128,  B = 4:   11.3 / 13.0 / 14.6 / 15.6 / 16.6             7.5 / 9.6 / 14.6 / 21.5 / 28.6
//                    B = 32:  12.9 / 15.2 / 20.1 / 27.8 / 36.0             7.6 / 9.9 / 15.0 / 22.6 / 30.4
//   40/8 bf16 d 64,  B = 16:  10.9 / 12.2 / 14.4 / 17.8 / 21.5             6.5 / 8.1 / 12.2 / 18.2 / 24.6
//                    B = 32:  12.1 / 14.3 / 18.9 / 26.5 / 34.0             6.7 / 8.7 / 13.5 / 21.1 / 28.4
// `over` is where the two meet, in pages over an equal share, by segments per workgroup:
// with one workgroup per CU whole segments leave CUs idle that could read, with two
// (half-size pages) they don't until half the workgroups are gone.
//   The general loop is slower a page, and slower again with the remainders that go with
// a longer stream (rlda_kernels.hip), 8 / 16 / 32 / 48 / 64 pages:
//   4 rows, 28/4 bf16 d 128, B = 4:   15.8 / 17.7 / 22.0 / 24.5 / 25.8    against   12.0 / 14.6 / 18.4 / 22.4 / 26.5
//                            B = 16:  16.3 / 17.4 / 18.6 / 20.1 / 21.2              12.1 / 14.8 / 18.7 / 23.2 / 27.4
//                            B = 32:  17.0 / 18.6 / 21.2 / 23.3 / 25.2              12.2 / 14.9 / 18.9 / 23.7 / 27.9
//   3 rows, 40/8 fp8 d 128,  B = 8:   12.3 / 12.8 / 13.5 / 14.3 / 14.9              9.4 / 11.0 / 13.5 / 16.5 / 19.5
//                            B = 24:  14.8 / 16.2 / 18.3 / 20.2 / 21.8              9.4 / 11.1 / 13.9 / 17.2 / 20.1
//   after a prompt pass, 16/1 bf16 d 64, B = 16:   17.3 / 18.7 / 19.5 / 20.6 / 21.2   14.9 / 16.2 / 18.0 / 20.3 / 22.7
//                                        B = 128:  19.0 / 19.5 / 20.7 / 22.1 / 22.8   15.9 / 17.5 / 19.6 / 22.2 / 24.4
// There equal shares that are the segments anyway (all of one length, as many as
// workgroups) cut nothing and stay without remainders: 4 rows, 40/8 fp8 d 128, B = 32,
// 64 / 112 pages 23.6 / 32.5 against 27.4 / 39.8.
//   Equal shares hold at least 4 pages (one a wave), and so many that the largest
// segment falls into at most 16 pieces, one batch of its final merge (17, where lengths
// differ and it begins inside a share); of segments above 300 pages at least
// sqrt(1.25 nbmax), where pages and pieces cost alike (a share's page 0.15 us, a piece
// 0.19 us).  us a call at d 128, one sequence of 64 / 112 / 188 pages: 8/1 heads bf16
// 14.4 / - / 16.5 with nbmax / 16 - 1 (18 to 22 pieces) and 13.1 / - / 15.0 so; 12/2 fp8
// - / 15.1 / - and - / 13.3 / - (12/2 bf16 in 256 shares 31.4).
//   Fewer shares are a multiple of the segments, so that segments of one length are cut
// alike.  Segments of unlike lengths are cut anywhere, and little fewer shares save less
// than the remainders of their longer streams cost, so those keep W unless 0.7 W or fewer
// do.  us a call with fewer shares less W shares, by shares / W, lengths within a factor of
// 3, 1 to 24 sequences of 120 to 1300 pages, mean and extremes: bf16 d 128 0.5 -2.5 (-3.5
// to -1.6), 0.6 -1.1 (-1.5 to -0.3), 0.7 to 0.8 +0.1 (-1.0 to 1.1), above +0.7 (-0.2 to
// 1.4); fp8 d 128 -2.7 (-3.5 to -0.9), -0.8 (-2.3 to 0.8), -0.1 (-1.6 to 1.8), +1.1 (0.4
// to 1.7); equal lengths up to W -1.7 (-5.6 to 0.3).
//   W workgroups (inv_ranges = 1 / W, or 0: the caller fixed the share count), nseg
// segments costing `cost` together, the largest of nb_max pages.
RLDA_HD Split split_of(SplitForm form, int W, float inv_ranges, int nseg, int cost, int nb_max) {
  if (!(inv_ranges > 0.f)) return {false, W};
  const float nb = (float)nb_max, fair = (float)cost * inv_ranges, segs = (float)nseg * inv_ranges;
  const float over = form == kSplitGeneral     ? __builtin_fmaxf(46.f - 96.f * segs, 20.f)
                     : form == kSplitFullPages ? __builtin_fmaxf(54.f - 72.f * segs, 26.f)
                                               : (form == kSplitHalfPages64 ? 78.f : 57.f) + __builtin_fmaxf(80.f * segs - 20.f, 0.f);
  const bool even = cost == (int64_t)nseg * (nb_max + kStartCost);   // all segments of one length
  Split s = {nseg <= W && nb - fair <= over && !(form == kSplitGeneral && even && nseg == W), W};
  const float least = __builtin_fmaxf(__builtin_fminf(0.0625f * (nb + (float)kStartCost), split_sqrt(1.25f * nb)), 4.f);
  if (fair < least) {
    const float n = (float)nseg * __builtin_ceilf((float)cost * split_rcp((float)nseg * least));
    if (n < (even ? 1.f : 0.7f) * (float)W) s.shares = (int)n;
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
