// Whole analysis of a short window by one workgroup (winfused.hip).
#pragma once
#include "pipeline.h"

namespace apo {

// Longest window one workgroup takes: its suffix sort keeps the window's token
// ranks, suffix ranks and suffix order in LDS, and its candidate sort up to two
// records per token (16 bytes of LDS per token in all, of the 160 KB).
constexpr uint32_t kFusedMax = 8192;
// Longest window one workgroup takes with its arrays in the workspace (positions
// and ranks in 16 bits, one array of them in LDS at a time).
constexpr uint32_t kFusedLongMax = 65536;
// Longest window that takes one workgroup where it is a batch's or the server's only
// one.  Up to here no content is slower than stage by stage before there was that
// form (a loop without substitutions 1.16 ms at either; in most windows the one workgroup is
// twice as fast); above, stage by stage, host-driven, is as fast for a loop with 5 %
// substitutions (30000 tokens: 0.70 and 0.70 ms; 65536: 1.48 and 0.80) and faster for
// one without (1.34 and 0.86; 2.85 and 0.96), 65536 random tokens 3.1 and 0.62.
constexpr uint32_t kFusedLone = 25600;
// Longest window of a large batch that shares a compute unit with another.
constexpr uint32_t kFusedMidMax = 32768;

// What one window's analysis reports to the host (pinned memory).
struct FusedInfo {
  uint32_t sigma, cands, maxl, m, accepted, rows, nhist;
  uint32_t hist[kMaxRounds];  // suffixes still grouped after each doubling round
  uint64_t stamp[kStages + 1];
};

// One window of n tokens (2 <= n < kFusedLongMax, `bits` 32 or 64; device
// memory or pinned host memory).  Rows and occurrences are written only when
// both fit (row_cap; occ_cap unless occ is null); `info` always is.  w: scratch
// arrays for n tokens.
void fused_window(const Workspace &w, const void *tok, int bits, uint32_t n, uint32_t min_len, void *rows,
                  uint32_t row_cap, void *occ, uint32_t occ_cap, FusedInfo *info, hipStream_t s);

// Copies what `info` reports into the run's info and the host mirrors of the
// per-round counts.
void fused_read(const FusedInfo &f, uint32_t n, Workspace &w, RunInfo &info);

// Batch of windows of at most kFusedLongMax 64-bit tokens each (offsets and
// order in w.d_off and w.d_order): rows of all windows packed in window order
// into w.rows, counts into w.win_rows, counters where finish_run reads them.
// Uses w.wflag.  With w.may_leave, batches of two or three windows may come out
// unfinished: CNT_WFLAG is then not 0.
// two: in two launches, where fused_in_two says so; either form is right for any
// windows.
bool fused_in_two(const uint64_t *off, uint32_t W);
void fused_batch(Workspace &w, const void *tok, uint32_t W, uint64_t longest, bool two, uint32_t min_len,
                 hipStream_t s);

}  // namespace apo
