// Launch interface of the one-kernel prefill (kda_prefill_fused.hip).
#pragma once
#include "kda_intra.h"

namespace kda {
namespace mfma {

// (sequence, head) pairs per batch of the grid: the scan workgroups of a batch wait for the per-chunk
// workgroups behind them, and about two batches' worth of them are resident at a time, each on half a
// compute unit.  Up to 128 pairs make one batch (128 pairs x 64 chunks: 376 us, as two batches of 64 421 us).  More are
// dealt out evenly in batches of at most 96, which is where two batches in flight do best (64 scan workgroups cannot take
// the slots as fast as the per-chunk role makes them, 192 and more leave that role too little of the device), and an
// uneven last batch is a chain with little beside it: us with batches of at most 128 / of at most 96, evenly: 144 pairs
// x 32 chunks 287 / 224, 160 x 128 1049 / 935, 192 x 64 597 / 556, 192 packed with the output gate (7200 chunks in all) 512 / 458,
// 256 x 64 751 / 740, 256 x 16 223 / 203, 256 x 512 5691 / 5713, 384 x 64 1114 / 1093.  Packed sequences, longest first, go
// whole into a batch, as many as fit, where that comes to five sixths of the 96 or more (32 heads, sequences of 512 to 8192 tokens, us as
// batches of 128 pairs / evenly / whole: eight sequences 958 / 944 / 925, 764 / 801 / 784 and 865 / 844 / 849 for three draws of
// their lengths, six 616 / - / 610 and 597 / - / 560, ten 1063 / 1056 / 1047 and 897 / 899 / 885; 40 heads, which make 80: four
// 770 / 697 / 695).  Otherwise evenly, too: with 64 heads whole sequences make batches of 64 (four sequences 1032 / 1020 / 1066 and 658 /
// 650 / 668; eight shorter ones 942 / 919 / 912 and 714 / 694 / 698).  A device with fewer compute units gets batches of a quarter of
// its workgroup slots, so that two batches never take more than half.
constexpr int kMaxSingleBatchPairs = 128, kMaxBatchPairs = 96;

// Chunks a workgroup of the per-chunk role works through.  Four: the fetch of each hides behind the one before, which is
// what counts where the per-chunk role sets the pace (a batch of 96 pairs or more on its own, ranges of a time split: 2^17
// tokens x 32 heads 2972 us, with one 3108) and in short calls (64 pairs x 16 chunks 56 us, with one 58).  One: the
// chunks are finished in just the order the scan wants them, which is what counts where its steps set the pace: several
// batches (192 x 64: 595 us with four, 556 with one), or one of fewer than 96 pairs and 32 chunks a pair or more (64 x 64:
// 233 and 217 us, 88 x 128: 549 and 504, 64 x 32: 114.5 and 112.5; at 24 chunks equal).
// But the grid of a packed call has a place for as many chunks of every sequence as the longest may have, and a workgroup that finds
// nothing at its place costs its launch, about 2 ns each, with batches of them ahead of the next batch's scan workgroups.  One chunk a
// workgroup means four times as many, so it is taken only while such places are at most half of all and at most kMostEmptyPlaces.
// us with four / with one: eight sequences of 5000 tokens x 32 heads 946 / 894, and without max_seqlen, 140 000 empty places, 1282 /
// 1538; twelve of 500 to 3000 without it 830 / 1016; forty of 100 to 300 x 2 heads without it 48 / 62; with it, of 512 to 8192 tokens
// x 32 heads: eight (11 500 empty) 972 / 925, nine (14 200) 998 / 972 and (15 000) 771 / 773, ten (16 700) 1047 / 1074 and (15 900) 885 / 908.
constexpr int kItemsPerWorkgroup = 4;
constexpr int kOrderedPairs = 96, kOrderedChunks = 32;
constexpr int64_t kMostEmptyPlaces = 14 * 1024;

// Time-split scan (kda_scan4_split.h): workspace areas and the cut of the chunk axis.
struct SplitArgs {
    float *E, *Tm, *Bm;          // [split_parts_cap(pairs, seg_chunks)][pairs][128][128] fp32 each
    uint32_t *flags;             // kSplitFlagsPerPair words per pair
    int64_t part_len, part0_len; // chunk indices of the first range and of every other one
    int64_t tail;                // chunks at the end of a range whose transition is tested for zero (<= both lengths)
    int parts;                   // 1: no time split
};

struct FusedArgs {
    const uint16_t *q, *k, *v, *log_alpha, *beta;
    const int32_t *cu;              // cu_seqlens or NULL
    const int32_t *order;           // packed calls in several batches: the sequences, longest first (NULL: as they come)
    const float *state_in;          // [N,H,dk,dv] or NULL (= zeros)
    float *state_out;               // [N,H,dk,dv] or NULL
    void *o;
    uint8_t *ws;                    // first slot of the segment
    uint32_t *ready;                // one flag per slot
    uint32_t *status;
    int64_t T;                      // tokens per batch row (fixed-length batches)
    int64_t pairs;                  // num_seqs * heads
    int64_t seg_chunks, seg_index;  // chunk indices per time segment, and which segment this launch works on
    int64_t launch_chunks;          // chunk indices this launch covers (<= seg_chunks)
    uint64_t wait_limit;            // ticks of the 100 MHz wall clock a scan workgroup waits for one slot
    int H, nb;
    float scale;
    uint32_t epoch;                 // value of a raised flag
    int producers;                  // 0: the per-chunk role does nothing (a diagnostic: every wait of the scan role then runs out)
    int per_wg, window;             // per-chunk role: chunks per workgroup, and workgroups that share a run of window * per_wg chunks
    RawParams raw;
    SplitArgs split;
    // output gate of Section 4 (kGate kernels only): o <- Sigmoid(g) * RMSNorm(o) * w
    const uint16_t *out_gate;       // gate logits [B,T,H,dv] bf16
    uint8_t *gate_ws;               // the same re-laid by the per-chunk role, kGateSlotBytes per slot
    const float *norm_w;            // [dv] or NULL (= ones)
    float rms_eps;
};

struct FusedLaunch {
    FusedArgs args;
    bool raw, scalar_gate, out_bf16, gate;
    bool reset_flags;               // clear num_flags words at args.ready and the status word first
    int64_t num_flags;
    int32_t *order_out;             // the first launch of such a call (the one that resets the flags) writes the order here, else NULL
    int num_seqs;
    bool reset_split;               // clear the counters of the time-split scan first (segments after the first)
    int64_t live_chunks;            // of the pairs * launch_chunks places for a chunk, how many hold one, as far as the host can tell (at least)
    int compute_units;              // of the device the launch goes to
};

// Plain scan: pairs per batch, and chunks a workgroup of the per-chunk role works through.
// heads: of a packed call whose sequences are taken longest first, else 0
int fused_batch_pairs(int64_t pairs, int compute_units, int heads);
int fused_chunks_per_workgroup(int64_t pairs, int batch_pairs, int64_t launch_chunks, int64_t live_chunks);
// Workgroups of a launch, and the two figures the kernel lays them out by (a.per_wg, a.window); a.nb, a.pairs, a.launch_chunks and
// a.split are given.
int64_t fused_workgroups(FusedArgs &a, int64_t live_chunks, int compute_units);
kda_status launch_prefill_fused(const FusedLaunch &L, hipStream_t stream);

}  // namespace mfma
}  // namespace kda
