// Internal interface between the host runtime (snn_api.hip) and the gfx950
// kernels (snn_kernels.hip). Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <type_traits>
#include <stdint.h>

namespace snn {

constexpr int kBlock = 256;          // threads per workgroup of the element kernels
constexpr int kNeuronBlock = 1024;   // threads per workgroup of the neuron update on large
                                     // networks (one list-scan status word per workgroup)
constexpr int kNeuronSmallN = 65536; // up to this many neurons the update takes kBlock threads
                                     // per workgroup
constexpr int kWave = 64;            // CDNA wavefront width
constexpr int kXcds = 8;             // XCDs of the device: workgroup b runs on XCD b mod 8
constexpr int kMaxPoisson = 32;
constexpr int kMaxSortRow = 16384;   // longest row the LDS row sort accepts
constexpr int kStdpBlock = 512;      // threads of the slice STDP kernel
constexpr int kStdpBatch = 512;      // rows whose segments are staged at once
constexpr int kStdpUnroll = 4;       // elements per thread with loads in flight
constexpr int kStdpWindow = kStdpBlock * kStdpUnroll;  // elements per segment map
constexpr int kGlobalMaxBlocks = 2048;
constexpr int kLdsBytes = 160 * 1024;
// slice widths are bounded by the 8-byte accumulators in LDS, so a slice-local
// index (compressed targets) always fits 16 bits
static_assert(kLdsBytes / 8 <= 65536, "slice-local index must fit 16 bits");
// Spike histories: hw 64-bit words per neuron (1 or 2), neuron-major; word 0
// bit b = step t-b, word 1 bit b = step t-64-b. A plastic row is forced once
// its last update is 64 hw steps old, so every window fits the history.
constexpr int kMaxHistWords = 2;
constexpr int kMaxAge = 64 * kMaxHistWords;

// Delivered inputs are accumulated exactly as 64-bit fixed-point integers with
// 32 fractional bits (sums of |x| < 2^31 mV, resolution 2^-32 mV); integer
// atomics make the sum independent of the order of the atomic updates.
constexpr float kFixScale = 4294967296.0f;        // 2^32
constexpr float kFixUnit = 2.3283064365386963e-10f; // 2^-32

// Per-block statistics slots of the STDP kernel.
enum StdpStat { kStRows = 0, kStForced = 1, kStSyn = 2, kStForcedSyn = 3, kStFields = 4 };

// Global counters.
enum GlobalStat { kGSpikes = 0, kGNaiveSyn = 1, kGSteps = 2, kGFields = 8 };

// Error bits raised by kernels (device int32, ORed).
enum DevError {
    kErrIndex = 1, kErrRowTooLong = 2, kErrWindow = 4, kErrRing = 8,
    kErrLookback = 16  // a list scan waited too long for an earlier workgroup
};

// Per-step scalars, kept on the device (one struct in the workspace). Every
// kernel of a step reads them there rather than from its launch arguments,
// and the neuron update advances the step index, so the launches of a step
// are the same whatever step they run (a captured step replays correctly).
struct StepClock {
    long long t;           // neuron updates run so far: the index of the next step
    int32_t input_forced;  // 1: the next neuron update reads the fp32 input `ain`
    int32_t n_parts;       // 0: it adds this many fixed-point partial sums instead
    long long pad_[2];
};

// Look-back status words of the list scans, one per workgroup (and step of
// a multi-step launch): bits 0-23 and 24-47 two counts, bits 48-61 the step
// they belong to (mod 2^14), bits 62-63 the kind: the workgroup's own counts
// (aggregate) or those of it and every workgroup before it (inclusive).
constexpr unsigned long long kStatusAgg = 1ull << 62;
constexpr unsigned long long kStatusInc = 2ull << 62;
constexpr int kLookbackSpins = 1 << 16;  // bound of the wait for an earlier workgroup (rounds)
constexpr int kLookbackDelay = 16;       // s_sleep units (64 clocks) before the first read

struct NeuronArgs {
    float *v;
    int32_t *ref;
    float *ie, *ii;
    uint64_t *hist;
    float *ypost;
    const int32_t *t_last;
    const long long *apart; // fixed-point partial inputs [n_parts][nacc][n]
    const float *ain;       // fp32 input [nacc][n], used when clk->input_forced
    int64_t part_stride;    // nacc * n
    int32_t max_parts;      // most partial sums a delivery writes (the chunk count)
    StepClock *clk;         // step index and input source (advanced by the update)
    uint64_t *mask;         // spikes emitted at t
    uint64_t *txmask;       // spikes transmitted at t (emitted at t-D+1)
    uint8_t *code;          // per neuron: 0 no spike in the last 64 steps, 1 + i one spike
                            // at step t-i, kCodeMulti more than one (see k_neuron)
    uint64_t *recent;       // neurons with a spike in the last 64 steps (hist != 0)
    int32_t n, n_exc, model, n_plastic_rows, dm1, ref_steps, poisson_len, hw;
    float k_m, v_th, v_reset, v_inf, d_e, d_i, j_ext, d_minus;
    uint32_t fire_thr;
    uint64_t seed;
    uint32_t poisson[kMaxPoisson];  // entries past poisson_len: the largest word
};

struct RowInfo;

// The lists k_neuron builds: spikes of step t (into the delay ring), forced
// plastic rows, and the snapshots of the rows to update at t. The lists are
// ascending: each workgroup's stretch starts at the counts of all earlier
// workgroups, which it learns by a decoupled look-back over their status
// words; the last workgroup publishes the counts and advances the step.
struct CompactArgs {
    int32_t *ring, *ring_cnt;      // delay ring: D lists of n and D counts; step t: slot t mod D
    // the number of rows transmitting at t (the count of ring slot
    // (t-D+1) mod D) at a fixed address, so that the synapse pass needs no
    // load that waits for the clock to find it
    int32_t *tx_cnt;
    int32_t *row_list, *row_cnt;   // forced plastic rows
    unsigned long long *status;    // look-back status words, one per workgroup
    // position of each neuron in the spike list of the step it last fired
    // (only D > 1 with plasticity): [D][n], slot of the step as in the ring
    int32_t *spk_pos;
    int64_t *gstats;
    int32_t n, nw, n_plastic_rows, hw, delay;
    // snapshots of the plastic rows to update at step t (see RowInfo): forced
    // rows aligned with row_list; transmitting rows aligned with the
    // delay-ring list of step t-D+1 (txinfo[r].k = that list's entry r)
    RowInfo *info;
    RowInfo *txinfo;
    const int64_t *row_ptr;
    const int32_t *pend;
    const uint64_t *hist;
    const int32_t *t_last;
    const float *xpre;
    int32_t *err;
    int64_t *info_stats;     // [gridDim.x][kStFields]
    // target-range segments of the forced rows (see StdpArgs::segb), when
    // segb is given: segment x < xparts of row k ends at pivot
    // piv[k][xcd_piv[x + 1]]
    int32_t *segb;
    const int32_t *piv;
    int32_t piv_stride, xparts;
    int32_t xcd_piv[kXcds + 1];
    float dpow[kMaxAge + 1];
};

// Snapshot of one row to bring up to date, taken before the synapse pass;
// the pass reads only snapshots, so the workgroup that commits t_last and
// xpre never races with another that still needs the old values.
struct RowInfo {
    long long rs;    // first edge of the row
    int32_t k;       // row (source neuron)
    int32_t len;     // plastic prefix length; 0 = nothing to do
    int32_t age_pre; // age (1 .. 64 hw) | pre << 8
    float xp0;       // pre trace at the previous update
    float xp_now;    // pre trace after this update
    int32_t pad;
};

struct RowInfoArgs {
    const int32_t *rows;     // list mode: rows to update; nullptr in flush mode
    const int32_t *row_cnt;
    int32_t n_rows_all;      // flush mode: rows 0 .. n_rows_all-1
    int32_t dm1, hw;
    const StepClock *clk;    // flush: rows are brought up to the last completed step
    const int64_t *row_ptr;
    const int32_t *pend;
    const uint64_t *hist;
    const int32_t *t_last;
    const float *xpre;
    RowInfo *info;
    int32_t *err;            // kErrWindow when a row fell more than 64 hw steps behind
    int64_t *stats;          // [gridDim.x][kStFields]
    float dpow[kMaxAge + 1]; // d_plus^i, i = 0..kMaxAge
};

struct StdpArgs {
    const RowInfo *info;
    const int32_t *row_cnt;  // list mode row count (nullptr: flush, n_rows_all)
    // tx_rows: the rows are the transmitted spikes of step t (info = their
    // snapshots, tx_cnt their count)
    int32_t tx_rows;
    const int32_t *tx_cnt;
    int32_t n_rows_all;
    int32_t n_info;  // entries of info (snapshot loads are clamped to it)
    int32_t *t_last;         // committed here: t_last = t, xpre = xp_now
    float *xpre;
    const StepClock *clk;    // t = clk->t - 1: the step whose neuron update ran last
    const int32_t *col;      // synapse targets (sorted per row)
    float *w;                // synapse weights
    const int32_t *piv;      // [n][S+1] delivery pivots, used at multiples of `mult`
    const uint64_t *hist;
    const float *ypost;
    int32_t n, n_slices, mult, width, n_groups, chunks, n_work, target_limit, hw;
    int32_t event;           // 1: replay only the set history bits; 0: every step (lazy only)
    float c_pot, c_dep, mu;
    int64_t *stats;          // [gridDim.x] weights written
    // row-wise layout: per-neuron history codes or the spike-recency bitmap
    // staged in LDS (at most one of them; both nullptr: gather everything)
    const uint8_t *code;
    const uint64_t *recent;
    int32_t nw;              // words of `recent`
    int32_t parts;           // row-wise layout: waves sharing one row (>= 1)
    // Forced rows partitioned by target range over the XCDs (xcd != 0): the
    // plastic targets are cut into xparts (2, 4 or 8) ranges of whole
    // slices, [xlo[x], xlo[x+1]); range x belongs to the 8 / xparts XCDs
    // b mod 8 in [x 8 / xparts, (x + 1) 8 / xparts), whose waves bring up
    // to date the entries of every forced row with targets in range x: the
    // target histories they gather stay in those XCDs' L2, and they stage
    // the history codes of range x only. The entries of forced row r (list
    // position) in range x are segb[8 r + x - 1] (0 for x = 0) ..
    // segb[8 r + x] - 1, boundaries moved to 128-byte lines of the weight
    // array so that no line is shared by two ranges (a target next to a
    // boundary may fall outside the range: it is gathered).
    int32_t xcd, xparts;
    const int32_t *segb;
    int32_t xlo[kXcds + 1];
    // the forced rows of a source block (SourceArgs): info holds row_cnt of
    // them, info2 the last step's (row_cnt2); histories from hq by the step
    // of each (RowInfo::pad) of the block's `steps`; nothing is committed
    const RowInfo *info2;
    const int32_t *row_cnt2;
    const uint64_t *hq, *hcode;
    int32_t steps;
    float dpow[kMaxAge + 1];
};

struct DeliverArgs {
    const int64_t *row_ptr;
    const int32_t *col;
    float *w;
    const int32_t *piv;      // [n][S+1]
    // the transmitted spikes of step t = clk->t - 1: delay-ring slot
    // (t - D + 1) mod D (a delay block: slots of its steps)
    const int32_t *ring, *ring_cnt;
    const int32_t *tx_cnt;   // the transmitted spikes' count of the step (see CompactArgs)
    StepClock *clk;
    long long *apart;        // fixed-point partial inputs [C][nacc][n]
    float *ain;              // fp32 input [nacc][n], written directly when C == 1
    int64_t part_stride;
    int32_t n, n_exc, width, n_slices, chunks, nacc, n_work, hw;
    const uint16_t *col16;   // compressed targets: slice-local indices (nullptr: read `col`)
    int32_t busy_chunks, busy_from;  // fused pass: workgroups per slice of steps from so many
                                     // spikes on (busy_chunks <= chunks: as in every step)
    int64_t *stats;          // [gridDim.x][2]: events delivered, weights written
    int32_t delay;
    // delay block (k_deliver_block): the inputs of its steps; n_work counts
    // the items (step, slice)
    long long *abatch;       // [steps][nacc][n]
    // plasticity of the transmitting rows, fused into slice delivery
    int32_t plastic;         // 0: no plastic rows
    int32_t event;           // as in StdpArgs
    const RowInfo *txinfo;   // aligned with the transmitted list
    const uint64_t *hist;
    const float *ypost;
    int32_t *t_last;
    float *xpre;
    float c_pot, c_dep, mu;
    float dpow[kMaxAge + 1];
};

// Naive plasticity (every plastic synapse every step, per-synapse traces).
struct NaiveArgs {
    const int64_t *row_ptr;
    const int32_t *pend;     // plastic prefix length per row
    const int32_t *col;
    float *w;
    float *sx_pre, *sx_post; // per-synapse pre and post traces
    const uint64_t *mask;    // spikes of step t (post)
    const uint64_t *txmask;  // spikes transmitted at t (pre)
    int32_t n_rows, nw;
    float d_plus, d_minus, c_pot, c_dep, mu;
    int64_t *stats;          // [gridDim.x] weights written
    int64_t *syn_count;      // synapse updates (one counter)
};

struct GraphArgs {
    int64_t *row_ptr;        // n+1
    int32_t *col;
    uint16_t *col16;         // compressed targets (encoded from col), or nullptr
    float *w;
    int32_t *piv;
    int32_t *pend;
    int32_t *err;
    int32_t *maxlen;
    uint64_t seed;
    int32_t n, n_exc, width, n_slices, plastic, fanout;
    uint32_t thr;
    float w_exc, w_inh;
};

// Building the rows by buckets of 2^shift consecutive rows (k_bucket_count,
// k_bucket_place, k_bucket_sort): of an edge list, or (fanout > 0) of rows of
// that many targets already in place, which are only sorted.
struct BucketArgs {
    const int32_t *src, *dst;
    const float *w;
    int64_t e;
    int64_t *start;   // [nb + 1]: first edge of each bucket (counted into start + 1, then scanned)
    int64_t *cursor;  // [nb]: next free place of each bucket
    int64_t stretch;  // edges per workgroup of the counting and placing kernels
    int32_t grid;     // their workgroups
    int32_t nb, shift, fanout;
    uint32_t scale;   // target range of a row: mulhi(target, scale)
};
constexpr int kBucketShift = 8;     // most rows per bucket: 2^8 (row in the top byte of a word)
constexpr int kBucketAim = 5120;    // edges per bucket aimed at
// fewest buckets aimed at: one workgroup of the sort fits a CU and costs about
// 6 us however few its edges (its ranges' counters), so small graphs take one
// round of up to 256 (2,000 rows of 20 edges: 172.8 us with 512, 155.5 with 128)
constexpr int kBucketFew = 128;
constexpr int kBucketCap = 12288;   // most edges a bucket can have (LDS: 8 B each)
constexpr int kBucketSubs = 8192;   // target ranges per bucket (LDS: 4 B each)
constexpr int kBucketMax = 32768;   // most buckets (LDS: 4 B each)
// The buckets for n rows and e edges, the longest row max_row if known (else
// 0); false where they do not fit (then: launch_edges_count and so on).
bool choose_buckets(BucketArgs &b, int32_t n, int64_t e, int64_t max_row);
hipError_t launch_bucket_count(hipStream_t s, const GraphArgs &a, const BucketArgs &b);
hipError_t launch_bucket_place(hipStream_t s, const GraphArgs &a, const BucketArgs &b);
hipError_t launch_bucket_sort(hipStream_t s, const GraphArgs &a, const BucketArgs &b);

// Several whole steps of a small network without plasticity in one launch of
// one workgroup (k_small_steps): neuron update, spike list into the delay
// ring, and delivery into an LDS accumulator that the next step's neuron
// update reads, so no step waits for a kernel boundary or an HBM round trip.
struct SmallArgs {
    int32_t *ring, *ring_cnt;   // delay ring: D lists of n, D counts
    int32_t delay;
    const int64_t *row_ptr;
    const int32_t *col;
    const float *w;
    long long *apart;           // after the last step: part 0 = the pending input
    int64_t *gstats;            // kGSpikes
    int64_t *dlv_stats;         // slot 0: events delivered
    // the list scans' status words, cleared at the end (the steps run here
    // leave stale step tags in them)
    unsigned long long *status;
    int32_t status_words;
    int32_t n_exc, nacc, steps;
    int32_t lds_rows;           // 1: the row pointers are staged in LDS (32 bits each)
};
// steps per launch from which staging the row pointers pays (one step reads
// each spike's pair once)
constexpr int kSmallStage = 4;
constexpr int kSmallBlock = 1024;
constexpr int kSmallRounds = 4;     // neurons per thread: n <= 4096
constexpr int kSmallMaxAcc = 8192;  // nacc * n accumulators (64 KiB of LDS)
constexpr int kSmallChunk = 4096;   // steps per launch

// One launch per step of a network without plasticity and D = 1
// (k_step_one): deliver the spikes of the step before, update the neurons.
struct StepOneArgs {
    const uint64_t *mask_in;  // spikes of the step to deliver (deliver != 0)
    uint64_t *mask_out;       // spikes of the step updated (last == 0)
    int32_t deliver, last;    // last: deliver only, and leave the state as after snn_step
    int32_t step;             // the step updated is clk->t + step; last: the call's steps
    int32_t gw, mult;         // targets per workgroup: mult slices
    int32_t n_slices;
    int32_t lg_team;          // log2 of the lanes that share one row
    const int64_t *row_ptr;
    const int32_t *col;
    const float *w;
    const int32_t *piv;       // [n][n_slices + 1]
    int32_t *ring, *ring_cnt, *tx_cnt;
    int32_t parts;            // workgroups per group of targets at most ...
    int32_t per_part;         // ... one for every per_part spikes of the step
    int32_t *arrived;         // [groups]: parts of the launch that have ended (0 before it)
    long long *apart;         // the parts' sums; part 0: the pending input after the last step
    int64_t *gstats, *dlv_stats;
    int32_t dlv_slots;
    unsigned long long *status;
    int32_t status_words;
};
constexpr int kOneMaxN = 65536;  // a mask word per thread
constexpr int kOneMaxW = 4096;   // targets per workgroup
constexpr int kOneMaxParts = 16;
// Work of a part: entries, and kOneRow more per row. An exchange of sums costs
// about 2.5 us and a workgroup adds 1.7 entries per ns: 5,003 neurons (250 spikes
// of 100 entries at most) take 10.4, 8.9, 8.3 and 7.6 us per step with 2,048, 4,096,
// 6,144 and 12,288; groups of 4,096 targets (62,500 neurons, 16 groups) do not
// tell them apart: 20.9 (27 whole, 20.0 separately).
constexpr int kOnePart = 12288;
constexpr int kOneRow = 6;
hipError_t launch_step_one(hipStream_t s, const NeuronArgs &a, const StepOneArgs &b);

// Delay-blocked steps of a network without plasticity and delay D >= 2
// (k_neuron_steps after k_deliver_block). The input of step t comes
// from the spikes of step t-D only, so the inputs of steps t0+1 .. t0+B
// (B <= D-1) depend on spikes already in the delay ring when step t0
// starts: one delivery launch computes all B of them, then one neuron
// launch runs steps t0 .. t0+B-1, each thread keeping its neuron's state in
// registers across the B steps.
struct BatchArgs {
    int32_t *ring, *ring_cnt;   // delay ring: D lists of n, D counts
    int32_t delay;
    unsigned long long *status; // [kBatchMax][status_stride] look-back status words (step
                                // k of the block: row k, one word per workgroup)
    int32_t status_stride;
    const long long *abatch;    // [B][nacc][n] fixed-point inputs of steps t0+1 .. t0+B
    long long *apart;           // partial 0 receives the input of step t0+B
    int64_t *gstats;            // kGSpikes
    int32_t *err;
    int32_t steps;
};
constexpr int kBatchMax = 16;  // steps per delay block
// steps per delay block for neuron model m (CUBA: two inputs per step)
constexpr int batch_steps_max(int m) { return m == 1 ? kBatchMax / 2 : kBatchMax; }
constexpr int64_t kBatchBytes = 256ll << 20;  // most workspace for a block's partial inputs

// Blocks of steps of a plastic network with D >= 2 (k_block_plan, then
// k_block_run). Delivery at step t sends the spikes emitted at t-D+1, and
// the weight of synapse k->j at t depends only on the pre spikes of k that
// arrived by t (emitted by t-D+1) and on the post spikes of j. So the rows
// to bring up to date and to deliver at each of the steps t0 .. t0+B-1
// (B <= D-1) follow from the histories when t0 starts, and a workgroup that
// owns a range of targets can run all B steps alone: the neuron update of
// its targets, then the plasticity and delivery of every listed row's
// entries that fall in its range, into an accumulator in LDS that its next
// neuron update reads. No workgroup waits for another within the block.
//   The plan (one thread per row) walks each row through the block's steps
// as the neuron update would (transmitting: history bit D-1 of the step;
// forced: idle for 64 hw steps), and writes each step's list of row updates
// (PbEvent), each workgroup's share placed by one atomic add per list, and
// commits t_last and x_pre after the block. A forced update that is its row's last
// event of the block delivers nothing and no later event of the block reads
// its weights: it goes to one more list, the deferred updates, which the run
// computes after the block's last step from the targets' histories at the
// update's step (the history at block start and the block's spike bits). A group finds a row's entries with
// targets in the group from the pivot table at group granularity
// (gpiv[k][g] = the row-relative first entry of row k with a target >=
// g gwidth, g = 0..n_groups; the pivot kernel with gwidth for the slice
// width). After the last
// block of a call, the deferred launch also rebuilds what the step-by-step
// path keeps per step: the delay-ring lists of the last D steps with their
// positions and the forced-row list of the last step, from masks the run and
// the plan leave; and clears the list scans' status words.
struct BlockClock {
    long long t0;          // the block's first step
    int32_t input_forced;  // the input of step t0, as the step clock said
    int32_t n_parts;
    long long pad_[2];
};
// One row to bring up to date (and deliver) at a step of a block.
struct PbEvent {
    int32_t rs;      // first edge of the row
    uint32_t lenf;   // plastic prefix length (bits 0-15), age (16-23), pre spike (24),
                     // transmitting (25), inhibitory source of a CUBA network (26),
                     // step in the block (27-30), an event at the step before too (31)
    float xp0;       // pre trace at the row's previous update
    int32_t k;       // the row
};
constexpr int kPbPlanBlock = 512;   // threads of the plan (one row each, a half wave per step's scan)
constexpr int kPbBlock = 512;       // threads of a target group's workgroup
constexpr int kPbMaxWidth = 256;    // most targets per group (one neuron per thread)
constexpr int kPbRecords = 4096;    // a block's records a workgroup holds in LDS
constexpr int kPbMaxN = 65536;      // largest network the blocks run
constexpr int kPbMaxSteps = kBatchMax - 1;  // steps per block: lists 0 .. B-1, deferred list B
constexpr int kPbDfPart = 8 * 64;   // entries per part of a deferred row (8 per lane)
static_assert(kPbPlanBlock / 32 >= kPbMaxSteps + 1, "a half wave per list scan");
static_assert(kPbMaxSteps < 16, "step in the block fits PbEvent::lenf");
struct BlockArgs {
    // plan
    const int64_t *row_ptr;
    const int32_t *pend;
    const uint64_t *hist;
    int32_t *t_last;
    float *xpre;
    unsigned long long *status;  // look-back words of the step-by-step kernels (the finish
    int32_t status_stride;       // clears them)
    PbEvent *ev;                 // [steps + 1][n]: step k's rows at ev + k n, the deferred
                                 // forced updates at ev + steps n
    int32_t *ev_cnt;             // [kBatchMax]: the lists' lengths (0 when the plan starts)
    int32_t *ev_cnt_next;        // [kBatchMax]: the other block's, cleared by the plan
    uint8_t *dcode;              // [n, padded to 16] run -> deferred: per target, the first
                                 // spike step of the block (bits 0-3), the latest spike before
                                 // it against a forced window (4-7)
    uint64_t *hq;                // [n][2 hw] run -> deferred: history words at block start,
                                 // then the block's spikes (bit 0: its last step)
    int32_t *df_cnt;             // run -> deferred: the deferred list's length
    uint64_t *dmask;             // [D + 1][mask words]: run -> lists, spikes of the last D steps
                                 // (row q: step t0 + B - 1 - q); plan -> lists, row D: the
                                 // forced rows of the block's last step
    int32_t fin_blocks;          // D + 1 after a call's last block: the deferred launch also
                                 // rebuilds the per-step lists; else 0
    int32_t n_cu;
    int32_t df_parts;            // parts of kDfPart entries of the longest row (deferred)
    BlockClock *bclk;            // written by the plan, read by the run
    StepClock *clk;              // read by the plan, advanced by the run
    int64_t *info_stats;         // plan: rows, forced rows, synapses (kStFields per slot)
    int32_t info_slots;
    int32_t *err;
    int32_t steps, n, n_exc, n_plastic_rows, hw, delay, nacc;
    // run
    const int32_t *col;
    const uint16_t *col16;       // compressed targets (slice-local), or nullptr
    float *w;
    const int32_t *gpiv;         // [n][n_groups + 1]
    int64_t n_edges;
    int32_t gwidth, width, n_groups;
    long long *apart;            // partial 0 receives the input of step t0 + B
    int64_t part_stride;
    int64_t *dlv_stats;          // [dlv_slots][2]: events delivered, weights written (transmitting rows)
    int32_t dlv_slots;
    int64_t *syn_stats;          // [syn_slots]: weights written (forced rows)
    int32_t syn_slots;
    int64_t *gstats;
    int32_t event;               // 1: replay only the set history bits; 0: every step
    float c_pot, c_dep, mu;
    // lists after the last block
    int32_t *ring, *ring_cnt, *spk_pos, *rows, *row_cnt;
    uint64_t *mask, *txmask, *recent;
    int32_t status_words;
    float dpow[kMaxAge + 1];
};
// Blocks of steps of a plastic network of Bernoulli sources with D = 1
// (k_source_steps, then k_source_run). A source fires on a counter-based draw
// that no input changes, so one launch runs the neuron update of B steps:
// each thread walks its neuron through them (spike, history, post trace) and
// its row through the updates of each step (transmitting, or forced by the
// history window), with t_last and x_pre carried in registers from one update
// to the next, and commits them after the block. It writes
//   - per step the rows to deliver or, forced and with a later event in the
//     block, to bring up to date only (ascending, with their snapshots; the
//     place of each chunk of rows in the list: `split`);
//   - the other forced rows of the block (all but the last step's) in one
//     list: no later event of the block reads their weights, so they can be
//     brought up to date at any time during it;
//   - each neuron's history words before the block with its spikes in it
//     (hq), and who fired at all in either (recent);
//   - the histories and post traces after the block's first step.
// The last step's lists, snapshots, counts, masks and the clock are those of
// the state, so after the block the state is that of the step-by-step path.
// k_source_run then runs the synapse part of all B steps: a workgroup owns a
// slice and a chunk of the rows through the block, so no workgroup waits for
// another.
struct SourceArgs {
    unsigned long long *status;  // [kBatchMax][status_stride]: step k's scan in row k
    int32_t status_stride;
    int32_t steps;               // B: 1 .. kSrcMaxSteps
    int32_t info_slots;          // statistics slots of CompactArgs::info_stats
    int32_t chunks;              // row chunks (of whole workgroups of k_source_steps)
    uint64_t *hist0;             // [n][hw], post traces [n]: after step 0 (B > 1)
    float *y0;
    uint64_t *hq;                // [n][2 hw]: history words before the block, then its spikes
                                 // (bit 0: the last step)
    uint64_t *code;              // [n]: the same in one word (src_code)
    uint64_t *recent;            // [nw]: fired in the block or in the history before it
    RowInfo *txinfo;             // [B-1][n]: the steps' lists; RowInfo::pad: step | kSrcTx
    RowInfo *dinfo;              // [n_plastic_rows]: forced rows without a later event
    int32_t *dcnt;               // their number
    int32_t *split;              // [kSrcMaxSteps][chunks + 1]
    int32_t *t_last;
    float *xpre;
};
constexpr int kSrcMaxChunks = 64;
constexpr int kSrcTx = 1 << 8;  // RowInfo::pad of a list entry: delivered (step: bits 0-7)
constexpr int kSrcMaxSteps = kBatchMax;  // steps per source block (one scan per half wave)

// The synapse part of a source block (k_source_run): delivery of work items
// (slice, chunk) on workgroups [0, nd), the listed forced rows on the others.
// 704 records of 16 B and a map of 5,632 entries beside a slice of 2,048 targets
// with 128-step histories are 80,384 of the 81,920 B that let two workgroups
// share a CU (each role's time is latency: 16 waves per CU instead of 8).
constexpr int kSrcRecs = 704;   // rows staged at once
constexpr int kSrcU = 11;       // entries per thread and window
constexpr int kSrcMaxW = 4096;  // targets per slice of the form for most networks
constexpr int kSrcWideW = 7168;  // targets per slice whose LDS a workgroup can have
constexpr int64_t kSrcMaxEdges = 1ll << 52;  // (first edge in 32 + 22 bits, signed)
struct SourceRunArgs {
    int32_t n, n_slices, width, chunks, n_work, steps, event;
    int64_t n_edges;
    const int32_t *col;
    const uint16_t *col16;
    float *w;
    const int32_t *piv;
    const uint64_t *hist0, *hq;
    const float *y0;
    const RowInfo *txinfo, *txlast;  // steps before the last; the last
    const int32_t *split;
    long long *apart;
    float *ain;
    StepClock *clk;
    int64_t *stats, *syn_stats, *gstats;
    int32_t stat_slots, syn_slots;
    float c_pot, c_dep, mu, d_minus;
    float dpow[kMaxAge + 1];
};
// LDS of a delivery workgroup
inline size_t source_run_lds(int width, int hw)
{
    return (size_t)kSrcRecs * 16 + (size_t)width * (8 + 8 * hw + 4) +
           (size_t)kSrcU * 512 * sizeof(uint16_t) + 512;
}
hipError_t launch_block_plan(hipStream_t s, const BlockArgs &b);
hipError_t launch_block_run(hipStream_t s, const NeuronArgs &a, const BlockArgs &b);
hipError_t launch_block_deferred(hipStream_t s, const BlockArgs &b);

// Optional events placed by a launch itself around the kernel
// (hipExtLaunchKernelGGL): its device time without marker or dispatch gaps.
struct KernelEvents {
    hipEvent_t start = nullptr, stop = nullptr;
};
// timed parts of a step: neuron update with its lists, plasticity, delivery
constexpr int kTimedParts = 3;
// k_source_steps (see SourceArgs) and its workgroups for n neurons
hipError_t launch_source_steps(hipStream_t s, const NeuronArgs &a, const CompactArgs &c,
                               const SourceArgs &b, KernelEvents ev = {});
int source_steps_grid(int32_t n);

// ---- launchers (k_*.hip); all enqueue on `s` and return the launch
// status of the last kernel they started.
hipError_t launch_init_state(hipStream_t s, float *v, int32_t *ref, float *ie, float *ii,
                             uint64_t *hist, float *ypost, int32_t *t_last, float *xpre,
                             int32_t n, int32_t hw);
hipError_t launch_fill_f32(hipStream_t s, float *p, int64_t count, float value);
hipError_t launch_fill_i64(hipStream_t s, int64_t *p, int64_t count, int64_t value);
hipError_t launch_fill_i32(hipStream_t s, int32_t *p, int64_t count, int32_t value);
hipError_t launch_fill_ll(hipStream_t s, long long *p, int64_t count, long long value);
hipError_t launch_copy_bytes(hipStream_t s, void *dst, const void *src, int64_t bytes);
// k_small_steps: steps a.t .. a.t + b.steps - 1 (a describes step a.t)
hipError_t launch_small_steps(hipStream_t s, const NeuronArgs &a, const SmallArgs &b,
                              KernelEvents ev = {});
hipError_t launch_neuron(hipStream_t s, const NeuronArgs &a, const CompactArgs &b,
                         KernelEvents ev = {});
// workgroups of k_neuron and k_neuron_steps for n neurons (one status word each)
int neuron_grid(int32_t n);
int neuron_steps_grid(int32_t n);
// k_neuron_steps: steps a.t .. a.t + b.steps - 1 (a describes step a.t)
hipError_t launch_neuron_steps(hipStream_t s, const NeuronArgs &a, const BatchArgs &b);
// pos[q n + ring[q n + r]] = r for every delay-ring slot q < d and r < its count
hipError_t launch_ring_positions(hipStream_t s, const int32_t *ring, const int32_t *cnt,
                                 int32_t *pos, int32_t n, int32_t d);
hipError_t launch_row_info(hipStream_t s, const RowInfoArgs &a, int64_t max_rows);
hipError_t launch_stdp(hipStream_t s, const StdpArgs &a, int blocks, size_t lds, KernelEvents ev = {});
hipError_t launch_stdp_rows(hipStream_t s, const StdpArgs &a, int blocks, KernelEvents ev = {});
hipError_t launch_stdp_naive(hipStream_t s, const NaiveArgs &a, int blocks, KernelEvents ev = {});
// k_probe_rows: measurement only (sink: one scratch word)
hipError_t launch_probe_rows(hipStream_t s, int blocks, const int64_t *row_ptr,
                             const int32_t *pend, const int32_t *col, float *w, int32_t n_rows,
                             int32_t n_plastic, uint64_t seed, int32_t write,
                             unsigned long long *sink, KernelEvents ev);
constexpr int kStdpRowsBlock = 1024;   // threads of the row-wise STDP kernel
constexpr int kStdpRowsUnroll = 8;     // synapses per lane and row part (64-step histories)
constexpr int kStdpRowsUnroll2 = 8;    // the same with 128-step histories (4: 28.3 against
                                       // 26.4 us for the stress network's fused pass)
constexpr int kStdpXcdUnroll = 4;      // the same in the target-range form (both lengths)
constexpr int kDlvBlock = 512;         // threads per workgroup of slice delivery
constexpr int kDlvBatch = 704;         // spikes whose segments slice delivery stages at once
                                       // (two per thread: 1,250 spikes over two chunks fit
                                       // one batch, 4.5 standard deviations above the mean)
constexpr int kDlvUnroll = 8;          // flattened elements per thread per window
constexpr int kDlvWindow = kDlvBlock * kDlvUnroll;
// Slice delivery's staging arrays, at the start of its dynamic LDS. MapT is
// the element type of the segment map: int, or uint16_t where LDS is tight
// (the fused pass with 128-step histories), at the cost of a few registers.
template <typename MapT>
struct DlvSharedT {
    long long start[kDlvBatch];        // segment starts (edge index)
    long long sh[kDlvBlock / 64];      // scan scratch
    unsigned long long written;        // weights written by the workgroup
    long long total;                   // the scan's running total between its rounds
    int off[kDlvBatch + 1];            // segment offsets in the batch
    // per segment: plastic elements (bits 0-17), row age (bits 18-25: the
    // replay window), inhibitory source of a CUBA network (bit 26)
    int info[kDlvBatch];
    // pre trace at the last update (the trace after this one, x0 d+^age + 1,
    // is computed where it is needed, as the neuron update computed it)
    float xp0[kDlvBatch];
    MapT map[kDlvWindow];              // element -> 1 + segment of the window (0: none)
    float dpow[kMaxAge + 1];           // decay table
    int shi[kDlvBlock / 64];           // scan scratch
    int nlong;                         // segments longer than the direct-map limit
    int pad_[1];
};
using DlvShared = DlvSharedT<int>;
using DlvShared16 = DlvSharedT<uint16_t>;
// the fused pass's map type: 16-bit with 128-step histories (two workgroups
// per CU on the stress network), else int
template <int HW>
using FusedMap = typename std::conditional<HW == 2, uint16_t, int>::type;
inline size_t fused_dlv_shared_bytes(int hw)
{
    return hw == 2 ? sizeof(DlvShared16) : sizeof(DlvShared);
}
static_assert(sizeof(DlvShared) % 16 == 0 && sizeof(DlvShared16) % 16 == 0,
              "the accumulators follow 16-byte aligned");
constexpr int kStoreLine = 32;         // weights per store line of the row-wise STDP (128 B)
constexpr int kStdpRowsSplit = 8;      // most waves that share one row


// LDS of the row-wise STDP workgroup's candidate queues (one per wave: target
// and weight of up to U x 64 synapses)
constexpr int stdp_rows_queue_bytes(int hw)
{
    return (kStdpRowsBlock / kWave) * (hw == 2 ? kStdpRowsUnroll2 : kStdpRowsUnroll) * kWave * 8;
}
// the per-neuron summary it stages beside the queues (160 KB of LDS per workgroup)
constexpr int kCodeMax = 163840 - stdp_rows_queue_bytes(1) - 1024;  // bytes of history codes
// The row-wise STDP kernel runs one workgroup per CU, and the fused synapse
// pass (k_synapse_pass) fills the slots of every CU (one or two workgroups
// per CU, as the LDS of both parts allows): both grids come from the CU
// count of the device (hipDeviceAttributeMultiprocessorCount).
constexpr int fused_queue_bytes(int hw)
{
    return (kDlvBlock / kWave) * (hw == 2 ? kStdpRowsUnroll2 : kStdpRowsUnroll) * kWave * 8;
}
constexpr int kRecentMaxWords = kCodeMax / 8;  // words of the spike-recency bitmap
constexpr uint8_t kCodeMulti = 255;    // history code: two or more spikes in the window
int stdp_static_bytes();  // static LDS of the slice STDP kernel (-1 on error)
// k_deliver_block: workgroups of kDlvBlock threads, kBdBlockMax for few items
constexpr int kBdBlockMax = 1024;
hipError_t launch_deliver_block(hipStream_t s, const DeliverArgs &a, int64_t n_edges);
hipError_t launch_deliver_lds(hipStream_t s, const DeliverArgs &a, int blocks, size_t lds, KernelEvents ev = {});
// k_synapse_pass: slice delivery on workgroups [0, nd) (nd a multiple of 8),
// forced-row STDP on ns more, kDlvBlock threads each; lds covers both
hipError_t launch_synapse_pass(hipStream_t s, const DeliverArgs &d, const StdpArgs &a, int nd,
                               int ns, size_t lds, KernelEvents ev = {});
// k_source_run: nd delivery workgroups (a multiple of 8), ns for the forced rows
hipError_t launch_source_run(hipStream_t s, const SourceRunArgs &d, const StdpArgs &a, int hw,
                             int nd, int ns, size_t lds, KernelEvents ev = {});
int source_run_static_bytes();  // static LDS of k_source_run (-1 on error)
hipError_t launch_deliver_global(hipStream_t s, const DeliverArgs &a, int blocks, KernelEvents ev = {});
int deliver_lds_static_bytes();  // static LDS of the slice kernel (-1 on error)
int synapse_pass_static_bytes();  // static LDS of the fused synapse pass (-1 on error)
// the fp32 input from the partial sums when clk->input_forced is 0 (then
// set to 1 by a second kernel, so that every workgroup reads the flag first)
hipError_t launch_materialize_input(hipStream_t s, const long long *apart, int64_t part_stride,
                                    StepClock *clk, float *ain, int64_t count);
// clk->t = t unless t < 0, the input flags unless input_forced < 0
hipError_t launch_set_clock(hipStream_t s, StepClock *clk, int64_t t, int32_t input_forced,
                            int32_t n_parts);
hipError_t launch_scan_i64(hipStream_t s, int64_t *data, int64_t count, int64_t *bsum);
hipError_t launch_graph_count_bernoulli(hipStream_t s, const GraphArgs &a);
hipError_t launch_graph_fill_bernoulli(hipStream_t s, const GraphArgs &a);
hipError_t launch_graph_fill_fanout(hipStream_t s, const GraphArgs &a);
hipError_t launch_edges_count(hipStream_t s, const GraphArgs &a, const int32_t *src,
                              const int32_t *dst, int64_t e);
hipError_t launch_edges_scatter(hipStream_t s, const GraphArgs &a, const int32_t *src,
                                const int32_t *dst, const float *w, int64_t e,
                                int64_t *cursor);
hipError_t launch_row_maxlen(hipStream_t s, const GraphArgs &a);
hipError_t launch_row_sort(hipStream_t s, const GraphArgs &a, int pow2len);
hipError_t launch_pivots(hipStream_t s, const GraphArgs &a);
// col16 from col (snn_config.compressed_targets): slice-local indices
hipError_t launch_encode_targets(hipStream_t s, const GraphArgs &a, int64_t n_edges);

}  // namespace snn
