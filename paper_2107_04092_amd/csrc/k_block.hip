// gfx950 kernels of a block of steps of a plastic network with D >= 2 (see
// BlockArgs): the plan of the block's rows, the target groups' run of its
// steps, and the per-step lists rebuilt after the last block.
//
// Built with -ffp-contract=off: the neuron update reproduces a fixed fp32
// operation order.
#include "snn_neuron.h"

#include <algorithm>

namespace snn {
namespace {

// ---------------------------------------------------------------------------
// The plan of steps t0 .. t0+B-1 (t0 = clk->t), one thread per row k.
//
// Row k transmits at t when it spiked at t-D+1, which the history word holds
// when the block starts (bit b = step t0-1-b, so bit D-2-q for t = t0+q). A
// plastic row is brought up to date when it transmits, or, idle, once its
// last update is 64 hw steps old (forced), exactly as the step-by-step
// neuron update decides; each such event is a snapshot of the row at its
// step, taken from the t_last and x_pre that the row's earlier events in the
// block left. A row is forced at most once per block (64 hw > B steps apart)
// and only before its first transmission; a forced update that is the row's
// last event of the block goes to the deferred list (list B) instead of its
// step's. The steps are walked twice: once for the event flags (each list's
// count in the workgroup, which one atomic add per list turns into the
// workgroup's place in the list), then for the snapshots (PbEvent), written
// at their positions. A list is ascending inside each workgroup's share; the
// shares come in the order the workgroups arrive, and no result depends on
// the order (the run accumulates in exact fixed point and every synapse's
// update is its own).

__global__ __launch_bounds__(kPbPlanBlock) void k_block_plan(BlockArgs b)
{
    constexpr int NWV = kPbPlanBlock / kWave;
    __shared__ uint64_t s_m[kBatchMax][NWV];
    __shared__ int s_lb[kBatchMax];
    __shared__ int s_wp[kBatchMax][NWV];  // events of list q in the waves before
    __shared__ int s_rq[NWV][kWave];      // a wave's lanes with an event
    __shared__ float s_dpow[kMaxAge + 1];
    __shared__ unsigned long long s_st[kStFields];
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int k = blockIdx.x * kPbPlanBlock + tid;
    const bool live = k < b.n;
    const bool plastic = k < b.n_plastic_rows;  // (n_plastic_rows <= n)
    const int B = b.steps, D = b.delay, hw = b.hw;
    // the row's values, then the clock: one round trip
    uint64_t h0 = 0ull;
    int64_t rs = 0;
    int tl0 = 0, pend_k = 0;
    float xp0 = 0.f;
    if (live) {
        h0 = b.hist[(int64_t)k * hw];
        rs = b.row_ptr[k];
    }
    if (plastic) {
        tl0 = b.t_last[k];
        xp0 = b.xpre[k];
        pend_k = b.pend[k];
    }
    const StepClock ck = load_clock(b.clk);
    const int64_t t0 = ck.t;
    if (blockIdx.x == 0 && tid == 0) {
        BlockClock bc{};
        bc.t0 = t0;
        bc.input_forced = ck.input_forced;
        bc.n_parts = ck.n_parts;
        *b.bclk = bc;
    }
    for (int q = tid; q <= kMaxAge; q += kPbPlanBlock) s_dpow[q] = b.dpow[q];
    if (tid < kStFields) s_st[tid] = 0ull;
    // the steps with an event, and the deferred one
    uint32_t evm = 0, fm = 0;
    {
        int tl = tl0;
        for (int q = 0; q < B; ++q) {  // uniform
            const int64_t t = t0 + q;
            const bool tx = live && ((h0 >> (D - 2 - q)) & 1ull);
            bool ev = tx;
            if (plastic) {
                if (tx) {
                    if (t - (int64_t)tl > 0) tl = (int)t;
                } else if (t - (int64_t)tl >= 64 * hw) {
                    ev = true;
                    fm |= 1u << q;
                    tl = (int)t;
                }
            }
            evm |= (uint32_t)ev << q;
        }
    }
    // (a forced update is the row's last event when no higher bit is set)
    const uint32_t dfm = fm != 0u && (evm >> (__ffs((int)fm))) == 0u ? fm : 0u;
    if (b.fin_blocks) {  // the forced rows of the call's last step, for the lists after it
        const uint64_t m = ballot64((fm >> (B - 1)) & 1u);
        const int word = blockIdx.x * NWV + wave;
        if (lane == 0 && word * kWave < b.n)
            b.dmask[(int64_t)D * ((b.n + kWave - 1) / kWave) + word] = m;
    }
    for (int q = 0; q <= B; ++q) {  // uniform
        const bool ev = q < B ? ((evm & ~dfm) >> q) & 1u : dfm != 0u;
        const uint64_t m = ballot64(ev);
        if (lane == 0) s_m[q][wave] = m;
    }
    __syncthreads();  // s_m, s_dpow, s_st
    // this workgroup's place in list tid; the other block's counts cleared
    // for the next plan (the launches that read them have ended)
    if (tid <= B) {
        int own = 0;
        for (int w = 0; w < NWV; ++w) {
            s_wp[tid][w] = own;
            own += __popcll(s_m[tid][w]);
        }
        s_lb[tid] = own ? atomicAdd(b.ev_cnt + tid, own) : 0;
    }
    if (blockIdx.x == 0 && tid < kBatchMax) b.ev_cnt_next[tid] = 0;
    __syncthreads();  // s_lb
    // the snapshots, at their positions (the workgroup's place in the list,
    // then earlier waves, then earlier lanes). A wave's rows with an event
    // are compacted first: a lane walks one such row's events in order (each
    // snapshot starts from the one before), with the wave's lanes busy.
    const uint64_t hm = ballot64(evm != 0u);
    if (evm != 0u) s_rq[wave][lane_rank(hm)] = lane;
    __builtin_amdgcn_wave_barrier();
    const int nq = (int)__popcll(hm);  // wave-uniform
    const int src = lane < nq ? s_rq[wave][lane] : lane;
    const int kr = blockIdx.x * kPbPlanBlock + wave * kWave + src;  // the lane's row
    const uint32_t r_evm = (uint32_t)__shfl((int)evm, src);
    const uint32_t r_dfm = (uint32_t)__shfl((int)dfm, src);
    const uint64_t r_h0 = (uint64_t)__shfl((long long)h0, src);
    const int64_t r_rs = (int64_t)__shfl((long long)rs, src);
    const int r_tl0 = __shfl(tl0, src), r_pend = __shfl(pend_k, src);
    const float r_xp0 = __shfl(xp0, src);
    const bool r_plastic = kr < b.n_plastic_rows;
    const uint64_t below = src == 0 ? 0ull : (~0ull >> (64 - src));
    int tl = r_tl0;
    float xp = r_xp0;
    long long n_rows = 0, n_forced = 0, n_syn = 0, n_fsyn = 0;
    for (uint32_t m = lane < nq ? r_evm : 0u; m; m &= m - 1u) {
        const int q = __ffs((int)m) - 1;
        const int64_t t = t0 + q;
        const int tx = (int)((r_h0 >> (D - 2 - q)) & 1ull);
        RowInfo ri = RowInfo{};
        int ok = 0;
        if (r_plastic) {
            ok = make_row_info_d(ri, kr, t, tl, r_rs, r_pend, xp, tx, hw,
                                 s_dpow[row_age_index(t, tl, hw)], b.err);
            if (ok) {
                tl = (int)t;
                xp = ri.xp_now;
                n_rows += 1;
                n_syn += ri.len;
                if (!tx) {
                    n_forced += 1;
                    n_fsyn += ri.len;
                }
            }
        }
        // nothing to bring up to date (ok == 0): the row is only delivered
        PbEvent pe;
        pe.rs = (int32_t)r_rs;
        pe.lenf = ok ? ((uint32_t)ri.len & 0xffffu) | ((uint32_t)(ri.age_pre & 0xff) << 16) |
                           ((uint32_t)((ri.age_pre >> 8) & 1) << 24)
                     : 0u;
        pe.lenf |= ((uint32_t)tx << 25) | ((uint32_t)(b.nacc == 2 && kr >= b.n_exc) << 26) |
                   ((uint32_t)q << 27) | (q > 0 ? ((r_evm >> (q - 1)) & 1u) << 31 : 0u);
        pe.xp0 = ok ? ri.xp0 : 0.f;
        pe.k = kr;
        const int lq = (r_dfm >> q) & 1u ? B : q;  // the list
        const int pos = s_lb[lq] + s_wp[lq][wave] + (int)__popcll(s_m[lq][wave] & below);
        // (the counts of a list never exceed n unless they did not start at 0)
        if (pos < b.n)
            b.ev[(int64_t)lq * b.n + pos] = pe;
        else
            atomicOr(b.err, kErrRing);
    }
    if (lane < nq && r_plastic && tl != r_tl0) {  // the row as its last event left it
        b.t_last[kr] = tl;
        b.xpre[kr] = xp;
    }
    n_rows = wave_sum_i64(n_rows);
    n_forced = wave_sum_i64(n_forced);
    n_syn = wave_sum_i64(n_syn);
    n_fsyn = wave_sum_i64(n_fsyn);
    if (lane == 0) {
        if (n_rows) atomicAdd(s_st + kStRows, (unsigned long long)n_rows);
        if (n_forced) atomicAdd(s_st + kStForced, (unsigned long long)n_forced);
        if (n_syn) atomicAdd(s_st + kStSyn, (unsigned long long)n_syn);
        if (n_fsyn) atomicAdd(s_st + kStForcedSyn, (unsigned long long)n_fsyn);
    }
    __syncthreads();  // s_st complete
    if (tid < kStFields && s_st[tid])
        add_stat(b.info_stats + (int64_t)(blockIdx.x % b.info_slots) * kStFields + tid,
                 (long long)s_st[tid]);
}

// ---------------------------------------------------------------------------
// The run of the block: workgroup of target group g (targets [g gw, g gw +
// gw), gw = gwidth, inside one slice), every step t = t0 + q:
//   (1) the neuron update of the group's targets (thread j: neuron g gw + j,
//       its state in registers from the first step to the last), with the
//       input of step t: the state's input at t0, afterwards the LDS
//       accumulator; the new history words and post traces go to LDS;
//   (2) the step's rows (the plan's list): of each, the entries with a target
//       in the group; the plastic ones brought up to date from the target's
//       history in LDS (a forced row: only those; its other entries are not
//       read), and a transmitting row's entries added to the accumulator
//       (64-bit fixed point, LDS atomics), which step t+1's neuron update
//       reads.
// A synapse belongs to the group of its target, so each weight is read and
// written by one workgroup only, and the steps of a workgroup are ordered by
// its barriers.
//
// What bounds it is the chain of one step (a step of the 25,000-neuron Brunel
// network has 700 entries per group), so everything that does not depend on
// the step before is taken out of it:
//   - the rows' records of all steps are loaded into LDS first (start of the
//     group's entries, plastic length, age, flags, pre trace), the entries
//     flattened over all of them by one scan, and a map from each flattened
//     entry to its record written once; a step only walks its stretch of the
//     map, with no staging of its own;
//   - the entries of step q+1 are loaded before those of step q are computed
//     (two register sets in turn), every slot from a valid address so that
//     the loads in flight are counted, not guessed. A row with an event in
//     both steps would be loaded before its store: the plan marks such a
//     record (late), and its weights are loaded again after the barrier;
//   - the external drive of several steps is drawn by all threads at once
//     (512 / gw steps), not by the neurons' threads inside the step;
// which leaves two barriers a step. A launch of up to 14 steps of that network: 91 -> 49 us
// (a scan, a map and five barriers per step before).
// Blocks with more records than LDS holds, or entries than the map, run in
// stretches of whole steps that fit; a step that does not fit by itself takes
// its records in portions, as many as have their entries in the map. A step of
// more entries than are loaded ahead loads each window while the one before is
// computed: busy states are bound by that stream (that network with 10% of its
// neurons firing per step on average, in bursts: 105 us per step with 8,192
// entries in flight and no look-ahead, 139 with 2,048, 89.5 now).
//
// At the end the state goes back, the accumulator becomes partial sum 0 (the
// input of step t0 + B), each target's history words at block start and its
// code for the deferred updates are written (see k_block_deferred), and
// workgroup 0 advances the step clock, which no workgroup of the run reads
// (they read the plan's copy).

constexpr int kPbU = 4;                       // entries per thread loaded ahead
constexpr int kPbAhead = kPbU * kPbBlock;     // ... per workgroup
constexpr int kPbMap = 16384;                 // entries of a stretch of steps
static_assert(kMaxSortRow <= kPbMap, "any one record fits the map");
static_assert(kPbRecords < 65536, "16-bit map (1 + record, 0: none)");
static_assert(kPbMap % (8 * kPbBlock) == 0, "whole 16-byte words per thread");
// a record's flags, as kept in LDS and with each loaded entry: age (bits
// 0-7), pre spike (8), delivered (9), inhibitory (10), late (11), step (12-15);
// a loaded entry also: present (16), odd edge index (17), plastic (18)
constexpr int kRfPre = 1 << 8, kRfTx = 1 << 9, kRfInh = 1 << 10, kRfLate = 1 << 11, kRfStep = 12;
constexpr int kEnIn = 1 << 16, kEnOdd = 1 << 17, kEnPlastic = 1 << 18;
// The graphs of the blocks (at most kPbMaxN rows of at most kMaxSortRow
// entries) have fewer than 2^31 edges: 32-bit edge indices.
static_assert((int64_t)kPbMaxN * kMaxSortRow < (1ll << 31), "32-bit edge index");

struct PbEntries {
    float wv[kPbU];     // weight as loaded
    uint32_t cv[kPbU];  // target as loaded (compressed: the 32-bit word holding it)
    int f[kPbU];        // flags
    int e[kPbU];        // edge
    float xp0[kPbU];    // pre trace at the row's previous update
};
// a queued update: weight, edge, pre trace (as bits), flags with the target in
// the group in bits 24-31
static_assert(kEnPlastic < 1 << 24 && kPbMaxWidth <= 256, "queue word");

template <int HW, bool CT>
__global__ __launch_bounds__(kPbBlock) void k_block_run(NeuronArgs a, BlockArgs b)
{
    constexpr int NWV = kPbBlock / kWave;
    // per record: first edge less its flattened index, flattened end of its
    // plastic entries, flags, pre trace
    __shared__ int r_base[kPbRecords], r_pend[kPbRecords], r_info[kPbRecords];
    __shared__ float r_xp0[kPbRecords];
    __shared__ __align__(16) uint16_t s_map[kPbMap];  // flattened entry -> record
    __shared__ int s_yoff[kBatchMax + 1];  // a stretch's first entry of each step, and its end
    __shared__ int4 s_q[NWV][kPbU * kWave];
    __shared__ uint64_t s_hist[kPbMaxWidth * HW];
    __shared__ float s_y[kPbMaxWidth];
    __shared__ float s_x[kPbBlock];  // external drive: [step of the draw][target]
    __shared__ long long s_acc[2 * kPbMaxWidth];
    __shared__ float s_dpow[kMaxAge + 1];
    __shared__ long long sh[NWV];
    __shared__ int shi[NWV];
    __shared__ int s_cnt[kBatchMax], s_base[kBatchMax + 1];
    __shared__ int s_fit[2];  // records, and their entries, that the map holds in full
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    // neighbouring groups (which read neighbouring entries of each row) on
    // one XCD: workgroup b runs on XCD b mod 8
    const int nb = gridDim.x;  // multiple of 8
    const int g = (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3);
    if (g >= b.n_groups) return;  // whole workgroup, before any barrier
    const int n = a.n, G = b.n_groups;
    const int glo = g * b.gwidth;
    const int wn = min(b.gwidth, n - glo);  // > 0
    const int cbase = CT ? glo % b.width : glo;  // subtracted from a loaded target
    const int i = glo + tid;
    const bool live = tid < wn;
    const int B = b.steps;
    const long long ne = (long long)b.n_edges;
    // the lists' lengths, the neuron state, the input of the first step and
    // the block clock: every load out before any is looked at
    static_assert(kBatchMax <= kWave, "one list per lane");
    const int cnt_l = b.ev_cnt[min(lane, kBatchMax - 1)];
    const int ic = live ? i : glo;
    NState st = {};
    float ae0 = 0.f, ai0 = 0.f;
    InputLoads in0;
    nstate_load<-1, HW>(a, ic, st);
    if (a.model != 2) input_issue(a, ic, in0);
    BlockClock bc;  // (vector loads, as in load_clock)
    bc.t0 = __hip_atomic_load(&b.bclk->t0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bc.input_forced =
        __hip_atomic_load(&b.bclk->input_forced, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bc.n_parts = __hip_atomic_load(&b.bclk->n_parts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int q = tid; q <= kMaxAge; q += kPbBlock) s_dpow[q] = b.dpow[q];
    {
        const int c = lane < B ? min(max(cnt_l, 0), n) : 0;
        const int upto = wave_incl_scan(c, 0, AddOp{});
        if (wave == 0 && lane < kBatchMax) {
            s_cnt[lane] = c;
            s_base[lane + 1] = upto;
            if (lane == 0) s_base[0] = 0;
        }
    }
    const int64_t t0 = bc.t0;
    if (a.model != 2) input_combine(a, in0, bc.input_forced, bc.n_parts, ic, ae0, ai0);
    const float c_pot = b.c_pot, c_dep = b.c_dep, mu = b.mu;
    const int32_t *__restrict__ col = b.col;
    const uint32_t *__restrict__ col32 = reinterpret_cast<const uint32_t *>(b.col16);
    float *__restrict__ wgt = b.w;
    long long events = 0, w_tx = 0, w_forced = 0, spikes = 0;
    uint32_t blk = 0u;  // the block's spikes (bit 0: the latest step)
    const bool driven = a.model == 0 && a.poisson_len > 0;
    const int gsh = 31 - __clz(b.gwidth);  // gwidth is 64, 128 or 256
    const int dsteps = kPbBlock >> gsh;    // steps per draw of the drive
    const uint64_t hs0 = st.h0, hs1 = st.h1;  // the history words at block start
    __syncthreads();  // s_base

    // the external drive of steps q .. q + dsteps - 1 (published by the next barrier)
    auto draw = [&](int q) {
        const int ds = tid >> gsh, j = tid & (b.gwidth - 1);
        s_x[tid] = drive(a, t0 + q + ds, min(glo + j, n - 1));
    };
    // LDS records 0 .. count - 1 (count <= kPbRecords) from the lists from
    // entry j0 of step q0 on (across the steps' lists in order): the row's
    // entries in the group (from the group pivots of the row, loaded once the
    // row is known), clamped to the graph (only a failed plan, which leaves
    // list entries unwritten, could point elsewhere). Their entries are
    // flattened: s_yoff[q], q = q0 .. q1, the first entry of each step, and
    // the map written as far as it reaches (read after the next barrier).
    // Returns the number of entries; begins with a barrier.
    auto load_records = [&](int q0, int q1, int j0, int count) -> int {
        constexpr int RU = kPbRecords / kPbBlock;
        static_assert(kPbRecords % kPbBlock == 0, "whole rounds of records");
        __syncthreads();  // every read of the records and the map before
        const int per = (count + kPbBlock - 1) / kPbBlock;  // records per thread, consecutive
        const int r0 = tid * per;
        int own = 0;
        int sb[kBatchMax];  // first record of the steps after q0's, from the first one loaded
#pragma unroll
        for (int z = 0; z < kBatchMax; ++z) sb[z] = s_base[z + 1] - s_base[q0] - j0;
        PbEvent pe[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            if (u >= per) break;  // uniform
            const int x = min(r0 + u, max(count - 1, 0));
            // its list: the steps that end at or before it are behind it
            int q = q0, first = -j0;
#pragma unroll
            for (int z = 0; z < kBatchMax; ++z)
                if (z >= q0 && z < B - 1 && sb[z] <= x) {
                    q = z + 1;
                    first = sb[z];
                }
            pe[u] = b.ev[(int64_t)q * n + min(max(x - first, 0), n - 1)];
        }
        constexpr int MW = kPbMap / (8 * kPbBlock);  // 16-byte map words per thread
        uint4 *mw = reinterpret_cast<uint4 *>(s_map) + tid * MW;  // consecutive
#pragma unroll
        for (int v = 0; v < MW; ++v) mw[v] = make_uint4(0u, 0u, 0u, 0u);
        int p0[RU], p1[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            if (u >= per) break;
            const int32_t *gp = b.gpiv + (int64_t)min(max(pe[u].k, 0), n - 1) * (G + 1) + g;
            p0[u] = gp[0];
            p1[u] = gp[1];
        }
        int len[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            if (u >= per) break;
            const int x = r0 + u;
            len[u] = 0;
            if (x >= count) continue;
            int sl = max(p1[u] - p0[u], 0);
            const uint32_t f = pe[u].lenf;
            const int plen = min(max((int)(f & 0xffffu) - p0[u], 0), sl);
            const int deliver = (f >> 25) & 1;
            if (!deliver) sl = plen;  // a forced row: its plastic entries only
            const long long st0 = min(max((long long)pe[u].rs + p0[u], 0ll), ne);
            sl = (int)min((long long)sl, ne - st0);
            len[u] = sl;
            r_base[x] = (int)st0;
            r_pend[x] = min(plen, sl);
            r_info[x] = (int)((f >> 16) & 0xff) | (((f >> 24) & 1) ? kRfPre : 0) |
                        (deliver ? kRfTx : 0) | (((f >> 26) & 1) ? kRfInh : 0) |
                        ((f >> 31) ? kRfLate : 0) | (int)(((f >> 27) & 15) << kRfStep);
            r_xp0[x] = pe[u].xp0;
            own += sl;
        }
        const long long incl = block_incl_scan_i64_n<kPbBlock>((long long)own, sh);
        // (the map was cleared before the scan's barriers)
        int y = (int)min(incl - own, (long long)INT32_MAX / 2);
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            if (u >= per) break;
            const int x = r0 + u;
            if (x >= count) continue;
            r_base[x] -= y;
            r_pend[x] += y;
            // the first record of a step: the step's first entry (and that of
            // empty steps before it)
            const int q = (r_info[x] >> kRfStep) & 15;
            const int pq = x == 0 ? q0 - 1 : (u == 0 ? 16 : (r_info[x - 1] >> kRfStep) & 15);
            if (pq < 16)
                for (int z = max(pq + 1, q0); z <= min(q, q1); ++z) s_yoff[z] = y;
            if (len[u] > 0 && y < kPbMap) s_map[y] = (uint16_t)(x + 1);  // marks its first entry
            if (y <= kPbMap && kPbMap < y + len[u]) {  // the first record not in it in full
                s_fit[0] = x;
                s_fit[1] = y;
            }
            y += len[u];
        }
        __syncthreads();  // the marks, r_info (the record before the thread's first)
        // the map: each entry's record is the last one marked up to it
        {
            uint32_t m[4 * MW];
            uint32_t top = 0u;
#pragma unroll
            for (int v = 0; v < MW; ++v) {
                const uint4 x = mw[v];
                m[4 * v] = x.x;
                m[4 * v + 1] = x.y;
                m[4 * v + 2] = x.z;
                m[4 * v + 3] = x.w;
            }
#pragma unroll
            for (int v = 0; v < 4 * MW; ++v) {
                const uint32_t lo = max(top, m[v] & 0xffffu);
                top = max(lo, m[v] >> 16);
                m[v] = lo | (top << 16);
            }
            const int inc = wave_incl_scan((int)top, 0, MaxOp{});
            if (lane == kWave - 1) shi[wave] = inc;
            __syncthreads();
            int ex = wave_shr1(inc, 0);
            for (int w = 0; w < wave; ++w) ex = max(ex, shi[w]);
            const uint32_t e0 = (uint32_t)ex;
#pragma unroll
            for (int v = 0; v < 4 * MW; ++v) {  // record = mark - 1 (before the first mark: 0)
                const uint32_t lo = max(e0, m[v] & 0xffffu), hi = max(e0, m[v] >> 16);
                m[v] = (lo ? lo - 1u : 0u) | ((hi ? hi - 1u : 0u) << 16);
            }
#pragma unroll
            for (int v = 0; v < MW; ++v)
                mw[v] = make_uint4(m[4 * v], m[4 * v + 1], m[4 * v + 2], m[4 * v + 3]);
        }
        if (r0 < count && r0 > 0) {
            const int q = (r_info[r0] >> kRfStep) & 15, pq = (r_info[r0 - 1] >> kRfStep) & 15;
            const int yf = (int)min(incl - own, (long long)INT32_MAX / 2);
            for (int z = max(pq + 1, q0); z <= min(q, q1); ++z) s_yoff[z] = yf;
        }
        long long total = 0;  // the waves' sums of the scan
#pragma unroll
        for (int w = 0; w < NWV; ++w) total += sh[w];
        return (int)min(total, (long long)INT32_MAX / 2);
    };
    // loads of the entries y0 + u kPbBlock + tid (u < kPbU) below y1: every
    // slot loads from a valid address, the results are looked at when the
    // entries are computed
    auto issue = [&](int y0, int y1, PbEntries &E) {
        static_assert(kPbU % 2 == 0, "two halves");
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h && y0 + kPbAhead / 2 >= y1) {  // uniform: the second half is empty
#pragma unroll
                for (int u = kPbU / 2; u < kPbU; ++u) E.f[u] = 0;
                break;
            }
#pragma unroll
            for (int u = h * kPbU / 2; u < (h + 1) * kPbU / 2; ++u) {
                const int y = y0 + u * kPbBlock + tid;
                const bool in = y < y1;
                const int r = in ? (int)s_map[y] : 0;
                const int e = in ? r_base[r] + y : 0;  // < n_edges
                E.cv[u] = CT ? col32[e >> 1] : (uint32_t)col[e];
                E.wv[u] = wgt[e];
                E.e[u] = e;
                E.xp0[u] = r_xp0[r];
                E.f[u] = in ? (r_info[r] & ((1 << kRfStep) - 1)) | kEnIn |
                                  ((e & 1) ? kEnOdd : 0) | (y < r_pend[r] ? kEnPlastic : 0)
                            : 0;
            }
        }
    };
    // weights of late records loaded again, once the step before is stored
    auto reload = [&](PbEntries &E) {
        bool any = false;
#pragma unroll
        for (int u = 0; u < kPbU; ++u) any = any || (E.f[u] & kRfLate);
        if (!ballot64(any)) return;  // wave-uniform
#pragma unroll
        for (int u = 0; u < kPbU; ++u)
            if (E.f[u] & kRfLate) E.wv[u] = wgt[E.e[u]];
    };
    // The entries of one window: a transmitting row's entry whose
    // weight does not change is delivered at once; the entries whose weight
    // changes (a pre spike, or a post spike of the target within the row's
    // window) go to the wave's queue, which is then updated 64 at a time
    // with every lane busy (the replay loops run over those entries only),
    // stored, and delivered where the row transmits.
    auto compute = [&](const PbEntries &E) {
        int4 *qq = s_q[wave];
        int qn = 0;
#pragma unroll
        for (int u = 0; u < kPbU; ++u) {
            const int f = E.f[u];
            if (!ballot64(f & kEnIn)) continue;  // an unused slot of the wave
            const uint32_t c = CT ? ((f & kEnOdd) ? E.cv[u] >> 16 : E.cv[u] & 0xffffu) : E.cv[u];
            const int j = (int)c - cbase;
            const bool ok = (f & kEnIn) && (unsigned)j < (unsigned)wn;
            if ((f & kEnIn) && !ok) atomicOr(b.err, kErrIndex);  // not this group's target
            bool cand = false;
            if (ok && (f & kEnPlastic)) {
                uint64_t m0, m1;
                window_masks(f & 0xff, m0, m1);
                const uint64_t h0 = s_hist[j * HW] & m0;
                const uint64_t h1 = HW == 2 ? s_hist[j * 2 + 1] & m1 : 0ull;
                cand = h0 || h1 || (f & kRfPre) || !b.event;
            }
            if (ok && !cand && (f & kRfTx)) {
                atomicAdd((unsigned long long *)(s_acc + j + ((f & kRfInh) ? kPbMaxWidth : 0)),
                          (unsigned long long)to_fix(E.wv[u]));
                ++events;
            }
            const uint64_t bl = ballot64(cand);
            if (cand) {
                qq[qn + lane_rank(bl)] =
                    make_int4(__float_as_int(E.wv[u]), E.e[u], __float_as_int(E.xp0[u]),
                              (f & 0xffffff) | (j << 24));
            }
            qn += (int)__popcll(bl);
        }
        __builtin_amdgcn_wave_barrier();
        for (int e0 = 0; e0 < qn; e0 += kWave) {  // wave-uniform
            const int e = e0 + lane;
            if (e >= qn) continue;
            const int4 p = qq[e];
            float w = __int_as_float(p.x);
            const int info = p.w, j = (int)((unsigned)p.w >> 24);
            const int age = info & 0xff, pre = (info & kRfPre) ? 1 : 0;
            uint64_t m0, m1;
            window_masks(age, m0, m1);
            const uint64_t h0 = s_hist[j * HW] & m0;
            const uint64_t h1 = HW == 2 ? s_hist[j * 2 + 1] & m1 : 0ull;
            const float yp = pre ? s_y[j] : 0.f;
            const float xp0 = __int_as_float(p.z);
            // the pre trace after this update, as the plan's snapshot has it
            const float xpn = __fadd_rn(__fmul_rn(xp0, s_dpow[age]), (float)pre);
            w = b.event ? stdp_synapse(w, h0, h1, age, pre, xp0, xpn, yp, s_dpow, c_pot, c_dep, mu)
                        : stdp_synapse_steps(w, h0, h1, age, pre, xp0, xpn, yp, s_dpow[1],
                                             c_pot, c_dep, mu);
            wgt[p.y] = w;
            if (pre)
                ++w_tx;
            else
                ++w_forced;
            if (info & kRfTx) {
                atomicAdd((unsigned long long *)(s_acc + j + ((info & kRfInh) ? kPbMaxWidth : 0)),
                          (unsigned long long)to_fix(w));
                ++events;
            }
        }
        __builtin_amdgcn_wave_barrier();  // the queue is rewritten next
    };
    // entries [y0, y1) but for the last window, which E holds afterwards, as it
    // holds the first one before: each window loaded while the one before is
    // computed
    auto windows = [&](int y0, int y1, PbEntries &E, PbEntries &F) {
        for (int y = y0 + kPbAhead; y < y1; y += kPbAhead) {  // uniform
            issue(y, y1, F);
            compute(E);
            E = F;
        }
    };
    auto neuron_step = [&](int q) {
        if (live) {
            float ae = 0.f, ai = 0.f;
            if (a.model != 2) {
                if (q == 0) {
                    ae = ae0;
                    ai = ai0;
                } else {
                    const long long se = s_acc[tid];
                    const long long si = b.nacc == 2 ? s_acc[kPbMaxWidth + tid] : 0;
                    if (!ballot64(!(fix_small(se) && fix_small(si)))) {  // any input in earnest
                        ae = from_fix_small(se);
                        ai = from_fix_small(si);
                    } else {
                        ae = from_fix(se);
                        ai = from_fix(si);
                    }
                }
            }
            int sp;
            if (a.model == 2)
                sp = neuron_dynamics<2>(a, i, t0 + q, ae, ai, st);
            else
                sp = lif_dynamics<-1>(a, ae, ai,
                                      driven ? s_x[((q & (dsteps - 1)) << gsh) + tid] : 0.f, st);
            neuron_record<-1, HW>(a, sp, st);
            spikes += sp;
            blk = (blk << 1) | (uint32_t)sp;
            s_hist[tid * HW] = st.h0;
            if (HW == 2) s_hist[tid * 2 + 1] = st.h1;
            s_y[tid] = st.y;
        }
        if (tid < kPbMaxWidth) {
            s_acc[tid] = 0;
            s_acc[kPbMaxWidth + tid] = 0;
        }
    };
    // the drive of the steps after step q, when step q used the last drawn
    // (after step q's first barrier)
    auto draw_next = [&](int q) {
        if (driven && ((q + 1) & (dsteps - 1)) == 0 && q + 1 < B) draw(q + 1);
    };

    PbEntries E0, E1;
    int most = kPbRecords;  // records of a step's portion loaded
    if (driven) draw(0);
    __syncthreads();  // s_x
    for (int q = 0; q < B;) {
        // the whole steps whose records fit
        int qe = q;
        while (qe < B && s_base[qe + 1] - s_base[q] <= kPbRecords) ++qe;
        int fit = 0;  // steps of the stretch
        if (qe > q) {
            const int cnt = s_base[qe] - s_base[q];
            const int total = load_records(q, qe, 0, cnt);
            if (tid == 0) {  // the steps after the last record
                const int lq = cnt > 0 ? (r_info[cnt - 1] >> kRfStep) & 15 : q - 1;
                for (int z = lq + 1; z <= qe; ++z) s_yoff[z] = total;
            }
            __syncthreads();  // s_yoff
            while (q + fit < qe && s_yoff[q + fit + 1] <= kPbMap) ++fit;
        }
        if (fit > 0) {
            const int qs = q, qx = q + fit;
            // one step: its entries loaded (E), the next step's loaded into F
            auto step = [&](int k, PbEntries &E, PbEntries &F) {
                neuron_step(k);
                __syncthreads();  // histories, traces, the cleared accumulator
                const int y0 = s_yoff[k], y1 = s_yoff[k + 1];
                const int z1 = k + 1 < qx ? s_yoff[k + 2] : y1;
                windows(y0, y1, E, F);
                issue(y1, z1, F);
                compute(E);
                draw_next(k);
                __syncthreads();  // every atomic and weight store of step k done
                reload(F);
            };
            issue(s_yoff[qs], s_yoff[qs + 1], E0);
            for (int k = qs; k < qx; k += 2) {
                step(k, E0, E1);
                if (k + 1 < qx) step(k + 1, E1, E0);
            }
            q = qx;
        } else {
            // a step that does not fit: its records in portions, as many as
            // have their entries in the map (one record always does), about
            // that many loaded for the next portion
            neuron_step(q);
            for (int j = 0; j < s_cnt[q];) {
                int m = min(s_cnt[q] - j, most);
                int total = load_records(q, q, j, m);
                __syncthreads();
                if (total > kPbMap) {  // uniform
                    m = s_fit[0];
                    total = s_fit[1];
                    most = min(m + m / 8 + 1, kPbRecords);
                } else if (total < kPbMap / 2) {
                    most = min(2 * most, kPbRecords);
                }
                issue(0, total, E0);
                windows(0, total, E0, E1);
                compute(E0);
                j += m;
            }
            __syncthreads();  // every atomic of step q done (and the neuron update published)
            draw_next(q);
            __syncthreads();  // s_x
            ++q;
        }
    }
    if (live) {
        nstate_store<-1, HW>(a, i, st);
        a.code[i] = hist_code(st.h0, st.h1);
        b.apart[i] = s_acc[tid];
        if (b.nacc == 2) b.apart[n + i] = s_acc[kPbMaxWidth + tid];
        uint64_t *hqi = b.hq + (int64_t)i * (2 * HW);
        hqi[0] = hs0;
        if (HW == 2) hqi[1] = hs1;
        hqi[HW] = blk;
        // the code of the deferred updates: the first step of the block with
        // a spike (15: none), and the bit L of the latest spike before it
        // against the window of a forced update at step q (L + q + 1 < 64 hw,
        // q < 15): 0 if always inside, 15 if never, else L - (64 hw - 16)
        const int first = blk ? B - 1 - (31 - __clz((int)blk)) : 15;
        const int last = hs0 ? __ffsll((long long)hs0) - 1
                             : (HW == 2 && hs1) ? 63 + __ffsll((long long)hs1) : 1 << 20;
        const int lc = last <= 64 * HW - 16 ? 0 : last >= 64 * HW - 1 ? 15 : last - (64 * HW - 16);
        b.dcode[i] = (uint8_t)(first | (lc << 4));
    }
    if (b.fin_blocks && wave * kWave < wn) {  // wave-uniform
        // the call's last block: the masks of its last step, and (b.dmask) the
        // spikes of the last D steps, which the lists are made from
        const int word = glo / kWave + wave, nw = (n + kWave - 1) / kWave;
        const uint64_t h0 = live ? st.h0 : 0ull, h1 = live ? st.h1 : 0ull;
        const uint64_t txm = ballot64((h0 >> (b.delay - 1)) & 1ull);
        const uint64_t rcm = ballot64((h0 | h1) != 0ull);
        uint64_t mine = 0ull;  // lane q: the spikes of step t0 + B - 1 - q
        for (int q = 0; q < b.delay; ++q) {
            const uint64_t m = ballot64((h0 >> q) & 1ull);
            if (lane == q) mine = m;
        }
        if (lane < b.delay) b.dmask[(int64_t)lane * nw + word] = mine;
        if (lane == 0) {
            b.mask[word] = mine;
            b.txmask[word] = txm;
            b.recent[word] = rcm;
        }
    }
    events = block_sum_i64_n<kPbBlock>(events, sh);
    w_tx = block_sum_i64_n<kPbBlock>(w_tx, sh);
    w_forced = block_sum_i64_n<kPbBlock>(w_forced, sh);
    spikes = block_sum_i64_n<kPbBlock>(spikes, sh);
    if (tid == 0) {
        int64_t *ds = b.dlv_stats + 2 * (int64_t)(g % b.dlv_slots);
        if (events) add_stat(ds, events);
        if (w_tx) add_stat(ds + 1, w_tx);
        if (w_forced) add_stat(b.syn_stats + (g % b.syn_slots), w_forced);
        if (spikes) add_stat(b.gstats + kGSpikes, spikes);
        if (g == 0) {
            add_stat(b.gstats + kGSteps, B);
            *b.df_cnt = b.ev_cnt[B];  // the deferred updates' count
            b.clk->t = t0 + B;
            b.clk->input_forced = 0;  // the next input is partial sum 0
            b.clk->n_parts = 1;
        }
    }
}

// ---------------------------------------------------------------------------
// The deferred forced updates of a block (the plan's list B), after its run,
// streamed by the whole device: one workgroup per CU, the rows' plastic
// entries (from each row's first 8-aligned entry on) cut into parts of
// kDfPart, spread over the waves (each lane 8 consecutive targets and
// weights in 16-byte loads), the next part loaded while the current one is
// computed.
//   An update at step t = t0 + q changes the synapses whose target spiked in
// the window (t - a, t] (every one without event-driven replay). The
// target's history word at t is its word at block start shifted up by q + 1
// steps, under the block's spike bits of steps t0 .. t (Sec. III-A's bit
// history). A forced update has the longest age, a = 64 hw (> q), so a
// synapse changes iff its target spiked in the block at a step <= q, or
// before the block at bit L of the start words with L + q + 1 < a: one byte
// per target holds both (the first spike step in the block; L against the
// last 15 bits of the window), staged in LDS. The synapses that pass are
// queued and brought up to date 64 at a time from the full words (hq), which
// decide exactly (an update of another age queues every entry).

constexpr int kDfBlock = 1024;
constexpr int kDfPart = kPbDfPart;      // entries per part of a row
constexpr int kDfU = kDfPart / kWave;   // entries per lane per part
static_assert(kDfU == 8, "two 16-byte loads of targets and of weights per lane");
static_assert(kPbMaxN <= 65536, "target in 16 bits of the queue word");

struct DfPart {
    int4 c[2];
    float4 w[2];
    long long base, lo, hi;  // first entry of the part (8-aligned), the row's plastic entries
    int age, qs;
    float xp0;
    int valid;
};

// After the last block of a call, the per-step lists of the step-by-step path,
// from the masks the run and the plan left (b.dmask): role q < D, the spike
// list of step t-1-q (t = clk->t) in ascending order into its ring slot, with
// its count and each neuron's position; role D, the forced rows of step t-1.
// Each also clears a share of the list scans' status words, so that no stale
// step tag matches a later scan. These workgroups join the last block's
// deferred launch (neither needs the other): a mask word per thread and one
// scan over the words, 25,000 neurons and D = 15: about no time of its own beside the
// deferred updates, against 28.4 us as a launch of its own that read the
// histories 1,024 neurons at a time (18.0 with eight loads in flight: one CU
// per list reads 200 KB).
__device__ __forceinline__ void finish_lists(const BlockArgs &b, int q, long long *sh)
{
    const int tid = threadIdx.x;
    const int n = b.n, D = b.delay;
    const int nw = (n + kWave - 1) / kWave;
    static_assert(kPbMaxN / kWave <= kDfBlock, "one mask word per thread");
    uint64_t m = tid < nw ? b.dmask[(int64_t)q * nw + tid] : 0ull;
    const int64_t t = load_clock(b.clk).t;
    for (int64_t x = (int64_t)q * kDfBlock + tid; x < b.status_words;
         x += (int64_t)(D + 1) * kDfBlock)
        b.status[x] = 0ull;
    if (q == 0 && tid < kBatchMax) {  // both blocks' list counts, for the next call's plans
        b.ev_cnt[tid] = 0;            // (the deferred updates read b.df_cnt)
        b.ev_cnt_next[tid] = 0;
    }
    const bool lists = q < D;
    const int own = (int)__popcll(m);
    const int incl = (int)block_incl_scan_i64_n<kDfBlock>(own, sh);
    const int slot = ring_slot(t - 1 - q, D);
    int32_t *list = lists ? b.ring + (int64_t)slot * n : b.rows;
    int32_t *pos = b.spk_pos + (int64_t)slot * n;  // (lists only)
    for (int r = incl - own; m; m &= m - 1ull, ++r) {  // r < n: one entry per neuron
        const int i = tid * kWave + __ffsll((long long)m) - 1;
        list[r] = i;
        if (lists) pos[i] = r;
    }
    if (tid == kDfBlock - 1) {
        if (lists)
            b.ring_cnt[slot] = incl;
        else
            *b.row_cnt = incl;
    }
}

template <int HW>
__global__ __launch_bounds__(kDfBlock) void k_block_deferred(BlockArgs b)
{
    constexpr int NWV = kDfBlock / kWave;
    constexpr int A = 64 * HW;  // the age of a forced update
    __shared__ uint8_t s_code[kPbMaxN];
    __shared__ int q_p[NWV][kDfPart];    // target (bits 0-15), entry in the part (16-24)
    __shared__ float q_w[NWV][kDfPart];  // weight
    __shared__ float s_dpow[kMaxAge + 1];
    __shared__ long long sh[NWV];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int n = b.n, B = b.steps;
    if ((int)blockIdx.x < b.fin_blocks) {  // whole workgroup, before any barrier
        finish_lists(b, blockIdx.x, sh);
        return;
    }
    const int block = blockIdx.x - b.fin_blocks, blocks = gridDim.x - b.fin_blocks;
    const int nd = min(max(*b.df_cnt, 0), n);
    const PbEvent *__restrict__ evd = b.ev + (int64_t)B * n;
    const int32_t *__restrict__ col = b.col;
    float *__restrict__ wgt = b.w;
    const uint64_t *__restrict__ hq = b.hq;
    const long long ne = (long long)b.n_edges;  // < 2^31
    const float c_pot = b.c_pot, c_dep = b.c_dep, mu = b.mu;
    // the targets' codes (padded to 16 bytes), loaded first: every later
    // load of the wave completes after them
    constexpr int kCodeLoads = kPbMaxN / 16 / kDfBlock;
    uint4 cl[kCodeLoads];
    const int ncv = (n + 15) / 16;
#pragma unroll
    for (int u = 0; u < kCodeLoads; ++u)
        cl[u] = reinterpret_cast<const uint4 *>(b.dcode)[min(u * kDfBlock + tid, ncv - 1)];
    // Items: part p of row r is item r P + p (P = parts of the longest
    // row); the wave takes items w0 + j stride, j = 0 .. nit - 1. Lane l
    // holds the record of the row of item (j & ~63) + l, read out for the
    // current item j (no load inside the part stream waits on a record).
    const int P = b.df_parts;
    const int stride = blocks * NWV;
    const int w0 = block * NWV + wave;
    const long long nitems = (long long)nd * P;
    const int nit = w0 < nitems ? (int)((nitems - 1 - w0) / stride + 1) : 0;
    PbEvent le = PbEvent{};
    int j = 0;
    long long base = 0, r_lo = 0, r_hi = 0;  // the current item's part, its row's entries
    int r_age = 0, r_qs = 0;
    float r_xp0 = 0.f;
    auto set_item = [&]() {  // j < nit
        if ((j & 63) == 0) {
            const long long it = w0 + (long long)(j + lane) * stride;
            le = j + lane < nit ? evd[it / P] : PbEvent{};
        }
        const int src = j & 63;
        const long long rs = __builtin_amdgcn_readlane(le.rs, src);
        const uint32_t f = (uint32_t)__builtin_amdgcn_readlane((int)le.lenf, src);
        r_xp0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(le.xp0), src));
        r_lo = min(max(rs, 0ll), ne);
        r_hi = min(r_lo + (long long)(f & 0xffffu), ne);
        base = (r_lo & ~7ll) + (long long)((w0 + (long long)j * stride) % P) * kDfPart;
        r_age = min((int)((f >> 16) & 0xff), kMaxAge);
        r_qs = (int)((f >> 27) & 15);
    };
    if (nit > 0) set_item();
    // the next part's loads, from a valid address whether or not the part
    // exists, so that every part issues the same loads
    auto issue = [&](DfPart &p) {
        p.valid = j < nit && base < r_hi;
        p.base = base;
        p.lo = r_lo;
        p.hi = r_hi;
        p.age = r_age;
        p.qs = r_qs;
        p.xp0 = r_xp0;
        // (entries up to 7 past the last edge lie in the next array of the
        // graph buffer; they are never used)
        const long long e0 = p.valid ? min(base + lane * kDfU, (r_hi - 1) & ~7ll) : 0ll;
        const int4 *cv = reinterpret_cast<const int4 *>(col + e0);
        const float4 *wv = reinterpret_cast<const float4 *>(wgt + e0);
        p.c[0] = cv[0];
        p.c[1] = cv[1];
        p.w[0] = wv[0];
        p.w[1] = wv[1];
        if (j < nit && ++j < nit) set_item();  // wave-uniform
    };
    DfPart P0, P1;
    issue(P0);
    issue(P1);
#pragma unroll
    for (int u = 0; u < kCodeLoads; ++u)
        if (u * kDfBlock + tid < ncv) reinterpret_cast<uint4 *>(s_code)[u * kDfBlock + tid] = cl[u];
    for (int x = tid; x <= kMaxAge; x += kDfBlock) s_dpow[x] = b.dpow[x];
    __syncthreads();
    long long written = 0;
    // The history words of the first kDfRounds rounds of the queue are
    // gathered before the next part's loads are issued (a wave's loads
    // complete in order: waiting for a later gather waits for every earlier
    // load), so that part loads while this one is brought up to date.
    constexpr int kDfRounds = 2;
    auto words_of = [&](int j, uint64_t &s0, uint64_t &s1, uint64_t &blk) {
        const uint4 *hj = reinterpret_cast<const uint4 *>(hq + (int64_t)j * (2 * HW));
        const uint4 v0 = hj[0];
        if (HW == 2) {
            const uint4 v1 = hj[1];
            s1 = (uint64_t)v0.z | ((uint64_t)v0.w << 32);
            blk = (uint64_t)v1.x | ((uint64_t)v1.y << 32);
        } else {
            s1 = 0ull;
            blk = (uint64_t)v0.z | ((uint64_t)v0.w << 32);
        }
        s0 = (uint64_t)v0.x | ((uint64_t)v0.y << 32);
    };
    // a part, then the next part's loads into p
    auto step = [&](DfPart &p) {
        if (!p.valid) {  // wave-uniform
            issue(p);
            return;
        }
        const int age = p.age, qs = min(p.qs, B - 1);
        const long long pbase = p.base;
        const float xp0 = p.xp0;
        const bool filt = b.event && age == A;  // the codes decide
        const int cj[kDfU] = {p.c[0].x, p.c[0].y, p.c[0].z, p.c[0].w,
                              p.c[1].x, p.c[1].y, p.c[1].z, p.c[1].w};
        const float wj[kDfU] = {p.w[0].x, p.w[0].y, p.w[0].z, p.w[0].w,
                                p.w[1].x, p.w[1].y, p.w[1].z, p.w[1].w};
        const long long e0 = pbase + lane * kDfU;
        bool cand[kDfU];
#pragma unroll
        for (int v = 0; v < kDfU; ++v) {
            const long long e = e0 + v;
            const bool in = e >= p.lo && e < p.hi;
            const bool okj = (unsigned)cj[v] < (unsigned)n;
            if (in && !okj) atomicOr(b.err, kErrIndex);
            const int c = s_code[okj ? cj[v] : 0];
            cand[v] = in && okj && (!filt || (c & 15) <= qs || (c >> 4) + qs < 15);
        }
        int *qp = q_p[wave];
        float *qw = q_w[wave];
        int qn = 0;
#pragma unroll
        for (int v = 0; v < kDfU; ++v) {
            const uint64_t bl = ballot64(cand[v]);
            if (cand[v]) {
                const int x = qn + lane_rank(bl);
                qp[x] = cj[v] | ((lane * kDfU + v) << 16);
                qw[x] = wj[v];
            }
            qn += (int)__popcll(bl);
        }
        __builtin_amdgcn_wave_barrier();
        uint64_t g0[kDfRounds], g1[kDfRounds], gb[kDfRounds];
        int gp[kDfRounds];
#pragma unroll
        for (int r = 0; r < kDfRounds; ++r) {  // every lane, clamped into the queue
            const int x = min(r * kWave + lane, max(qn - 1, 0));
            gp[r] = qn > 0 ? qp[x] : 0;
            words_of(gp[r] & 0xffff, g0[r], g1[r], gb[r]);
        }
        issue(p);
        uint64_t m0, m1;
        window_masks(age, m0, m1);
        const int sft = B - 1 - qs;
        const float xpn = __fadd_rn(__fmul_rn(xp0, s_dpow[age]), 0.f);  // no pre spike
        auto update = [&](int x, int pk, uint64_t s0, uint64_t s1, uint64_t blk) {
            const uint64_t h0 = ((s0 << (qs + 1)) | (blk >> sft)) & m0;
            const uint64_t h1 = HW == 2 ? ((s1 << (qs + 1)) | (s0 >> (63 - qs))) & m1 : 0ull;
            if (b.event && !(h0 | h1)) return;  // unchanged
            float w = qw[x];
            w = b.event ? stdp_synapse(w, h0, h1, age, 0, xp0, xpn, 0.f, s_dpow, c_pot, c_dep, mu)
                        : stdp_synapse_steps(w, h0, h1, age, 0, xp0, xpn, 0.f, s_dpow[1], c_pot,
                                             c_dep, mu);
            wgt[pbase + (pk >> 16)] = w;
            ++written;
        };
#pragma unroll
        for (int r = 0; r < kDfRounds; ++r) {
            const int x = r * kWave + lane;
            if (x < qn) update(x, gp[r], g0[r], g1[r], gb[r]);
        }
        for (int x0 = kDfRounds * kWave; x0 < qn; x0 += kWave) {  // wave-uniform; rare
            const int x = x0 + lane;
            if (x >= qn) continue;
            const int pk = qp[x];
            uint64_t s0, s1, blk;
            words_of(pk & 0xffff, s0, s1, blk);
            update(x, pk, s0, s1, blk);
        }
        __builtin_amdgcn_wave_barrier();  // the queue is rewritten next
    };
    while (P0.valid || P1.valid || j < nit) {  // wave-uniform
        step(P0);
        step(P1);
    }
    written = block_sum_i64_n<kDfBlock>(written, sh);
    if (tid == 0 && written) add_stat(b.syn_stats + (block % b.syn_slots), written);
}

template <int HW, bool CT>
hipError_t launch_run(hipStream_t s, const NeuronArgs &a, const BlockArgs &b)
{
    const int grid = (b.n_groups + 7) / 8 * 8;
    hipLaunchKernelGGL((k_block_run<HW, CT>), dim3(grid), dim3(kPbBlock), 0, s, a, b);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_block_plan(hipStream_t s, const BlockArgs &b)
{
    if (b.steps < 1 || b.steps > kPbMaxSteps || b.steps > b.delay - 1 || b.n < 1 ||
        b.n > kPbMaxN || b.ev_cnt == b.ev_cnt_next)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_block_plan, dim3(blocks_for(b.n, kPbPlanBlock)), dim3(kPbPlanBlock), 0,
                       s, b);
    return hipGetLastError();
}

hipError_t launch_block_run(hipStream_t s, const NeuronArgs &a, const BlockArgs &b)
{
    if (b.steps < 1 || b.steps > kPbMaxSteps || b.gwidth < 1 || b.gwidth > kPbMaxWidth ||
        b.n_edges < 1 || b.n_edges > INT32_MAX ||
        b.width % b.gwidth != 0 || (int64_t)b.n_groups * b.gwidth < a.n ||
        (int64_t)(b.n_groups - 1) * b.gwidth >= a.n || a.n != b.n || b.nacc < 1 || b.nacc > 2 ||
        b.dlv_slots < 1 || b.syn_slots < 1)
        return hipErrorInvalidValue;
    const bool ct = b.col16 != nullptr;
    if (a.hw == 2) return ct ? launch_run<2, true>(s, a, b) : launch_run<2, false>(s, a, b);
    return ct ? launch_run<1, true>(s, a, b) : launch_run<1, false>(s, a, b);
}

hipError_t launch_block_deferred(hipStream_t s, const BlockArgs &b)
{
    if (b.steps < 1 || b.steps > kPbMaxSteps || b.n < 1 || b.n > kPbMaxN || b.n_edges < 1 ||
        b.n_edges > INT32_MAX || b.n_cu < 1 || b.syn_slots < 1 || (b.hw != 1 && b.hw != 2) ||
        b.df_parts < 1 || b.df_parts > (kMaxSortRow + 7 + kDfPart - 1) / kDfPart ||
        (b.fin_blocks != 0 && b.fin_blocks != b.delay + 1) || b.delay < 2 || b.delay > 64)
        return hipErrorInvalidValue;
    // one workgroup per CU, those of the lists among them
    const int grid =
        b.fin_blocks + (int)std::min<int64_t>(
                           std::max(b.n_cu - b.fin_blocks, 1),
                           ((int64_t)b.n * b.df_parts + kDfBlock / kWave - 1) / (kDfBlock / kWave));
    if (b.hw == 2)
        hipLaunchKernelGGL(k_block_deferred<2>, dim3(grid), dim3(kDfBlock), 0, s, b);
    else
        hipLaunchKernelGGL(k_block_deferred<1>, dim3(grid), dim3(kDfBlock), 0, s, b);
    return hipGetLastError();
}

}  // namespace snn
