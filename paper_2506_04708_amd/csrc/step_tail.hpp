// step_tail.hpp -- step_tail_kernel: everything that follows the row kernel, in one launch, for small batches (paper
// Sec. 3.2, 4.1, 4.2).
#pragma once
#include "draft.hpp"
#include "path_pass.hpp"

namespace stand {

// ---------------------------------------------------------------------------------------------
// A step's dependent part costs a small batch more than its rows.  As separate launches (exact sums, finish + claims,
// apply, draft) every part pays 2 to 3 us for its start, reads again what the part before it wrote, and waits for the last
// workgroup of that part.  Here they are one launch:
//
//   workgroups [0, B)   a trajectory each
//   the others          exact partial sums of the path rows (they follow the path themselves): a wave takes one of the
//                       row's `nsub` ranges of vectors, with at most a few vectors per lane
//
// and inside a trajectory's workgroup the waves take what depends on different things:
//
//   first wave          the token: replay of the stop node, resampled token, the new context
//   last wave           claims of the table slots (they need the path's tokens only)
//   the others          observations of the path rows, then the merge records, then the replay of the other path nodes
//
// so that the longest chain is path, sums, token, draft, with claims and applies beside it.  The replay of the other path nodes
// is a check that no result waits for, but it reads the pending draft, which the same workgroup overwrites when all its waves have
// joined: it comes before that and in this workgroup, the waves without records first.  The summing workgroups read nothing that
// this launch overwrites, and wait for nothing.
//   - A partial sum is one self-validating word (top bit set; the row kernel before has cleared the words).  The ranges
//     are so small that the wave which draws the token finds it by itself, with one more look at one range.
//   - Between claims and applies, and between applies and the draft's lookups, the trajectories meet at a counter
//     (cleared by the row kernel as well, so that a recorded launch can be replayed).  A third one counts observations: only
//     a slot that several records have claimed needs those of others.
//   - Inside a workgroup the waves meet at counters in shared memory until all of them join for the draft.
//   - Waits are bounded by the handle's wait limit (TailWait).  When all waves of a trajectory have joined, its waits are over:
//     one of them that ran out is counted there, the trajectory's outputs are void, its context stays and nothing is drafted.
// The first B workgroups are resident from the start and take at most an eighth of what the stream's compute units hold at
// once (plan_tail_places; asked for every call, a stream may be masked to a few of them): the summing workgroups, which wait
// for nothing, have room, with launches of other handles beside it as well.
//
// Bound by latency: of the 13 us of one launch for 1 x 32 rows x 152 064 (clock readings), the path is known at 1.6, the last
// sum is stored at 1.9, seen at 3 (a word travels about 1 us from one workgroup to another), the token is there at 8.6 and the
// draft takes the last 4.5; claims end at 4.1, applies at 7.
// Steps, separate launches / one launch, us:
// 1 x 16 rows x 32 000 fp32 27.9 / 22.5, 1 x 32 x 152 064 bf16 32.4 / 25.5, 8 x 32 x 128 256 47.1 / 41.4,
// 6 x 40 x 50 257 by verify, update and draft 62.3 / 55.0, 32 x 64 x 152 064 with long paths 149.9 / 148.0; verify of
// 12 x 48 x 32 003 fp32 37.6 / 33.7.
// Then, with what waits for nothing moved off the chains (the stop node's tests left by the row kernel, a range looked at once,
// the draft's constants formed before the waves join and its root taken by an idle wave, claims met without observations, upper
// nodes replayed by waves that are done, a wave's next record requested while one is folded; with what the row kernel gained at the
// same time): 1 x 16 22.9 / 22.3, 1 x 32 25.0 / 23.4, 8 x 32 42.0 / 39.2, with long paths 47.9 / 44.7, 24 x 20 x 50 000 42.7 / 38.1,
// 32 x 64 with long paths 147.3 / 144.9, chains of 32 nodes all accepted, x 32 000, 1 trajectory 54.4 / 54.6, 12 76.5 / 73.3.
// The arguments are read again in each phase (fresh_args): kept from the start they were 361 spilled scalar registers.
// ---------------------------------------------------------------------------------------------
constexpr int kTailThreads = 1024, kTailWaves = kTailThreads / 64;
// Most trajectories.  (63 x 15 rows x 198 592 130.0 / 128.1 us; beyond, the first workgroups would be more than an eighth of
// the device, and the launches saved are few per cent of such steps.)
constexpr int kTailBatch = 64;
constexpr int kSubMax = 512, kSubPerLane = kSubMax / 64;   // most ranges of a row
constexpr unsigned long long kSumThere = 1ull << 63;   // set in a partial sum (a row's sum is below 2^63)

struct StepTailArgs {
    PathArgs path;
    MergeArgs mg;
    DraftArgs draft;
    unsigned long long *part;   // [B][W][nsub]
    unsigned *bar;              // [kTailCounters] trajectories whose claims are made, records applied, observations written
    const StagedTest *staged;   // [B*N][K] what the row kernel has left of the nodes' tests, or NULL
    int nsub;                   // ranges of a row: a multiple of kTailWaves
    int row_slots;              // path rows that have summing workgroups of their own (longer paths loop)
    unsigned wait_units;        // bound of every wait in units of wait_clock
    int merge, drafts;          // a verification: neither; an update: merge; a step: both  (words: as bytes they would be vector
                                // loads, whose wait is one for every store before them as well)
    const int32_t *given_tok;   // [B][W] tokens committed instead of the emitted ones, or NULL (an update: its tokens)
    int32_t *ctx_tail;
    long long *ctx_len;
};

struct SmallTail {
    int path[kMaxDepth + 2];
    int len, ok;                // ok: 0 once a wait of the trajectory has run out (TailWait)
    int arrived[2], met;        // waves that have written their observations / applied their records; all claims are made
    int32_t seq[kMaxOrder + kMaxDepth + 2];   // context tail (oldest first), then the committed tokens
    long long had;                            // length of the context before
    long long slot[kMaxOrder * (kMaxDepth + 1)];   // table slot of each record of the trajectory
    alignas(16) unsigned long long P[kSubMax];   // masses of the ranges; then, while the token is located, the vectors of one
    alignas(16) unsigned long long scratch[kTailWaves][2 * kMaxK];
};
// Per node: outcome + 1, drafted children << 6, first child + 1 << 12 (a node has at most kMaxK children).
struct TailStage { int32_t *word; float *m; int32_t *tok; };
constexpr size_t kTailFixed = (sizeof(SmallTail) + 15) & ~(size_t)15;
constexpr size_t tail_shared_bytes(int N) { return kTailFixed + (size_t)(3 * N + 3) / 4 * 16 + draft_shared_bytes(N, kTailWaves); }
static_assert(2 * ((tail_shared_bytes(kMaxNodes) + 1279) / 1280 * 1280) <= 160 * 1024, "two workgroups per compute unit");
__device__ __forceinline__ TailStage tail_stage(char *smem, int N)
{
    int32_t *w = (int32_t *)(smem + kTailFixed);
    return TailStage{w, (float *)(w + N), w + 2 * N};
}
__device__ __forceinline__ int stage_outcome(int32_t w) { return (w & 63) - 1; }
__device__ __forceinline__ int stage_drafted(int32_t w) { return (w >> 6) & 63; }
__device__ __forceinline__ int stage_first(int32_t w) { return (w >> 12) - 1; }

// follows the accepted path (one thread, after the staging)
__device__ __forceinline__ int tail_walk(const TailStage &st, int D, int *path)
{
    int cur = 0, len = 0;
    for (;;) {
        path[len++] = cur;
        const int32_t w = st.word[cur];
        const int acc = stage_outcome(w);
        if (acc < 0 || len > D) return len;
        cur = stage_first(w) + acc;
    }
}

// Range `sub` of a row's vectors.
struct SubRange { int v0, v1; };
__device__ __forceinline__ int sub_vectors(const RowGeom &g, int nsub) { return (g.nvec + nsub - 1) / nsub; }
__device__ __forceinline__ SubRange sub_range(const RowGeom &g, int per, int sub)
{
    const int v0 = sub * per < g.nvec ? sub * per : g.nvec;
    return SubRange{v0, v0 + per < g.nvec ? v0 + per : g.nvec};
}

__device__ __forceinline__ bool still_ok(const SmallTail *ts)
{
    return __hip_atomic_load(&ts->ok, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0;
}
// The device's constant clock in units of 64 ticks (32 bits of them are 45 minutes at 100 MHz).
constexpr int kWaitShift = 6;
__device__ __forceinline__ unsigned wait_clock() { return (unsigned)(wall_clock64() >> kWaitShift); }
// A wait: whether it, not satisfied yet, goes on for another poll.  It ends after `units` of that clock or kWaitMaxPolls polls,
// and as soon as another wait of the trajectory has run out.
struct TailWait {
    unsigned since = wait_clock(), now = since;
    unsigned polls = 0u;
    __device__ __forceinline__ bool goes_on(SmallTail *ts, unsigned units)
    {
        // (the clock is far away: its reading is looked at after the next poll)
        if (now - since < units && ++polls < kWaitMaxPolls && __builtin_amdgcn_readfirstlane(still_ok(ts) ? 1 : 0)) {
            now = wait_clock();
            return true;
        }
        __hip_atomic_store(&ts->ok, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return false;
    }
};

// Lane l waits for the partial sums of ranges [l * q, l * q + q), q = ranges per lane, of path row j.
// request() asks for them once, wait() asks again until they are there.
struct SubSums {
    unsigned long long v[kSubPerLane];
    const unsigned long long *p;
    int q, here;               // ranges per lane (uniform), ranges of this lane
    __device__ __forceinline__ void ask()
    {
#pragma unroll
        for (int k = 0; k < kSubPerLane; ++k)
            if (k < q) v[k] = ld_agent(p + (k < here ? k : 0));
    }
    __device__ __forceinline__ void request(const StepTailArgs &A, int b, int j, int per_lane, int lane)
    {
        q = per_lane;
        const int at = lane * q < A.nsub ? lane * q : 0;   // (a lane without ranges looks at the first one)
        here = A.nsub - lane * q;
        p = A.part + ((size_t)b * A.path.R + j) * A.nsub + at;
#pragma unroll
        for (int k = 0; k < kSubPerLane; ++k) v[k] = kSumThere;
        ask();
    }
    __device__ __forceinline__ void wait(SmallTail *ts, unsigned units)
    {
        TailWait w;
#pragma clang loop unroll(disable)
        for (;;) {
            bool all = true;
#pragma unroll
            for (int k = 0; k < kSubPerLane; ++k)
                if (k < q) all &= (v[k] & kSumThere) != 0ull;
            if (__all(all) || !w.goes_on(ts, units)) break;
            __builtin_amdgcn_s_sleep(1);
            ask();
        }
#pragma unroll
        for (int k = 0; k < kSubPerLane; ++k) v[k] = k < q && k < here ? v[k] & ~kSumThere : 0ull;
    }
};
__device__ __forceinline__ unsigned long long lane_total(const SubSums &s)
{
    unsigned long long t = 0ull;
#pragma unroll
    for (int k = 0; k < kSubPerLane; ++k)
        if (k < s.q) t += s.v[k];
    return t;
}

// A node's proposal as it enters its accept tests (lane i: stored id i, -1 if there is none, and what StagedTest says).
template <int DT>
__device__ __forceinline__ StagedTest tail_node_tests(const StepTailArgs &A, int b, size_t row, int nch, int fc, int lane, int32_t &my_id)
{
    const PathArgs &a = A.path;
    StagedTest t{0.0f, 0.0f, 0.0f, -1};
    my_id = -1;
    if (A.staged) {
        if (lane < a.K) { my_id = a.draft_qid[row * a.K + lane]; t = A.staged[row * a.K + lane]; }
        if ((uint32_t)my_id >= (uint32_t)a.V) my_id = -1;
        return t;
    }
    float mu = 0.0f;
    int32_t ch = -1;
    if (lane < a.K) { my_id = a.draft_qid[row * a.K + lane]; mu = a.draft_qmu[row * a.K + lane]; }
    if (lane < nch && lane < kMaxK && fc >= 0 && fc + lane < a.N) ch = a.draft_tok[(size_t)b * a.N + fc + lane];
    if ((uint32_t)my_id >= (uint32_t)a.V) { my_id = -1; mu = 0.0f; }  // never index outside the row
    else t.l = load_scalar<DT>((const char *)a.logits + row * (size_t)a.V * VecTraits<DT>::ES, my_id);
    const NodeTests n = node_tests_prepare(lane, a.K, my_id, mu, nch, ch, a.seed, (uint32_t)b, a.step, fc);
    t.w = n.w; t.om = n.om; t.pos = n.pos;
    return t;
}

template <int DT>
__device__ __forceinline__ void tail_sums(int i, SmallTail *ts, char *smem)
{
    constexpr int ES = VecTraits<DT>::ES;
    const StepTailArgs &A = fresh_args<StepTailArgs>();
    const PathArgs &a = A.path;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int groups = A.nsub / kTailWaves;
    // row slots are the slowest: the workgroups of the root rows, which every path has, are first
    const int j = i / (groups * a.B), b = i / groups % a.B, sub = i % groups * kTailWaves + wave;
    const TailStage st = tail_stage(smem, a.N);
    int len = 0;   // (not followed yet)
    for (int jj = j; jj < a.R; jj += A.row_slots) {
        int node;
        float m;
        if (a.mode != 0) {
            node = commit_row_of(a, b, jj);
            if (node < 0) continue;   // (the same in the whole workgroup)
            m = a.src_m[b * a.R + jj];
        } else if (jj == 0) {
            node = 0;
            m = a.src_m[b * a.N];
        } else {
            if (len == 0) {
                for (int u = tid; u < a.N; u += kTailThreads) {
                    st.word[u] = (a.outcome[(size_t)b * a.N + u] + 1) | ((a.tree.first_child[u] + 1) << 12);
                    st.m[u] = a.src_m[(size_t)b * a.N + u];
                }
                __syncthreads();
                if (tid == 0) ts->len = tail_walk(st, a.tree.D, ts->path);
                __syncthreads();
                len = ts->len;
            }
            if (jj >= len) return;
            node = ts->path[jj];
            m = st.m[node];
        }
        node = __builtin_amdgcn_readfirstlane(node);
        const char *rowp = (const char *)a.logits + (size_t)(b * a.N + node) * (size_t)a.V * ES;
        const RowGeom g = row_geom<DT>(rowp, a.V);
        const int per = sub_vectors(g, A.nsub);
        const SubRange r = sub_range(g, per, sub);
        unsigned long long S;
        if (per <= 64) S = thread_exact_partial<DT, 1>(rowp, g, r.v0, r.v1, sub == 0, m, a.c, lane, 64, a.fx_shift);
        else S = thread_exact_partial<DT, 4>(rowp, g, r.v0, r.v1, sub == 0, m, a.c, lane, 64, a.fx_shift);
        S = wave_sum_u64(S);
        if (lane == 0) st_agent(&A.part[((size_t)b * a.R + jj) * A.nsub + sub], S | kSumThere);
    }
}

// The stop row of trajectory b by its first wave: replay of the node's accept tests with exact probabilities and the
// resampled token, which is returned.  The same arithmetic as finish_stop_row, in ranges instead of segments.
template <int DT>
__device__ __forceinline__ int32_t tail_token(const StepTailArgs &A, SmallTail *ts, const TailStage &stage, int b, int len, int q, int lane)
{
    constexpr int ES = VecTraits<DT>::ES, EPV = VecTraits<DT>::EPV;
    const PathArgs &a = A.path;
    const int node = __builtin_amdgcn_readfirstlane(ts->path[len - 1]);
    const int32_t word = __builtin_amdgcn_readfirstlane(stage.word[node]);
    const int nch = stage_drafted(word);
    const float m = uniform_f32(stage.m[node]);
    const size_t row = (size_t)b * a.N + node;
    const char *rowp = (const char *)a.logits + row * (size_t)a.V * ES;
    const RowGeom g = row_geom<DT>(rowp, a.V);
    const int per = sub_vectors(g, A.nsub);
    // ---- before the sums are needed: the node's proposal, the row's edges, the tests and the position's random bits
    int32_t my_id = -1;
    StagedTest mine_t{0.0f, 0.0f, 0.0f, -1};
    if (nch > 0) mine_t = tail_node_tests<DT>(A, b, row, nch, stage_first(word), lane, my_id);
    const int32_t top0 = a.src_top_idx[row * a.K];
    int edge_id = -1;
    if (lane < g.head) edge_id = lane;
    else if (lane < g.head + g.ntail) edge_id = g.tail0 + (lane - g.head);
    const unsigned long long edge_f =
        edge_id >= 0 ? fixed_mass(exact_exp2(scaled_offset(load_scalar<DT>(rowp, edge_id), m, a.c)), a.fx_shift) : 0ull;
    const Philox4 ph = philox_group(a.seed, (uint32_t)b, a.step, (uint32_t)node, 0u, kStreamBonus);
    unsigned long long u = ((unsigned long long)ph.x << 32) | ph.y;
    asm volatile("" : "+v"(u));   // (here: these instructions cost nothing while the sums are on their way)
    const float my_e = my_id >= 0 ? exact_exp2(scaled_offset(mine_t.l, m, a.c)) : 0.0f;
    const bool has_edge = g.head + g.ntail > 0;  // rows that start on a 16-byte boundary have none
    const unsigned long long edge_all = has_edge ? wave_sum_u64(edge_f) : 0ull;
    const NodeTests tests{mine_t.w, mine_t.om, mine_t.pos};
    const bool in_sub = my_id >= g.head && my_id < g.tail0;
    const int my_sub = in_sub ? ((my_id - g.head) / EPV) / per : -1;

    // (asked for not before they are needed: they are there by now, and an answer that came too early would be a second question)
    SubSums part;
    part.request(A, b, len - 1, q, lane);
    part.wait(ts, A.wait_units);
    const unsigned long long S = wave_sum_u64(lane_total(part));
    const float s = normaliser_from_fixed(S, a.fx_shift);
    // ---- residual at the stop node
    bool support = nch > 0;
    float my_r = 0.0f, rho = 1.0f;
    if (support) {
        const NodeResult nr = wave_node_outcome(lane, a.K, tests, my_e / s, nch, false, 0.0f, a.onehot);
        my_r = (lane < a.K && my_id >= 0) ? nr.r : 0.0f;
        rho = nr.rho;
        if (lane == 0 && nr.accepted != -1 && still_ok(ts)) atomicAdd(&a.stats[kStatMismatch], 1ull);  // the stop node rejects all
        // a residual that is not a distribution any more (the normalising mass underflowed) is not used
        const float rs = wave_tree_sum(my_r);
        if (!(rs <= 2.0f) || !(rho < __builtin_inff())) support = false;
    }
    // ---- integer masses (unit 2^-(40 - fx_shift) / s * rho): support token i weighs floor(r_i * (S / rho)),
    // a token outside the support the term it contributes to S
    unsigned long long my_g = 0ull, g_inc = 0ull, gsum = 0ull, T = 0ull, edge_m = 0ull, head_m = 0ull;
    for (int attempt = 0; attempt < 2; ++attempt) {
        unsigned long long my_f = 0ull;
        my_g = 0ull;
        const bool mine = support && lane < a.K && my_id >= 0;
        if (mine) {
            const double ratio = (double)S / (double)rho;
            my_g = (unsigned long long)((double)my_r * ratio);
            my_f = fixed_mass(my_e, a.fx_shift);
        }
        if (has_edge) {
            bool edge_in_support = false;
            if (support)
                for (int i = 0; i < a.K; ++i) edge_in_support |= __builtin_amdgcn_readlane(my_id, i) == edge_id;
            edge_m = (edge_id >= 0 && !edge_in_support) ? edge_f : 0ull;
            head_m = wave_sum_u64(lane < g.head ? edge_m : 0ull);
        }
        // the ranges' masses without the support (and, in the first range, without the edges)
#pragma unroll
        for (int k = 0; k < kSubPerLane; ++k)
            if (k < q) ts->P[lane * q + k] = part.v[k] - (lane == 0 && k == 0 ? edge_all : 0ull);
        __builtin_amdgcn_wave_barrier();
        if (mine && in_sub) atomicAdd(&ts->P[my_sub], 0ull - my_f);
        __builtin_amdgcn_wave_barrier();
        g_inc = wave_inclusive_scan_u64(my_g);
        gsum = readlane_u64(g_inc, 63);
        T = S + gsum - wave_sum_u64(my_f);
        if (!support || T != 0ull) break;
        support = false;  // the residual vanished: draw from the target itself
    }
    unsigned long long t = __umul64hi(u, T);
    if (t < gsum) return __builtin_amdgcn_readlane(my_id, __ffsll((long long)__ballot(t < g_inc)) - 1);
    t -= gsum;
    // the layout after the support: head elements, ranges, tail elements, each in id order
    auto edge_token = [&](bool head, unsigned long long rem) {
        const unsigned long long em = head == (lane < g.head) ? edge_m : 0ull;
        const unsigned long long einc = wave_inclusive_scan_u64(em);
        const int w = __ffsll((long long)__ballot(rem < einc)) - 1;
        return w >= 0 ? __builtin_amdgcn_readlane(edge_id, w) : top0;
    };
    if (t < head_m) return edge_token(true, t);
    t -= head_m;
    unsigned long long pv[kSubPerLane], mine_total = 0ull;
#pragma unroll
    for (int k = 0; k < kSubPerLane; ++k)
        if (k < q) { pv[k] = ts->P[lane * q + k]; mine_total += pv[k]; }
    const unsigned long long inc = wave_inclusive_scan_u64(mine_total);
    const int win = __ffsll((long long)__ballot(t < inc)) - 1;
    if (win < 0) return edge_token(false, t - readlane_u64(inc, 63));
    // in the winning lane: which of its ranges
    unsigned long long rem = t - (inc - mine_total);
    int sub = -1;
#pragma unroll
    for (int k = 0; k < kSubPerLane; ++k)
        if (k < q && sub < 0) {
            if (rem < pv[k]) sub = lane * q + k;
            else rem -= pv[k];
        }
    sub = __builtin_amdgcn_readlane(sub, win);
    rem = readlane_u64(rem, win);
    // ---- locate the token inside the range: every lane owns a contiguous run of vectors, so lane order is id order; then
    // every lane an element of the winning run
    const SubRange r = sub_range(g, per, sub < 0 ? 0 : sub);
    const int cpt = (per + 63) / 64;
    const int r0 = r.v0 + lane * cpt < r.v1 ? r.v0 + lane * cpt : r.v1, r1 = r0 + cpt < r.v1 ? r0 + cpt : r.v1;
    const unsigned long long within = __ballot(support && lane < a.K && in_sub && my_sub == sub);   // stored ids in this range
    constexpr int kBatch = 4;
    uint4 *run = (uint4 *)ts->P;   // a range of up to kBatch vectors per lane is looked at twice: the second time here
    static_assert(sizeof(ts->P) >= 64 * kBatch * sizeof(uint4), "a range in shared memory");
    unsigned long long sum = 0ull;
    const int last = r1 > r0 ? r1 - 1 : (r.v1 > 0 ? r.v1 - 1 : 0);
    for (int k0 = 0; k0 < cpt; k0 += kBatch) {
        uint4 w[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
            if (k0 + k < cpt) w[k] = g.vp[r0 + k0 + k < last ? r0 + k0 + k : last];
        double acc = kWhole;
        whole_begin();
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            if (k0 + k >= cpt) continue;   // uniform
            const int e0 = g.head + (r0 + k0 + k) * EPV;
            uint32_t without = 0u;
            for (unsigned long long left = within; left; left &= left - 1) {
                const uint32_t d = (uint32_t)(__builtin_amdgcn_readlane(my_id, __ffsll((long long)left) - 1) - e0);
                if (d < (uint32_t)EPV) without |= 1u << d;
            }
            if (k0 == 0) run[lane * kBatch + k] = w[k];
            add_exact_terms<DT>(w[k], r0 + k0 + k < r1 ? without : ~0u, m, a.c, (uint32_t)a.fx_shift << 23, acc);
        }
        whole_end();
        sum += (unsigned long long)__double_as_longlong(acc) & 0xFFFFFFFFFFFFFull;
    }
    const unsigned long long finc = wave_inclusive_scan_u64(sum);
    const int who = __ffsll((long long)__ballot(rem < finc)) - 1;
    if (who >= 0) {
        rem -= readlane_u64(finc, who) - readlane_u64(sum, who);
        const int first = g.head + __builtin_amdgcn_readlane(r0, who) * EPV, n = (__builtin_amdgcn_readlane(r1, who) - __builtin_amdgcn_readlane(r0, who)) * EPV;
        __builtin_amdgcn_wave_barrier();
        for (int base = 0; base < n; base += 64) {
            const int id = first + base + lane;
            const bool in = base + lane < n;
            const float x = cpt <= kBatch ? load_scalar<DT>(run + who * kBatch, in ? base + lane : 0) : load_scalar<DT>(rowp, in ? id : first);
            unsigned long long f = in ? fixed_mass(exact_exp2(scaled_offset(x, m, a.c)), a.fx_shift) : 0ull;
            for (unsigned long long left = within; left; left &= left - 1)
                if (__builtin_amdgcn_readlane(my_id, __ffsll((long long)left) - 1) == id) f = 0ull;
            const unsigned long long einc = wave_inclusive_scan_u64(f);
            const unsigned long long hit = __ballot(rem < einc);
            if (hit) return first + base + __ffsll((long long)hit) - 1;
            rem -= readlane_u64(einc, 63);
        }
    }
    // not reachable while the partial sums describe this row; keep the output a valid token
    if (lane == 0 && still_ok(ts)) atomicAdd(&a.stats[kStatMismatch], 1ull);
    return top0;
}

// A counter in shared memory at which the waves of a workgroup meet without the first one.
// Returns (in lane 0) how many had arrived before.
__device__ __forceinline__ int wave_arrive(int *counter, int lane)
{
    publish_fence();   // what this wave stored is complete
    return lane == 0 ? __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0;
}
__device__ __forceinline__ void wave_await(const int *counter, int target)
{
    // (every wave of the workgroup is resident and arrives, at the latest when its own bounded waits have ended)
    while (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < target) __builtin_amdgcn_s_sleep(1);
    consume_fence();
}
// The trajectories' workgroups meet (called by one wave of each).
__device__ __forceinline__ void tail_meet(const StepTailArgs &A, int which, SmallTail *ts, int lane)
{
    const unsigned B = (unsigned)A.path.B;
    if (B == 1) return;
    if (lane == 0) {
        atomicAdd(&A.bar[which], 1u);
        TailWait w;
        while (ld_agent(&A.bar[which]) < B && w.goes_on(ts, A.wait_units)) __builtin_amdgcn_s_sleep(1);
    }
    consume_fence();
}
// Waits until every trajectory's observations are there.
__device__ __forceinline__ bool tail_observed(const StepTailArgs &A, SmallTail *ts, int lane)
{
    if (lane == 0) {
        TailWait w;
        while (ld_agent(&A.bar[2]) < (unsigned)A.path.B && w.goes_on(ts, A.wait_units)) __builtin_amdgcn_s_sleep(1);
    }
    consume_fence();
    return still_ok(ts);
}

template <int DT>
__device__ __forceinline__ void tail_trajectory(int b, SmallTail *ts, char *smem)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kControl = kTailWaves - 1;   // claims the slots
    const int N = fresh_args<StepTailArgs>().path.N;
    const TailStage stage = tail_stage(smem, N);
    const DraftShared dsm = draft_shared_carve(smem + kTailFixed + (size_t)(3 * N + 3) / 4 * 16, N, kTailWaves);
    // where the summing waves share a SIMD with these, the longer chain goes first
    __builtin_amdgcn_s_setprio(3);
    int len, mode, level_reg = 0, n_given = 0;
    int32_t ctx = 0;            // lanes 0..7: context tail, oldest first; lanes 8 + j: given token j (first and control wave)
    long long ctx_len = 0;
    {
        // ---- everything that is known before the launch is requested at once
        const StepTailArgs &A = fresh_args<StepTailArgs>();
        const PathArgs &a = A.path;
        mode = a.mode;
        if (A.merge && (wave == 0 || wave == kControl)) {
            if (lane < kMaxOrder) ctx = A.ctx_tail[(size_t)b * kMaxOrder + lane];
            else if (A.given_tok && lane < kMaxOrder + a.W) ctx = A.given_tok[(size_t)b * a.W + (lane - kMaxOrder)];
            ctx_len = A.ctx_len[b];
        }
        if (mode != 0) {
            n_given = clamp_len(a.commit_len[b], a.W);
            if (tid < a.W) ts->path[tid] = commit_row_of(a, b, tid);
        } else {
            if (A.drafts) level_reg = lane < a.tree.D + 2 ? a.tree.level_start[lane] : 0;
            for (int u = tid; u < N; u += kTailThreads) {
                const size_t at = (size_t)b * N + u;
                const int fc = a.tree.first_child[u];
                stage.word[u] = (a.outcome[at] + 1) | (a.draft_has[at] << 6) | ((fc + 1) << 12);
                stage.m[u] = a.src_m[at];
                stage.tok[u] = a.draft_tok[at];
                if (A.drafts) {
                    dsm.info[u] = (fc << 8) | a.tree.nchild[u];
                    if (u > 0) dsm.tok[u] = -1;
                    dsm.has[u] = 0;
                }
            }
            if (A.drafts) {
                if (tid <= kMaxOrder) dsm.n_hit[tid] = 0u;
                if (tid >= 1 && tid < kMaxDepth + 2) dsm.live[tid] = 0;
            }
        }
        if (tid == 0) { ts->ok = 1; ts->arrived[0] = ts->arrived[1] = 0; ts->met = 0; }
        asm volatile("" : "+v"(level_reg));
        __syncthreads();
        if (mode == 0 && tid == 0) ts->len = tail_walk(stage, a.tree.D, ts->path);
        if (mode != 0 && tid == 0) ts->len = n_given;
        __syncthreads();
        len = __builtin_amdgcn_readfirstlane(ts->len);
    }
    const int q = (fresh_args<StepTailArgs>().nsub + 63) / 64;   // ranges per lane that waits for a row's sums
    // waves [first, kControl) finish rows and apply records
    const int first = mode == 0 ? 1 : 0;

    if (wave == kControl) {
        const StepTailArgs &A = fresh_args<StepTailArgs>();
        const PathArgs &a = A.path;
        if (A.merge) {
            const int W = a.W;
            const MergeArgs &mg = A.mg;
            const int NO = mg.omax - mg.omin + 1, per_traj = mg.R * NO;
            // context tail and committed tokens in one line (the last one, which no key contains, may be still to come)
            int32_t v = ctx;
            const int jt = lane - kMaxOrder;
            if (!A.given_tok && jt >= 0) v = jt + 1 < len ? stage.tok[ts->path[jt + 1]] : 0;
            if (lane < kMaxOrder + W) ts->seq[lane] = v;
            if (lane == 0) ts->had = ctx_len;
            __builtin_amdgcn_wave_barrier();
            for (int i = lane; i < ((per_traj + 63) & ~63); i += 64) {
                int outcome = kClaimNone;
                if (i < per_traj) {
                    const int n = mg.omin + i % NO, j = i / NO;
                    long long slot = -1;
                    if (j < len && ctx_len + j >= n && ts->path[j] >= 0) {
                        int32_t newest[kMaxOrder];
#pragma unroll
                        for (int k = 0; k < kMaxOrder; ++k) newest[k] = k < n ? ts->seq[kMaxOrder + j - 1 - k] : 0;
                        outcome = claim_slot(mg, b * per_traj + i, n, fingerprint_newest_first(n, newest), slot);
                    }
                    st_agent(&mg.rec_slot[b * per_traj + i], slot);
                    ts->slot[i] = slot;
                }
                count_claims(mg, outcome, lane);
            }
            if (mode != 0) {
                // the context of an update: the last tokens of tail and commit
                const int32_t t = __shfl(v, (lane & (kMaxOrder - 1)) + len);
                if (lane < kMaxOrder) A.ctx_tail[(size_t)b * kMaxOrder + lane] = t;
                if (lane == 0) A.ctx_len[b] = ctx_len + len;
            }
        }
    } else if (wave >= first) {
        const StepTailArgs &A = fresh_args<StepTailArgs>();
        const PathArgs &a = A.path;
        if (mode == 0 && wave == kControl - 1) {   // (few paths are so long that it has a row)
            const int W = a.W;
            if (lane < W) {
                a.out_node[(size_t)b * W + lane] = lane < len ? ts->path[lane] : -1;
                // (the last emitted token, position len - 1, is written by the first wave)
                if (lane + 1 < len) a.out_tok[(size_t)b * W + lane] = stage.tok[ts->path[lane + 1]];
                else if (lane >= len) a.out_tok[(size_t)b * W + lane] = -1;
            }
            if (lane < len) atomicAdd(&a.node_count[ts->path[lane]], 1ull);  // paper Sec. 4.3: acceptance statistics per node
            if (lane == 0) {
                a.out_len[b] = len;
                // accept tests along the path: rank + 1 at every accepted node, all children at the stop node
                unsigned long long tests = (unsigned long long)stage_drafted(stage.word[ts->path[len - 1]]);
                for (int k = 0; k + 1 < len; ++k) tests += (unsigned long long)(stage_outcome(stage.word[ts->path[k]]) + 1);
                atomicAdd(&a.stats[kStatTokens], (unsigned long long)len);
                atomicAdd(&a.stats[kStatTests], tests);
                if (len > a.late_len) atomicAdd(&a.stats[kStatLatePaths], 1ull);
            }
        }
        // observations (a verification leaves none)
        for (int j = wave - first; A.merge && j < len; j += kControl - first) {
            const int node = __builtin_amdgcn_readfirstlane(ts->path[j]);
            if (node < 0) continue;
            const size_t src = mode == 0 ? (size_t)b * a.N + node : (size_t)b * a.R + j;
            int32_t id = 0;
            float l = 0.0f;
            if (lane < a.K) { id = a.src_top_idx[src * a.K + lane]; l = a.src_top_l[src * a.K + lane]; }
            const float m = mode == 0 ? stage.m[node] : a.src_m[src];
            SubSums part;
            part.request(A, b, j, q, lane);
            part.wait(ts, A.wait_units);
            const unsigned long long S = wave_sum_u64(lane_total(part));
            write_observation(a, b, j, id, l, m, normaliser_from_fixed(S, a.fx_shift), lane);
        }
    }
    if (fresh_args<StepTailArgs>().merge && wave >= first) {
        // ---- every trajectory's claims, this one's observations; then its records (a wave without one waits for neither)
        const StepTailArgs &A = fresh_args<StepTailArgs>();
        const MergeArgs &mg = A.mg;
        const int NO = mg.omax - mg.omin + 1, rec0 = b * mg.R * NO;
        if (wave == kControl) {
            publish_fence();   // the claims are complete
            tail_meet(A, 0, ts, lane);
            if (lane == 0) __hip_atomic_store(&ts->met, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else if (wave_arrive(&ts->arrived[0], lane) == kControl - first - 1 && lane == 0) {
            atomicAdd(&A.bar[2], 1u);   // the last of them: the trajectory's observations are complete
        }
        const int n_rec = len * NO;
        int i = wave - first;
        if (i < n_rec) {
            wave_await(&ts->met, 1);
            long long slot = ts->slot[i];
            ClaimedRecord r;
            if (slot >= 0) r.request_slot(mg, rec0 + i, slot, lane);
            wave_await(&ts->arrived[0], kControl - first);
            if (still_ok(ts)) {
                if (slot >= 0) r.request_observation(mg, lane);
                while (i < n_rec) {
                    // (the next record is on its way while this one is folded)
                    i += kTailWaves - first;
                    const long long next_slot = i < n_rec ? ts->slot[i] : -1;
                    ClaimedRecord next;
                    if (next_slot >= 0) { next.request_slot(mg, rec0 + i, next_slot, lane); next.request_observation(mg, lane); }
                    if (slot >= 0) apply_claimed(mg, r, lane, ts->scratch[wave], [&] { return tail_observed(A, ts, lane); });
                    slot = next_slot;
                    r = next;
                }
            } else {
                for (; i < n_rec; i += kTailWaves - first) {
                    slot = ts->slot[i];
                    if (slot >= 0 && lane == 0) release_claimed(mg, slot);
                }
            }
        }
        if (A.drafts) {
            wave_arrive(&ts->arrived[1], lane);
            if (wave == kControl) {
                wave_await(&ts->arrived[1], kTailWaves - first);
                tail_meet(A, 1, ts, lane);   // every record is applied before the first lookup
            }
        }
    }
    if (mode == 0 && wave >= first && wave < kControl) {
        // ---- replay of the path nodes above the stop node, the first ones by the waves with the fewest records.  What it reads of
        // the pending draft is overwritten behind the barrier below.  (Sum before node: together they need more registers
        // than there are.)  Where waves without records waited for the claims as well / as it is: 1 x 16 rows 23.1 / 22.7 us,
        // 1 x 32 24.6 / 24.4, 8 x 32 39.2 / 39.2.
        const StepTailArgs &A = fresh_args<StepTailArgs>();
        const PathArgs &a = A.path;
        for (int j = kControl - 1 - wave; j + 1 < len; j += kControl - first) {
            const int node = __builtin_amdgcn_readfirstlane(ts->path[j]);
            float s;
            {
                SubSums part;
                part.request(A, b, j, q, lane);
                part.wait(ts, A.wait_units);
                s = normaliser_from_fixed(wave_sum_u64(lane_total(part)), a.fx_shift);
            }
            if (!still_ok(ts)) break;   // (the sum may not be the whole one; the trajectory is void)
            UpperReplay replay;
            replay.request<DT>(a, b, node, lane);
            replay.run(a, b, stage.m[node], s, stage_outcome(stage.word[node]), lane);
        }
    }
    if (wave == 0 && mode == 0) {
        const StepTailArgs &A = fresh_args<StepTailArgs>();
        const PathArgs &a = A.path;
        const int32_t token = tail_token<DT>(A, ts, stage, b, len, q, lane);
        if (lane == 0) a.out_tok[(size_t)b * a.W + (len - 1)] = token;
        if (A.drafts) {
            // the new context: the last tokens of tail and commit
            const int jt = lane - kMaxOrder;
            int32_t v = ctx;
            if (!A.given_tok && jt >= 0 && jt < len) v = jt + 1 < len ? stage.tok[ts->path[jt + 1]] : token;
            const int32_t t = __shfl(v, (lane & (kMaxOrder - 1)) + len);
            const long long now = ctx_len + len;
            if (lane < kMaxOrder) {
                dsm.recent[0][kMaxOrder - 1 - lane] = t;
                if (lane == kMaxOrder - 1) { dsm.tok[0] = now > 0 ? t : -1; dsm.live[0] = now > 0 && t >= 0; }
                A.ctx_tail[(size_t)b * kMaxOrder + lane] = t;   // (the control wave has read the old one before the path was followed)
            }
            if (lane == 0) { *dsm.clen = now; A.ctx_len[b] = now; }
        }
    }
    const bool drafts = fresh_args<StepTailArgs>().drafts != 0;
    // (after this barrier every wave has joined: no wait of this trajectory is left)
    if (drafts) draft_run<kTailThreads>(fresh_args<StepTailArgs>().draft, b, dsm, level_reg, [] { __syncthreads(); });
    else __syncthreads();
    if (__builtin_expect(!still_ok(ts), 0)) {
        // (not reachable while the other workgroups run)
        const StepTailArgs &A = fresh_args<StepTailArgs>();
        if (tid == 0) atomicAdd(&A.path.stats[kStatWaitExpired], 1ull);
        if (A.path.mode == 0) {
            const size_t at = (size_t)b * A.path.W;
            if (tid < A.path.W) { A.path.out_tok[at + tid] = -1; A.path.out_node[at + tid] = -1; }
            if (tid == 0) A.path.out_len[b] = 0;
        }
        if (A.merge) {   // (the context as it was)
            if (tid < kMaxOrder) A.ctx_tail[(size_t)b * kMaxOrder + tid] = ts->seq[tid];
            if (tid == 0) A.ctx_len[b] = ts->had;
        }
        if (!drafts) return;
        for (int u = tid; u < N; u += kTailThreads) {
            A.draft.draft_tok[(size_t)b * N + u] = -1;
            A.draft.draft_has[(size_t)b * N + u] = 0;
            if (A.draft.out_tok) A.draft.out_tok[(size_t)b * N + u] = -1;
        }
    }
}

// (64 registers: two workgroups per compute unit)
template <int DT>
__global__ __launch_bounds__(kTailThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void step_tail_kernel(StepTailArgs A)
{
    extern __shared__ __align__(16) char tail_smem[];
    SmallTail *ts = (SmallTail *)tail_smem;
    const int B = A.path.B;
    if ((int)blockIdx.x < B) tail_trajectory<DT>((int)blockIdx.x, ts, tail_smem);
    else tail_sums<DT>((int)blockIdx.x - B, ts, tail_smem);
}

}  // namespace stand
