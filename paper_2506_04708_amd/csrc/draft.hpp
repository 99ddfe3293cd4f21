// draft.hpp -- draft_kernel: multi-level lookup and Gumbel-Top-K along the static tree (paper Sec. 4.2).
#pragma once
#include <type_traits>

#include "wave_ops.hpp"

namespace stand {

// ---------------------------------------------------------------------------------------------
// Draft (paper Sec. 4.2): one workgroup per trajectory, tree levels in sequence, one wave per node.
// ---------------------------------------------------------------------------------------------
struct DraftArgs {
    char *table;
    uint64_t mask;
    int slot_bytes, K, max_probe;
    int B, W, omin, omax;
    uint64_t seed, step;
    TreeDev tree;
    int32_t *ctx_tail;
    long long *ctx_len;
    const int32_t *append_tok;   // [B][W] tokens to append to the contexts first, or NULL
    const int32_t *append_len;   // [B]
    int32_t *draft_tok, *draft_has, *draft_qid;
    float *draft_qmu;
    int32_t *out_tok;  // caller's copy, may be NULL
    unsigned long long *stats;
    int mode;          // 0: Gumbel-Top-K, 1: sequential multinomial without replacement, 2: largest means
    int32_t *recent_out;  // [B][N][kMaxOrder] or NULL: the recent tokens of every drafted node (all-nodes update)
};

constexpr int kDraftThreads = 1024;  // 16 waves: the nodes of a tree level are looked up side by side

// Shared memory of one trajectory's draft, sized for a tree of N nodes.
struct DraftShared {
    int32_t (*recent)[kMaxOrder];    // [N][kMaxOrder] recent[u][i]: the token i positions before the end of the
                                     // sequence that ends at node u (recent[u][0] is the node's own token), so a
                                     // key is read without walking up the tree; 16-byte aligned
    unsigned long long (*keys)[kMaxK];  // [waves][kMaxK] scores of the node a wave is ranking; 16-byte aligned
    long long *clen;
    unsigned *n_hit;                 // [kMaxOrder + 1] lookups answered by order n; [0]: misses
    int32_t *live;                   // [kMaxDepth + 2] a node of this tree level has a token
    int32_t *tok;                    // [N]
    int32_t *info;                   // [N] first child << 8 | number of children
    int32_t *has;                    // [N] children drafted
};
constexpr size_t draft_shared_fixed(int waves) { return (size_t)waves * kMaxK * 8 + 16 + 48 + 144; }
constexpr size_t draft_shared_bytes(int N, int waves) { return (size_t)N * (kMaxOrder + 3) * 4 + draft_shared_fixed(waves); }
__device__ __forceinline__ DraftShared draft_shared_carve(char *base, int N, int waves)
{
    DraftShared s;
    s.recent = (int32_t(*)[kMaxOrder])base;  base += (size_t)N * kMaxOrder * 4;
    s.keys = (unsigned long long(*)[kMaxK])base;  base += (size_t)waves * kMaxK * 8;
    s.clen = (long long *)base;              base += 16;
    s.n_hit = (unsigned *)base;              base += 48;
    s.live = (int32_t *)base;                base += 144;
    s.tok = (int32_t *)base;                 base += (size_t)N * 4;
    s.info = (int32_t *)base;                base += (size_t)N * 4;
    s.has = (int32_t *)base;
    return s;
}

// How a node's work is spread over the lanes of a wave: in each row of 16 lanes, G groups of 16 / G lanes hold the same
// 16 / G candidates (all values of a candidate are in one row, so that they move by data-parallel primitives, never
// through shared memory).  G = 4 for K <= 16, else 2.
template <int G>
struct CandLayout {
    static constexpr int kPerRow = 16 / G, kSlots = 4 * kPerRow;   // candidates per row, and of the wave
    static __device__ __forceinline__ int candidate(int lane) { return (lane >> 4) * kPerRow + (lane & (kPerRow - 1)); }
    static __device__ __forceinline__ int group(int lane) { return (lane & 15) / kPerRow; }
    static __device__ __forceinline__ int lane_of(int cand) { return cand / kPerRow * 16 + cand % kPerRow; }
    static constexpr int banks(int g) { return G == 4 ? 1 << g : 3 << (2 * g); }   // lanes of group g as banks of 4 lanes
    // combined over the groups of a row: rotations by 8 and, with four groups, 4 lanes
    static __device__ __forceinline__ int any_of_groups(int x)
    {
        x |= __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, true);
        if (G == 4) x |= __builtin_amdgcn_update_dpp(0, x, 0x124, 0xF, 0xF, true);
        return x;
    }
    static __device__ __forceinline__ int sum_of_groups(int x)
    {
        x += __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, true);
        if (G == 4) x += __builtin_amdgcn_update_dpp(0, x, 0x124, 0xF, 0xF, true);
        return x;
    }
};

// The value eight lanes further in the row of 16: the two halves of a row exchange theirs.
__device__ __forceinline__ uint32_t other_half(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128 /* row_ror:8 */, 0xF, 0xF, true);
}

// `uniform` of a token that lanes l and l ^ 8 both hold: each runs one of the two multiplications of a round (the same
// integers as philox4x32_10: lane 0..7 of a row holds words 0 and 3 of the state, lane 8..15 words 2 and 1), so that a
// round is one multiplication and one exchange long instead of two multiplications.
__device__ __forceinline__ float uniform_by_halves(uint64_t seed, uint32_t b, uint64_t step, uint32_t node, uint32_t token,
                                                   uint32_t stream, bool upper)
{
    uint32_t x = upper ? (uint32_t)step : token >> 2;
    uint32_t y = upper ? node | (stream << 24) : b | ((uint32_t)(step >> 32) << 20);
    const uint32_t mul = upper ? 0xCD9E8D57u : 0xD2511F53u;
    uint32_t key = upper ? (uint32_t)(seed >> 32) : (uint32_t)seed;
    const uint32_t key_step = upper ? 0xBB67AE85u : 0x9E3779B9u;
    asm volatile("" : "+v"(key));   // (the ten keys are formed on the way: kept from node to node they would take ten registers)
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p = (uint64_t)mul * x;
        uint32_t t = other_half(y) ^ key;
        asm("" : "+v"(t));   // (formed beside the multiplication: regrouped, the round would be two instructions longer)
        x = other_half((uint32_t)(p >> 32)) ^ t;
        y = (uint32_t)p;
        key += key_step;
    }
    // words 0..3 of the result: x of the lower, y of the upper, x of the upper, y of the lower lane
    const uint32_t mine = (token & 1u) ? y : x, other = other_half(mine);
    const bool want_upper = ((token ^ (token >> 1)) & 1u) != 0u;
    return word_to_uniform(want_upper == upper ? mine : other);
}

// Levels of the draft of trajectory b (see draft_trajectory): tree levels in sequence, one wave per node.  join(): called by all
// threads once what does not need the root's token is formed; that token is in `sm` when it returns.
template <int NT, int G, typename Join>
__device__ __forceinline__ void draft_levels(const DraftArgs &a, int b, const DraftShared &sm, int level_reg, const Join &join)
{
    using L = CandLayout<G>;
    constexpr int kMaxRounds = kMaxOrder / G;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int32_t *tok = sm.tok;
    int32_t(*recent)[kMaxOrder] = sm.recent;
    unsigned long long *keys = sm.keys[wave];
    const int N = a.tree.N, K = a.K, NO = a.omax - a.omin + 1;
    const int cand = L::candidate(lane), grp = L::group(lane);
    const bool upper = (lane & 8) != 0, has_cand = cand < K;
    // Lane j < omax of every row forms the term of the token omax - 1 - j positions back; the fingerprint of the last
    // n = omax - j tokens is then the sum over lanes j, j + 1, ... (three data-parallel moves), so that lane 0 holds the
    // longest order.
    const int j16 = lane & 15, n = a.omax - j16;
    unsigned long long term_mul = 0ull;
#pragma unroll
    for (int i = 0; i < kMaxOrder; ++i) term_mul = n == i + 1 ? fingerprint_multiplier(i) : term_mul;
    const unsigned long long order_term = (unsigned long long)(uint32_t)n * 0x2545F4914F6CDD1DULL;
    const bool order_lane = n >= a.omin && j16 < a.omax;
    const int rounds = (NO + G - 1) / G;  // <= kMaxRounds
    const unsigned payload = 16u + 4u * (unsigned)(has_cand ? cand : 0);   // where the lane's candidate stands in a slot
    unsigned my_hits = 0u;   // lane n <= kMaxOrder: lookups of this wave answered by order n; lane 0: misses
    int32_t *qid_out = a.draft_qid + (size_t)b * N * K;
    float *qmu_out = a.draft_qmu + (size_t)b * N * K;
    // the first node of a level falls to the second wave: the first one may have just found the root's token
    const int turn = (wave + NT / 64 - 1) & (NT / 64 - 1);
    const int D = a.tree.D;
    join();
    const long long clen = (long long)readlane_u64((unsigned long long)*sm.clen, 0);
    for (int d = 0; d < D; ++d) {
        // values read from shared memory that are the same in every lane go to scalar registers
        const int lo = __builtin_amdgcn_readlane(level_reg, d), hi = __builtin_amdgcn_readlane(level_reg, d + 1);
        // the wave's first node of the level is read together with the flag that ends the tree
        int live = sm.live[d];
        int u = lo + turn;
        int4 r_lo, r_hi;
        int32_t my_recent;
        int info, my_tok;
        auto read_node = [&](int at) {
            r_lo = *(const int4 *)&recent[at][0]; r_hi = *(const int4 *)&recent[at][4];
            my_recent = recent[at][(n - 1) & (kMaxOrder - 1)];
            info = sm.info[at]; my_tok = tok[at];
        };
        read_node(u < N ? u : 0);
        asm volatile("" : "+v"(live), "+v"(info), "+v"(my_tok), "+v"(my_recent));  // (one round trip, not one after the branch)
        if (!__builtin_amdgcn_readfirstlane(live)) break;  // a level without a drafted node ends the tree (the same in every wave)
        for (; u < hi; u += NT / 64) {
            if (u != lo + turn) read_node(u);
            info = __builtin_amdgcn_readfirstlane(info);
            const int nch = info & 0xFF, first = info >> 8;
            if (nch == 0 || __builtin_amdgcn_readfirstlane(my_tok) < 0) continue;
            // ---- multi-level lookup (paper Sec. 4.2).  The home slot of every order is read together with its
            // payload in one round trip; only a key that was displaced by linear probing needs further probes.
            unsigned long long fp;
            {
                unsigned long long acc = term_mul * ((unsigned long long)(uint32_t)my_recent + 1u);
                acc += dpp_fetch_u64<0x101, 0xF>(acc);  // row_shl:1
                acc += dpp_fetch_u64<0x102, 0xF>(acc);  // row_shl:2
                acc += dpp_fetch_u64<0x104, 0xF>(acc);  // row_shl:4
                fp = fmix64(acc + order_term);
                fp = fp ? fp : 1ull;
            }
            // (an order that is not looked up reads the table's first slot: no branch around the loads, which would make
            // them two round trips)
            const bool looked_up = order_lane && clen + d >= n;
            const unsigned long long home = looked_up ? (fp & a.mask) * (unsigned long long)(unsigned)a.slot_bytes : 0ull;
            const unsigned long long home_fp = ld_agent((const unsigned long long *)(a.table + home));
            const uint32_t home_cnt = ld_agent((const uint32_t *)(a.table + home + 8));
            // lane group g of round r fetches the payload of order omax - (r * G + g)
            int32_t pid[kMaxRounds] = {};
            uint32_t pmu[kMaxRounds] = {};
            const int home_lo = (int)(uint32_t)home, home_hi = (int)(uint32_t)(home >> 32);
            auto fetch = [&](auto round) {
                constexpr int r = decltype(round)::value;
                int at_lo = 0, at_hi = 0;
                auto take = [&](auto group) {   // (row_newbcast: lane r * G + g of the row, to the lanes of group g)
                    constexpr int g = decltype(group)::value;
                    at_lo = __builtin_amdgcn_update_dpp(at_lo, home_lo, 0x150 + r * G + g, 0xF, L::banks(g), false);
                    at_hi = __builtin_amdgcn_update_dpp(at_hi, home_hi, 0x150 + r * G + g, 0xF, L::banks(g), false);
                };
                take(std::integral_constant<int, 0>{});
                take(std::integral_constant<int, 1>{});
                if constexpr (G == 4) {
                    take(std::integral_constant<int, 2>{});
                    take(std::integral_constant<int, 3>{});
                }
                const char *at = a.table + (((unsigned long long)(uint32_t)at_hi << 32) | (uint32_t)at_lo) + payload;
                pid[r] = ld_agent((const int32_t *)at);
                pmu[r] = ld_agent((const uint32_t *)(at + 4 * K));
            };
            fetch(std::integral_constant<int, 0>{});
            if (rounds > 1) fetch(std::integral_constant<int, 1>{});
            if constexpr (kMaxRounds > 2) {
                if (rounds > 2) fetch(std::integral_constant<int, 2>{});
                if (rounds > 3) fetch(std::integral_constant<int, 3>{});
            }
            asm volatile("" :: "v"(home_fp), "v"(home_cnt));   // (all have arrived here, whichever are used below)
#pragma unroll
            for (int r = 0; r < kMaxRounds; ++r) asm volatile("" :: "v"(pid[r]), "v"(pmu[r]));
            bool hit = looked_up && home_fp == fp && home_cnt > 0;
            unsigned long long slot = fp & a.mask;
            const bool displaced = looked_up && lane < 16 && home_fp != fp && home_fp != 0ull;
            if (__builtin_expect(__ballot(displaced) != 0ull, 0)) {
                if (displaced) {
                    for (int i = 1; i < a.max_probe; ++i) {  // displaced key: keep probing
                        const uint64_t s = (fp + (uint64_t)i) & a.mask;
                        const SlotHeader *h = slot_header(a.table, s, a.slot_bytes);
                        const unsigned long long cur = ld_agent(&h->fp);
                        if (cur == fp) { if (ld_agent(&h->count) > 0) { hit = true; slot = s; } break; }
                        if (cur == 0ull) break;
                    }
                }
            }
            const unsigned long long hits = __ballot(hit) & 0xFFFFull;   // (the rows hold the same)
            if (!hits) {
                my_hits += lane == 0 ? 1u : 0u;
                continue;
            }
            const int win = __ffsll((long long)hits) - 1;  // lowest lane = longest order
            my_hits += lane == a.omax - win ? 1u : 0u;
            int32_t id;
            float mu;
            if (__builtin_expect((__ballot(slot == (fp & a.mask)) >> win) & 1ull, 1)) {
                // the payload fetched with the home slot is the entry's: from the winning order's group to all groups
                const int r_win = win / G;
                int32_t t_id = pid[0];
                uint32_t t_mu = pmu[0];
#pragma unroll
                for (int r = 1; r < kMaxRounds; ++r) if (r == r_win) { t_id = pid[r]; t_mu = pmu[r]; }
                const bool from = grp == win % G;
                id = L::any_of_groups(from ? t_id : 0);
                mu = u2f((uint32_t)L::any_of_groups(from ? (int)t_mu : 0));
            } else {
                const char *at = a.table + readlane_u64(slot, win) * (unsigned long long)(unsigned)a.slot_bytes + payload;
                id = ld_agent((const int32_t *)at);
                mu = u2f(ld_agent((const uint32_t *)(at + 4 * K)));
                asm volatile("" : "+v"(id), "+v"(mu));
            }
            // (stored here, so that the acknowledgements have the ranking to arrive before the next level's loads are waited for)
            if (has_cand && grp == 0) { qid_out[u * K + cand] = id; qmu_out[u * K + cand] = mu; }
            const bool usable = has_cand && mu > 0.0f;
            const int ncand = __popcll(__ballot(usable && grp == 0));
            int rank = kMaxK;  // child rank of this lane's candidate (>= nch: not drafted)
            if (a.mode == 1) {
                // ---- sequential sampling without replacement (the ablation's plain stochastic
                // drafting): draw j takes the first remaining candidate, in stored order, whose
                // running sum of mu exceeds U_j * (sum of the remaining mu).  Lane i holds candidate i here.
                const float u_l = lane < nch ? uniform(a.seed, (uint32_t)b, a.step, (uint32_t)u, (uint32_t)lane, kStreamDraft) : 0.0f;
                const float mu_l = __shfl(mu, L::lane_of(lane & (L::kSlots - 1)));
                bool left = lane < K && mu_l > 0.0f;
                const int draws = nch < ncand ? nch : ncand;
                for (int j = 0; j < draws; ++j) {
                    const float mleft = left ? mu_l : 0.0f;
                    const float z = wave_tree_sum(mleft);
                    const float t = u2f((uint32_t)__builtin_amdgcn_readlane((int)f2u(u_l), j)) * z;
                    float acc = 0.0f;
                    int pick = -1, last = -1;
                    const unsigned long long left_mask = __ballot(left);
                    for (int i = 0; i < K; ++i) {
                        const float mi = u2f((uint32_t)__builtin_amdgcn_readlane((int)f2u(mleft), i));
                        if (!((left_mask >> i) & 1ull)) continue;  // uniform
                        last = i;
                        acc = acc + mi;
                        if (pick < 0 && t < acc) pick = i;
                    }
                    if (pick < 0) pick = last;
                    if (lane == pick) { rank = j; left = false; }
                }
                rank = __shfl(rank, cand);
            } else {
                // ---- Gumbel-Top-K (paper Sec. 4.2): score = ln mu - ln(-ln U), the largest scores in
                // order; deterministic drafting (Sec. 3.1): the largest means themselves
                unsigned long long key;
                if (a.mode == 2) key = rank_key(mu, (uint32_t)id);
                else {
                    // ln mu in the upper half of a row while the lower one takes ln U
                    const float U = uniform_by_halves(a.seed, (uint32_t)b, a.step, (uint32_t)u, (uint32_t)id, kStreamDraft, upper);
                    const float lnx = exact_log(upper ? (mu > 0.0f ? mu : 1.0f) : U);
                    const float ln_mu = u2f(other_half(f2u(lnx)));
                    const float g = exact_log(upper ? 1.0f : -lnx);
                    key = rank_key(ln_mu - g, (uint32_t)id);   // (in the lower half)
                }
                // each group compares the candidate with its share of the scores; an empty place holds key 0, which is
                // above no key
                if (grp == 0) keys[cand] = usable ? key : 0ull;
                __builtin_amdgcn_wave_barrier();
                const unsigned long long mine = keys[cand];
                constexpr int share = L::kSlots / G;   // 4 or 16
                const unsigned long long *ks = keys + grp * share;
                rank = 0;
#pragma unroll
                for (int q = 0; q < share; ++q) rank += ks[q] > mine ? 1 : 0;
                rank = L::sum_of_groups(rank);
                __builtin_amdgcn_wave_barrier();
            }
            if (usable && grp == 0 && rank < nch) {
                const int child = first + rank;
                tok[child] = id;
                *(int4 *)&recent[child][0] = make_int4(id, r_lo.x, r_lo.y, r_lo.z);
                *(int4 *)&recent[child][4] = make_int4(r_lo.w, r_hi.x, r_hi.y, r_hi.z);
                sm.live[d + 1] = 1;
            }
            if (lane == 0) sm.has[u] = ncand < nch ? ncand : nch;
        }
        __syncthreads();
    }
    // (counted per workgroup: hundreds of lookups of a launch would add to the same line one after the other)
    if (my_hits) atomicAdd(&sm.n_hit[lane], my_hits);
    __syncthreads();
}

// The draft of trajectory b by the NT threads of the calling workgroup (all of them call this).
//
// Bound by the instructions of ONE wave per tree level, one level after the other, and one round trip to the table per
// level.  So a node's dependent chain is kept short: its values never leave the rows of 16 lanes that hold them
// (CandLayout: exchanges by data-parallel primitives, not through shared memory), the two multiplications of a Philox
// round run side by side (53 cycles a round instead of 107), ln mu is taken beside ln U, header and payload of every
// order are requested without a branch between them (which had made two round trips of them), a node's outputs are stored
// before its ranking, and nothing in the level loop waits for a store.  With clock readings between the parts a level of a
// warm 64-node tree went from about 4 700 to 2 900 cycles (and with the constants formed before the first level is waited for:
// draft and packing of 32 such trees 18.3 -> 17.3 us); draft of 32 such trees 19.7 -> 15.0 us, steps of 32 x 64 rows
// x 152 064 154.3 -> 149.9 us (separate launches) and 116.9 -> 114.3 us (one launch), of 8 x 32 49.3 -> 47.1 us.
// (Table entries are read past the XCD's own caches in every launch form: in the one-launch step other workgroups
// have just written them, and as ordinary loads they made no repeated call faster and the first call after other work
// 6 us slower.)
// draft_prepare brings the tree and the context (after appending the committed tokens) into shared memory: it needs none
// of the table, so a caller that waits for other workgroups' updates calls it meanwhile.  Returns what draft_run takes.
template <int NT>
__device__ __forceinline__ int draft_prepare(const DraftArgs &a, int b, const DraftShared &sm)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int32_t *tok = sm.tok;
    int32_t(*recent)[kMaxOrder] = sm.recent;
    const int N = a.tree.N;
    // ---- everything that is read from memory is requested at once.  Lane d of every wave holds the first node of level d
    // (D + 2 <= 33 entries).  Context tail of this trajectory, after appending the tokens committed by this step: lane
    // i < 8 of the second wave holds the stored tail, lane 8 + j the j-th committed token (W <= 32); the new tail is the
    // last eight of the first 8 + n lanes.
    const bool appends = a.append_tok != nullptr;
    int32_t ctx = 0, n = 0;
    long long len = 0;
    if (wave == 1) {
        if (lane < kMaxOrder) ctx = a.ctx_tail[(size_t)b * kMaxOrder + lane];
        else if (appends && lane < kMaxOrder + a.W) ctx = a.append_tok[(size_t)b * a.W + (lane - kMaxOrder)];
        if (appends) n = a.append_len[b];
        len = a.ctx_len[b];
    }
    int level_reg = lane < a.tree.D + 2 ? a.tree.level_start[lane] : 0;
    for (int u = tid; u < N; u += NT) {
        sm.info[u] = (a.tree.first_child[u] << 8) | a.tree.nchild[u];  // (a leaf's first child, -1, is not looked at)
        if (u > 0) tok[u] = -1;  // the root's token is set with the context below
        sm.has[u] = 0;
    }
    if (tid <= kMaxOrder) sm.n_hit[tid] = 0u;
    if (tid >= 1 && tid < kMaxDepth + 2) sm.live[tid] = 0;
    if (wave == 1) {
        n = clamp_len(n, a.W);
        len += n;
        const int32_t t = __shfl(ctx, (lane & (kMaxOrder - 1)) + n);
        if (lane < kMaxOrder) {
            recent[0][kMaxOrder - 1 - lane] = t;
            if (appends) a.ctx_tail[(size_t)b * kMaxOrder + lane] = t;
            if (lane == kMaxOrder - 1) { tok[0] = len > 0 ? t : -1; sm.live[0] = len > 0 && t >= 0; }
        }
        if (lane == 0) {
            if (appends) a.ctx_len[b] = len;
            *sm.clen = len;
        }
    }
    asm volatile("" : "+v"(level_reg));   // (here: waited for inside the loop, it would wait for the stores of every level)
    return level_reg;
}

// (`sm` as draft_prepare, or whatever else has filled it, leaves it; join() ends with a barrier)
template <int NT, typename Join>
__device__ __forceinline__ void draft_run(const DraftArgs &a, int b, const DraftShared &sm, int level_reg, const Join &join)
{
    const int tid = threadIdx.x, N = a.tree.N;
    const int32_t *tok = sm.tok;
    const int32_t(*recent)[kMaxOrder] = sm.recent;
    if (a.K <= 16) draft_levels<NT, 4>(a, b, sm, level_reg, join);
    else draft_levels<NT, 2>(a, b, sm, level_reg, join);
    if (tid <= a.omax) {
        const unsigned c = sm.n_hit[tid];
        if (c) atomicAdd(&a.stats[tid == 0 ? (int)kStatMisses : (int)kStatHits + tid], (unsigned long long)c);
    }
    for (int u = tid; u < N; u += NT) {
        a.draft_tok[(size_t)b * N + u] = tok[u];
        a.draft_has[(size_t)b * N + u] = sm.has[u];
        if (a.out_tok) a.out_tok[(size_t)b * N + u] = tok[u];
    }
    if (a.recent_out)
        for (int i = tid; i < N * kMaxOrder; i += NT)
            if (tok[i / kMaxOrder] >= 0) a.recent_out[(size_t)b * N * kMaxOrder + i] = recent[i / kMaxOrder][i % kMaxOrder];
}

template <int NT>
__device__ __forceinline__ void draft_trajectory(const DraftArgs &a, int b, const DraftShared &sm)
{
    const int level_reg = draft_prepare<NT>(a, b, sm);
    draft_run<NT>(a, b, sm, level_reg, [] { __syncthreads(); });
}

__global__ __launch_bounds__(kDraftThreads) void draft_kernel(DraftArgs a)
{
    __shared__ __align__(16) char smem[draft_shared_bytes(kMaxNodes, kDraftThreads / 64)];
    draft_trajectory<kDraftThreads>(a, (int)blockIdx.x, draft_shared_carve(smem, a.tree.N, kDraftThreads / 64));
}

}  // namespace stand
