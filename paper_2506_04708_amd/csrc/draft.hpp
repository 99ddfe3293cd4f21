// draft.hpp -- draft_kernel: multi-level lookup and Gumbel-Top-K along the static tree (paper Sec. 4.2).
#pragma once
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

__device__ __forceinline__ unsigned long long fingerprint_multiplier_of_lane(int lane)
{
    unsigned long long m = 0ull;
#pragma unroll
    for (int i = 0; i < kMaxOrder; ++i) m = lane == i ? fingerprint_multiplier(i) : m;
    return m;
}

// The draft of trajectory b by the NT threads of the calling workgroup (all of them call this).
//
// Bound by the instructions of ONE wave per tree level, one level after the other: with clock readings between the
// parts, a level of a warm 64-node tree took 7 700 cycles, of which a wave waited 300 for memory; the rest was the
// fingerprint (570), one address computation per order and payload half (1 300), the selection of the winning
// order's payload (750), Philox and three logarithms (1 650), sixteen readlane comparisons (570) and the copies of
// the recent tokens (680).  So the work of a node is spread over the lanes a K-entry payload leaves idle: each order
// is one lane up to its slot's address; payloads of 64 / KP orders arrive with one pair of loads (KP = K rounded up to
// 8, 16 or 32 lanes); ln mu is taken by the upper 32 lanes while the lower ones take ln U; the ranking compares in
// 64 / KP groups of lanes against scores in shared memory.  Draft and packing of 32 such trees, back to back:
// 31.3 -> 21.3 us; the one-launch step of 32 x 64 rows, which ends with its draft: 126 -> 117.6 us.
// (Table entries are read past the XCD's own caches in every launch form: in the one-launch step other workgroups
// have just written them, and as ordinary loads they made no repeated call faster and the first call after other work
// 6 us slower.)
template <int NT>
__device__ __forceinline__ void draft_trajectory(const DraftArgs &a, int b, const DraftShared &sm)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int32_t *tok = sm.tok;
    int32_t(*recent)[kMaxOrder] = sm.recent;
    unsigned long long *keys = sm.keys[wave];
    const int N = a.tree.N, K = a.K;
    // lane d of every wave holds the first node of level d (D + 2 <= 33 entries)
    const int level_reg = lane < a.tree.D + 2 ? a.tree.level_start[lane] : 0;
    for (int u = tid; u < N; u += NT) {
        sm.info[u] = (a.tree.first_child[u] << 8) | a.tree.nchild[u];  // (a leaf's first child, -1, is not looked at)
        if (u > 0) tok[u] = -1;  // the root's token is set with the context below
        sm.has[u] = 0;
    }
    if (tid <= kMaxOrder) sm.n_hit[tid] = 0u;
    if (tid >= 1 && tid < kMaxDepth + 2) sm.live[tid] = 0;
    if (wave == 1) {
        // Context tail of this trajectory, after appending the tokens committed by this step.  Lane i < 8 holds
        // the stored tail, lane 8 + j the j-th committed token (W <= 32), all requested at once: the new tail is
        // the last eight of the first 8 + n lanes.
        int32_t v = 0;
        if (lane < kMaxOrder) v = a.ctx_tail[(size_t)b * kMaxOrder + lane];
        else if (a.append_tok && lane < kMaxOrder + a.W) v = a.append_tok[(size_t)b * a.W + (lane - kMaxOrder)];
        const int n = a.append_tok ? clamp_len(a.append_len[b], a.W) : 0;
        const long long len = a.ctx_len[b] + n;
        const int32_t t = __shfl(v, (lane & (kMaxOrder - 1)) + n);
        if (lane < kMaxOrder) {
            recent[0][kMaxOrder - 1 - lane] = t;
            if (a.append_tok) a.ctx_tail[(size_t)b * kMaxOrder + lane] = t;
            if (lane == kMaxOrder - 1) { tok[0] = len > 0 ? t : -1; sm.live[0] = len > 0 && t >= 0; }
        }
        if (lane == 0) {
            if (a.append_tok) a.ctx_len[b] = len;
            *sm.clen = len;
        }
    }
    __syncthreads();
    const long long clen = (long long)readlane_u64((unsigned long long)*sm.clen, 0);
    const int NO = a.omax - a.omin + 1;
    const unsigned long long term_mul = fingerprint_multiplier_of_lane(lane);
    const int kp_shift = K <= 8 ? 3 : (K <= 16 ? 4 : 5);  // lanes per payload: 8, 16 or 32
    const int li = lane & ((1 << kp_shift) - 1), grp = lane >> kp_shift;
    const int per_round = 64 >> kp_shift, per_round_shift = 6 - kp_shift;
    const int rounds = (NO + per_round - 1) >> per_round_shift;  // <= kMaxRounds
    constexpr int kMaxRounds = kMaxOrder / 2;
    const int half = lane & 31;  // candidates are held twice: lanes 0..K-1 and 32..32+K-1
    int32_t *qid_out = a.draft_qid + (size_t)b * N * K;
    float *qmu_out = a.draft_qmu + (size_t)b * N * K;
    for (int d = 0; d < a.tree.D; ++d) {
        // values read from shared memory that are the same in every lane go to scalar registers
        const int lo = __builtin_amdgcn_readlane(level_reg, d), hi = __builtin_amdgcn_readlane(level_reg, d + 1);
        if (!__builtin_amdgcn_readfirstlane(sm.live[d])) break;  // a level without a drafted node ends the tree (the same in every wave)
        for (int u = lo + wave; u < hi; u += NT / 64) {
            const int4 r_lo = *(const int4 *)&recent[u][0], r_hi = *(const int4 *)&recent[u][4];
            const int32_t my_recent = recent[u][lane & (kMaxOrder - 1)];
            const int info = __builtin_amdgcn_readfirstlane(sm.info[u]);
            const int nch = info & 0xFF, first = info >> 8;
            if (nch == 0 || __builtin_amdgcn_readfirstlane(tok[u]) < 0) continue;
            // ---- multi-level lookup (paper Sec. 4.2): lane n - 1 takes order n.  The home slot of every
            // order is read together with its payload in one round trip; only a key that was displaced by linear
            // probing needs further probes.  Lane i < 8 forms the term of the token i positions back; the sum of
            // the first n terms of the fingerprint is then an inclusive scan over the lanes (three data-parallel
            // moves inside a row of 16 lanes), so no lane multiplies more than once.
            unsigned long long fp = 0ull;
            {
                const int n = lane + 1;
                unsigned long long acc = term_mul * ((unsigned long long)(uint32_t)my_recent + 1u);
                acc += dpp_fetch_u64<0x111, 0xF>(acc);  // row_shr:1
                acc += dpp_fetch_u64<0x112, 0xF>(acc);  // row_shr:2
                acc += dpp_fetch_u64<0x114, 0xF>(acc);  // row_shr:4
                acc += (unsigned long long)(uint32_t)n * 0x2545F4914F6CDD1DULL;
                const unsigned long long hsh = fmix64(acc);
                if (n >= a.omin && n <= a.omax && clen + d >= n) fp = hsh ? hsh : 1ull;
            }
            const char *home = fp ? a.table + (fp & a.mask) * (unsigned long long)(unsigned)a.slot_bytes : nullptr;
            unsigned long long home_fp = 0ull;
            uint32_t home_cnt = 0;
            if (fp) {
                home_fp = ld_agent(&((const SlotHeader *)home)->fp);
                home_cnt = ld_agent(&((const SlotHeader *)home)->count);
            }
            // lane group g of round r fetches the payload of order omax - (r * per_round + g)
            int32_t pid[kMaxRounds];
            float pmu[kMaxRounds];
#pragma unroll
            for (int r = 0; r < kMaxRounds; ++r) {
                pid[r] = -1; pmu[r] = 0.0f;
                if (r < rounds) {
                    const int oi = (r << per_round_shift) + grp;
                    const unsigned long long at = shfl_u64((unsigned long long)home, (a.omax - 1 - oi) & 63);
                    if (oi < NO && at && li < K) {
                        pid[r] = ld_agent((const int32_t *)(at + 16) + li);
                        pmu[r] = ld_agent((const float *)(at + 16) + K + li);
                    }
                }
            }
            long long hit_slot = -1;
            if (fp) {
                if (home_fp == fp) { if (home_cnt > 0) hit_slot = (long long)(fp & a.mask); }
                else if (home_fp != 0ull) {
                    for (int i = 1; i < a.max_probe; ++i) {  // displaced key: keep probing
                        const uint64_t slot = (fp + (uint64_t)i) & a.mask;
                        const SlotHeader *h = slot_header(a.table, slot, a.slot_bytes);
                        const unsigned long long cur = ld_agent(&h->fp);
                        if (cur == fp) { if (ld_agent(&h->count) > 0) hit_slot = (long long)slot; break; }
                        if (cur == 0ull) break;
                    }
                }
            }
            const unsigned long long hits = __ballot(hit_slot >= 0);
            if (!hits) {
                if (lane == 0) atomicAdd(&sm.n_hit[0], 1u);
                continue;
            }
            const int win = 63 - __builtin_clzll(hits);  // highest lane = longest order
            const long long slot = (long long)readlane_u64((unsigned long long)hit_slot, win);
            const unsigned long long win_fp = readlane_u64(fp, win);
            if (lane == 0) atomicAdd(&sm.n_hit[win + 1], 1u);
            int32_t id = -1;
            float mu = 0.0f;
            if ((unsigned long long)slot == (win_fp & a.mask)) {
                // the payload fetched with the home slot is the entry's
                const int oi = a.omax - 1 - win, r_win = oi >> per_round_shift;
                const int src = ((oi & (per_round - 1)) << kp_shift) + half;
                int32_t t_id = pid[0];
                float t_mu = pmu[0];
#pragma unroll
                for (int r = 1; r < kMaxRounds; ++r) if (r == r_win) { t_id = pid[r]; t_mu = pmu[r]; }
                t_id = __shfl(t_id, src & 63);
                t_mu = __shfl(t_mu, src & 63);
                if (half < K) { id = t_id; mu = t_mu; }
            } else if (half < K) {
                id = ld_agent(&slot_ids(a.table, (uint64_t)slot, a.slot_bytes)[half]);
                mu = ld_agent(&slot_mu(a.table, (uint64_t)slot, a.slot_bytes, K)[half]);
            }
            const bool cand = lane < K && mu > 0.0f;
            int rank = kMaxK;  // child rank of this lane's candidate (>= nch: not drafted)
            if (a.mode == 1) {
                // ---- sequential sampling without replacement (the ablation's plain stochastic
                // drafting): draw j takes the first remaining candidate, in stored order, whose
                // running sum of mu exceeds U_j * (sum of the remaining mu)
                const float u_l = lane < nch ? uniform(a.seed, (uint32_t)b, a.step, (uint32_t)u, (uint32_t)lane, kStreamDraft) : 0.0f;
                bool left = cand;
                const int ncand_all = __popcll(__ballot(cand));
                const int draws = nch < ncand_all ? nch : ncand_all;
                for (int j = 0; j < draws; ++j) {
                    const float mleft = left ? mu : 0.0f;
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
            } else {
                // ---- Gumbel-Top-K (paper Sec. 4.2): score = ln mu - ln(-ln U), the largest scores in
                // order; deterministic drafting (Sec. 3.1): the largest means themselves
                unsigned long long key;
                if (a.mode == 2) key = rank_key(mu, (uint32_t)id);
                else {
                    const float U = uniform(a.seed, (uint32_t)b, a.step, (uint32_t)u, (uint32_t)id, kStreamDraft);
                    const float lnx = exact_log(lane < 32 ? U : (mu > 0.0f ? mu : 1.0f));
                    const float ln_mu = __shfl_xor(lnx, 32);
                    const float g = exact_log(lane < 32 ? -lnx : 1.0f);
                    key = rank_key(ln_mu - g, (uint32_t)id);
                }
                // lane group g counts, for candidate li, the larger ones among every group's share of the scores;
                // lanes without a candidate hold key 0, which is above no key
                if (lane < kMaxK) keys[lane] = cand ? key : 0ull;
                __builtin_amdgcn_wave_barrier();
                const unsigned long long mine = keys[li];
                rank = 0;
                const int share = 1 << (2 * kp_shift - 6);  // KP * KP / 64: 1, 4 or 16 scores per group
                const unsigned long long *ks = keys + grp * share;
                if (kp_shift == 3) rank += ks[0] > mine ? 1 : 0;
                else {
                    for (int q = 0; q < share; q += 4) {
                        const unsigned long long k0 = ks[q], k1 = ks[q + 1], k2 = ks[q + 2], k3 = ks[q + 3];
                        rank += (k0 > mine ? 1 : 0) + (k1 > mine ? 1 : 0) + (k2 > mine ? 1 : 0) + (k3 > mine ? 1 : 0);
                    }
                }
                rank += __shfl_xor(rank, 32);
                if (kp_shift <= 4) rank += __shfl_xor(rank, 16);
                if (kp_shift == 3) rank += __shfl_xor(rank, 8);
                __builtin_amdgcn_wave_barrier();
            }
            if (cand && rank < nch) {
                const int child = first + rank;
                tok[child] = id;
                *(int4 *)&recent[child][0] = make_int4(id, r_lo.x, r_lo.y, r_lo.z);
                *(int4 *)&recent[child][4] = make_int4(r_lo.w, r_hi.x, r_hi.y, r_hi.z);
                sm.live[d + 1] = 1;
            }
            const int ncand = __popcll(__ballot(cand));
            if (lane == 0) sm.has[u] = ncand < nch ? ncand : nch;
            if (lane < K) { qid_out[u * K + lane] = id; qmu_out[u * K + lane] = mu; }
        }
        __syncthreads();
    }
    // (counted per workgroup: hundreds of lookups of a launch would add to the same line one after the other)
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

__global__ __launch_bounds__(kDraftThreads) void draft_kernel(DraftArgs a)
{
    __shared__ __align__(16) char smem[draft_shared_bytes(kMaxNodes, kDraftThreads / 64)];
    draft_trajectory<kDraftThreads>(a, (int)blockIdx.x, draft_shared_carve(smem, a.tree.N, kDraftThreads / 64));
}

}  // namespace stand
