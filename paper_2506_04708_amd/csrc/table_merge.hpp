// table_merge.hpp -- the n-gram table's update: slot claims, merge_apply_kernel, context append (paper Sec. 4.1).
#pragma once
#include "wave_ops.hpp"

namespace stand {

// ---------------------------------------------------------------------------------------------
// Table merge (paper Sec. 4.1): claim a slot per record, then apply the records of each slot in
// record order (b, then position, then order ascending).
// ---------------------------------------------------------------------------------------------
struct MergeArgs {
    char *table;
    uint64_t mask;
    int slot_bytes, K, max_probe;
    int B, W, omin, omax;
    const int32_t *ctx_tail;          // [B][kMaxOrder], newest token last
    const long long *ctx_len;         // [B]
    const int32_t *commit_tok;        // [B][W]
    const int32_t *commit_row;        // [B][W] or NULL (then every j < len is valid)
    const int32_t *commit_len;        // [B]
    int N;
    int R;                            // record slots per trajectory: W, or N in all-nodes mode
    bool all_nodes;                   // record (b, j, n) observes drafted node j under its path's context
    bool replace;                     // an existing entry becomes the newest observation (no running mean)
    const int32_t *draft_tok;         // [B][N]
    const int32_t *depth;             // [N]
    const int32_t *recent;            // [B][N][kMaxOrder] recent[.][i]: token i positions before the end of node's sequence
    long long *rec_slot;              // [B*R*NO]
    const int32_t *obs_idx;
    const float *obs_p;
    unsigned long long *stats;
};

// transient use of the slot header between claiming and applying the records of one merge
constexpr uint32_t kTagShift = 8, kTagMax = 0x7FFFFFu, kMultiBit = 0x80000000u;

__device__ __forceinline__ int clamp_len(int len, int W) { return len < 0 ? 0 : (len > W ? W : len); }

enum ClaimOutcome { kClaimNone = 0, kClaimInsert, kClaimMerge, kClaimDrop };

// claims a table slot for merge record rec, whose key of order n has fingerprint fp; run by one thread
__device__ __forceinline__ int claim_slot(const MergeArgs &a, int rec, int n, unsigned long long fp, long long &slot_out)
{
    for (int i = 0; i < a.max_probe; ++i) {
        const uint64_t slot = (fp + (uint64_t)i) & a.mask;
        SlotHeader *h = slot_header(a.table, slot, a.slot_bytes);
        const unsigned long long old = atomicCAS(&h->fp, 0ull, fp);
        if (old == 0ull || old == fp) {
            // Until the records are applied the order word also carries the smallest record
            // number that claimed the slot (stored inverted, so that atomicMax keeps it), and
            // the top bit of the count word says that more than one record did.
            const uint32_t tag = ((kTagMax - (uint32_t)rec) << kTagShift) | (uint32_t)n;
            const uint32_t before = atomicMax(&h->order, tag);
            if (before >> kTagShift) atomicOr(&h->count, kMultiBit);
            slot_out = (long long)slot;
            return old == 0ull ? kClaimInsert : kClaimMerge;
        }
    }
    return kClaimDrop;
}

// claims the table slot of merge record rec = (b, position j, order n); run by one thread
__device__ __forceinline__ int merge_claim_record(const MergeArgs &a, int rec)
{
    const int NO = a.omax - a.omin + 1;
    if (rec >= a.B * a.R * NO) return kClaimNone;
    int outcome = kClaimNone;
    const int n = a.omin + rec % NO;
    const int j = (rec / NO) % a.R;
    const int b = rec / (NO * a.R);
    long long slot_out = -1;
    const long long base_len = a.ctx_len[b];
    bool valid;
    if (a.all_nodes) {
        valid = a.draft_tok[(size_t)b * a.N + j] >= 0 && base_len + a.depth[j] >= n;
    } else {
        const int len = clamp_len(a.commit_len[b], a.W);
        valid = j < len && base_len + j >= n;
        if (valid && a.commit_row) {
            const int r = a.commit_row[(size_t)b * a.W + j];
            valid = r >= 0 && r < a.N;
        }
    }
    if (valid) {
        int32_t key[kMaxOrder];
        for (int i = 0; i < n; ++i) {
            if (a.all_nodes) {
                // the last n tokens of context ++ path to node j, as the draft kernel left them
                key[i] = a.recent[((size_t)b * a.N + j) * kMaxOrder + (n - 1 - i)];
                continue;
            }
            const int back = n - i;  // this token is `back` positions before token j
            // positions before j: commit tokens j-1, j-2, ... then the context tail
            key[i] = (back <= j) ? a.commit_tok[(size_t)b * a.W + (j - back)]
                                 : a.ctx_tail[(size_t)b * kMaxOrder + (kMaxOrder - (back - j))];
        }
        outcome = claim_slot(a, rec, n, fingerprint(n, key), slot_out);
    }
    st_agent(&a.rec_slot[rec], slot_out);
    return outcome;
}

// Adds the outcomes of a wave's claims to the statistics.  (One device-wide addition per record made the claims of an
// update of 672 rows, 2688 records on one address, take 40 us.)
__device__ __forceinline__ void count_claims(const MergeArgs &a, int outcome, int lane)
{
    const int ins = __popcll(__ballot(outcome == kClaimInsert)), mrg = __popcll(__ballot(outcome == kClaimMerge));
    const int drp = __popcll(__ballot(outcome == kClaimDrop));
    if (lane == 0) {
        if (ins) atomicAdd(&a.stats[kStatInserts], (unsigned long long)ins);
        if (mrg) atomicAdd(&a.stats[kStatMerges], (unsigned long long)mrg);
        if (drp) atomicAdd(&a.stats[kStatDrops], (unsigned long long)drp);
    }
}


// One wave per record, kMergeWaves records per workgroup.  The lowest record that claimed a slot (its leader, named in
// the slot header by the claim) applies all records of that slot in record order; the other records' waves leave at
// once.  A slot claimed by one record only needs no search for followers.  The waves of a workgroup do not interact.
// A record that exists costs some 700 instructions, and those that exist are the first positions of each trajectory:
// consecutive records therefore go to different workgroups, small ones (sixteen consecutive records per workgroup left
// most compute units idle: step 32 x 64 rows with deep paths 156.5 -> 155.3 us, update of 32 x 21 rows 88 -> 83).
constexpr int kMergeWaves = 4;
constexpr int kFollowGroups = 16;

// The entry stored in a slot, lane i < K its i-th place.  Only the slot's leader writes it, so it may be requested as soon as
// the slot is known.
struct StoredEntry { int32_t id; float mu; };
__device__ __forceinline__ StoredEntry request_entry(const MergeArgs &a, long long slot, int lane)
{
    StoredEntry e{-1, 0.0f};
    if (lane < a.K) {
        e.id = ld_agent(&slot_ids(a.table, (uint64_t)slot, a.slot_bytes)[lane]);
        e.mu = ld_agent(&slot_mu(a.table, (uint64_t)slot, a.slot_bytes, a.K)[lane]);
    }
    return e;
}

// Takes back what the claim of a record that will not be applied left in its slot's header (one lane): no later merge or
// lookup sees it.
__device__ __forceinline__ void release_claimed(const MergeArgs &a, long long slot)
{
    SlotHeader *h = slot_header(a.table, (uint64_t)slot, a.slot_bytes);
    atomicAnd(&h->order, (1u << kTagShift) - 1u);
    atomicAnd(&h->count, ~kMultiBit);
}

// A record that has claimed a slot, as a wave asks for what it needs: the slot (header and stored entry, once every claim is made)
// and its observation (lanes 32 .. 32 + K - 1).
struct ClaimedRecord {
    int rec;
    long long slot;
    StoredEntry e;
    uint32_t order_word, count;
    int32_t o_id;
    float o_p;
    __device__ __forceinline__ void request_slot(const MergeArgs &a, int record, long long claimed, int lane)
    {
        rec = record; slot = claimed;
        const SlotHeader *h = slot_header(a.table, (uint64_t)slot, a.slot_bytes);
        order_word = ld_agent(&h->order);
        count = ld_agent(&h->count);
        e = request_entry(a, slot, lane);
    }
    __device__ __forceinline__ void request_observation(const MergeArgs &a, int lane)
    {
        o_id = -1; o_p = 0.0f;
        if (lane >= 32 && lane < 32 + a.K) {
            const size_t at = (size_t)(rec / (a.omax - a.omin + 1)) * a.K + (lane - 32);
            o_id = ld_agent(&a.obs_idx[at]);
            o_p = ld_agent(&a.obs_p[at]);
        }
    }
};

// Applies a record by one wave (all 64 lanes call this; scratch: 2 * kMaxK words of shared memory, 16-byte aligned, owned by
// the wave).  Does nothing unless the record leads its slot.  others_there(): whether the observations of other
// trajectories' records are there (a caller may wait for them; without them the claim is released).
// Folding one observation into an entry was 2 600 (K = 10) to 6 700 cycles (K = 32) of readlanes; with ids and keys read
// from shared memory, four and two per access, K compares and 2 K 64-bit compares remain.
struct AlwaysThere { __device__ __forceinline__ bool operator()() const { return true; } };
template <typename OthersThere = AlwaysThere>
__device__ __forceinline__ void apply_claimed(const MergeArgs &a, const ClaimedRecord &r, int lane, unsigned long long *scratch,
                                              const OthersThere &others_there = OthersThere())
{
    const int rec = r.rec;
    const long long slot = r.slot;
    const int NO = a.omax - a.omin + 1;
    const int nrec = a.B * a.R * NO;
    const int K = a.K;
    SlotHeader *h = slot_header(a.table, (uint64_t)slot, a.slot_bytes);
    int32_t *ids = slot_ids(a.table, (uint64_t)slot, a.slot_bytes);
    float *mus = slot_mu(a.table, (uint64_t)slot, a.slot_bytes, K);
    const uint32_t order_word = r.order_word;
    uint32_t count = r.count;
    int32_t e_id = r.e.id;
    float e_mu = r.e.mu;
    // lanes 0..K-1: stored entry; lanes 32..32+K-1: observation
    const int32_t o_id = r.o_id;
    const float o_p = r.o_p;
    if (kTagMax - (order_word >> kTagShift) != (uint32_t)rec) return;  // another record leads this slot
    const bool multi = (count & kMultiBit) != 0u;
    count &= ~kMultiBit;
    if (multi && !others_there()) {
        if (lane == 0) release_claimed(a, slot);
        return;
    }
    if (count == 0) { e_id = -1; e_mu = 0.0f; }

    auto apply = [&](int32_t o_id, float o_p) {
        if (count == 0 || a.replace) {
            // first sight, or a table that keeps only the newest observation: the entry is the observation
            const int32_t id2 = __shfl(o_id, 32 + (lane & 31));
            const float p2 = __shfl(o_p, 32 + (lane & 31));
            if (lane < K) { e_id = id2; e_mu = p2; }
        } else {
            const float cf = (float)count;
            const float denom = cf + 1.0f;
            const int32_t id = lane < 32 ? e_id : o_id;
            bool act = (lane & 31) < K;
            // where the other list (stored ids: lanes 0.., observed ids: lanes 32..) holds this id; ids are distinct
            int32_t *ids_l = (int32_t *)scratch;
            ids_l[lane] = act ? id : (lane < 32 ? -1 : -2);
            __builtin_amdgcn_wave_barrier();
            const int4 *others = (const int4 *)(ids_l + (lane < 32 ? 32 : 0));
            int at = -1;
            for (int q = 0; q < K; q += 4) {
                const int4 v = others[q >> 2];
                if (v.x == id) at = q;
                if (v.y == id) at = q + 1;
                if (v.z == id) at = q + 2;
                if (v.w == id) at = q + 3;
            }
            const float o_at = __shfl(o_p, 32 + (at & 31));
            float val;
            if (lane < 32) { float t = cf * e_mu; t = t + (at >= 0 ? o_at : 0.0f); val = t / denom; }
            else { float t = cf * 0.0f; t = t + o_p; val = t / denom; act = act && at < 0; }
            const unsigned long long key = act ? rank_key(val, (uint32_t)id) : 0ull;
            __builtin_amdgcn_wave_barrier();
            scratch[lane] = key;   // (lanes without an entry hold key 0, which is above no key)
            __builtin_amdgcn_wave_barrier();
            int rank = 0;
            for (int q = 0; q < K; q += 2) {
                const ulonglong2 k0 = *(const ulonglong2 *)&scratch[q], k1 = *(const ulonglong2 *)&scratch[32 + q];
                rank += (k0.x > key ? 1 : 0) + (k0.y > key ? 1 : 0) + (k1.x > key ? 1 : 0) + (k1.y > key ? 1 : 0);
            }
            __builtin_amdgcn_wave_barrier();
            if (act && rank < K) scratch[rank] = ((unsigned long long)f2u(val) << 32) | (uint32_t)id;
            __builtin_amdgcn_wave_barrier();  // the wave's own part of shared memory: no other wave is involved
            if (lane < K) { e_id = (int32_t)(uint32_t)scratch[lane]; e_mu = u2f((uint32_t)(scratch[lane] >> 32)); }
            __builtin_amdgcn_wave_barrier();
        }
        count++;
    };

    apply(o_id, o_p);
    if (multi) {
        // the later records of this slot, in record order (kFollowGroups groups of 64 record slots are read per
        // round trip: a step of 128 trajectories has thousands of record slots)
        for (int base = rec + 1; base < nrec; base += 64 * kFollowGroups) {
            unsigned found = 0u;   // bit q: the lane's record slot of group q is such a record
#pragma unroll
            for (int q = 0; q < kFollowGroups; ++q) {
                const int r = base + 64 * q + lane;
                found |= (r < nrec ? ld_agent(&a.rec_slot[r]) : -1ll) == slot ? 1u << q : 0u;
            }
            if (!__ballot(found != 0u)) continue;
#pragma unroll 1
            for (int q = 0; q < kFollowGroups; ++q) {
                unsigned long long hits = __ballot((found >> q) & 1u);
                while (hits) {
                    const int bit = __ffsll((long long)hits) - 1;
                    hits &= hits - 1;
                    const int jb = (base + 64 * q + bit) / NO;  // = b * R + j
                    int32_t f_id = -1;
                    float f_p = 0.0f;
                    if (lane >= 32 && lane < 32 + K) { f_id = ld_agent(&a.obs_idx[(size_t)jb * K + (lane - 32)]); f_p = ld_agent(&a.obs_p[(size_t)jb * K + (lane - 32)]); }
                    apply(f_id, f_p);
                }
            }
        }
    }
    if (lane < K) { st_agent(&ids[lane], e_id); st_agent(&mus[lane], e_mu); }
    if (lane == 0) { st_agent(&h->count, count); st_agent(&h->order, order_word & ((1u << kTagShift) - 1u)); }
}

// apply_claimed for a record whose slot is still to be looked up; does nothing unless it exists.
__device__ __forceinline__ void apply_record(const MergeArgs &a, int rec, int lane, unsigned long long *scratch)
{
    const long long slot = ld_agent(&a.rec_slot[rec]);
    if (slot < 0) return;
    ClaimedRecord r;
    r.request_slot(a, rec, slot, lane);
    r.request_observation(a, lane);
    apply_claimed(a, r, lane, scratch);
}

// Appends the committed tokens of trajectory b to its context tail (one thread).
__device__ __forceinline__ void append_context(const MergeArgs &a, int b, int32_t *ctx_tail, long long *ctx_len)
{
    const int len = clamp_len(a.commit_len[b], a.W);
    int32_t t[kMaxOrder];
#pragma unroll
    for (int i = 0; i < kMaxOrder; ++i) {
        // the last kMaxOrder tokens of tail ++ commit
        const int at = i + len;
        t[i] = at < kMaxOrder ? ctx_tail[(size_t)b * kMaxOrder + at] : a.commit_tok[(size_t)b * a.W + (at - kMaxOrder)];
    }
#pragma unroll
    for (int i = 0; i < kMaxOrder; ++i) ctx_tail[(size_t)b * kMaxOrder + i] = t[i];
    ctx_len[b] += len;
}

// Blocks [0, apply_blocks) apply the records; with ctx_tail set, the blocks after them append the committed tokens to
// the contexts (stand_update; the claims, which read the contexts as they were, are in an earlier launch).
__global__ __launch_bounds__(64 * kMergeWaves) void merge_apply_kernel(MergeArgs a, int apply_blocks, int32_t *ctx_tail, long long *ctx_len)
{
    __shared__ __align__(16) unsigned long long scratch[kMergeWaves][2 * kMaxK];
    if ((int)blockIdx.x >= apply_blocks) {
        const int b = ((int)blockIdx.x - apply_blocks) * 64 * kMergeWaves + (int)threadIdx.x;
        if (b < a.B) append_context(a, b, ctx_tail, ctx_len);
        return;
    }
    const int NO = a.omax - a.omin + 1;
    const int nrec = a.B * a.R * NO;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int rec = wave * apply_blocks + (int)blockIdx.x;
    if (rec >= nrec) return;
    apply_record(a, rec, lane, scratch[wave]);
}

}  // namespace stand
