// path_tail.hpp -- path_tail_kernel: what follows the exact sums of a step of ONE trajectory, in one workgroup
// (paper Sec. 3.2, 4.1, 4.2).
#pragma once
#include "draft.hpp"
#include "path_pass.hpp"

namespace stand {

// With one trajectory nothing that follows the exact sums needs another workgroup: the rows of the path are finished
// and the records' slots claimed, the records applied and the next tree drafted by the waves of one workgroup, with
// workgroup barriers where a larger batch has kernel boundaries.  Bound by the chain of dependent instructions and
// round trips, which the two launches and their first loads only lengthened: steps of 1 x 16 rows 30.1 -> 28.3 us, of
// 1 x 32 rows 33.3 -> 32.0 us when it was taken in (today 28.6 .. 29.6 and 31 .. 33, from box to box).
constexpr int kTailThreads = 1024;

struct PathTailArgs {
    PathArgs path;       // verification, accepted-path update, B = 1
    MergeArgs mg;
    DraftArgs draft;
};

template <int DT>
__global__ __launch_bounds__(kTailThreads) void path_tail_kernel(PathTailArgs A)
{
    static_assert(kTailThreads == kFinishThreads && kTailThreads == kDraftThreads, "one workgroup runs all parts");
    __shared__ FinishShared fin;
    __shared__ __align__(16) unsigned long long scratch[kTailThreads / 64][2 * kMaxK];
    __shared__ __align__(16) char smem[draft_shared_bytes(kMaxNodes, kTailThreads / 64)];
    const PathArgs &a = A.path;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kWaves = kTailThreads / 64, kClaimWaves = kMaxOrder * (kMaxDepth + 1) / 64;
    const int NO = A.mg.omax - A.mg.omin + 1;
    StopRow st;
    st.request(a, 0, lane, wave == 0);
    // the other waves: first the claims (the last kClaimWaves of them, one record per thread), then the rows above
    // the stop row; the first wave is at the stop row's replay meanwhile
    if (wave >= kWaves - kClaimWaves) {
        const int rec = tid - 64 * (kWaves - kClaimWaves);
        count_claims(A.mg, rec < A.mg.R * NO ? merge_claim_record(A.mg, rec) : (int)kClaimNone, lane);
    } else if (wave > 0) {
        for (int j = wave - 1; j + 1 < st.len; j += kWaves - kClaimWaves - 1) {
            const unsigned long long part = lane < a.nseg ? ld_agent(&a.seg_part[(size_t)j * kSegMax + lane]) : 0ull;
            const int node = a.out_node[j];
            finish_row<DT, kTailThreads>(a, fin, 0, j, node, false, a.src_m[node], 0, -1, 0, -1, 0.0f, 0.0f, -1, part, lane, 0);
        }
    }
    finish_row<DT, kTailThreads>(a, fin, 0, st.j, st.node, true, st.m, st.nch, st.fc, st.len, st.my_id, st.my_mu, st.my_l, st.ch,
                                 st.part, tid, wave);
    // claims and observations are complete before the first record is applied
    publish_fence();
    __syncthreads();
    consume_fence();
    for (int i = wave; i < st.len * NO; i += kWaves) apply_record(A.mg, i, lane, scratch[wave]);
    // every record is applied before the first lookup
    publish_fence();
    __syncthreads();
    consume_fence();
    draft_trajectory<kTailThreads>(A.draft, 0, draft_shared_carve(smem, A.draft.tree.N, kTailThreads / 64));
}

}  // namespace stand
