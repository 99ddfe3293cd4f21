// row_parts.hpp -- row_parts_kernel: the row pass for few rows, and for short rows however many (paper Sec. 4.1, 3.2).  Every
// row is split over workgroups that hold their part in registers; a row that fits one is its only part.
#pragma once
#include "row_pass.hpp"

namespace stand {

// ---------------------------------------------------------------------------------------------
// With few rows the row pass is bound by latency: by how many compute units pull at a row, and by what a row costs
// after its last byte has arrived (lists of sixteen waves gathered and pruned one after the other, kept vectors read
// again).  Here a row is split over P workgroups of kPartThreads threads.  Each holds its part in registers, at most R
// 16-byte vectors per lane, all requested at once, so that
//   - the part's maximum is known before its first exponential (no running reference);
//   - no candidate list is kept while streaming: the K-th largest of the 64 maxima of 8-lane groups is a lower bound
//     of the part's K-th largest element, and it is tight: 64 ln(64 / (64 - K)) elements reach it on average (11 for
//     K = 10, 44 for K = 32); the vectors that hold them go to shared memory, where every thread takes an element;
//   - nothing is read twice.
// Where a launch fills the device, what bounds it after its last byte are the vector instructions of all its waves (eight to a
// SIMD: 100 more in each are 1.6 us), so what is not done per element is kept short: the arguments are read again in the later
// phases instead of spilled from the start (up to 90 scalar registers), streamed and plain loads are two kernels instead of
// two branches that meet in moves (of all this the least: 8 x 32 x 128 256 40.0 / 39.6, 1 x 32 x 152 064 25.9 / 25.7, verify of
// 12 x 48 x 32 003 fp32 31.7 / 31.4), and candidates are not taken apart in the registers that happen to hold them (200 of 800
// instructions).  Steps, with all this before / as it is, us: 8 x 32 rows x 128 256 bf16 41.4 / 39.8, 24 x 20 x 50 000 42.9 / 40.8,
// verify of 2 x 40 x 150 000 fp32, K = 32 39.0 / 37.4, update and draft of 4 x 32 x 152 064 47.8 / 44.8 (its rows without the fast
// normaliser, which an update does not use).  Vectors taken one by one as they arrive, relative to a reference that is
// raised on the way, were slower (40.3 / 40.8): the phases of a unit's four workgroups overlap as it is.
// The last workgroup of a row to finish (a counter that its last user sets back to zero, so a recorded launch can be
// replayed) merges the parts: the largest of the parts' bounds cuts the candidates again, one wave ranks them exactly
// while another runs the node's accept tests.
// Masked vocabularies (-inf, or the type's lowest value) and quantised logits make whole parts equal to their own bound.
// Where more than kPartTies lanes of a wave are at or above the bound, the part collects all that exceeds it, but of what
// equals it each wave takes only the lowest ids, as many as can be among the K best (it meets its elements in id order):
// row pass over 256 rows of 257 KB whose upper half is masked 27 us, without a mask 19; with the streaming scan for
// all such parts, which orders every tie, 154.  Only more than kPartList elements above the bound are still left to the
// scan of row_pass.hpp.
// ---------------------------------------------------------------------------------------------
constexpr int kTicketStride = 32;                    // words between two rows' counters: a cache line each
constexpr int kPartKeys = 64;                        // candidate keys a part hands over
constexpr int kPartList = kPartsMax * kPartKeys;     // candidates collected in shared memory
// Vectors collected in shared memory.  Where more hold an element at the bound, though few lanes of a wave (rows of which 6 to 24 of
// every 64 vectors lie above the others), the part is fetched again; candidates taken out of the registers / as it is, verifications,
// us: 300 rows x 32 768 bf16, K = 25, ordinary rows 17.6 / 16.8, 2 of 64 46.0 / 29.7, 5 48.1 / 34.3, 6 48.4 / 49.5, 24 56.6 / 57.3;
// 256 x 128 256, K = 32, 29.4 / 27.3, 77.8 / 49.4, 73.9 / 50.0, 74.8 / 77.1, 86.9 / 89.6
constexpr int kPartVecs = 384;
constexpr int kPartTies = 32;                        // more lanes of a wave than this at or above the bound: most elements there equal it
constexpr int kPartTied = 1 << 20;                   // added to the count of candidates by such a wave

struct PartHead { float m, s, theta; int cnt; };     // maximum, fast sum relative to it, bound, candidates of a part

struct RowPartsArgs {
    RowPassArgs r;
    int P, per;                    // parts per row, vectors per part (<= kPartThreads * R)
    unsigned *ticket;              // [rows or row slots][kTicketStride] parts that have finished; back at zero after the launch
    PartHead *head;                // [slots * P]
    unsigned long long *keys;      // [slots * P][kPartKeys]
    // update mode: the rows are those of the commits (slot (j, b)) and there are no accept tests
    bool commit, all_nodes;
    int W, R;
    const int32_t *commit_row, *commit_len;
    float *pr_m;                   // [B*R]
    int32_t *pr_top_idx;           // [B*R][K]
    float *pr_top_l;               // [B*R][K]
};

struct PartShared {
    float bins[64];                // maxima of groups of 8 lanes
    int above[64];                 // number of bins above each
    float wmax[kPartWaves], wsum[kPartWaves];
    int n_vec, n, n_row, last;     // vectors that reach the bound, candidates of the part, then of the row
    union {
        int rank[kPartList];
        struct { uint4 vec[kPartVecs]; int vec_at[kPartVecs]; };   // those vectors and their places in the row
    };
    union {
        unsigned long long list[kPartList + 8];
        RowShared<kPartWaves> scan;  // the streaming scan's own memory (ties)
    };
    unsigned long long top[kMaxK];
};

// Adds to rank[i] the number of keys among list[j0..j1) that are larger than key i (n distinct keys; one wave).
__device__ __forceinline__ void rank_against(const unsigned long long *list, int *rank, int n, int j0, int j1, int lane)
{
    for (int base = 0; base < n; base += 64) {
        const int i = base + lane;
        const unsigned long long mine = i < n ? list[i] : ~0ull;
        int c = 0;
        int jj = j0;
        for (; jj + 4 <= j1; jj += 4) {
            const unsigned long long k0 = list[jj], k1 = list[jj + 1], k2 = list[jj + 2], k3 = list[jj + 3];
            c += (k0 > mine ? 1 : 0) + (k1 > mine ? 1 : 0) + (k2 > mine ? 1 : 0) + (k3 > mine ? 1 : 0);
        }
        for (; jj < j1; ++jj) c += list[jj] > mine ? 1 : 0;
        if (c) atomicAdd(&rank[i], c);   // (c is 0 for lanes without a key)
    }
}

// More candidates than kPartCut (quantised logits, short parts): every wave keeps the K best of its eighth of the list, so
// that the ranking of all against all, which grows with the square, sees at most kPartWaves * K.  Called by all threads.
// (Update of 144 rows of 500 000 fp32 logits, 31 parts each, K = 32: 339 -> 160 us; K = 8: 118 and 120.)
constexpr int kPartCut = 256;
__device__ __forceinline__ int cut_list(unsigned long long *list, int n, int K, int lane, int wave)
{
    static_assert(kPartCut >= kPartWaves * kMaxK, "an eighth of the list holds K keys");
    constexpr int kHeld = (kPartList / kPartWaves + 63) / 64;
    const int lo = n * wave / kPartWaves, hi = n * (wave + 1) / kPartWaves;
    unsigned long long mine[kHeld];
    int rank[kHeld];
#pragma unroll
    for (int q = 0; q < kHeld; ++q) {
        const int i = lo + 64 * q + lane;
        mine[q] = i < hi ? list[i] : ~0ull;
        rank[q] = i < hi ? 0 : kMaxK;
    }
#pragma unroll 4
    for (int j = lo; j < hi; ++j) {
        const unsigned long long k = list[j];
#pragma unroll
        for (int q = 0; q < kHeld; ++q) rank[q] += k > mine[q] ? 1 : 0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kHeld; ++q)
        if (rank[q] < K) list[wave * K + rank[q]] = mine[q];
    __syncthreads();
    return kPartWaves * K;
}

template <int AUX, int R>
__device__ __forceinline__ void load_part(uint4 (&w)[R], __amdgpu_buffer_rsrc_t rsrc, int tid)
{
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const stream_u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (q * kPartThreads + tid) * 16, 0, AUX);
        w[q] = make_uint4(t.x, t.y, t.z, t.w);
    }
}

// (64 registers leave room for four workgroups per compute unit, so that their phases overlap: 256 rows of 257 KB
// take 19.7 us; with 116 registers and two workgroups 21.2)
template <int DT, int R, bool STREAMED>
__global__ __launch_bounds__(kPartThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void row_parts_kernel(RowPartsArgs a)
{
    constexpr int ES = VecTraits<DT>::ES, EPV = VecTraits<DT>::EPV;
    __shared__ __align__(16) PartShared sm;
    const RowPassArgs &r = a.r;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // grid (parts, trajectories, nodes or commit positions): all trajectories' rows of node 0 first
    const int part = blockIdx.x, b = blockIdx.y, j = blockIdx.z;
    const int V = r.V, K = r.K, P = a.P;
    const bool commit = a.commit;
    const float c = r.c;
    // (the later phases read the arguments again: kept from the start they were up to 90 spilled scalar registers, a tenth of
    // the vector instructions of a wave)
    auto late = []() -> const RowPartsArgs & { return fresh_args<RowPartsArgs>(); };
    int node = j;
    if (a.commit) {
        if (a.all_nodes) node = r.draft_tok[(size_t)b * r.N + j] >= 0 ? j : -1;
        else {
            int cl = a.commit_len[b];
            cl = cl < 0 ? 0 : (cl > a.W ? a.W : cl);
            node = j < cl ? a.commit_row[(size_t)b * a.W + j] : -1;
        }
        if (node < 0 || node >= r.N) {  // (the same for all parts of the row)
            if (part == 0) late().r.clear.row(b, j);
            return;
        }
    }
    node = __builtin_amdgcn_readfirstlane(node);
    const int row = b * r.N + node;
    const char *rowp = (const char *)r.logits + (size_t)row * (size_t)r.V * ES;
    const RowGeom g = row_geom<DT>(rowp, r.V);
    const int v0 = part * a.per < g.nvec ? part * a.per : g.nvec;
    const int v1 = v0 + a.per < g.nvec ? v0 + a.per : g.nvec;

    // ---- the whole part is requested at once (buffer loads: a lane past the part's end gets zeros)
    uint4 w[R];
    {
        const __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc((void *)(g.vp + v0), (short)0, (v1 - v0) * 16, 0x00020000);
        load_part<STREAMED ? 2 : 0>(w, rsrc, tid);
        if (part == 0) late().r.clear.row(b, j);
    }
    // elements of the row before its first and after its last aligned vector: one per lane of the first wave
    auto edge_of_lane = [&]() {
        int id = -1;
        if (wave == 0) {
            if (part == 0 && lane < g.head) id = lane;
            if (part == P - 1 && lane >= 32 && lane - 32 < g.ntail) id = g.tail0 + lane - 32;
        }
        return id;
    };
    const int edge_id = edge_of_lane();
    const float edge_val = edge_id >= 0 ? load_scalar<DT>(rowp, edge_id) : -__builtin_inff();
    // ---- maxima
    float cm[R], lm = edge_val;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        float x[EPV];
        unpack<DT>(w[q], x);
        float m1 = x[0];
#pragma unroll
        for (int e = 1; e < EPV; ++e) m1 = fmaxf(m1, x[e]);
        cm[q] = v0 + q * kPartThreads + tid < v1 ? m1 : -__builtin_inff();
        lm = fmaxf(lm, cm[q]);
    }
    float x8 = fmaxf(lm, dpp_fetch_f32<0xB1>(lm));     // quad_perm [1,0,3,2]
    x8 = fmaxf(x8, dpp_fetch_f32<0x4E>(x8));           // quad_perm [2,3,0,1]
    x8 = fmaxf(x8, dpp_fetch_f32<0x141>(x8));          // row_half_mirror: groups of 8 lanes
    const float wm = wave_max_f32(x8);

    // ---- the wave's share of the fast normaliser, relative to its maximum.  The exponent of a term is
    // fma(l, c, nb); the rounding of nb shifts every exponent by the same dlt, which is taken out at the end
    // (see wave_row_stream).
    const bool none = wm == -__builtin_inff();         // (no vector, or masked throughout: adds nothing)
    const float m_ref = none ? 0.0f : wm;
    float dlt;
    const float nb = fast_offset(m_ref, c, dlt);
    float s_t = edge_id >= 0 ? fast_exp2(__builtin_fmaf(edge_val, c, nb)) : 0.0f;
    if (!commit)   // (an update takes its rows' exact sums only)
#pragma unroll
    for (int q = 0; q < R; ++q) {
        float x[EPV];
        // (unpacked again: kept from the maxima, the elements would take eight registers per vector and half the waves)
        asm volatile("" : "+v"(w[q].x), "+v"(w[q].y), "+v"(w[q].z), "+v"(w[q].w));
        unpack<DT>(w[q], x);
        float e = 0.0f;
#pragma unroll
        for (int k = 0; k < EPV; ++k) e += fast_exp2(__builtin_fmaf(x[k], c, nb));
        s_t += v0 + q * kPartThreads + tid < v1 ? e : 0.0f;
    }
    s_t = wave_sum_f32(s_t);
    if ((lane & 7) == 0) sm.bins[wave * 8 + (lane >> 3)] = x8;
    if (lane == 0) { sm.wmax[wave] = none ? -3.402823466e38f : wm; sm.wsum[wave] = s_t * fast_exp2(dlt); }
    if (wave == 0) { sm.above[lane] = 0; if (lane == 0) { sm.n_vec = 0; sm.n = 0; sm.n_row = 0; } }
    __syncthreads();

    // ---- K-th largest of the 64 bins: every wave compares all bins with eight of them
    const float my_bin = sm.bins[lane];
    {
        const float4 o0 = *(const float4 *)&sm.bins[wave * 8], o1 = *(const float4 *)&sm.bins[wave * 8 + 4];
        const int c = (o0.x > my_bin) + (o0.y > my_bin) + (o0.z > my_bin) + (o0.w > my_bin) +
                      (o1.x > my_bin) + (o1.y > my_bin) + (o1.z > my_bin) + (o1.w > my_bin);
        atomicAdd(&sm.above[lane], c);
    }
    __syncthreads();
    const float theta = -wave_max_f32(sm.above[lane] < K ? -my_bin : -__builtin_inff());

    float pm, ps;   // the part's maximum and sum (in the waves that use them)
    if (wave < 2 || P == 1) {
        const float wm_l = lane < kPartWaves ? sm.wmax[lane] : -3.402823466e38f;
        pm = wave_max_f32(wm_l);
        ps = wave_sum_f32(lane < kPartWaves ? sm.wsum[lane] * fast_exp2((wm_l - pm) * c) : 0.0f);
    }

    // ---- the vectors that reach the bound go to shared memory, then every thread takes an element of them
    {
        unsigned long long reach[R], any = 0ull;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            reach[q] = __ballot(v0 + q * kPartThreads + tid < v1 && cm[q] >= theta);
            any |= reach[q];
        }
        if (__popcll(any) > kPartTies) {
            if (lane == 0) atomicAdd(&sm.n_vec, kPartTied);
        } else if (any) {
#pragma unroll
            for (int q = 0; q < R; ++q) {
                if (!reach[q]) continue;
                int base = 0;
                if (lane == 0) base = atomicAdd(&sm.n_vec, __popcll(reach[q]));
                const int at = __builtin_amdgcn_readfirstlane(base) + lane_prefix_count(reach[q]);
                if (((reach[q] >> lane) & 1ull) && at < kPartVecs) { sm.vec[at] = w[q]; sm.vec_at[at] = v0 + q * kPartThreads + tid; }
            }
        }
    }
    if (edge_id >= 0 && edge_val >= theta) {
        const int at = atomicAdd(&sm.n, 1);
        sm.list[at] = rank_key(edge_val, (uint32_t)edge_id);
    }
    __syncthreads();
    // the node's proposal, for the wave that runs the accept tests if this workgroup is the row's last (asked for here, where
    // the part's registers are free)
    NodeProposal prop;
    if (!commit && wave == 1) prop.request(late().r, row, node, lane);
    int n = sm.n_vec;
    if (__builtin_expect(n <= kPartVecs, 1)) {
        for (int i = tid; i < n * EPV; i += kPartThreads) {
            const float x = load_scalar<DT>(sm.vec, i);
            if (x >= theta) {
                const int at = atomicAdd(&sm.n, 1);   // (at most kPartVecs * EPV)
                if (at < kPartList) sm.list[at] = rank_key(x, (uint32_t)(g.head + sm.vec_at[i / EPV] * EPV + i % EPV));
            }
        }
        __syncthreads();
        n = sm.n;
    } else n = kPartTied;
    if (__builtin_expect(n >= kPartTied, 0)) {
        // again, without most of what equals the bound (the part is fetched a second time: kept until here it would cost
        // the registers of a fourth workgroup per compute unit)
        __syncthreads();  // every wave has seen n
        if (tid == 0) sm.n = 0;
        __syncthreads();
        const __amdgpu_buffer_rsrc_t rsrc =
            __builtin_amdgcn_make_buffer_rsrc((void *)(g.vp + v0), (short)0, (v1 - v0) * 16, 0x00020000);
        uint4 next[1];
        load_part<0>(next, rsrc, tid);
        auto collect = [&](const uint4 &ws, int q, unsigned which) {   // `which` elements of the lane's vector q, ws, join the list
            float x[EPV];
            unpack<DT>(ws, x);
            int at = atomicAdd(&sm.n, __popc(which));
            const int id0 = g.head + (v0 + q * kPartThreads + tid) * EPV;
            while (which) {
                const int k = __ffs((int)which) - 1;
                which &= which - 1u;
                float xv = x[0];
#pragma unroll
                for (int e = 1; e < EPV; ++e) xv = k == e ? x[e] : xv;
                if (at < kPartList) sm.list[at] = rank_key(xv, (uint32_t)(id0 + k));
                ++at;
            }
        };
        int left = K;   // elements equal to the bound that the wave may still take
#pragma unroll 1
        for (int q = 0; q < R; ++q) {
            const uint4 ws = next[0];
            load_part<0>(next, rsrc, (q + 1) * kPartThreads + tid);
            unsigned in = 0u, equal = 0u;
            if (v0 + q * kPartThreads + tid < v1) {
                float x[EPV];
                unpack<DT>(ws, x);
#pragma unroll
                for (int k = 0; k < EPV; ++k) {
                    in |= x[k] > theta ? 1u << k : 0u;
                    equal |= x[k] == theta ? 1u << k : 0u;
                }
            }
            if (q == 0 || (left > 0 && __ballot(equal != 0u))) {
                const int c = __popc(equal), upto = (int)wave_inclusive_scan_u64((unsigned long long)c);
                const int total = __builtin_amdgcn_readlane(upto, 63);
                int all = total;
                if (q == 0) {
                    // the waves' first vectors follow each other in the row, and all others follow them
                    if (lane == 0) sm.rank[wave] = total;
                    __syncthreads();
                    all = 0;
                    for (int o = 0; o < kPartWaves; ++o) {
                        left -= o < wave ? sm.rank[o] : 0;
                        all += sm.rank[o];
                    }
                }
                const int keep = left - (upto - c);   // what the lower lanes leave
                for (int d = c; d > keep && d > 0; --d) equal &= ~(0x80000000u >> __clz((int)equal));
                in |= equal;
                left = (q == 0 ? K : left) - all;
            }
            if (in) collect(ws, q, in);
        }
        const int id = edge_of_lane();   // (again: registers, as above)
        const float val = id >= 0 ? load_scalar<DT>(rowp, id) : -__builtin_inff();
        if (id >= 0 && val >= theta) {
            const int at = atomicAdd(&sm.n, 1);
            if (at < kPartList) sm.list[at] = rank_key(val, (uint32_t)id);
        }
        __syncthreads();
        n = sm.n;
    }
    if (__builtin_expect(n > kPartList, 0)) {
        // too many above the bound: the streaming scan over this part (edges included) finds its K best
        __syncthreads();  // every wave has seen n
        const int base = part == 0 ? 0 : g.head + v0 * EPV;
        const int end = part == P - 1 ? V : g.head + v1 * EPV;
        const void *sub = rowp + (size_t)base * ES;
        WaveScan *wsc = &sm.scan.wsh[wave];
        const WavePartial wp = wave_row_stream<DT>(sub, end - base, c, K, wsc, lane, wave, kPartWaves);
        if (lane == 0) sm.scan.part_cnt[wave] = wp.cnt;
        __syncthreads();
        if (wave == 0) {
            const int cnt = gather_wave_records<DT, kPartWaves>(&sm.scan, lane, K);
            wave_row_finish<DT>(sub, end - base, K, wsc, sm.scan.ebuf, lane, cnt);
            const unsigned long long key = lane < K ? wsc->top[lane] - (unsigned long long)base : 0ull;  // (the low word counts ids down)
            __builtin_amdgcn_wave_barrier();
            if (lane < K) sm.list[lane] = key;
        }
        n = K;   // more than kPartList elements: the part has K
        __syncthreads();
    }
    if (__builtin_expect(n > kPartCut, 0)) n = cut_list(sm.list, n, K, lane, wave);
    // (here and not where their data arrive: the part's registers are free, and the other waves are handing over)
    if (wave == 1 && !commit) {
        const RowPassArgs &r = late().r;
        prop.template request_logits<DT>(r, b, rowp, lane);
        prop.prepare(r, b, lane);
    }
    if (P > 1) {
        if (n > kPartKeys) {
            // more than a part hands over: its K best
            for (int i = tid; i < n; i += kPartThreads) sm.rank[i] = 0;
            __syncthreads();
            rank_against(sm.list, sm.rank, n, n * wave / kPartWaves, n * (wave + 1) / kPartWaves, lane);
            __syncthreads();
            for (int i = tid; i < n; i += kPartThreads)
                if (sm.rank[i] < K) sm.top[sm.rank[i]] = sm.list[i];
            __syncthreads();
            if (tid < K) sm.list[tid] = sm.top[tid];
            n = K;
        }
        // ---- hand over; the row's last workgroup goes on
        const RowPartsArgs &a = late();
        const int slot = j * a.r.B + b;
        const size_t first = (size_t)slot * P, at = first + part;
        if (wave == 0) {
            __builtin_amdgcn_wave_barrier();
            if (lane < n) st_agent(&a.keys[at * kPartKeys + lane], sm.list[lane]);
            if (lane < 4) {
                const uint32_t v = lane == 0 ? f2u(pm) : (lane == 1 ? f2u(ps) : (lane == 2 ? f2u(theta) : (uint32_t)n));
                st_agent((uint32_t *)&a.head[at] + lane, v);
            }
            publish_fence();
            if (lane == 0) {
                unsigned *tk = &a.ticket[(size_t)slot * kTicketStride];
                const unsigned before = atomicAdd(tk, 1u);
                sm.last = before == (unsigned)P - 1u;
                if (sm.last) st_agent(tk, 0u);
            }
        }
        __syncthreads();
        if (!sm.last) return;
        consume_fence();
        // every wave looks at all heads; wave w fetches the keys of parts w, w + 8, ... (whole records: their
        // lengths arrive with the same round trip)
        PartHead h;
        h.m = -3.402823466e38f; h.s = 0.0f; h.theta = -__builtin_inff(); h.cnt = 0;
        if (lane < P) {
            const uint32_t *p = (const uint32_t *)&a.head[first + lane];
            h.m = u2f(ld_agent(p)); h.s = u2f(ld_agent(p + 1)); h.theta = u2f(ld_agent(p + 2)); h.cnt = (int)ld_agent(p + 3);
        }
        constexpr int kRounds = kPartsMax / kPartWaves;
        unsigned long long k[kRounds];
#pragma unroll
        for (int q = 0; q < kRounds; ++q) {
            const int p = q * kPartWaves + wave;
            k[q] = p < P ? ld_agent(&a.keys[(first + p) * kPartKeys + lane]) : 0ull;
        }
        pm = wave_max_f32(h.m);
        const float bound = wave_max_f32(h.theta);
        ps = wave_sum_f32(h.s * fast_exp2((h.m - pm) * c));
#pragma unroll
        for (int q = 0; q < kRounds; ++q) {
            const int p = q * kPartWaves + wave;
            if (p < P) {
                const int c = __builtin_amdgcn_readlane(h.cnt, p);
                const bool in = lane < c && rank_key_value(k[q]) >= bound;
                const unsigned long long bal = __ballot(in);
                int base = 0;
                if (lane == 0 && bal) base = atomicAdd(&sm.n_row, __popcll(bal));
                base = __builtin_amdgcn_readfirstlane(base);
                if (in) { sm.list[base + lane_prefix_count(bal)] = k[q]; sm.rank[base + lane_prefix_count(bal)] = 0; }
            }
        }
        __syncthreads();
        n = sm.n_row;
        if (__builtin_expect(n > kPartCut, 0)) n = cut_list(sm.list, n, K, lane, wave);
    } else {
        for (int i = tid; i < n; i += kPartThreads) sm.rank[i] = 0;
        __syncthreads();
    }
    // ---- one wave runs the accept tests, the others rank the candidates
    const float m = pm + 0.0f;  // (no negative zero)
    if (wave == 1) {
        if (!commit) {
            prop.stage(late().r, row, lane);
            prop.template outcome<DT>(late().r, b, row, rowp, lane, m, ps);
        }
    } else {
        const int who = wave == 0 ? 0 : wave - 1;
        rank_against(sm.list, sm.rank, n, n * who / (kPartWaves - 1), n * (who + 1) / (kPartWaves - 1), lane);
    }
    __syncthreads();
    if (!commit && __builtin_expect(fast_sum_void(m, c), 0)) ps = wave_row_plain_sum<DT>(rowp, V, m, c, lane);
    const RowPartsArgs &e = late();
    const size_t o = (size_t)(commit ? b * e.R + j : row) * K;
    for (int i = tid; i < n; i += kPartThreads) {
        const int at = sm.rank[i];
        if (at >= K) continue;
        const unsigned long long key = sm.list[i];
        const float l = rank_key_value(key);
        if (commit) {
            e.pr_top_idx[o + at] = (int32_t)rank_key_id(key);
            e.pr_top_l[o + at] = l;
        } else {
            e.r.top_idx[o + at] = (int32_t)rank_key_id(key);
            e.r.top_l[o + at] = l;
            e.r.top_p[o + at] = exact_exp2(scaled_offset(l, m, c)) / ps;
        }
    }
    if (tid == 0) {
        if (commit) e.pr_m[b * e.R + j] = m;
        else { e.r.row_m[row] = m; e.r.row_s[row] = ps; }
    }
}

}  // namespace stand
