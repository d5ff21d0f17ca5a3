// Optimal level and capacity-constrained placement of a batch of queries.
//
// One workgroup of 1024 threads.  The level of query q is the number of
// thresholds at or below its best score.  Placement runs rounds r = 0..L:
// every unassigned query applies to the r-th entry of its preference list
// [lam, lam-1, .., 0, lam+1, .., L]; a level accepts applicants in query
// order while it has places left.  Within a round, levels do not interact,
// so each 1024-query chunk computes every applicant's rank among the
// applicants of its level with one wave ballot per level (prefix counts in
// lane order) plus per-wave totals summed in wave order; chunks run in
// query order.  Ranks therefore never depend on atomic ordering, and the
// result is deterministic.  A placement of rank t at level p lands on the
// level's instances ordered by (queue desc, index asc), each filled up to
// its capacity.
#include "apc_internal.h"
#include "route_plan.h"

namespace apc {
namespace {

constexpr int NT = 1024;
constexpr int NWAVE = NT / 64;

// The table is a kernel argument.  Kernel-argument memory is read through
// uncached paths, so every per-lane (dynamically indexed) read of it would be
// a full memory round trip; the kernels copy it into LDS once instead.
// All of a thread's loads are issued before its stores: one round trip.
static_assert(sizeof(AssignTable) % 4 == 0, "table copied as 32-bit words");
template <int NTHR>
__device__ inline void table_to_lds(const AssignTable& src, AssignTable& dst, int tid)
{
    constexpr int W = (int)(sizeof(AssignTable) / 4), PER = (W + NTHR - 1) / NTHR;
    const uint32_t* s = reinterpret_cast<const uint32_t*>(&src);
    uint32_t* d = reinterpret_cast<uint32_t*>(&dst);
    uint32_t v[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i] = tid + i * NTHR < W ? s[tid + i * NTHR] : 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (tid + i * NTHR < W) d[tid + i * NTHR] = v[i];
    __syncthreads();
}

__global__ __launch_bounds__(NT) void k_assign(const AssignTable targ, const float* __restrict__ top_score,
                                                int32_t ld, int32_t b, int32_t* __restrict__ opt_level,
                                                int32_t* __restrict__ out_level,
                                                int32_t* __restrict__ out_inst,
                                                int32_t* __restrict__ out_slot,
                                                int32_t* __restrict__ inst_fill)
{
    __shared__ int used[APC_MAX_LEVELS + 1];
    __shared__ int wcnt[NWAVE][APC_MAX_LEVELS + 1];
    __shared__ AssignTable t;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    table_to_lds<NT>(targ, t, tid);
    const int L = t.L;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

    for (int q = tid; q < b; q += NT) {
        const float best = top_score[(int64_t)q * ld];
        int lam = 0;
        for (int l = 0; l < L; ++l) lam += best >= t.theta[l];
        opt_level[q] = lam;
        out_level[q] = -1;
        out_slot[q] = -1;
    }
    if (tid <= L) used[tid] = 0;
    __syncthreads();

    for (int r = 0; r <= L; ++r) {
        for (int base = 0; base < b; base += NT) {
            const int q = base + tid;
            int want = -1;
            if (q < b && out_level[q] < 0) {
                const int lam = opt_level[q];
                want = r <= lam ? lam - r : r;
            }
            int pre = 0;
            for (int p = 0; p <= L; ++p) {
                const uint64_t m = __ballot(want == p);
                if (want == p) pre = __popcll(m & lt_mask);
                if (lane == 0) wcnt[wave][p] = __popcll(m);
            }
            __syncthreads();
            if (want >= 0) {
                int rank = used[want] + pre;
                for (int w = 0; w < wave; ++w) rank += wcnt[w][want];
                if (rank < t.level_cap[want]) {
                    out_level[q] = want;
                    out_slot[q] = rank;           // admission rank until the instance pass below
                }
            }
            __syncthreads();
            if (tid <= L) {
                int tot = 0;
                for (int w = 0; w < NWAVE; ++w) tot += wcnt[w][tid];
                const int u = used[tid] + tot;
                used[tid] = u < t.level_cap[tid] ? u : t.level_cap[tid];
            }
            __syncthreads();
        }
    }

    for (int q = tid; q < b; q += NT) {
        const int p = out_level[q];
        int inst = -1, slot = -1;
        if (p >= 0) {
            const int rank = out_slot[q];
            for (int j = t.level_first[p]; j < t.level_first[p + 1]; ++j)
                if (rank < t.ord_cum[j] + t.ord_cap[j]) {
                    inst = t.ord_inst[j];
                    slot = rank - t.ord_cum[j];
                    break;
                }
        }
        out_inst[q] = inst;
        out_slot[q] = slot;
    }
    for (int p = 0; p <= L; ++p)
        for (int j = t.level_first[p] + tid; j < t.level_first[p + 1]; j += NT) {
            int f = used[p] - t.ord_cum[j];
            f = f < 0 ? 0 : (f > t.ord_cap[j] ? t.ord_cap[j] : f);
            inst_fill[t.ord_inst[j]] = f;
        }
}

// The same for up to NTB queries, thread tid's query in its registers: no
// global-memory round trip per round.  The block is sized to the batch.  Each
// round takes two barriers: after the per-wave ballots, and after the ranks,
// which read the level counts of the rounds before (used[cur]) while threads
// p <= L write the counts after this round into the other buffer.  The rounds
// stop once one has no applicant (every query placed; later rounds would change
// nothing).
template <int NTB>
__global__ __launch_bounds__(NTB) void k_assign_reg(const AssignTable targ, const float* __restrict__ top_score,
                                                    int32_t ld, int32_t b, int32_t* __restrict__ opt_level,
                                                    int32_t* __restrict__ out_level,
                                                    int32_t* __restrict__ out_inst,
                                                    int32_t* __restrict__ out_slot,
                                                    int32_t* __restrict__ inst_fill)
{
    constexpr int NT = NTB, NWAVE = NTB / 64;
    __shared__ int used[2][APC_MAX_LEVELS + 1];
    __shared__ int wcnt[NWAVE][APC_MAX_LEVELS + 2];          // [L + 1]: the wave has an applicant
    __shared__ AssignTable t;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool mine = tid < b;
    const float best = mine ? top_score[(int64_t)tid * ld] : 0.f;   // issued before the table copy
    table_to_lds<NT>(targ, t, tid);
    const int L = t.L;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int lam = 0, lev = -1, rk = -1;
    if (mine)
        for (int l = 0; l < L; ++l) lam += best >= t.theta[l];
    if (tid <= L) used[0][tid] = 0;
    int cur = 0;
    for (int r = 0; r <= L; ++r) {
        int want = -1;
        if (mine && lev < 0) want = r <= lam ? lam - r : r;
        int pre = 0;
        for (int p = 0; p <= L; ++p) {
            const uint64_t m = __ballot(want == p);
            if (want == p) pre = __popcll(m & lt_mask);
            if (lane == 0) wcnt[wave][p] = __popcll(m);
        }
        const bool wave_any = __ballot(want >= 0) != 0;
        if (lane == 0) wcnt[wave][L + 1] = wave_any;
        __syncthreads();
        bool any = false;
#pragma unroll
        for (int w = 0; w < NWAVE; ++w) any |= wcnt[w][L + 1] != 0;
        if (!any) break;                                      // uniform: no applicant
        if (want >= 0) {
            int rank = used[cur][want] + pre;
#pragma unroll
            for (int w = 0; w < NWAVE; ++w) rank += w < wave ? wcnt[w][want] : 0;
            if (rank < t.level_cap[want]) {
                lev = want;
                rk = rank;
            }
        }
        if (tid <= L) {
            int tot = used[cur][tid];
#pragma unroll
            for (int w = 0; w < NWAVE; ++w) tot += wcnt[w][tid];
            const int cap = t.level_cap[tid];
            used[cur ^ 1][tid] = tot < cap ? tot : cap;
        }
        __syncthreads();
        cur ^= 1;
    }
    if (mine) {
        int inst = -1, slot = -1;
        if (lev >= 0) {
            for (int j = t.level_first[lev]; j < t.level_first[lev + 1]; ++j)
                if (rk < t.ord_cum[j] + t.ord_cap[j]) {
                    inst = t.ord_inst[j];
                    slot = rk - t.ord_cum[j];
                    break;
                }
        }
        opt_level[tid] = lam;
        out_level[tid] = lev;
        out_inst[tid] = inst;
        out_slot[tid] = slot;
    }
    for (int p = 0; p <= L; ++p)
        for (int j = t.level_first[p] + tid; j < t.level_first[p + 1]; j += NT) {
            int f = used[cur][p] - t.ord_cum[j];
            f = f < 0 ? 0 : (f > t.ord_cap[j] ? t.ord_cap[j] : f);
            inst_fill[t.ord_inst[j]] = f;
        }
}

// Position of level j in the preference list of level i, and its inverse.
__device__ inline int pref_pos(int i, int j) { return j == i ? 0 : (j < i ? i - j : j); }
__device__ inline int pref_at(int i, int pos) { return pos == 0 ? i : (pos <= i ? i - pos : pos); }

// Ranks of a batch's values v[c] (0..L, others: none) among equal ones in query
// order, query q = c NTB + tid.  A segment is the 64 queries of a wavefront in a
// chunk.  The lanes with a lane's value are found by a ballot per bit of it
// (six for up to 33 levels, where a ballot per level took up to 33), the first
// of them stores their count; seg[p][g] is then, after one scan per level (a
// wavefront each), the count before segment g.  total[p]: the counts.  Four
// barriers whatever the number of chunks.
template <int QPT, int NTB>
struct Ranks {
    static constexpr int NWAVE = NTB / 64, NSEG = QPT * NWAVE;
    static constexpr int LD = NSEG + 1;
    int seg[APC_MAX_LEVELS + 1][LD];
    int total[APC_MAX_LEVELS + 1];
};
template <int QPT, int NTB>
__device__ inline void rank_levels(Ranks<QPT, NTB>& rk, const int (&v)[QPT], int n, int tid, int (&rank)[QPT])
{
    typedef Ranks<QPT, NTB> R;
    const int lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < n * R::LD; i += NTB) rk.seg[i / R::LD][i % R::LD] = 0;
    const int bits = 32 - __builtin_clz(n);                        // of values 0..n - 1, and n: none
    __syncthreads();
#pragma unroll
    for (int c = 0; c < QPT; ++c) {
        const int x = v[c] < 0 ? n : v[c];
        uint64_t same = ~0ull;
        for (int i = 0; i < bits; ++i) {
            const uint64_t m = __ballot((x >> i) & 1);
            same &= (x >> i) & 1 ? m : ~m;
        }
        rank[c] = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        if (v[c] >= 0 && rank[c] == 0) rk.seg[v[c]][c * R::NWAVE + wave] = __popcll(same);
    }
    __syncthreads();
    if constexpr (QPT == 1) {
        // few segments: every query adds the counts of the wavefronts before its own
        if (v[0] >= 0) {
#pragma unroll
            for (int w = 0; w < R::NWAVE; ++w) rank[0] += w < wave ? rk.seg[v[0]][w] : 0;
        }
        if (tid < n) {
            int t = 0;
#pragma unroll
            for (int w = 0; w < R::NWAVE; ++w) t += rk.seg[tid][w];
            rk.total[tid] = t;
        }
        __syncthreads();
    } else {
        for (int p = wave; p < n; p += R::NWAVE) {                 // uniform per wavefront
            constexpr int PER = (R::NSEG + 63) / 64;
            int x[PER], sum = 0;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int g = lane * PER + i;
                x[i] = g < R::NSEG ? rk.seg[p][g] : 0;
                sum += x[i];
            }
            int inc = sum;
#pragma unroll
            for (int m = 1; m < 64; m *= 2) {
                const int o = __shfl_up(inc, m, 64);
                if (lane >= m) inc += o;
            }
            int run = inc - sum;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int g = lane * PER + i;
                if (g < R::NSEG) rk.seg[p][g] = run;
                run += x[i];
            }
            if (lane == 63) rk.total[p] = inc;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < QPT; ++c)
            if (v[c] >= 0) rank[c] += rk.seg[v[c]][c * R::NWAVE + wave];
    }
}

// The flow x[i n + p] (queries of optimal level i placed at level p) of the
// rounds placement, by one wavefront, lane p holding level p.  In round r level
// i wants level i - r (r <= i) or r (r > i), in query order.  What a level has
// left is always the last of its queries: each round takes a prefix of them.
// So a round is a minimum of demand and places per level, except for level r
// itself, which the levels below r and level 2 r all want: where they ask for
// more than it has, the first in query order win, and the query at which the
// places run out is found from the counts before each segment and the levels of
// that segment's queries.
template <int QPT, int NTB>
__device__ inline void rounds_flow(const Ranks<QPT, NTB>& rk, const uint8_t* lam, const AssignTable& t, int lane, int* x)
{
    static_assert(QPT > 1, "reads the counts before each segment, which rank_levels leaves only for several queries per thread");
    constexpr int NSEG = Ranks<QPT, NTB>::NSEG;
    const int L = t.L, n = L + 1;
    int done = 0;                                                  // of this level's queries
    int rem = lane <= L ? rk.total[lane] : 0, room = lane <= L ? t.level_cap[lane] : 0;
    for (int r = 0; r <= L; ++r) {
        if (!__ballot(rem > 0)) break;                             // every query placed
        // single sources: level lane + r into level lane
        const int from = lane + r;
        const bool one = lane <= L && from <= L && (lane != r || r == 0);
        const int want = __shfl(rem, from & 63, 64);
        const int take = one ? (want < room ? want : room) : 0;
        if (one) x[from * n + lane] = take;
        // level r >= 1: sources below r and 2 r
        const bool src = r > 0 && lane <= L && (lane < r || lane == 2 * r);
        int ask = src ? rem : 0;
        int total = ask;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) total += __shfl_xor(total, m, 64);
        const int places = __builtin_amdgcn_readlane(room, r);
        if (r > 0 && total > places) {                             // uniform
            // segments whose preceding applicants fit (a prefix): the last one is where places run out
            constexpr int PER = (NSEG + 63) / 64;
            int c[PER];
#pragma unroll
            for (int j = 0; j < PER; ++j) c[j] = 0;
            for (int i = 0; i <= L; ++i)
                if (i < r || i == 2 * r) {
                    const int d = __builtin_amdgcn_readlane(done, i);
#pragma unroll
                    for (int j = 0; j < PER; ++j) {
                        const int over = rk.seg[i][j * 64 + lane < NSEG ? j * 64 + lane : 0] - d;
                        c[j] += over > 0 ? over : 0;
                    }
                }
            int g = 0;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const uint64_t fit = __ballot(j * 64 + lane < NSEG && c[j] <= places);
                if (fit) g = j * 64 + 63 - __builtin_clzll(fit);
            }
            const int mine = lam[g * 64 + lane];                   // 255 past the batch
            const int start = lane <= L ? rk.seg[lane][g] : 0;     // this level's count before the segment
            const int ahead = src && start > done ? start - done : 0;   // its applicants before the segment
            int before = ahead;
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) before += __shfl_xor(before, m, 64);
            uint64_t apps = 0;                                     // the segment's applicants
            for (int i = 0; i <= L; ++i)
                if (i < r || i == 2 * r) {
                    const int d = __builtin_amdgcn_readlane(done, i), s0 = __builtin_amdgcn_readlane(start, i);
                    const uint64_t m = __ballot(mine == i);
                    const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    apps |= __ballot(mine == i && s0 + rank >= d);
                }
            const int nth = __builtin_amdgcn_mbcnt_hi((uint32_t)(apps >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)apps, 0u));
            const uint64_t won = apps & __ballot(nth < places - before);
            ask = ahead;
            for (int i = 0; i <= L; ++i)
                if (i < r || i == 2 * r) {
                    const int c1 = __popcll(won & __ballot(mine == i));
                    if (lane == i) ask += c1;
                }
        }
        if (src) x[lane * n + r] = ask;
        // what is left
        const int gone = __shfl(take, (lane - r) & 63, 64);        // by level lane - r
        if (src) {
            rem -= ask;
            done += ask;
        } else if (lane <= L && lane >= r) {
            rem -= gone;
            done += gone;
        }
        const int got = total < places ? total : places;
        if (lane == r && r > 0) room -= got;
        else room -= take;
    }
}

// Placement by rounds (MODE 2) or by a route plan x (queries of optimal level i
// served at level j): read from the caller (MODE 0; negative entries count as
// 0) or the optimal one, built from the batch's level histogram H, the places
// per level and K (one thread per level, then one per plan entry) and written
// out (MODE 1).  The rounds are a plan too, whose flow one wavefront finds
// (rounds_flow).  Same query ownership as k_assign_reg.  Pass 1 ranks every
// query among the queries of its own level in index order, which also yields
// H.  A query of level i with rank s takes the first level j of its preference
// list [i, i-1, .., 0, i+1, .., L] where s falls below the running sum of
// x[i][.]; the position pos of j in that list is its round.  A level admits in
// (round, index) order while it has places, so a query's admission rank is the
// number of queries routed to j in earlier rounds (from the realised flow) plus
// its rank inside group (j, pos).  Only group (j, j) mixes queries of several
// levels; pass 2 ranks its members, the others are ranked by their offset in
// their level's quota.
// 16,384 queries, 10 levels: the rounds 281 us as k_assign_reg does them, with
// several queries per thread (two barriers and a ballot per level for each of 16
// chunks in every round), 63 here; the call by plan 61 us with a barrier pair
// per chunk, 42 now.
enum { PLAN_GIVEN = 0, PLAN_OPTIMAL = 1, PLAN_ROUNDS = 2 };
template <int QPT, int NTB, int MODE>
__global__ __launch_bounds__(NTB) void k_assign_plan(const AssignTable targ, const float* __restrict__ top_score,
                                                     int32_t ld, int32_t b, int32_t* __restrict__ plan,
                                                     int32_t* __restrict__ opt_level,
                                                     int32_t* __restrict__ out_level,
                                                     int32_t* __restrict__ out_inst,
                                                     int32_t* __restrict__ out_slot,
                                                     int32_t* __restrict__ inst_fill)
{
    constexpr int NT = NTB, NL = APC_MAX_LEVELS + 1;
    __shared__ Ranks<QPT, NTB> rkl;
    __shared__ uint8_t lams[MODE == PLAN_ROUNDS ? QPT * NTB : 1];
    __shared__ int xs[NL * NL];
    __shared__ int fs[NL * NL];                              // realised flow, level i -> level j
    __shared__ int gb[NL * NL];                              // [j * n + pos]: places before group (j, pos)
    __shared__ int cum[NL * NL];                             // [i * n + pos]: queries of level i placed up to position pos
    __shared__ int used[NL];                                 // places taken per level
    __shared__ PlanWork w;
    __shared__ unsigned long long multi;                     // bit j: group (j, j) has members
    __shared__ AssignTable t;
    const int tid = threadIdx.x;
    float best[QPT];
#pragma unroll
    for (int c = 0; c < QPT; ++c) {
        const int q = c * NT + tid;
        best[c] = q < b ? top_score[(int64_t)q * ld] : 0.f;
    }
    table_to_lds<NT>(targ, t, tid);
    const int L = t.L, n = L + 1;
    int lam[QPT], rs[QPT], dr[QPT], ik[QPT], rk[QPT];
#pragma unroll
    for (int c = 0; c < QPT; ++c) {
        const int q = c * NT + tid;
        lam[c] = q < b ? 0 : -1;
        rk[c] = -1;
    }
    for (int l = 0; l < L; ++l) {
        const float th = t.theta[l];
#pragma unroll
        for (int c = 0; c < QPT; ++c)
            lam[c] += lam[c] >= 0 && best[c] >= th;
    }
    if constexpr (MODE == PLAN_ROUNDS) {
#pragma unroll
        for (int c = 0; c < QPT; ++c) lams[c * NT + tid] = (uint8_t)lam[c];   // 255 past the batch
    }
    // Pass 1: rank among the queries of the same level; the histogram.
    rank_levels<QPT, NTB>(rkl, lam, n, tid, rs);
    // The plan.
    if constexpr (MODE == PLAN_ROUNDS) {
        for (int e = tid; e < n * n; e += NT) xs[e] = 0;
        __syncthreads();
        if (tid < 64) rounds_flow<QPT, NTB>(rkl, lams, t, tid, xs);
    } else if constexpr (MODE == PLAN_OPTIMAL) {
        if (tid <= L) plan_level_own(L, rkl.total, t.level_cap, tid, w);
        __syncthreads();
        if (tid < L) plan_level_flow(L, tid, w);
        if (tid == L) w.n[L] = 0;
        __syncthreads();
        if (tid <= L) plan_level_intervals(L, tid, w);
        __syncthreads();
        for (int e = tid; e < n * n; e += NT) {
            const int v = plan_entry(e / n, e % n, w);
            xs[e] = v;
            plan[e] = v;
        }
    } else {
        for (int e = tid; e < n * n; e += NT) {
            const int v = plan[e];
            xs[e] = v < 0 ? 0 : v;
        }
    }
    __syncthreads();
    // Realised flow: how many of level i's queries the plan sends to level j
    // (the row's quotas taken in preference order until the level runs out).
    const int* H = rkl.total;
    for (int e = tid; e < n * n; e += NT) {
        const int i = e / n, j = e - i * n, pj = pref_pos(i, j);
        int64_t before = 0;
        for (int pos = 0; pos < pj; ++pos) before += xs[i * n + pref_at(i, pos)];
        int64_t f = (int64_t)H[i] - before;
        f = f < 0 ? 0 : (f > xs[e] ? xs[e] : f);
        fs[e] = (int)f;
        // queries of level i that go to positions up to pj (its quotas' running sum, at most H)
        const int64_t upto = before + xs[e];
        cum[i * n + pj] = upto < H[i] ? (int)upto : H[i];
    }
    if (tid == 0) multi = 0ull;
    __syncthreads();
    // Places at level j taken before group (j, pos), i.e. by earlier positions.
    for (int e = tid; e < n * n; e += NT) {
        const int j = e / n, pos = e - j * n;
        int base = 0;
        for (int i = 0; i <= L; ++i) base += pref_pos(i, j) < pos ? fs[i * n + j] : 0;
        gb[e] = base;
    }
    if (tid <= L) {
        int tot = 0;
        int mixed = 0;                                       // members of group (tid, tid)
        for (int i = 0; i <= L; ++i) {
            tot += fs[i * n + tid];
            mixed += tid > 0 && pref_pos(i, tid) == tid ? fs[i * n + tid] : 0;
        }
        if (mixed) atomicOr(&multi, 1ull << tid);
        used[tid] = tot < t.level_cap[tid] ? tot : t.level_cap[tid];
    }
    // Destination, position and rank inside its group (j, pos).  A group with
    // pos != j holds queries of one level i only (i = j + pos, or i = j for
    // pos = 0), in index order, so the rank is the offset in i's quota.  Group
    // (j, j) gathers the moves up from every level below j (and the move down
    // from level 2j): ranked by ballots below.
#pragma unroll
    for (int c = 0; c < QPT; ++c) {
        dr[c] = -1;
        ik[c] = -1;
        if (lam[c] >= 0) {
            // the first position whose running sum passes the rank (the sums rise with it)
            const int i = lam[c];
            const int* row = cum + i * n;
            int lo = 0, hi = L;
            if (rs[c] < row[L]) {
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (rs[c] < row[mid]) hi = mid;
                    else lo = mid + 1;
                }
                const int pos = lo, j = pref_at(i, pos);
                dr[c] = j | (pos << 8);
                if (pos != j || j == 0) ik[c] = rs[c] - (pos > 0 ? row[pos - 1] : 0);
            }
        }
    }
    __syncthreads();
    const unsigned long long mm = multi;
    if (mm) {                                                 // uniform
        int g[QPT], r2[QPT];
#pragma unroll
        for (int c = 0; c < QPT; ++c) g[c] = dr[c] >= 0 && ik[c] < 0 ? (dr[c] & 0xff) : -1;
        rank_levels<QPT, NTB>(rkl, g, n, tid, r2);
#pragma unroll
        for (int c = 0; c < QPT; ++c)
            if (g[c] >= 0) ik[c] = r2[c];
    }
    // Admission rank at the level: earlier groups, then the rank in the group.
#pragma unroll
    for (int c = 0; c < QPT; ++c) {
        rk[c] = -1;
        if (dr[c] >= 0) {
            const int j = dr[c] & 0xff, pos = dr[c] >> 8;
            const int rank = gb[j * n + pos] + ik[c];
            if (rank < t.level_cap[j]) rk[c] = rank;
        }
    }
#pragma unroll
    for (int c = 0; c < QPT; ++c) {
        const int q = c * NT + tid;
        if (q >= b) continue;
        const int p = rk[c] >= 0 ? (dr[c] & 0xff) : -1;
        int inst = -1, slot = -1;
        if (p >= 0) {
            for (int j = t.level_first[p]; j < t.level_first[p + 1]; ++j)
                if (rk[c] < t.ord_cum[j] + t.ord_cap[j]) {
                    inst = t.ord_inst[j];
                    slot = rk[c] - t.ord_cum[j];
                    break;
                }
        }
        opt_level[q] = lam[c];
        out_level[q] = p;
        out_inst[q] = inst;
        out_slot[q] = slot;
    }
    for (int p = 0; p <= L; ++p)
        for (int j = t.level_first[p] + tid; j < t.level_first[p + 1]; j += NT) {
            int f = used[p] - t.ord_cum[j];
            f = f < 0 ? 0 : (f > t.ord_cap[j] ? t.ord_cap[j] : f);
            inst_fill[t.ord_inst[j]] = f;
        }
}

template <int MODE>
hipError_t launch_plan_t(const AssignTable& t, const float* top_score, int32_t ld, int32_t b, int32_t* plan,
                         int32_t* opt_level, int32_t* out_level, int32_t* out_inst, int32_t* out_slot,
                         int32_t* inst_fill, hipStream_t s)
{
    if constexpr (MODE != PLAN_ROUNDS) {                     // (up to NT queries the rounds have k_assign_reg)
        if (b <= NT) {
            if (b <= 256)
                k_assign_plan<1, 256, MODE><<<1, 256, 0, s>>>(t, top_score, ld, b, plan, opt_level, out_level, out_inst, out_slot, inst_fill);
            else
                k_assign_plan<1, NT, MODE><<<1, NT, 0, s>>>(t, top_score, ld, b, plan, opt_level, out_level, out_inst, out_slot, inst_fill);
            return hipGetLastError();
        }
    }
    if (b <= 4 * NT)
        k_assign_plan<4, NT, MODE><<<1, NT, 0, s>>>(t, top_score, ld, b, plan, opt_level, out_level, out_inst, out_slot, inst_fill);
    else if (b <= 16 * NT)
        k_assign_plan<16, NT, MODE><<<1, NT, 0, s>>>(t, top_score, ld, b, plan, opt_level, out_level, out_inst, out_slot, inst_fill);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_assign(const AssignTable& t, const float* top_score, int32_t ld, int32_t b,
                         int32_t* opt_level, int32_t* out_level, int32_t* out_inst,
                         int32_t* out_slot, int32_t* inst_fill, hipStream_t s)
{
    if (b <= 256)
        k_assign_reg<256><<<1, 256, 0, s>>>(t, top_score, ld, b, opt_level, out_level, out_inst, out_slot, inst_fill);
    else if (b <= NT)
        k_assign_reg<NT><<<1, NT, 0, s>>>(t, top_score, ld, b, opt_level, out_level, out_inst, out_slot, inst_fill);
    else if (b <= 16 * NT)                               // several queries per thread: the rounds as a plan
        return launch_plan_t<PLAN_ROUNDS>(t, top_score, ld, b, nullptr, opt_level, out_level, out_inst, out_slot,
                                          inst_fill, s);
    else
        k_assign<<<1, NT, 0, s>>>(t, top_score, ld, b, opt_level, out_level, out_inst, out_slot, inst_fill);
    return hipGetLastError();
}

hipError_t launch_assign_plan(const AssignTable& t, bool planned, const float* top_score, int32_t ld, int32_t b,
                              int32_t* plan, int32_t* opt_level, int32_t* out_level, int32_t* out_inst,
                              int32_t* out_slot, int32_t* inst_fill, hipStream_t s)
{
    static_assert(16 * NT == APC_MAX_ROUTED_BATCH, "largest routed batch");
    return planned ? launch_plan_t<PLAN_OPTIMAL>(t, top_score, ld, b, plan, opt_level, out_level, out_inst, out_slot, inst_fill, s)
                   : launch_plan_t<PLAN_GIVEN>(t, top_score, ld, b, plan, opt_level, out_level, out_inst, out_slot, inst_fill, s);
}

}  // namespace apc
