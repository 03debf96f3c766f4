// Resident searches: one workgroup runs one query from its roots to its end.
//
// On a graph of small degree (roads, grids) a query's frontier is a few
// hundred to a few thousand entries, and a batch in global rounds is bound by
// the rounds themselves: two launches each, and in each a chain of dependent
// accesses to lines that any XCD may have written. Here a query lives on one
// compute unit:
//   - a round takes three workgroup barriers (three more for each further
//     batch of candidates) instead of two kernel boundaries;
//   - its distance words are only ever touched by that workgroup, so plain
//     loads and stores serve, and the words stay in one XCD's L2;
//   - its frontier (two queues by round parity) is in LDS, with a spill area
//     in memory for the entries beyond.
// A batch is one launch; the queries do not wait for each other.
// Rounds of the whole chip / resident, ms: one query on a 256^2 grid 2.25 /
// 0.66, 64 on it 7.7 / 1.35, 256 BiD-A* on a 2048^2 lattice 69.8 / 44.8, 100
// A* on an 800 x 600 one 22.6 / 10.6, 48 BiDS on a directed one 24.4 / 6.9,
// all distances on 1024^2 27.2 / 13.0. What bounds a query: its rounds, one
// after the other, about 5 us each when small (a chain of three barriers, three
// dependent accesses to memory and the LDS lists between), and 400 to 470
// arcs a microsecond on one compute unit beyond; a batch lasts as long as its
// longest query.
//
// Distances are 32-bit words, the two copies of a bidirectional query side by
// side (8 bytes a vertex, half of the round kernels' packed word): a frontier
// entry stores the distance it was added with, and is stale when the
// vertex's word is lower, so no stamp is needed. A vertex lowered twice in a
// round (by two batches of its candidates) has two entries, the first stale.
//
// The search is Algorithm 2 with the rules of Table 2, as in the round
// kernels: a round extracts the entries whose key is within the threshold
// (the others are carried, by their stored distance and heuristic term),
// repeats the meeting check of each, prunes, and relaxes its arcs; a
// successful relaxation does the meeting check at once, prunes and adds. The
// check at extraction sees every lowering of the rounds before (stores of the
// workgroup, ordered by the barrier), which covers two copies that became
// exact in the same round. The bound of a round is the query's mu at its
// start.
//
// A round has three parts, each packed for what follows (16 waves share four
// SIMDs: instructions count as much as the chain of accesses):
//   1. the queue is read; entries within the threshold are listed as the
//      round's candidates. Entries far above it go to a far list that is read
//      again only when the threshold comes near (with a heuristic four
//      entries in five wait, most of them for long);
//   2. the candidates are checked and pruned, and their arcs relaxed as one
//      list, an arc a lane. A lowered vertex is a bid (vertex, distance);
//      bids for one vertex meet in LDS: a global atomic minimum with its old
//      value costs about 950 cycles (it is executed at the memory side even at
//      workgroup scope: 4 cycles each on one CU alone, 25 when all CUs do it),
//      a minimum in LDS about a tenth;
//   3. the smallest bid of a vertex stores its distance (a plain store: no
//      other workgroup writes these words), and is pruned and added.
#include "resident.h"

namespace ppsp {

namespace {

constexpr int RES_WAYS = 5;             // 64-arc steps of a wave in flight (64 vertices of a road network have 262 arcs)
constexpr uint32_t SIDE_BIT = 0x80000000u;
constexpr uint32_t NO_KEY = 0xFFFFFFFFu;      // no entry; as a bound: none
constexpr uint32_t REACH = 4;           // the near queue reaches step / REACH past the threshold (2 to 8 measured the same,
                                        // 1: 3% slower, no far list: 9%)
constexpr uint32_t MAX_KEY = 0xFFFFFFFEu;     // keys are held in 32 bits, clamped here

__device__ __forceinline__ uint32_t mbcnt(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

// Row shifts, then row broadcasts: lane 63 ends with the whole wave's result.
#define PPSP_DPP(x, none, ctrl, rows) ((uint32_t)__builtin_amdgcn_update_dpp((int)(none), (int)(x), ctrl, rows, 0xf, false))
// *to = min(*to, x of every lane), one LDS atomic per row of 16 lanes.
__device__ __forceinline__ void wave_min_to(uint32_t *to, uint32_t x) {
    if (__ballot(x != NO_KEY) == 0) return;
    x = min(x, PPSP_DPP(x, NO_KEY, 0x111, 0xf));
    x = min(x, PPSP_DPP(x, NO_KEY, 0x112, 0xf));
    x = min(x, PPSP_DPP(x, NO_KEY, 0x114, 0xf));
    x = min(x, PPSP_DPP(x, NO_KEY, 0x118, 0xf));
    if ((__lane_id() & 15u) == 15u) atomicMin(to, x);
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {    // inclusive sums
    x += PPSP_DPP(x, 0, 0x111, 0xf);
    x += PPSP_DPP(x, 0, 0x112, 0xf);
    x += PPSP_DPP(x, 0, 0x114, 0xf);
    x += PPSP_DPP(x, 0, 0x118, 0xf);
    x += PPSP_DPP(x, 0, 0x142, 0xa);
    x += PPSP_DPP(x, 0, 0x143, 0xc);
    return x;
}
#undef PPSP_DPP

// Keeps the compiler from moving the load of `a` behind a branch on `b`.
#define PPSP_TOGETHER(a, b) asm volatile("" : "+v"(a), "+v"(b))

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long x) {
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

// Orders this wave's LDS accesses (its lanes exchange data through LDS).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Loads at a 32-bit byte offset: one address instruction each.
template <class T>
__device__ __forceinline__ T load_at(const void *base, uint32_t offset) {
    T x;
    __builtin_memcpy(&x, (const char *)base + offset, sizeof(T));
    return x;
}

// What a round hands to the next.
struct __attribute__((aligned(16))) Handover {
    uint32_t near, cand;                // near entries for the next round; candidates of this one (one atomic adds to both)
    uint32_t mk0, mk1;                  // the entries' smallest keys by side
    unsigned long long mu;              // the round's smallest (meeting distance, vertex)
    uint32_t stop, pad;                 // time is up
};
// The far list.
struct __attribute__((aligned(16))) FarList { uint32_t n, mk0, mk1, pad; };

}  // namespace

// B threads a query. LDS for 1,024 with a heuristic: 30 KB queues and keys,
// 8 KB candidates, 21 KB extracted entries and owners of arcs, 32 KB bids, 64 KB
// bid tables, in all 155.2 of a unit's 160; for 512 half of it, so that two
// workgroups share a unit.
template <int B, bool PAIR, bool HEUR, bool REV>
__global__ __launch_bounds__(B) void k_resident(ResidentArgs A) {
    constexpr uint32_t KIND = PAIR ? (HEUR ? K_BIDA_F : K_2DIST) : (HEUR ? K_ASTAR : K_DIST);
    constexpr uint32_t CAP = B + B / 4;                   // entries of a near queue in LDS (the rest: spill area)
    constexpr uint32_t CAND = 4 * B;                      // candidates of a round (more wait)
    constexpr uint32_t BIDS = 2 * B;                      // bids of B candidates (beyond: their candidate waits)
    constexpr uint32_t NW = B / 64;                       // waves
    constexpr uint32_t TAB = 4 * B;                       // slots of a bid table
    __shared__ uint2 lq[2][CAP];                          // near queues by round parity: (vertex | side, distance)
    __shared__ uint32_t lk[2][HEUR ? CAP : 1];            // keys (without a heuristic: a multiple of the distance)
    __shared__ uint16_t s_idx[CAND];                      // candidates: places in the queue
    __shared__ uint4 s_ext[B];                            // extracted: (vertex | side, distance, first arc less its place in
                                                          // its wave's list of arcs, candidate)
    __shared__ uint8_t s_owner[B / 64][64 * RES_WAYS];    // a wave's candidate of each arc of the list's current part
    __shared__ uint4 s_bid[BIDS];                         // (vertex | side, distance, the other copy's, candidate)
    __shared__ unsigned long long s_tab[2][TAB];          // smallest bids: 15 - batch (4 bits), distance, vertex | side
    __shared__ Handover s_hand[3];                        // read, written and reset in turn
    __shared__ FarList s_far[2];
    __shared__ uint32_t s_nbid, s_err;
    __shared__ unsigned long long s_stat[RS_N];
    static_assert(sizeof(lq) + sizeof(lk) + sizeof(s_idx) + sizeof(s_ext) + sizeof(s_owner) + sizeof(s_bid) +
                  sizeof(s_tab) + sizeof(s_hand) + sizeof(s_far) + sizeof(s_nbid) + sizeof(s_err) + sizeof(s_stat) <=
                  160 * B, "a unit's 160 KB hold one workgroup of 1,024 threads or two of 512");

    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid / 64), q = blockIdx.x;
    const SearchDesc sd = A.sd[PAIR ? 2 * q : q];
    const uint32_t n = A.n;
    uint32_t *D = A.D + (uint64_t)q * n * (PAIR ? 2 : 1);
    // spill area: two near queues beyond LDS, two far lists
    uint4 *spill = A.spill + (uint64_t)q * 4 * A.spcap;
    const uint64_t d0 = A.delta[PAIR ? 2 * q : q], d1 = PAIR ? A.delta[2 * q + 1] : d0;
    const bool has_pair = sd.pend > sd.pbeg;
    const Partner part = has_pair ? A.partners[sd.pbeg] : Partner{TARGET_BIT, 0};
    const uint32_t target = has_pair ? part.other & ~TARGET_BIT : NO_KEY;      // one-sided searches

    // the forward heuristic term: h_t - h_s, or h_t for one-sided A*
    auto hterm = [&](int2 p) -> int32_t {
        const int32_t ht = (int32_t)heur(p.x, p.y, sd.tx, sd.ty, A.ws2, A.fb);
        return PAIR ? ht - (int32_t)heur(p.x, p.y, sd.sx, sd.sy, A.ws2, A.fb) : ht;
    };
    auto clamp = [](uint64_t k) { return (uint32_t)min(k, (uint64_t)MAX_KEY); };
    auto dist_key = [&](uint32_t d) { return PAIR ? (d > 0x7FFFFFFFu ? MAX_KEY : min(2u * d, MAX_KEY)) : min(d, MAX_KEY); };
    struct Entry { uint32_t v, d, key; };
    auto get = [&](uint32_t par, uint32_t k) -> Entry {
        if (k < CAP) {
            const uint2 x = lq[par][k];
            return {x.x, x.y, HEUR ? lk[par][k] : dist_key(x.y)};
        }
        const uint4 x = spill[(uint64_t)par * A.spcap + (k - CAP)];
        return {x.x, x.y, x.z};
    };
    auto put = [&](uint32_t par, uint32_t k, const Entry &e) {
        if (k < CAP) {
            lq[par][k] = make_uint2(e.v, e.d);
            if (HEUR) lk[par][k] = e.key;
        } else if (k - CAP < A.spcap) {
            spill[(uint64_t)par * A.spcap + (k - CAP)] = make_uint4(e.v, e.d, e.key, 0u);
        }
    };

    uint64_t th0 = 0, th1 = 0, mu = INF64;
    uint32_t bnd = NO_KEY, T0 = 0, T1 = 0;                 // near entries have keys up to T0, T1
    bool ex0 = false, ex1 = false;
    if (tid < 3) s_hand[tid] = {0, 0, NO_KEY, NO_KEY, INF64, 0, 0};
    if (tid < 2) s_far[tid] = {0, NO_KEY, NO_KEY, 0};
    if (tid == 0) s_nbid = s_err = 0;
    if (tid < (uint32_t)RS_N) s_stat[tid] = 0;
    {
        // Init(): the roots at distance 0
        const uint32_t s = sd.src, t = PAIR ? A.sd[2 * q + 1].src : 0;
        th0 = key_of(KIND, 0, HEUR ? hterm(A.xy[s]) : 0);
        th1 = PAIR ? key_of(KIND, 0, HEUR ? -hterm(A.xy[t]) : 0) : 0;
        __syncthreads();
        if (tid == 0) {
            put(0, 0, {s, 0u, clamp(th0)});
            D[PAIR ? 2ull * s : s] = 0;
            if (PAIR) {
                put(0, 1, {t | SIDE_BIT, 0u, clamp(th1)});
                D[2ull * t + 1] = 0;
            }
            s_hand[0].near = PAIR ? 2 : 1;
            s_hand[0].mk0 = clamp(th0);
            if (PAIR) s_hand[0].mk1 = clamp(th1);
        }
    }
    uint32_t c_ent = 0, c_sv = 0, c_se = 0, c_succ = 0, c_keep = 0, status = RES_DONE;
    unsigned long long t_begin = wall_clock64();           // of the first workgroup (tid 0 only)
    if (tid == 0 && A.ticks) t_begin = min(t_begin, atomicMin(A.t_begin, t_begin));
    uint32_t r = 0, gen = 0;                               // round; bid tables: 16 batches between clears
    uint32_t cur = 0, nxt = 1, rst = 2;                    // handover slots: this round's input, its output, the one reset
    uint32_t far = 0;                                      // the far list in use
    for (;; r++) {
        __syncthreads();
        const Handover hin = s_hand[cur];
        const FarList fin = s_far[far];
        const uint32_t cnt = uniform(hin.near), nfar = HEUR ? uniform(fin.n) : 0u;
        const uint32_t m0 = uniform(HEUR ? min(hin.mk0, fin.mk0) : hin.mk0);
        const uint32_t m1 = uniform(HEUR ? min(hin.mk1, fin.mk1) : hin.mk1);
        mu = min(mu, (uint64_t)uniform((uint32_t)(hin.mu >> 32)) << 32 | uniform((uint32_t)hin.mu));
        if (tid == 0) {
            s_hand[rst] = {0, 0, NO_KEY, NO_KEY, INF64, 0, 0};
            s_nbid = 0;
            // from the first round on: a launch of many short queries has few others (every round: single queries
            // and all distances of a source 1 to 1.5% slower)
            if (A.ticks && (r & 7) == 0 && wall_clock64() - t_begin > A.ticks) s_hand[nxt].stop = 1;
        }
        // Liveness, termination and bound (Table 2; a side that ran dry while
        // nothing could be pruned has covered its component, Appendix B), and
        // the thresholds, the same in every lane.
        const bool live0 = m0 != NO_KEY, live1 = PAIR && m1 != NO_KEY;
        if (r && bnd == NO_KEY) {
            ex0 = ex0 || !live0;
            ex1 = ex1 || (PAIR && !live1);
        }
        const bool found = mu != INF64;
        if ((!live0 && !live1) || (!sd.noprune && !found && (ex0 || ex1))) break;
        if (cnt > CAP + A.spcap || nfar > A.spcap) { status = RES_SPILL; break; }
        if (uniform(hin.stop)) { status = RES_TIMEOUT; break; }
        bnd = !sd.noprune && found ? (uint32_t)(mu >> 32) : NO_KEY;
        if (r) {
            // a clamped smallest key: extract everything
            if (live0) th0 = m0 == MAX_KEY ? INF64 : step_threshold(A.theta_mode, th0, m0, d0);
            if (live1) th1 = m1 == MAX_KEY ? INF64 : step_threshold(A.theta_mode, th1, m1, d1);
        }
        const uint32_t t0 = clamp(th0), t1 = clamp(th1);
        const uint32_t in = r & 1, out = in ^ 1;
        // the threshold passed the near queue's reach: the far list is read again
        const bool refill = HEUR && ((live0 && t0 > T0) || (live1 && t1 > T1) || r == 0);
        if (refill) {
            if (live0) T0 = clamp((uint64_t)t0 + min(d0, (uint64_t)1 << 32) / REACH);
            if (live1) T1 = clamp((uint64_t)t1 + min(d1, (uint64_t)1 << 32) / REACH);
        }
        const uint32_t fout = refill ? far ^ 1 : far;
        uint32_t k0 = NO_KEY, k1 = NO_KEY, f0 = NO_KEY, f1 = NO_KEY;   // smallest keys this lane adds: near, far; by side
        auto meet = [&](uint32_t d, uint32_t oth, uint32_t v) {      // UpdateDistance
            uint32_t sum = d;
            if (PAIR) {
                if (oth == INF32) return;
                sum = d + oth;
                if (sum < d || sum == INF32) { s_err = 1; return; }
            } else if (v != target) {
                return;
            }
            if (sum < (uint32_t)(s_hand[nxt].mu >> 32)) atomicMin(&s_hand[nxt].mu, ((unsigned long long)sum << 32) | v);
        };
        // the lanes of `mask` take consecutive places from *ctr
        auto reserve = [&](uint32_t *ctr, uint64_t mask) {
            uint32_t pos = 0;
            if (lane == 0) pos = atomicAdd(ctr, (uint32_t)__popcll(mask));
            return uniform(pos) + mbcnt(mask);
        };
        // Add: to the near queue or the far list
        auto add = [&](bool yes, const Entry &e) {
            const bool side = PAIR && (e.v & SIDE_BIT);
            const bool fr = HEUR && yes && e.key > (side ? T1 : T0) && e.key < bnd, nr = yes && !fr;
            if (const uint64_t m = __ballot(nr)) {
                const uint32_t pos = reserve(&s_hand[nxt].near, m);
                if (nr) {
                    put(out, pos, e);
                    if (side) k1 = min(k1, e.key); else k0 = min(k0, e.key);
                }
            }
            if (!HEUR) return;
            if (const uint64_t m = __ballot(fr)) {
                const uint32_t pos = reserve(&s_far[fout].n, m);
                if (fr) {
                    if (pos < A.spcap) spill[(uint64_t)(2 + fout) * A.spcap + pos] = make_uint4(e.v, e.d, e.key, 0u);
                    if (side) f1 = min(f1, e.key); else f0 = min(f0, e.key);
                }
            }
        };

        // 1. Extract: an entry above the threshold (or beyond the candidate
        // list) waits for a later round.
        for (uint32_t base = wave * 64; base < cnt; base += B) {
            const uint32_t k = base + lane;
            Entry e = {0, 0, 0};
            if (k < cnt) e = get(in, k);
            const bool side = PAIR && (e.v & SIDE_BIT);
            const bool far_off = k < cnt && e.key > (side ? t1 : t0) && e.key < bnd;
            const uint64_t mc = __ballot(k < cnt && !far_off), mw = __ballot(far_off);
            unsigned long long pos = 0;
            if (lane == 0)
                pos = atomicAdd((unsigned long long *)&s_hand[nxt], (unsigned long long)__popcll(mc) << 32 | (uint32_t)__popcll(mw));
            const uint32_t pw = uniform((uint32_t)pos), pc = uniform((uint32_t)(pos >> 32));
            if (k < cnt) {
                if (far_off) {
                    put(out, pw + mbcnt(mw), e);
                    if (side) k1 = min(k1, e.key); else k0 = min(k0, e.key);
                    c_keep++;
                } else if (pc + mbcnt(mc) < CAND) {
                    s_idx[pc + mbcnt(mc)] = (uint16_t)k;
                }
                c_ent++;
            }
            if (pc + (uint32_t)__popcll(mc) > CAND) add(k < cnt && !far_off && pc + mbcnt(mc) >= CAND, e);
        }
        if (refill) {
            for (uint32_t base = wave * 64; base < nfar; base += B) {
                uint4 x = make_uint4(0, 0, 0, 0);
                if (base + lane < nfar) x = spill[(uint64_t)(2 + far) * A.spcap + base + lane];
                c_ent += base + lane < nfar;
                c_keep += base + lane < nfar;
                add(base + lane < nfar, {x.x, x.y, x.z});
            }
        }
        if ((gen & 15u) == 0)
            for (uint32_t k = tid; k < TAB; k += B) s_tab[0][k] = s_tab[1][k] = INF64;
        __syncthreads();
        const uint32_t cand = min(uniform(s_hand[nxt].cand), CAND);
        if (refill && tid == 0) s_far[far] = {0, NO_KEY, NO_KEY, 0};
        // B candidates at a time
        for (uint32_t c0 = 0;; c0 += B) {
            // 2. Check and prune the candidates, and bid for the heads of their arcs.
            const unsigned long long tag = (unsigned long long)(15u - (gen & 15u)) << 60;
            // An even share for each wave, but 32 candidates (two steps of
            // arcs) before more than the four waves of the four SIMDs take
            // part: a wave costs its instructions however few its lanes. (An
            // even share alone, and of the bids below: 8 BiD-A* queries on
            // 1024^2 15.9 ms instead of 15.0, one query on a 256^2 grid 0.32
            // instead of 0.305.)
            const uint32_t batch = min(cand - c0, (uint32_t)B);
            const uint32_t share = max((batch + NW - 1) / NW, min(32u, (batch + 3) / 4));
            const uint32_t first = min(wave * share, batch), mine = min(share, batch - first), base = c0 + first;
            if (mine) {
                Entry e = {0, 0, 0};
                uint32_t rb = 0, deg = 0;
                if (lane < mine) {
                    e = get(in, s_idx[base + lane]);
                    const uint32_t u = e.v & ~SIDE_BIT;
                    const bool side = PAIR && (e.v & SIDE_BIT);
                    const uint2 row = load_at<uint2>((REV && side) ? A.in_row_ptr : A.row_ptr, 4u * u);
                    uint32_t own, oth = INF32;
                    if (PAIR) {
                        const uint2 w = load_at<uint2>(D, 8u * u);
                        own = side ? w.y : w.x;
                        oth = side ? w.x : w.y;
                    } else {
                        own = load_at<uint32_t>(D, 4u * u);
                    }
                    uint32_t r0 = row.x, r1 = row.y;
                    PPSP_TOGETHER(r0, own);                // both loads before the first use of either
                    if (own >= e.d) {                      // else lowered since: a fresher entry exists
                        meet(e.d, oth, u);
                        if (e.key < bnd) {                 // Prune
                            rb = r0;
                            deg = r1 - r0;
                            c_sv++;
                            c_se += deg;
                        }
                    }
                }
                const uint32_t end = wave_scan(deg), off = end - deg;
                const uint32_t total = uniform((uint32_t)__builtin_amdgcn_readlane((int)end, 63));
                if (deg) s_ext[wave * 64 + lane] = make_uint4(e.v, e.d, rb - off, base + lane);
                for (uint32_t w0 = 0; w0 < total; w0 += 64 * RES_WAYS) {
                    for (uint32_t j = max(off, w0); j < min(end, w0 + 64 * RES_WAYS); j++)
                        s_owner[wave][j - w0] = (uint8_t)lane;
                    wave_lds_sync();
                    uint32_t from[RES_WAYS], sb[RES_WAYS], du[RES_WAYS];
                    uint2 arc[RES_WAYS];
#pragma unroll
                    for (int k = 0; k < RES_WAYS; k++) {
                        arc[k] = make_uint2(0, 0);
                        from[k] = sb[k] = du[k] = 0;
                        if (w0 + 64 * k + lane < total) {
                            const uint4 x = s_ext[wave * 64 + s_owner[wave][64 * k + lane]];
                            sb[k] = x.x & SIDE_BIT;
                            du[k] = x.y;
                            from[k] = x.w;
                            arc[k] = load_at<uint2>((REV && sb[k]) ? A.in_arcs : A.arcs, 8u * (x.z + (w0 + 64 * k + lane)));
                        }
                    }
                    uint32_t own[RES_WAYS], oth[RES_WAYS], over = 0;
#pragma unroll
                    for (int k = 0; k < RES_WAYS; k++) {
                        own[k] = 0;
                        oth[k] = INF32;
                        if (w0 + 64 * k + lane < total) {
                            // possibly stale: never below the truth
                            if (PAIR) {
                                const uint2 w = load_at<uint2>(D, 8u * arc[k].x);
                                own[k] = sb[k] ? w.y : w.x;
                                oth[k] = sb[k] ? w.x : w.y;
                            } else {
                                own[k] = load_at<uint32_t>(D, 4u * arc[k].x);
                            }
                        }
                    }
                    uint64_t low[RES_WAYS];
                    uint32_t nlow = 0;
#pragma unroll
                    for (int k = 0; k < RES_WAYS; k++) {
                        const uint32_t c = du[k] + arc[k].y;
                        if (w0 + 64 * k + lane < total) over |= (uint32_t)(c < du[k]) | (uint32_t)(c == INF32);
                        low[k] = __ballot(c >= du[k] && c < own[k]);
                        nlow += (uint32_t)__popcll(low[k]);
                        du[k] = c;
                    }
                    if (over) s_err = 1;                   // past 32 bits
                    if (nlow == 0) continue;
                    uint32_t pos = 0;
                    if (lane == 0) pos = atomicAdd(&s_nbid, nlow);
                    pos = uniform(pos);
                    const bool full = pos + nlow > BIDS;
#pragma unroll
                    for (int k = 0; k < RES_WAYS; k++) {
                        const uint32_t at = pos + mbcnt(low[k]);
                        if ((low[k] >> lane & 1) && at < BIDS) {
                            const uint32_t v = arc[k].x | sb[k];
                            s_bid[at] = make_uint4(v, du[k], oth[k], from[k]);
                            const unsigned long long b = tag | (unsigned long long)du[k] << 28 | (v >> 4 & 0x8000000u) | arc[k].x;
                            atomicMin(&s_tab[0][(v ^ v >> 20) & (TAB - 1)], b);
                            atomicMin(&s_tab[1][(v * 2654435761u) >> 16 & (TAB - 1)], b);
                        }
                        // no room for a bid: its candidate runs again in the next round
                        if (full) {
                            bool left = (low[k] >> lane & 1) && at >= BIDS;
                            const uint64_t before = __ballot(left) & ((1ull << lane) - 1);
                            const uint32_t last = __shfl(from[k], before ? 63 - __clzll((long long)before) : 0, 64);
                            left = left && (!before || last != from[k]);   // once for its arcs of this step
                            Entry e2 = {0, 0, 0};
                            if (left) e2 = get(in, s_idx[from[k]]);
                            add(left, e2);
                        }
                        pos += (uint32_t)__popcll(low[k]);
                    }
                }
            }
            __syncthreads();
            const uint32_t nbid = min(uniform(s_nbid), BIDS);
            // 3. The smallest bid of a vertex is its new distance.
            for (uint32_t b0 = wave * 64; b0 < nbid; b0 += B) {
                Entry e = {0, 0, 0};
                bool app = false, again = false;
                if (b0 + lane < nbid) {
                    const uint4 x = s_bid[b0 + lane];
                    const uint32_t v = x.x & ~SIDE_BIT;
                    const unsigned long long b = tag | (unsigned long long)x.y << 28 | (x.x >> 4 & 0x8000000u) | v;
                    // a slot speaks for the vertex it holds; where neither holds this one, the bid is made again
                    const unsigned long long own_bits = 0xF00000000FFFFFFFull;
                    unsigned long long *slot = &s_tab[0][(x.x ^ x.x >> 20) & (TAB - 1)], w = *slot;
                    if ((w ^ b) & own_bits) {
                        slot = &s_tab[1][(x.x * 2654435761u) >> 16 & (TAB - 1)];
                        w = *slot;
                    }
                    again = ((w ^ b) & own_bits) != 0;
                    // equal bids: one of them takes the slot (its distance becomes infinity, which no bid has)
                    app = w == b && atomicCAS(slot, b, b | 0xFFFFFFFFull << 28) == b;
                    if (app) {
                        c_succ++;
                        meet(x.y, x.z, v);
                        *(uint32_t *)((char *)D + (PAIR ? 8u * v + (x.x & SIDE_BIT ? 4u : 0u) : 4u * v)) = x.y;
                        uint32_t key;
                        if (HEUR) {
                            const int32_t h = hterm(load_at<int2>(A.xy, 8u * v));
                            key = clamp(key_of(KIND, x.y, PAIR && (x.x & SIDE_BIT) ? -h : h));
                        } else {
                            key = dist_key(x.y);
                        }
                        e = {x.x, x.y, key};
                        app = key < bnd;                   // Prune before Add
                    }
                    if (again) e = get(in, s_idx[x.w]);
                }
                add(app || again, e);
            }
            gen++;
            if (c0 + B >= cand) break;
            // the next batch: its bids start from an empty list
            __syncthreads();
            if (tid == 0) s_nbid = 0;
            if ((gen & 15u) == 0)
                for (uint32_t k = tid; k < TAB; k += B) s_tab[0][k] = s_tab[1][k] = INF64;
            __syncthreads();
        }
        wave_min_to(&s_hand[nxt].mk0, k0);
        if (PAIR) wave_min_to(&s_hand[nxt].mk1, k1);
        if (HEUR) wave_min_to(&s_far[fout].mk0, f0);
        if (HEUR && PAIR) wave_min_to(&s_far[fout].mk1, f1);
        far = fout;
        const uint32_t z = cur;
        cur = nxt;
        nxt = rst;
        rst = z;
    }
    const unsigned long long v[5] = {wave_sum(c_ent), wave_sum(c_sv), wave_sum(c_se), wave_sum(c_succ), wave_sum(c_keep)};
    if (lane == 0)
        for (int k = 0; k < 5; k++) atomicAdd(&s_stat[RS_ENTRIES + k], v[k]);
    __syncthreads();
    if (tid == 0) {
        s_stat[RS_ROUNDS] = r;
        s_stat[RS_STATUS] = status | (s_err ? (uint32_t)RES_OVERFLOW : 0u);
        if (has_pair) A.mu[part.pair] = mu;
    }
    __syncthreads();
    if (tid < (uint32_t)RS_N) A.qstat[(uint64_t)q * RS_N + tid] = s_stat[tid];
}

// ---- host-side launcher ----

template <bool PAIR, bool HEUR, bool REV>
static hipError_t launch_t(const ResidentArgs &A, int threads, hipStream_t st) {
    if (threads == 1024) k_resident<1024, PAIR, HEUR, REV><<<A.nquery, 1024, 0, st>>>(A);
    else k_resident<512, PAIR, HEUR, REV><<<A.nquery, 512, 0, st>>>(A);
    return hipGetLastError();
}

hipError_t launch_resident(const ResidentArgs &A, bool pair, bool heur, bool rev, int threads, hipStream_t st) {
    if (A.nquery == 0) return hipSuccess;
    if (pair) {
        if (rev) return heur ? launch_t<true, true, true>(A, threads, st) : launch_t<true, false, true>(A, threads, st);
        return heur ? launch_t<true, true, false>(A, threads, st) : launch_t<true, false, false>(A, threads, st);
    }
    return heur ? launch_t<false, true, false>(A, threads, st) : launch_t<false, false, false>(A, threads, st);
}

}  // namespace ppsp
