// Max/min selection with searches run ahead of their turn (included by
// bfs.hip, whose levels, barriers and keys it uses).
//
// The method's pivots follow one another: pivot t + 1 is the argmax of m, and
// m needs the pruned BFS of pivot t.  Run one by one, the selection is a chain
// of BFS levels (6,400 on a 100k-node geometric graph with k = 200) on a chip
// that is otherwise idle.  But the next few pivots can be foretold: they are
// the current largest values of m that lie far from one another.  So a round
// runs the searches of the coming pivot and of the foretold ones at once, one
// workgroup each, and only its longest search is waited for.
//
// Exactness does not rest on the guess.  A search from c that prunes by an
// older m (m only falls) visits a superset of the nodes the current m would
// admit, at their exact distances; its list of (node, distance) is applied to
// m only when the argmax names c, and min() drops the superfluous entries.  A
// wrong guess costs idle workgroups, never a pivot.
//
// Guessing: from the local maxima of m that reach 3/4 of the largest (2,400 of
// 860k nodes on a mesh), take greedily the largest min(m, bound on the
// distance to the candidates taken so far).  The bound is the largest
// |d(l, u) - d(l, v)| over the landmarks l = pivots 0, 1, 2, whose full rows
// more workgroups compute beside the first rounds.  On a 100k-node geometric
// graph, k = 200, 38 rounds remain, on a 150k-node mesh, k = 150, 25.  The
// guessing stops when it does not pay.
//
// Bound by the chain of levels of the first, hardly foretold pivots (35 of
// the 52 ms of searches on the 3.25M-node mesh).  Measured, against the
// searches one by one: 100k-node geometric graph, k = 200, 12.5 -> 8.4 ms;
// mesh of 150k nodes, k = 150, 18.2 -> 9.2 ms; 700k, k = 64, 46.7 -> 22.8; 3.25M,
// k = 100, 133 -> 78 ms.  8 workers: 4 and 16 took 5 to 20 % longer on the
// smaller graphs.  For which graphs and k: ahead_workers.
#pragma once

namespace ssm {

constexpr int kAheadMax = 16;      // workers at most
constexpr int kAheadWorkers = 8;   // by default
// Smallest graph: below, a round's overhead (about 40 us for the guess, 8 us
// per pivot) eats the levels saved: a 30k-node lattice, k = 60, 3.5 against
// 3.4 ms.
constexpr int kAheadMinN = 40000, kAheadMaxRow = 64;
// where the visited bits do not fit in LDS: the workers' workgroups, of one search at most, of a landmark's
constexpr int kAheadGroups = 32, kAheadGroupMax = 16, kAheadMarkGroup = 8;
constexpr int kXcds = 8;           // workgroups of a launch go to the XCDs in turn
constexpr int kAheadMarks = 3;     // landmarks: pivots 0, 1, 2
constexpr int kAheadRec = 8192;    // candidate records kept per round at most
constexpr int kAheadIds = 1024;    // of them from one workgroup's slice
constexpr int kAheadMarkBits = 20; // a landmark distance in a record (larger ones saturate)
// control words, a line apart: pivots decided, landmark rows complete (bits),
// records of the round, landmark rows this step may use, list
// lengths; per group its level counters and its barrier
constexpr int kAcKnown = 0, kAcReady = 32, kAcRec = 64, kAcMask = 96, kAcLen = 128, kAcGrp = 160,
              kAcInts = kAcGrp + 32 * (kAheadMax + kAheadMarks);
constexpr int kAcOver = 1 << 30;  // kAcKnown once the selection has ended

__host__ __device__ constexpr int ahead_pass(int state) { return state == kRsStamps ? 8 : 2; }
__host__ __device__ constexpr int ahead_block(int state) { return state == kRsStamps ? 512 : kBfsBlock; }

// The same search by a group of G workgroups, for graphs whose visited bits do
// not fit in LDS: the levels of k_select_grid, with the list itself as the
// queue.  stamp[u] is lowered to base + distance by an agent-scope minimum; a
// group's searches use falling bases (a span above any distance apart), so a
// value above base + distance belongs to an older search, or to none, and
// nothing is cleared between searches.  cnt: three counters that the levels
// use in turn for the nodes they append, 0 on entry, with the source in place
// and stamped.  bar: the group's barrier; beat: the counter of sync_search that
// the other workgroups wait at.  Returns the number of nodes found, or -1 when a
// barrier was aborted.
template <int W, bool FULL>
__device__ __forceinline__ int ahead_search_grp(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                const int* __restrict__ ell, int G, int member, int* stamp, int base,
                                                const int* m, unsigned long long* list, int* cnt,
                                                unsigned long long* bar, unsigned long long& epoch,
                                                unsigned long long* beat) {
    constexpr int VW = W / 4;
    const int gt = member * (int)blockDim.x + (int)threadIdx.x, sub = gt % VW, grp = gt / VW,
              ngrp = G * (int)blockDim.x / VW;
    int at = 0, next = 1;
    for (int dv = 1; next > at; ++dv) {
        int* tail = &cnt[dv % 3];
        if (gt == 0) {
            store_agent(&cnt[(dv + 1) % 3], 0);  // last read two levels ago
            if (dv % kBeatLevels == 0) atomicAdd(beat, kBeat);
        }
        auto take = [&](const int (&u)[4]) {
            int old[4], mv[4];
            bool ok[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                ok[j] = (unsigned)u[j] < (unsigned)n;
                mv[j] = !FULL && ok[j] ? load_agent(&m[u[j]]) : kInf;
                old[j] = ok[j] ? atomicMin(&stamp[u[j]], base + dv) : 0;
            }
            uint64_t mk[4];
            int tot = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                ok[j] = ok[j] && old[j] > base + dv && mv[j] > dv;
                mk[j] = __ballot(ok[j]);
                tot += __popcll(mk[j]);
            }
            if (tot == 0) return;
            int slot = 0;
            if (lane_id() == 0) slot = atomicAdd(tail, tot);
            slot = next + __builtin_amdgcn_readfirstlane(slot);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (ok[j])
                    store_agent(&list[slot + mask_rank(mk[j])],
                                (unsigned long long)(unsigned)u[j] | ((unsigned long long)(unsigned)dv << 32));
                slot += __popcll(mk[j]);
            }
        };
        const int len = next - at;
        for (int b0 = 0; b0 < len; b0 += ngrp) {  // uniform
            const int qi = b0 + grp;
            const int v = qi < len ? (int)(unsigned)__hip_atomic_load(&list[at + qi], __ATOMIC_RELAXED,
                                                                      __HIP_MEMORY_SCOPE_AGENT)
                                   : -1;
            int4 nb = make_int4(-1, -1, -1, -1);
            if ((unsigned)v < (unsigned)n) nb = *(const int4*)(ell + (size_t)v * W + 4 * sub);
            const int u[4] = {nb.x, nb.y, nb.z, nb.w};
            take(u);
            // a row longer than W: its lanes walk the CSR tail
            const bool more = __shfl(nb.w, (lane_id() / VW) * VW + VW - 1) == kEllMore;
            if (__ballot(more) != 0) {  // uniform per wave
                int e = 0, e1 = 0;
                if (more) {
                    e = rp[v] + W - 1 + sub;
                    e1 = rp[v + 1];
                }
                while (__ballot(e < e1) != 0) {
                    int t[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) t[j] = e + j * VW < e1 ? ci[e + j * VW] : -1;
                    take(t);
                    e += 4 * VW;
                }
            }
        }
        if (!sync_count(bar, epoch, G)) return -1;
        at = next;
        next = min(next + load_agent(tail), n);
    }
    return next;
}

// Workers 0 .. S-1 search; two more compute the full rows
// of pivots 1 and 2 (landmarks) as soon as those are known and leave.  Every
// workgroup follows the same decisions (pivots, candidates, their workers)
// from data that all of them read after the same barrier; only worker w
// searches from candidate slot w.  Per pivot: its list lowers m (each
// workgroup a share; with state bytes every workgroup also applies the whole
// list to its own bytes), a barrier (values below 127 come from the own bytes
// and need none), each workgroup's argmax over its slice of the nodes, a
// barrier.  The last pivot needs no search.  m, the lists, the rows and the
// records pass between workgroups by agent-scope accesses alone, as sync_search
// requires.  t0 = 0: from pivot `first` with m = infinity; t0 = 1: pivots 0
// and 1 are known and m holds pivot 0's distances.  After pivot 0 the form
// goes on alone only where it pays (status[1] = 0): a mean frontier
// n / (eccentricity + 1) of at most max_front, else it leaves with pivot 1
// known, m current and status[1] = 1; a frontier twice as wide ends it during
// pivot 0's search, with nothing changed and status[1] = 2.
//
// One workgroup per worker: all of them on XCD 0 (workgroups go to the XCDs in
// turn, the others leave at once), so that the rows one search read are in the
// L2 of the next (5 % on a 150k-node mesh).  With groups (kRsStamps) the
// kAheadGroups workgroups divide evenly over a round's searches (the early
// ones, wide and not foretold, get kAheadGroupMax), and the pivot's own search
// lowers m itself, as k_select_grid does.  The searches beside it then see m
// falling, which keeps them exact: a node whose distance lies below the m that
// this pivot leaves is never pruned, nor is any node on its shortest paths;
// whatever else they list, at its distance or above, min() drops.
template <int W, int STATE>
__global__ __launch_bounds__(ahead_block(STATE)) void k_select_ahead(
    int n, const int* __restrict__ rp, const int* __restrict__ ci, const int* __restrict__ ell, int t0, int k,
    int first, int* pivots, int* m, unsigned long long* lists, int* gq, int* marks, unsigned long long* rec, int* ctl,
    unsigned long long* keys, int* status, unsigned long long* bar, int S, int max_front, int span, int polls) {
    constexpr int kBlk = ahead_block(STATE);
    constexpr int R = 8;            // records per thread
    constexpr int kRec = R * kBlk;  // records kept per round
    __shared__ __align__(16) unsigned char pool[STATE == kRsStamps ? 4 * ((ahead_pass(STATE) + 1) * kBlk + kAheadIds) : kSelPool];
    __shared__ unsigned long long s_red[kBlk / kWave];
    __shared__ int s_cid[kAheadMax], s_clen[kAheadMax];  // per worker: the candidate searched, its list's length
    __shared__ int s_cand[kAheadMax];
    __shared__ int s_new, s_n, s_base, s_c[kAheadMarks + 1];
    __shared__ unsigned long long s_key;
    __shared__ int s_runs[kAheadMax];  // searches run from each slot (groups)
    int* lheavy = (int*)pool;
    unsigned* bits = (unsigned*)(lheavy + kHeavyCap);
    unsigned char* m8 = (unsigned char*)bits;
    // the visited set's bytes, then the queue (the rest of the pool, at least 4096 ints)
    const int set_bytes = STATE == kRsStamps ? 0 : STATE == kRsBytes ? (n + 15) & ~15 : ((n + 31) / 32 * 4 + 15) & ~15;
    int* lq = STATE == kRsStamps ? (int*)pool : (int*)((unsigned char*)bits + set_bytes);
    const int cap = (kSelPool - 4 * kHeavyCap - set_bytes) / 4;
    const int tid = threadIdx.x;
    // NB workgroups are the workers', b is this one's rank; then come the landmarks'
    constexpr bool kGroups = STATE == kRsStamps;
    if (!kGroups && blockIdx.x % kXcds != 0) return;
    const int b = kGroups ? blockIdx.x : blockIdx.x / kXcds, NB = kGroups ? kAheadGroups : S;
    const bool lead = b == 0 && tid == 0;
    int* myq = gq + (size_t)b * 2 * n;  // not with groups
    // group q's level counters and barrier
    auto gcnt = [&](int q) { return ctl + kAcGrp + 32 * q; };
    auto gbar = [&](int q) { return (unsigned long long*)(ctl + kAcGrp + 32 * q + 16); };
    unsigned long long gepoch = 0;

    if (b >= NB) {  // a landmark's full row
        constexpr int GL = kGroups ? kAheadMarkGroup : 1;
        const int f = (b - NB) / GL + 1, member = (b - NB) % GL;
        if (f >= kAheadMarks) return;
        if (tid == 0) {
            int known = 0;
            for (long long polls = 0; polls < kBarPolls && known <= f; ++polls) {
                known = load_agent(&ctl[kAcKnown]);
                __builtin_amdgcn_s_sleep(8);
            }
            s_n = known > f && known < kAcOver ? load_agent(&pivots[f]) : -1;
        }
        __syncthreads();
        const int src = s_n;
        if (src < 0) return;
        int* row = marks + (size_t)f * n;
        if constexpr (STATE == kRsStamps) {  // the row is its own stamps, infinite on entry
            unsigned long long* list = lists + (size_t)(S + f - 1) * n;
            if (member == 0 && tid == 0) {
                store_agent(&row[src], 0);
                store_agent(&list[0], (unsigned long long)(unsigned)src);
            }
            unsigned long long* bf = gbar(kAheadMax + f);
            if (!sync_count(bf, gepoch, GL)) return;
            if (ahead_search_grp<W, true>(n, rp, ci, ell, GL, member, row, 0, m, list, gcnt(kAheadMax + f), bf, gepoch,
                                          bar) < 0)
                return;
        } else {
            ring_search<W, kRsFull>(n, rp, ci, ell, src, lq, cap, lheavy, bits, m, RowSink{row}, myq);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
        }
        if (member == 0 && tid == 0) atomicOr(&ctl[kAcReady], 1 << f);
        return;
    }
    unsigned epoch = 0;
#define SYNC_OR_LEAVE()                               \
    do {                                              \
        if (!sync_search(bar, epoch, NB, polls)) {    \
            if (lead) {                               \
                store_agent(&status[2], 1);           \
                store_agent(&ctl[kAcKnown], kAcOver); \
            }                                         \
            return;                                   \
        }                                             \
    } while (0)
    const int per = ((n + NB - 1) / NB + 15) & ~15;  // this workgroup's slice of the nodes
    const int lo = (int)min((long long)n, (long long)b * per), hi = min(n, lo + per);
    // value of node i from this worker's state
    auto value = [&](int i) {
        if (STATE == kRsBytes) {
            const int b = m8[i] & 0x7f;
            if (b < kM7Sat) return b;
        }
        return load_agent(&m[i]);
    };
    if (tid < kAheadMax) {
        s_cid[tid] = -1;
        s_runs[tid] = 0;
    }
    if (STATE == kRsBytes)
        for (int i = tid; i < ((n + 15) & ~15); i += blockDim.x) m8[i] = i < n ? (unsigned char)kM7Sat : 0;
    int p = t0 == 0 ? first : load_agent(&pivots[1]);
    int top = kInf;  // m[p]
    int mask = 0;    // landmark rows that may be used
    if (t0 == 1) {
        top = load_agent(&m[p]);
        for (int i = lo + tid; i < hi; i += blockDim.x) store_agent(&marks[i], load_agent(&m[i]));
        if (lead) atomicOr(&ctl[kAcReady], 1);
        mask = 1;
        SYNC_OR_LEAVE();
    }
    __syncthreads();
    int rounds = 0, hits = 0;
    bool ahead = S > 1;
    for (int t = t0; t < k; ++t) {
        if (lead) {
            if (t0 == 0 || t > 1) store_agent(&pivots[t], p);
            __builtin_amdgcn_s_waitcnt(0);  // the pivot is visible before its count
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            store_agent(&ctl[kAcKnown], t + 1);
        }
        if (t + 1 >= k && t != 0) break;
        int slot = -1;
        for (int q = 0; q < S; ++q)
            if (s_cid[q] == p) slot = q;
        const bool direct = slot < 0;  // searched in its turn
        if (slot >= 0) {
            ++hits;
        } else {  // a new round
            int nc = 1;
            if (ahead && t > 0 && t + 2 < k) {
                // records of the local maxima of m (of a level stretch its
                // lowest ids; over the padded row) with
                // m >= theta, each workgroup its slice
                const int theta = max(1, (int)((long long)top * 3 / 4));
                if (tid == 0) s_n = 0;
                __syncthreads();
                // kPass nodes per thread and pass; those with m >= theta wait
                // in lq until a workgroup's worth of rows can be read at once
                constexpr int kPass = ahead_pass(STATE), kWait = (kPass + 1) * kBlk;  // lq: waiting ids, the maxima's
                int waiting = 0;
                for (int i1 = lo; i1 < hi || waiting > 0;) {  // uniform
                    if (i1 < hi && waiting < kBlk) {  // leaves at most kWait - 1 waiting
                        if (tid == 0) s_base = waiting;
                        __syncthreads();
                        int mv[kPass];
#pragma unroll
                        for (int j = 0; j < kPass; ++j) {
                            const int i = i1 + j * kBlk + tid;
                            mv[j] = i < hi ? value(i) : -1;
                        }
#pragma unroll
                        for (int j = 0; j < kPass; ++j)
                            if (mv[j] >= theta) lq[atomicAdd(&s_base, 1)] = i1 + j * kBlk + tid;
                        i1 += kPass * kBlk;
                        __syncthreads();
                        waiting = s_base;
                        __syncthreads();
                        if (waiting < kBlk && i1 < hi) continue;
                    }
                    const int take = min(waiting, kBlk);
                    waiting -= take;
                    if (tid < take) {
                        const int v = lq[waiting + tid], mv = value(v);
                        const int4* row = (const int4*)(ell + (size_t)v * W);
                        int4 nb[W / 4];
#pragma unroll
                        for (int a = 0; a < W / 4; ++a) nb[a] = row[a];
                        bool best = true;  // no neighbour larger, nor equal with a lower id
#pragma unroll
                        for (int a = 0; a < W / 4; ++a) {
                            const int u[4] = {nb[a].x, nb[a].y, nb[a].z, nb[a].w};
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const int x = (unsigned)u[j] < (unsigned)n ? u[j] : v, mx = value(x);
                                best = best && (mx < mv || (mx == mv && x >= v));
                            }
                        }
                        if (best) {
                            const int at = atomicAdd(&s_n, 1);
                            if (at < kAheadIds) lq[kWait + at] = v;
                        }
                    }
                    __syncthreads();
                }
                __syncthreads();
                const int found = s_n, mine = min(found, kAheadIds);
                if (tid == 0) s_base = atomicAdd(&ctl[kAcRec], mine);  // slots for exactly the records written below
                __syncthreads();
                const int base = s_base;
                for (int q = tid; q < mine && base + q < kRec; q += blockDim.x) {
                    const int v = lq[kWait + q];
                    unsigned long long l[kAheadMarks];
#pragma unroll
                    for (int a = 0; a < kAheadMarks; ++a)
                        l[a] = mask >> a & 1
                                   ? (unsigned)min(load_agent(&marks[(size_t)a * n + v]), (1 << kAheadMarkBits) - 1)
                                   : 0u;
                    store_agent(&rec[2 * (base + q)],
                                (unsigned long long)(unsigned)v | ((unsigned long long)(unsigned)value(v) << 32));
                    store_agent(&rec[2 * (base + q) + 1],
                                l[0] | (l[1] << kAheadMarkBits) | (l[2] << (2 * kAheadMarkBits)));
                }
                SYNC_OR_LEAVE();
                const int have = min(load_agent(&ctl[kAcRec]), kRec);
                int rv[R], rm[R], ra[R], rb[R], rc[R];
                constexpr unsigned kMk = (1u << kAheadMarkBits) - 1;
                if (tid == 0) s_c[0] = -1;
                __syncthreads();
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const int at = tid + q * kBlk;
                    rm[q] = -1;
                    rv[q] = ra[q] = rb[q] = rc[q] = 0;
                    if (at < have) {
                        const unsigned long long a =
                            __hip_atomic_load(&rec[2 * at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const unsigned long long b =
                            __hip_atomic_load(&rec[2 * at + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        rv[q] = (int)(unsigned)a;
                        rm[q] = (int)(unsigned)(a >> 32);
                        ra[q] = (int)((unsigned)b & kMk);
                        rb[q] = (int)((unsigned)(b >> kAheadMarkBits) & kMk);
                        rc[q] = (int)((unsigned)(b >> (2 * kAheadMarkBits)) & kMk);
                        if (rv[q] == p) {
                            s_c[0] = p;
                            s_c[1] = ra[q];
                            s_c[2] = rb[q];
                            s_c[3] = rc[q];
                        }
                    }
                }
                __syncthreads();
                const int most = min(S, k - 1 - t);
                bool go = s_c[0] == p;
                while (go && nc < most) {  // uniform
                    const int ca = s_c[1], cb = s_c[2], cc = s_c[3];
                    unsigned long long best = 0;
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int lb = max(abs(ra[q] - ca), max(abs(rb[q] - cb), abs(rc[q] - cc)));
                        rm[q] = min(rm[q], lb);
                        if (rm[q] >= 0) best = key_max(best, argmax_key(rm[q], rv[q]));
                    }
                    best = block_max(best, s_red);
                    const int bm = (int)(best >> 32), bv = (int)(0xffffffffu - (unsigned)(best & 0xffffffffu));
                    go = bm >= theta;  // below, a node without a record may be larger
                    if (go) {
                        if (tid == 0) s_cand[nc] = bv;
                        ++nc;
#pragma unroll
                        for (int q = 0; q < R; ++q)
                            if (rm[q] == bm && rv[q] == bv) {
                                s_c[1] = ra[q];
                                s_c[2] = rb[q];
                                s_c[3] = rc[q];
                            }
                        __syncthreads();
                    }
                }
                if (nc > 1) ++rounds;
                if (rounds >= 8 && 2 * hits < rounds) ahead = false;  // the graph's pivots are not foretold
            }
            __syncthreads();
            if (tid == 0) {  // workers for the candidates without a search: idle ones first
                s_cand[0] = p;
                int keep = 0, fresh = 0;
                for (int j = 0; j < nc; ++j)
                    for (int q = 0; q < S; ++q)
                        if (s_cid[q] == s_cand[j]) {
                            keep |= 1 << q;
                            s_cand[j] = -1;
                        }
                for (int j = 0; j < nc; ++j) {
                    if (s_cand[j] < 0) continue;
                    int at = -1;
                    for (int q = S - 1; q >= 0; --q)
                        if (!(keep >> q & 1) && (at < 0 || s_cid[q] < 0 || s_cid[at] >= 0)) at = q;
                    keep |= 1 << at;
                    fresh |= 1 << at;
                    s_cid[at] = s_cand[j];
                }
                s_new = fresh;
            }
            __syncthreads();
            const int fresh = s_new;
            if constexpr (kGroups) {
                // the workgroups divided evenly over the searches
                const int nf = __popc(fresh);
                int gsize = min(NB, kAheadGroupMax);
                while (gsize * nf > NB) gsize /= 2;
                int q = -1, left = b / gsize;  // this workgroup's search: the left-th fresh slot
                for (int a = 0; a < S; ++a)
                    if ((fresh >> a & 1) && left-- == 0) q = a;
                if (q >= 0) {
                    const int src = s_cid[q], member = b % gsize, base = 0x7fffffff - (s_runs[q] + 1) * span;
                    int* stamp = gq + (size_t)q * n;
                    unsigned long long* list = lists + (size_t)q * n;
                    gepoch = 0;  // the barrier was cleared after its last search
                    if (member == 0 && tid == 0) {
                        if (src == p)
                            store_agent(&m[src], 0);
                        else
                            store_agent(&stamp[src], base);
                        store_agent(&list[0], (unsigned long long)(unsigned)src);
                        for (int a = 0; a < 3; ++a) store_agent(&gcnt(q)[a], 0);
                    }
                    int len = -1;
                    if (sync_count(gbar(q), gepoch, gsize))
                        len = src == p ? ahead_search_grp<W, true>(n, rp, ci, ell, gsize, member, m, 0, m, list,
                                                                   gcnt(q), gbar(q), gepoch, bar)
                                       : ahead_search_grp<W, false>(n, rp, ci, ell, gsize, member, stamp, base, m,
                                                                    list, gcnt(q), gbar(q), gepoch, bar);
                    if (len < 0) {  // aborted
                        if (tid == 0) {
                            store_agent(&status[2], 1);
                            store_agent(&ctl[kAcKnown], kAcOver);
                        }
                        return;
                    }
                    if (member == 0 && tid == 0) store_agent(&ctl[kAcLen + q], len);
                }
                __syncthreads();
                if (tid < S && (fresh >> tid & 1)) ++s_runs[tid];
            } else if (fresh >> b & 1) {
                const int len = ring_search<W, STATE>(n, rp, ci, ell, s_cid[b], lq, cap, lheavy, bits, m,
                                                       ListSink{lists + (size_t)b * n}, myq,
                                                       t == 0 && max_front < INT_MAX / 2 ? 2 * max_front : INT_MAX,
                                                       nullptr, Pages(), nullptr, bar);
                if (tid == 0) store_agent(&ctl[kAcLen + b], len);
            }
            SYNC_OR_LEAVE();
            if (lead) store_agent(&ctl[kAcRec], 0);  // read by all before this round's searches
            if (kGroups && b == 0 && tid < S) store_agent(gbar(tid), 0ull);  // for the next round's groups
            if (tid < S && (fresh >> tid & 1)) s_clen[tid] = load_agent(&ctl[kAcLen + tid]);
            __syncthreads();
            for (int q = 0; q < S; ++q)
                if (s_cid[q] == p) slot = q;
        }
        const int len = min(s_clen[slot], n);
        __syncthreads();
        if (len < 0) {  // a frontier too wide to go on (t = 0, uniform)
            if (lead) store_agent(&status[1], 2);
            break;
        }
        if (tid == 0) s_cid[slot] = -1;
        if (t == 0 && len < n) {  // disconnected (uniform)
            if (lead) {
                store_agent(&status[0], 1);
                store_agent(&ctl[kAcKnown], kAcOver);
            }
            return;
        }
        // the list lowers m
        const unsigned long long* list = lists + (size_t)slot * n;
        auto lower = [&](unsigned long long e, bool share) {
            const int v = (int)(unsigned)e, d = (int)(unsigned)(e >> 32);
            if (share) {
                atomicMin(&m[v], d);
                if (t == 0) store_agent(&marks[v], d);
            }
            if (STATE == kRsBytes) {
                const int b = m8[v];
                if (d < b) m8[v] = (unsigned char)d;  // d < 127 here
            }
        };
        if (STATE == kRsBytes) {
            for (int q0 = tid; q0 < len; q0 += 4 * kBlk) {
                unsigned long long e[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    e[j] = __hip_atomic_load(&list[min(q0 + j * kBlk, len - 1)], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (q0 + j * kBlk < len) lower(e[j], (q0 / kBlk + j) % S == b);
            }
        } else {
            // with groups a search that was not ahead has lowered m itself
            for (int q = b * kBlk + tid; q < (kGroups && direct ? 0 : len); q += NB * kBlk)
                lower(__hip_atomic_load(&list[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), true);
        }
        if (t == 0 && lead) atomicOr(&ctl[kAcReady], 1);  // complete at the barrier, used after it
        // state bytes are this worker's own; only values of 127 and above are read from the shared m
        if (STATE != kRsBytes || top >= kM7Sat)
            SYNC_OR_LEAVE();
        else
            __syncthreads();
        // argmax of m, each worker over its slice
        unsigned long long best = 0;
        if (STATE == kRsBytes) {
            const uint4* w16 = (const uint4*)(m8 + lo);
            int bv = -1, bi = 0;
            for (int q = tid; q < (hi - lo + 15) / 16; q += blockDim.x) {
                const uint4 x = w16[q];
                const unsigned part[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                for (int a = 0; a < 4; ++a) {
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const int val = (int)((part[a] >> (8 * b)) & 127u);
                        if (val > bv) {  // bytes past n are 0
                            bv = val;
                            bi = lo + 16 * q + 4 * a + b;
                        }
                    }
                }
            }
            if (bv >= 0) best = argmax_key(bv, bi);
            best = block_max(best, s_red);
            if ((int)(best >> 32) >= kM7Sat) {  // uniform: the saturated nodes' values are in m
                unsigned long long b2 = 0;
                for (int i = lo + tid; i < hi; i += blockDim.x)
                    if ((m8[i] & 0x7f) >= kM7Sat) b2 = key_max(b2, argmax_key(load_agent(&m[i]), i));
                best = block_max(b2, s_red);
            }
        } else {
            for (int i0 = lo + 4 * tid; i0 < hi; i0 += 4 * 4 * blockDim.x) {
                int4 q[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i = i0 + 4 * j * (int)blockDim.x;
                    q[j] = i + 4 <= hi ? load_agent4(m + i) : make_int4(-1, -1, -1, -1);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int i = i0 + 4 * j * (int)blockDim.x;
                    if (q[j].x >= 0) best = key_max(best, argmax_key(q[j].x, i));
                    if (q[j].y >= 0) best = key_max(best, argmax_key(q[j].y, i + 1));
                    if (q[j].z >= 0) best = key_max(best, argmax_key(q[j].z, i + 2));
                    if (q[j].w >= 0) best = key_max(best, argmax_key(q[j].w, i + 3));
                }
            }
            for (int i = lo + (hi - lo) / 4 * 4 + tid; i < hi; i += blockDim.x)
                best = key_max(best, argmax_key(load_agent(&m[i]), i));
            best = block_max(best, s_red);
        }
        if (tid == 0) {
            store_agent(&keys[b], best);
            if (b == 0) store_agent(&ctl[kAcMask], load_agent(&ctl[kAcReady]));
        }
        SYNC_OR_LEAVE();
        if (tid < kWave) {
            const unsigned long long b = keys_max(keys, NB);
            if (tid == 0) {
                s_key = b;
                s_n = load_agent(&ctl[kAcMask]);
            }
        }
        __syncthreads();
        top = (int)(s_key >> 32);
        p = (int)(0xffffffffu - (unsigned)(s_key & 0xffffffffu));
        mask = s_n;
        __syncthreads();
        if (t == 0 && k > 2 && n / (top + 1) > max_front) {  // uniform
            if (lead) {
                store_agent(&pivots[1], p);
                store_agent(&status[1], 1);
            }
            break;
        }
    }
#undef SYNC_OR_LEAVE
    if (lead) store_agent(&ctl[kAcKnown], kAcOver);
}

}  // namespace ssm
