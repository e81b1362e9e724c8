// Level-synchronous searches of one workgroup whose queue is the list of the
// nodes found (included by bfs.hip, whose padded-row levels it uses): the
// selection's pruned searches (select_ahead.h) and the BFS rows of large
// graphs.
#pragma once

namespace ssm {

// How a search holds its visited set and reads m: a state byte per node in LDS
// (bits 0-6 min(m, 127), bit 7 visited), LDS visited bits and global m,
// visited bits alone (a landmark's full search, a BFS row); where the bits do
// not fit in LDS, a stamped distance per node in memory (ahead_search_grp), or,
// for a BFS row, the visited bits of the pages of ids that the search is in.
enum RingState { kRsBytes = 0, kRsBits = 1, kRsFull = 2, kRsStamps = 3, kRsPaged = 4 };

// Paged visited bits.  A neighbour of level l lies on level l - 1, l or l + 1,
// so the bits of the levels l - 1 and l and of the nodes claimed for l + 1
// decide as the whole set would, and only the pages (128 ids) that those
// nodes lie in need bits.  A table of 16-bit entries names each page's bits in
// a pool (0: none yet).  When the pool runs short, all of it is cleared and
// the last two levels are put back.  A 3.25M-node mesh numbered by rows has up
// to 4,000 pages in use and gains about 30 per level.  A search whose
// last two levels alone fill the pool (wide levels, or a numbering that spreads
// them) or whose next level finds it empty (the pool's second counter) is left
// at its last complete level, the others of the launch soon after, and k_bfs_grp
// takes the rows up from there.
constexpr int kPagedBytes = 133120;  // table, pool and two counters: pages taken, pages refused
constexpr int kPagesSpare = 512;     // pages kept free when a level starts
constexpr int kPageShift = 7;        // log2 ids per page
// Nodes whose page table is at most 53,248 bytes.  Larger graphs would need pages
// of 256 ids, too few for their levels: 100 rows of a 6M-node lattice took 63.6 ms
// with them, on two workgroups each 61.8.
constexpr int kPagedMaxN = 3407488;

struct Pages {
    int tab, count;  // table words, pages in the pool
    // `most` (tuning) takes fewer pages than fit.
    __host__ explicit Pages(int n, int most = 65535)
        : tab(((n >> kPageShift) + 2) / 2), count(std::min((kPagedBytes / 4 - 2 - tab) >> (kPageShift - 5), most)) {}
    __device__ Pages() : tab(0), count(0) {}  // for the searches without pages
    __device__ __forceinline__ unsigned* pool(unsigned* set) const { return set + 2 + tab; }
    __device__ __forceinline__ unsigned short* table(unsigned* set) const { return (unsigned short*)(set + 2); }
    // The word of node u's bit in page e - 1 of the pool.
    __device__ __forceinline__ unsigned* word(unsigned* set, int u, unsigned e) const {
        return pool(set) + (((e - 1) << (kPageShift - 5)) + ((u & ((1 << kPageShift) - 1)) >> 5));
    }
    // Clears everything (call with the whole workgroup, barriers around).
    __device__ __forceinline__ void clear(unsigned* set) const {
        for (int w = threadIdx.x; w < kPagedBytes / 4; w += blockDim.x) set[w] = 0u;
    }
    // The page's entry after taking one from the pool (0: the pool is empty).
    __device__ __forceinline__ unsigned take(unsigned* set, int page) const {
        const unsigned mine = atomicAdd(&set[0], 1u) + 1u;
        if (mine > (unsigned)count) {
            set[1] = 1u;
            return 0;
        }
        unsigned* word = set + 2 + page / 2;
        const int sh = 16 * (page & 1);
        unsigned w = *word;
        for (;;) {  // ends: every failed swap means that one of the two entries was set
            const unsigned e = (w >> sh) & 0xffffu;
            if (e) return e;  // another lane's; this one's page stays unused until the next clearing
            const unsigned was = atomicCAS(word, w, w | (mine << sh));
            if (was == w) return mine;
            w = was;
        }
    }
    // Marks node u, whose page has entry e: true if it was not marked (or has no page).
    __device__ __forceinline__ bool mark(unsigned* set, int u, unsigned e) const {
        if (e == 0) e = take(set, u >> kPageShift);
        if (e == 0) return false;
        const unsigned bit = 1u << (u & 31);
        return !(atomicOr(word(set, u, e), bit) & bit);
    }
};

// Where a search's nodes go besides the frontier: the list of (node,
// distance) pairs in order of discovery, or a full distance row.
struct ListSink {
    unsigned long long* p;
    __device__ __forceinline__ void put(int at, int u, int d) const {
        store_agent(&p[at], (unsigned long long)(unsigned)u | ((unsigned long long)(unsigned)d << 32));
    }
};
struct RowSink {  // read by other workgroups of the launch
    int* p;
    __device__ __forceinline__ void put(int, int u, int d) const { store_agent(&p[u], d); }
};
struct PlainRowSink {
    int* p;
    __device__ __forceinline__ void put(int, int u, int d) const { p[u] = d; }
};

// A search's queue: the nodes in order of discovery, in LDS up to `cap`
// entries (the rest in global memory).  A level's frontier is the stretch
// [at, at + its size), the next one is appended behind it, so the queue is
// also the list of the search's nodes: it goes to the sink in bulk (flush),
// not node by node.  On gfx950 a wave's wait for a load also waits for the
// stores it issued before, and a store that bypasses the caches takes as long
// as a level: stored at discovery, the list cost 14 us per pivot on a
// 100k-node geometric graph.
constexpr int kRingLevels = 128;  // levels between flushes at most
constexpr int kRingStopLooks = 16;  // flushes between looks at the other searches' call to stop
constexpr int kBeatLevels = 1024;   // levels between a search's signs of life
constexpr int kRingLeft = -2;       // ring_search: left at a complete level, to be taken up from there
constexpr int kRingPool = 155648;  // LDS of a search: long rows, visited set, queue

struct RingFrontier : Frontier {
    int cap, at, next;  // LDS entries; queue positions of the current and the next frontier
};

__device__ __forceinline__ int split(const RingFrontier& f) { return max(0, f.cap - f.at); }

__device__ __forceinline__ int ring_get(const RingFrontier& f, const int* q, int pos) {
    return pos < f.cap ? ((const __attribute__((address_space(3))) int*)q)[pos]
                       : ((const __attribute__((address_space(1))) int*)f.gnxt)[pos - f.cap];
}

__device__ __forceinline__ void ring_set(const RingFrontier& f, int* q, int pos, int u) {
    if (pos < f.cap)
        q[pos] = u;
    else
        f.gnxt[pos - f.cap] = u;
}

__device__ __forceinline__ void put(const RingFrontier& f, int slot, int u) {
    ring_set(f, f.lnxt, f.next + slot, u);
}

// Claims u[0..N) for distance dv; ok[j] is set where this lane claimed u[j]
// and m lies above dv.  m is only read: it changes between the rounds.
template <int STATE, int N>
__device__ __forceinline__ void ring_claim(const int (&u)[N], bool (&ok)[N], int n, unsigned* bits, const int* m,
                                            int dv, const Pages& pg) {
    if (STATE == kRsBytes) {
        unsigned char* m8 = (unsigned char*)bits;
        unsigned old[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            ok[j] = (unsigned)u[j] < (unsigned)n;  // padding, continuation mark
            old[j] = ok[j] ? atomicOr((unsigned*)(m8 + (u[j] & ~3)), 0x80u << (8 * (u[j] & 3))) : 0u;
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const unsigned ob = (old[j] >> (8 * (u[j] & 3))) & 0xffu;
            int mv = (int)(ob & 0x7fu);
            ok[j] = ok[j] && !(ob & 0x80u);
            if (dv < kM7Sat) {  // uniform; a saturated byte means m >= 127 > dv
                ok[j] = ok[j] && mv > dv;
            } else {
                if (ok[j] && mv >= kM7Sat) mv = load_agent(&m[u[j]]);
                ok[j] = ok[j] && mv > dv;
            }
        }
    } else if (STATE == kRsPaged) {
        unsigned e[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {  // the entries in flight together
            ok[j] = (unsigned)u[j] < (unsigned)n;
            e[j] = pg.table(bits)[ok[j] ? u[j] >> kPageShift : 0];
        }
        bool any = false;
#pragma unroll
        for (int j = 0; j < N; ++j) any = any || (ok[j] && e[j] == 0);
        if (any) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (ok[j] && e[j] == 0) {
                    e[j] = pg.table(bits)[u[j] >> kPageShift];
                    if (e[j] == 0) e[j] = pg.take(bits, u[j] >> kPageShift);
                    ok[j] = e[j] != 0;
                }
        }
        unsigned old[N];
#pragma unroll
        for (int j = 0; j < N; ++j)
            old[j] = ok[j] ? atomicOr(pg.word(bits, u[j], e[j]), 1u << (u[j] & 31)) : ~0u;
#pragma unroll
        for (int j = 0; j < N; ++j) ok[j] = ok[j] && !(old[j] & (1u << (u[j] & 31)));
    } else {
        int mv[N];
        if (STATE == kRsBits) {  // m in flight beside the claims
#pragma unroll
            for (int j = 0; j < N; ++j) mv[j] = (unsigned)u[j] < (unsigned)n ? load_agent(&m[u[j]]) : 0;
        }
        claim(u, ok, bits, n);
        if (STATE == kRsBits) {
#pragma unroll
            for (int j = 0; j < N; ++j) ok[j] = ok[j] && mv[j] > dv;
        }
    }
}

// wave_levels for this search: levels whose frontier one wave covers in
// one pass, in wave 0 alone, until the queue or the level starts ls want a
// flush.
template <int W, int STATE>
__device__ __forceinline__ int ring_wave_levels(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                 const int* __restrict__ ell, unsigned* bits, const int* m, int* q,
                                                 RingFrontier& f, int len, int d0, int* ls, int& nl, const Pages& pg) {
    constexpr int G = W / 4;
    const int lane = lane_id(), sub = lane % G;
    while (len > 0 && len <= wave_level_nodes<W>() && (STATE != kRsBytes || d0 + nl + 1 < kM7Sat) &&
           nl < kRingLevels && f.next <= f.cap / 2 &&
           (STATE != kRsPaged || (int)bits[0] <= pg.count - kPagesSpare)) {
        const int at = f.at + lane / G;  // below cap: the frontier ends at f.next
        const int v = lane / G < len ? q[at] : -1;
        int4 nb = make_int4(-1, -1, -1, -1);
        if ((unsigned)v < (unsigned)n) nb = *(const int4*)(ell + (size_t)v * W + 4 * sub);
        const int dv = d0 + nl + 1;
        int cnt = 0;
        const int u[4] = {nb.x, nb.y, nb.z, nb.w};
        bool ok[4];
        ring_claim<STATE>(u, ok, n, bits, m, dv, pg);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t mk = __ballot(ok[j]);
            if (ok[j]) put(f, cnt + mask_rank(mk), u[j]);
            cnt += __popcll(mk);
        }
        uint64_t hm = __ballot(sub == G - 1 && nb.w == kEllMore);
        while (hm) {  // long rows: the whole wave over each tail, 64 arcs at a time
            const int src_lane = __builtin_ctzll(hm);
            hm &= hm - 1;
            const int h = __shfl(v, src_lane);
            const int e1 = rp[h + 1];
            for (int e = rp[h] + W - 1 + lane; __any(e < e1); e += kWave) {
                const int t[1] = {e < e1 ? ci[e] : -1};
                bool okt[1];
                ring_claim<STATE>(t, okt, n, bits, m, dv, pg);
                const uint64_t mk = __ballot(okt[0]);
                if (okt[0]) put(f, cnt + mask_rank(mk), t[0]);
                cnt += __popcll(mk);
            }
        }
        __builtin_amdgcn_wave_barrier();
        len = cnt;
        ++nl;
        f.at = f.next;
        f.next += cnt;
        if (lane == 0) ls[nl] = f.at;
    }
    return len;
}

// BFS from src in one workgroup through the nodes whose distance lies below m
// (kRsFull: all of them); every node found goes to the sink with its distance.
// q: the LDS queue of cap entries, lheavy: the long-row list, bits: the
// visited set (state bytes: flags clear on entry and on return).  gq holds
// 2 n ints (queue overflow, long rows).  Returns the number of nodes found, -1
// as soon as a frontier is wider than `widest` or more than n nodes were found,
// or kRingLeft where the pages ran out, which sets *stop, or *stop was set.
// *end (thread 0): the largest distance (left: the last complete level, all of
// it at the sink as well) and the nodes found.  beat: sync_search's counter, told
// that the search goes on.  Ends past a barrier.
template <int W, int STATE, class Sink>
__device__ __forceinline__ int ring_search(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                            const int* __restrict__ ell, int src, int* q, int cap, int* lheavy,
                                            unsigned* bits, const int* m, Sink sink, int* gq, int widest = INT_MAX,
                                            int2* end = nullptr, Pages pg = Pages(), int* stop = nullptr,
                                            unsigned long long* beat = nullptr) {
    __shared__ int2 s_slot[3];
    __shared__ int s_wave[4];
    __shared__ int s_ls[kRingLevels + 2];  // queue positions where the levels since the last flush start
    if (STATE == kRsPaged)
        pg.clear(bits);
    else if (STATE != kRsBytes)
        for (int w = threadIdx.x; w < (n + 31) / 32; w += blockDim.x) bits[w] = 0u;
    __syncthreads();
    if (threadIdx.x == 0) {
        if (STATE == kRsBytes)
            ((unsigned char*)bits)[src] |= 0x80;
        else if (STATE == kRsPaged)
            pg.mark(bits, src, 0);
        else
            bits[src >> 5] |= 1u << (src & 31);
        q[0] = src;
        s_ls[0] = 0;
        s_slot[0] = s_slot[1] = s_slot[2] = make_int2(0, 0);
    }
    __syncthreads();
    RingFrontier f;
    f.lnxt = q;
    f.gnxt = gq;
    f.cnt = nullptr;
    f.lheavy = lheavy;
    f.gheavy = gq + n;
    f.cap = cap;
    f.at = 0;
    f.next = 1;
    int total = 1, len = 1;       // nodes found; size of the current frontier
    int base = 0, d0 = 0, nl = 0;  // flushed: nodes, levels; complete levels since
    int step = 0;                  // block levels run: their counters rotate
    int flushes = 0;
    while (len > 0) {
        const int before = f.next;
        if (len <= wave_level_nodes<W>() && (STATE != kRsBytes || d0 + nl + 1 < kM7Sat) && f.next <= cap / 2) {
            if (threadIdx.x < kWave) {
                RingFrontier g = f;
                int l = nl;
                const int left = ring_wave_levels<W, STATE>(n, rp, ci, ell, bits, m, q, g, len, d0, s_ls, l, pg);
                if (threadIdx.x == 0) {
                    s_wave[0] = left;
                    s_wave[1] = l;
                    s_wave[2] = g.at;
                    s_wave[3] = g.next;
                }
            }
            __syncthreads();
            len = s_wave[0];
            nl = s_wave[1];
            f.at = s_wave[2];
            f.next = s_wave[3];
            __syncthreads();
        } else {
            level_begin(s_slot, step++, f);
            const int dv = d0 + nl + 1, lds = split(f);
            f.lcur = q + f.at;
            f.gcur = gq + (lds > 0 ? 0 : f.at - cap);
            len = ell_level_auto<W>(n, rp, ci, ell, len, f, [&](const auto& u, auto& ok) {
                ring_claim<STATE>(u, ok, n, bits, m, dv, pg);
            });
            ++nl;
            f.at = f.next;
            f.next += len;
            if (threadIdx.x == 0) s_ls[nl] = f.at;
        }
        total += f.next - before;
        if (len > widest) return -1;  // uniform
        // Paged bits forget the levels before the last, which no arc leads back
        // to in a symmetric graph.  In one that is not (the caller's error) a
        // node can be found again, for ever on a one-way cycle.
        if (STATE == kRsPaged && total > n) return -1;  // uniform
        bool full = false, over = false;
        if (STATE == kRsPaged) {
            over = bits[1] != 0;  // the level just run lacks nodes; over implies full
            full = (int)bits[0] > pg.count - kPagesSpare;
            __syncthreads();  // both read before the next level takes pages
        }
        if (len == 0 || nl >= kRingLevels || f.next > cap / 2 || full) {  // flush the complete levels (uniform)
            __syncthreads();
            bool leave = over;  // uniform
            if (STATE == kRsPaged && !over && full && len > 0) {  // the last complete level and the current frontier stay marked
                pg.clear(bits);
                __syncthreads();
                for (int pos = s_ls[nl - 1] + (int)threadIdx.x; pos < f.next; pos += blockDim.x) {
                    const int u = ring_get(f, q, pos);
                    pg.mark(bits, u, pg.table(bits)[u >> kPageShift]);
                }
                __syncthreads();
                leave = (int)bits[0] > pg.count - kPagesSpare;  // two levels alone fill the pool
            }
            if (STATE == kRsPaged && leave) {
                if (threadIdx.x == 0) store_agent(stop, 1);
            } else if (STATE == kRsPaged && len > 0 && ++flushes % kRingStopLooks == 0) {
                if (threadIdx.x == 0) s_wave[0] = load_agent(stop);
                __syncthreads();
                leave = s_wave[0] != 0;
            }
            for (int l = threadIdx.x / kWave; l < nl; l += blockDim.x / kWave)
                for (int pos = s_ls[l] + lane_id(); pos < s_ls[l + 1]; pos += kWave)
                    sink.put(base + pos, ring_get(f, q, pos), d0 + l);
            if (STATE == kRsPaged && leave) {  // uniform
                if (!over)
                    for (int pos = f.at + (int)threadIdx.x; pos < f.next; pos += blockDim.x)
                        sink.put(base + pos, ring_get(f, q, pos), d0 + nl);
                if (threadIdx.x == 0) *end = over ? make_int2(d0 + nl - 1, total - len) : make_int2(d0 + nl, total);
                __syncthreads();
                return kRingLeft;
            }
            if (beat && threadIdx.x == 0 && (d0 + nl) / kBeatLevels != d0 / kBeatLevels) atomicAdd(beat, kBeat);
            base += f.at;
            d0 += nl;
            nl = 0;
            __syncthreads();
            for (int c = 0; c < len; c += blockDim.x) {  // the current frontier to the front
                const int i = c + (int)threadIdx.x;
                const int u = i < len ? ring_get(f, q, f.at + i) : 0;
                __syncthreads();
                if (i < len) ring_set(f, q, i, u);
                __syncthreads();
            }
            f.at = 0;
            f.next = len;
            if (threadIdx.x == 0) s_ls[0] = 0;
            __syncthreads();
        }
    }
    if (end && threadIdx.x == 0) *end = make_int2(d0 - 1, total);
    if (STATE == kRsBytes) {
        uint4* w16 = (uint4*)bits;
        for (int w = threadIdx.x; w < (n + 15) / 16; w += blockDim.x) {
            uint4 x = w16[w];
            x.x &= 0x7f7f7f7fu;
            x.y &= 0x7f7f7f7fu;
            x.z &= 0x7f7f7f7fu;
            x.w &= 0x7f7f7f7fu;
            w16[w] = x;
        }
    }
    __syncthreads();
    return total;
}

// Block b: BFS from pivots[b] into dist[b][*] (pre-set to -1) on one workgroup
// (gq: 2 n ints per block).  reached[b] = nodes found, or -1 (the graph is not
// symmetric); from[b] = -1, or the level at which the search was left; *ecc_max
// = largest eccentricity of the complete rows; *stop: 0 on entry.
template <int W>
__global__ __launch_bounds__(kBfsBlock) void k_bfs_ring(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                        const int* __restrict__ ell, const int* __restrict__ pivots,
                                                        int* dist, int* gq, int* reached, int* from, int* ecc_max,
                                                        int* stop, Pages pg) {
    __shared__ __align__(16) unsigned char pool[kRingPool];
    __shared__ int2 s_end;
    int* lheavy = (int*)pool;
    unsigned* bits = (unsigned*)(lheavy + kHeavyCap);
    int* q = (int*)((unsigned char*)bits + kPagedBytes);
    const int b = blockIdx.x;
    const int found = ring_search<W, kRsPaged>(n, rp, ci, ell, pivots[b], q, (kRingPool - 4 * kHeavyCap - kPagedBytes) / 4,
                                            lheavy, bits, nullptr, PlainRowSink{dist + (size_t)b * n},
                                            gq + (size_t)b * 2 * n, INT_MAX, &s_end, pg, stop);
    if (threadIdx.x == 0) {
        reached[b] = found == kRingLeft ? s_end.y : found;
        from[b] = found == kRingLeft ? s_end.x : -1;
        if (found > 0) atomicMax(ecc_max, s_end.x);
    }
}

}  // namespace ssm
