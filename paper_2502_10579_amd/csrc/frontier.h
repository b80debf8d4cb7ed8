// Frontier plumbing shared by the bound solver and the multi-snapshot relaxer.
//
// An iteration's improvements only set a byte flag per vertex of the next
// frontier (an idempotent plain store), so no vertex is listed twice and no
// counter is hit per improvement.  A compaction kernel turns the flags into
// the next work list in vertex order, clearing the flags it reads, with one
// packed 64-bit counter reservation per block (items in the high word, edges
// in the low word) so that the list and the running edge offsets stay in the
// same order.
//
// Counters are double-buffered by iteration parity p: the compaction of
// iteration i zeroes the item counter of parity p ^ 1 (the previous
// iteration's, whose readers have finished) and adds into parity p, whose
// deferral counters the expansion before it has reset; the expansion of
// iteration i reads cnt[p],
// tells the next compaction whether it produced work, and publishes its item
// count to a host-mapped slot, so the host never has to synchronise the
// stream to learn when a loop has drained.  A compaction that finds the
// previous expansion empty returns at once, so iterations issued past the end
// cost one launch.  In a sparse iteration the bound solves' expansion may
// instead append its improved vertices to the next work list itself (into
// cnt[p ^ 1], zeroed by the compaction before it); the next compaction then
// skips its scan.  A run of small iterations is done by one launch (Team,
// below).
#pragma once

#include "evq_internal.h"

namespace evq {

// What an expansion publishes for the host, in one 64-bit word: the frontier
// items it processed (low word), the iterations it ran, and whether the loop
// is done (nothing was left to process, now or for the next launch) or has
// failed (a team gave up, see Team).
constexpr unsigned long long kSlotDone = 1ull << 63;
constexpr unsigned long long kSlotFailed = 1ull << 62;
__host__ __device__ inline unsigned long long slot_word(uint32_t items, uint32_t iters, bool done) {
    return (done ? kSlotDone : 0ull) | ((unsigned long long)iters << 32) | items;
}

struct FrontierCounters {
    unsigned long long packed[2];  // (items << 32) | edges, by parity
    uint32_t far[2];               // ids left flagged (for a later threshold or bucket), by parity
    uint32_t fmin[2];              // smallest order key among the ids left for a later threshold, by parity
    uint32_t thr;                  // near/far threshold of the bound solves (order keys below it are near)
    uint32_t delta;                // threshold step (0: every id is near)
    uint32_t heavy;                // with delta > 0: only ids with at least this many edges are gated (0: all)
    uint32_t kall[2];              // smallest order key over the compacted ids with edges, by parity (heavy > 0)
    uint32_t status[2];            // for the compaction of parity q: bit 0 the expansion before it had work
                                   // or deferred ids, bit 1 it appended the next list itself, bit 2 a team
                                   // left that list (its count is Team::result)
    uint32_t flip[2];              // the bound solves' item sets at host parity q are those of q ^ flip[q]
                                   // (a team that ran an even number of iterations moves them)
    // Bucketed schedule with light and heavy edges (bound solves of SSSP):
    uint32_t bdelta;               // bucket width (0: off)
    uint32_t bthr[2];              // the bucket's upper key bound set by the compaction of parity q
    uint32_t near[2];              // the expansion of parity q improved a vertex below bthr[q]
    uint32_t nmin[2];              // smallest value it wrote at or above bthr[q]
};
static_assert(sizeof(FrontierCounters) <= 128, "frontier counters share a 128-byte control slot");

__device__ __forceinline__ uint32_t items_of(unsigned long long x) { return (uint32_t)(x >> 32); }
__device__ __forceinline__ uint32_t edges_of(unsigned long long x) { return (uint32_t)x; }

// Next-frontier membership is one byte per id: marking is an idempotent plain
// byte store, so an improvement costs no second atomic.
__device__ __forceinline__ void mark(uint8_t* __restrict__ flags, uint32_t v) { flags[v] = 1; }

// Bytes of the flag array for n ids (a multiple of the 8 ids a lane reads).
inline uint64_t flag_bytes(uint64_t n) { return (n + 7) & ~uint64_t(7); }

// Item parity and count of the iteration of host parity h.  Both counts are
// read beside the flip, not after it: a kernel that calls this before its first
// store waits for one access, and takes the values through the scalar cache.
__device__ __forceinline__ unsigned long long read_list(const FrontierCounters* c, int h, int& p) {
    const uint32_t f = c->flip[h];
    const unsigned long long x0 = c->packed[0], x1 = c->packed[1];
    p = h ^ (int)uniform(f);
    return p ? x1 : x0;
}

// Expansion prologue (count x of item parity p, from read_list): tell the
// next compaction (host parity h ^ 1) whether there was work and whether this
// expansion appends the next list itself (`appends`, the same on every block),
// publish the item count to the host slot.
// When nothing was near but ids were deferred, the threshold moves to the
// smallest deferred order key plus delta, so the next compaction releases the
// best of them.  When only heavy ids are gated, the threshold also follows the
// frontier: it rises to the smallest key of this iteration's ids plus delta,
// so a heavy id is expanded once its value is within delta of the best one
// still moving (and, with positive steps, close to final).
__device__ __forceinline__ void expand_prologue(FrontierCounters* c, int h, int p, unsigned long long x,
                                                unsigned long long* slot, bool appends = false) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const uint32_t f = c->far[p];
        uint64_t t = c->thr;
        if (items_of(x) == 0 && f) t = (uint64_t)c->fmin[p] + c->delta;
        if (c->heavy && c->kall[p] != 0xFFFFFFFFu) {
            const uint64_t u = (uint64_t)c->kall[p] + c->delta;
            t = u > t ? u : t;
        }
        c->thr = t > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)t;
        c->status[h ^ 1] = (x != 0ull || f ? 1u : 0u) | (appends ? 2u : 0u);
        c->flip[h ^ 1] = (uint32_t)(h ^ p);
        // the other parity's deferral counters, last read by the compaction
        // before this expansion, start afresh for the next compaction
        c->far[p ^ 1] = 0u;
        c->fmin[p ^ 1] = 0xFFFFFFFFu;
        c->kall[p ^ 1] = 0xFFFFFFFFu;
        const uint32_t n = items_of(x) + f;
        __hip_atomic_store(slot, slot_word(n, n ? 1u : 0u, n == 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// A team: up to kTeamBlocks blocks of one launch (the bound solves' compaction,
// or the relaxation's k_relax_team) that run a loop's small iterations
// themselves, with a barrier of their own between iterations instead of a
// kernel boundary.
//
// What bounds a small iteration is latency: two launches of 2.4 us each and
// their start and drain (10-12 us an iteration as launches, whatever its
// size), against 1.6-1.8 us for a barrier over 64 blocks and about 2 us for the
// chain of dependent accesses of an expansion.  The batched loops, whose
// streams fill one another's gaps, gained nothing (4.79 against 4.76 ms) and go
// without; single queries' figures are below.
//
// Members are the candidate blocks (every kTeamEvery-th block of the grid) that
// are running when the first of them, after a short wait, closes the
// registration; so every member is resident and the barrier cannot wait for a
// block that has yet to start.  Blocks that come later find the registration
// closed and leave.  Nothing depends on where the members run: all they share
// goes through agent-scope relaxed atomic loads, stores and read-modify-writes,
// and a member's accesses have completed (s_waitcnt) before it arrives at the
// barrier.  An agent-scope fence would do as well but writes the L2 back (7.6
// us a barrier of 32 blocks against 1.3).
//
// The dispatcher deals consecutive blocks to the 8 XCDs in turn, so every
// eighth block would put a team on one L2.  That buys next to nothing (64
// blocks, a store per thread: 1.7 us a barrier, 1.8 from every 1st, 2nd or 4th
// block) and takes a launch of 512 blocks, which callers on several streams pay
// for.  Microseconds a query without teams, from every 8th, every 2nd and every
// block: 4096 vertices, one caller 350, 267, 245, 250, eight callers 87, 101,
// 68, 64; 150001 vertices 295, 236, 236, 242 and 103, 108, 98, 99; 2^20
// vertices 995, 929, 929, 938 and 640, 675, 640, 636.
//
// A team takes a list only if it is no more than kTeamRounds rounds of each
// member (a tile of edges, or its lane groups' tasks), and hands a longer one
// to the launches.  On an idle device all 64 candidates register, and the rule
// changes nothing; where other streams fill it (the mid query from 2, 4 or 8
// threads) teams of any size from one block up were counted, and without the
// rule one block would run 64 tiles an iteration that a launch spreads over the
// device.  1, 2, 4 and 64 rounds measured the same in those calls, so 4 bounds
// the worst case at about what the two launches of an iteration cost.
//
// Every wait is bounded.  A member whose wait runs out leaves, the others'
// next wait runs out too, and the lists are then in no known state: the
// expansion's launch that follows finds the team begun and not ended
// (team_end) and reports it to the host, which fails the call, instead of
// expanding them.
struct Team {
    uint32_t reg;     // members registered; bit 31: closed
    uint32_t n;       // their number, once closed
    uint32_t err;     // a wait ran out
    uint32_t began;   // tag of the last launch whose list a team took
    uint32_t ran;     // ... and of the last that a team ran to its end
    uint32_t pad0[27];
    uint32_t arrive;  // barrier arrivals so far
    uint32_t pad1[31];
    uint32_t gen;     // barriers completed
    uint32_t pad2[31];
    // (items << 32) | edges of the lists: iteration k reads [k % 3], appends into
    // [(k + 1) % 3] and clears [(k + 2) % 3], which iteration k - 1 read
    unsigned long long packed[3];
    unsigned long long result;  // count of the list the team left
};
constexpr uint32_t kTeamBlocks = 64;
constexpr uint32_t kTeamEvery = 2;
constexpr uint32_t kTeamGrid = kTeamBlocks * kTeamEvery;  // blocks of a launch with room for a whole team
constexpr uint32_t kTeamIters = 1024;      // most iterations of one launch
constexpr uint32_t kTeamRounds = 4;        // most rounds of a member in an iteration
constexpr uint32_t kTeamSpins = 1u << 24;  // polls of a wait (seconds); past them the member gives up
constexpr uint64_t kTeamBytes = 1024;      // control bytes of a team
static_assert(sizeof(Team) <= kTeamBytes, "team control block");

__device__ __forceinline__ void team_reset(Team* t) {  // one thread, in a launch before the team's
    t->reg = t->n = t->err = t->arrive = t->gen = 0u;
    t->packed[0] = t->packed[1] = t->packed[2] = 0ull;
}

template <typename T>
__device__ __forceinline__ T shared_load(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void shared_store(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// End of a team's launch at host parity h, by one thread: after k iterations the
// current list has count x and item parity q; `items` were processed.  What the
// next launches read is written to places that this launch's late blocks do
// not look at, or whose change only tells them to leave.  `tag` (never 0)
// tells the rest of this iteration's launches that a team has run it.
__device__ __forceinline__ void team_leave(FrontierCounters* c, Team* t, uint32_t tag, int h, int q,
                                           unsigned long long x, uint32_t items, uint32_t k, unsigned long long* slot) {
    t->result = x;
    t->ran = tag;
    c->status[h ^ 1] = x ? 5u : 4u;
    c->flip[h ^ 1] = (uint32_t)(q ^ h ^ 1);
    __hip_atomic_store(slot, slot_word(items, k, x == 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// How the team of the launch tagged `tag` fared, read by the expansion's launch
// after it: there was none (or tag is 0), it ran the iteration and published,
// or it began and did not end.
enum class TeamEnd { kNone, kRan, kGaveUp };
__device__ __forceinline__ TeamEnd team_end(const Team* t, uint32_t tag) {
    if (tag == 0) return TeamEnd::kNone;
    const uint32_t began = t->began, ran = t->ran;
    if (began != tag) return TeamEnd::kNone;
    return ran == tag ? TeamEnd::kRan : TeamEnd::kGaveUp;
}

// The launch at host parity h found that the team before it gave up; one
// thread.  No list is left for the launches already issued.
__device__ __forceinline__ void team_report(FrontierCounters* c, int h, unsigned long long* slot) {
    c->packed[0] = c->packed[1] = 0ull;
    c->status[h ^ 1] = 0u;
    __hip_atomic_store(slot, kSlotFailed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// What the host lays down for teams.
struct TeamRules {
    uint32_t place;   // which of every kTeamEvery blocks are the candidates
    uint32_t spins;   // polls of a wait before a member gives up
    uint32_t blocks;  // most members (at most kTeamBlocks)
};

struct TeamRun {
    uint32_t rank, n, gen, spins;
};

// Every thread of a block calls it; true for the members' blocks, unless the
// list's `work` is more than kTeamRounds rounds of `round` for each of them (then
// they leave it to the launches; all see the same number).  tag (not 0): this
// launch's.
__device__ __forceinline__ bool team_join(Team* t, const TeamRules& rules, uint32_t work, uint32_t round, uint32_t tag,
                                          TeamRun& r) {
    if (blockIdx.x % kTeamEvery != rules.place || blockIdx.x / kTeamEvery >= rules.blocks) return false;
    __shared__ uint32_t s_rank, s_n;
    if (threadIdx.x == 0) {
        uint32_t rank = kNone, n = 0;
        const uint32_t k = shared_load(&t->reg) >> 31 ? 1u << 31 : atomicAdd(&t->reg, 1u);
        if (!(k >> 31)) {
            rank = k;
            if (k == 0) {
                for (uint32_t i = 0; i < 32u && shared_load(&t->reg) < rules.blocks; ++i) __builtin_amdgcn_s_sleep(1);
                n = atomicOr(&t->reg, 1u << 31);
                if (work <= n * kTeamRounds * round) t->began = tag;
                shared_store(&t->n, n);
            } else {
                for (uint32_t i = 0; i < rules.spins && n == 0; ++i) n = shared_load(&t->n);
                if (n == 0) rank = kNone;
            }
            if (work > n * kTeamRounds * round) rank = kNone;
        }
        s_rank = rank;
        s_n = n;
    }
    __syncthreads();
    r.rank = s_rank;
    r.n = s_n;
    r.gen = 0;
    r.spins = rules.spins;
    return r.rank != kNone;
}

// Barrier over the team; every thread of every member calls it.  False: a
// member did not arrive in time (the caller leaves without publishing; see
// team_end).
__device__ __forceinline__ bool team_barrier(Team* t, TeamRun& r) {
    __shared__ uint32_t s_ok;
    __builtin_amdgcn_s_waitcnt(0);  // this wave's loads, stores and atomics have completed
    __syncthreads();
    ++r.gen;
    if (threadIdx.x == 0) {
        uint32_t ok = 1;
        if (__hip_atomic_fetch_add(&t->arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == r.n * r.gen) {
            shared_store(&t->gen, r.gen);
        } else {
            uint32_t i = 0;
            while (shared_load(&t->gen) < r.gen)
                if (++i >= r.spins || shared_load(&t->err)) {
                    shared_store(&t->err, 1u);
                    ok = 0;
                    break;
                }
        }
        s_ok = ok;
    }
    __syncthreads();
    return s_ok != 0;
}

// Compaction prologue (host parity h, item parity p, status st of this
// iteration): zero the other item parity's counters (the previous iteration's,
// read only by kernels that have finished) for the next iteration, clear this
// parity's bucket reports for the expansion that follows, and say whether the
// scan can be skipped: the previous expansion had no work and deferred nothing
// (no flag can be set), it appended the next list itself, or a team left one
// (its count is put in place here).  The first compaction of a loop scans,
// unless its list is there already.
__device__ __forceinline__ bool compaction_skips(FrontierCounters* c, int p, uint32_t st, Team* team = nullptr) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        c->packed[p ^ 1] = 0ull;
        if (team && (st & 4u)) c->packed[p] = team->result;
        c->near[p] = 0u;
        c->nmin[p] = 0xFFFFFFFFu;
    }
    return st != 1u;
}

// Largest i in [0, n) with off[i] <= x (off ascending, off[0] == 0), found by
// the whole wave with a 64-ary search.  Every lane must call it.
// SHARED: off is written by other blocks of this launch (a team's list).
template <bool SHARED = false>
__device__ __forceinline__ uint32_t wave_search(const uint32_t* off, uint32_t n, uint32_t x) {
    auto at = [&](uint32_t i) { return SHARED ? shared_load(off + i) : off[i]; };
    uint32_t lo = 0, hi = n;  // answer in [lo, hi)
    const uint32_t lane = lane_id();
    while (hi - lo > 64) {
        const uint32_t step = (hi - lo + 63) / 64;
        const uint32_t idx = lo + lane * step;
        const bool ok = idx < hi && at(idx) <= x;
        const uint64_t b = __ballot(ok);
        const uint32_t last = 63u - (uint32_t)__clzll((unsigned long long)b);  // lane 0 is always ok
        const uint32_t nlo = lo + last * step;
        const uint32_t nhi = nlo + step < hi ? nlo + step : hi;
        lo = nlo;
        hi = nhi;
    }
    const uint32_t idx = lo + lane;
    const bool ok = idx < hi && at(idx) <= x;
    const uint64_t b = __ballot(ok);
    return lo + 63u - (uint32_t)__clzll((unsigned long long)b);
}

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Flag compaction shared by the frontier loops.  A block of kCompactBlock
// threads takes kCompactIds consecutive ids (8 flag bytes per lane), stages
// the flagged ids and their flag bytes in LDS, reads every id's work size with
// all loads in flight at once, rewrites the flag bytes, and reserves (items,
// edges) for the whole block with one packed atomic.
// size_of(id, flag, items, edges, key, aux) gives an id's work (items and
// edges, zero for none), may keep two words of what it read in aux for emit,
// and returns the flag byte the id keeps: 0 clears it; an id left flagged is
// counted in *far and, unless size_of leaves key at 0xFFFFFFFF, its order key
// enters the minimum *fmin.  emit(id, item, edge, items, edges, aux) writes an
// id's work.  Ids appear in ascending order within a block.  With kall
// non-null, size_of gives every id with edges its order key and the smallest
// of them enters the minimum *kall.  post() runs on every thread of the block
// after each group of ids has been emitted (and the block synchronised),
// before the next group is compacted.
struct NoPost {
    __device__ void operator()() const {}
};
constexpr int kCompactBlock = 512;
constexpr int kCompactWaves = kCompactBlock / 64;
constexpr int kIdsPerWave = 512;
constexpr int kCompactIds = kCompactWaves * kIdsPerWave;
constexpr int kIdSteps = kIdsPerWave / 64;

template <typename SizeFn, typename EmitFn, typename PostFn = NoPost>
__device__ __forceinline__ void compact_flags(uint8_t* __restrict__ flags, uint32_t n, unsigned long long* cnt,
                                              uint32_t* far, uint32_t* fmin, SizeFn size_of, EmitFn emit,
                                              uint32_t* kall = nullptr, PostFn post = PostFn()) {
    __shared__ uint32_t ids[kCompactWaves][kIdsPerWave];
    __shared__ uint8_t fbyte[kCompactWaves][kIdsPerWave];  // flag byte of each listed id
    __shared__ uint2 nflag[kCompactWaves][64];             // the wave's new flag bytes, in id order
    __shared__ uint32_t wtot[kCompactWaves][5];
    __shared__ unsigned long long bbase;
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    uint2* __restrict__ f8 = reinterpret_cast<uint2*>(flags);
    uint8_t* const nf8 = reinterpret_cast<uint8_t*>(nflag[wave]);
    for (uint64_t b0 = (uint64_t)blockIdx.x * kCompactIds; b0 < n; b0 += (uint64_t)gridDim.x * kCompactIds) {
        const uint32_t w0 = (uint32_t)b0 + wave * kIdsPerWave;  // first id of this wave
        const uint32_t g0 = w0 + lane * 8;                       // first id of this lane
        uint2 fl = make_uint2(0u, 0u);
        if (g0 < n) fl = f8[g0 >> 3];
        uint32_t word = 0;  // bit k: id g0 + k is flagged
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            word |= ((fl.x >> (8 * k)) & 0xFFu) ? (1u << k) : 0u;
            word |= ((fl.y >> (8 * k)) & 0xFFu) ? (1u << (k + 4)) : 0u;
        }
        const uint32_t pc = (uint32_t)__popc(word);
        const uint32_t incl = wave_incl_scan(pc);
        const uint32_t tot = lane_value(incl, 63);
        uint32_t id[kIdSteps], ni[kIdSteps], ne[kIdSteps], pi[kIdSteps], pe[kIdSteps];
        uint2 aux[kIdSteps];
#pragma unroll
        for (int s = 0; s < kIdSteps; ++s) {
            id[s] = ni[s] = ne[s] = pi[s] = pe[s] = 0;
            aux[s] = make_uint2(0u, 0u);
        }
        uint32_t ti = 0, te = 0, tf = 0, tk = 0xFFFFFFFFu, ta = 0xFFFFFFFFu;
        if (tot) {
            nflag[wave][lane] = make_uint2(0u, 0u);
            uint32_t k = incl - pc;
            for (uint32_t m = word; m; m &= m - 1) {
                const uint32_t b = (uint32_t)__builtin_ctz(m);
                ids[wave][k] = g0 + b;
                fbyte[wave][k] = (uint8_t)(((b < 4 ? fl.x : fl.y) >> (8 * (b & 3))) & 0xFFu);
                ++k;
            }
            wave_lds_sync();
            uint32_t nf = 0, kmin = 0xFFFFFFFFu, amin = 0xFFFFFFFFu;
            // the steps past the wave's count (tot, wave-uniform) are skipped
#pragma unroll
            for (int s = 0; s < kIdSteps; ++s) {
                if (s * 64u >= tot) break;
                const uint32_t j = s * 64 + lane;
                if (j < tot) {
                    id[s] = ids[wave][j];
                    uint32_t key = 0xFFFFFFFFu;
                    const uint32_t kept = size_of(id[s], (uint32_t)fbyte[wave][j], ni[s], ne[s], key, aux[s]);
                    amin = key < amin ? key : amin;
                    if (kept) {  // its flag stays set
                        ++nf;
                        kmin = key < kmin ? key : kmin;
                        nf8[id[s] - w0] = (uint8_t)kept;
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < kIdSteps; ++s) {
                if (s * 64u >= tot) break;
                const uint32_t a = wave_incl_scan(ni[s]), b = wave_incl_scan(ne[s]);
                pi[s] = ti + a - ni[s];
                pe[s] = te + b - ne[s];
                ti += lane_value(a, 63);
                te += lane_value(b, 63);
            }
            tf = wave_sum(nf);
            tk = wave_min(kmin);
            if (kall) ta = wave_min(amin);
            wave_lds_sync();
            if (word) f8[g0 >> 3] = nflag[wave][lane];
        }
        if (lane == 0) {
            wtot[wave][0] = ti;
            wtot[wave][1] = te;
            wtot[wave][2] = tf;
            wtot[wave][3] = tk;
            wtot[wave][4] = ta;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long sum = 0;
            uint32_t fsum = 0, kmin = 0xFFFFFFFFu, amin = 0xFFFFFFFFu;
            for (int w = 0; w < kCompactWaves; ++w) {
                sum += ((unsigned long long)wtot[w][0] << 32) | wtot[w][1];
                fsum += wtot[w][2];
                kmin = wtot[w][3] < kmin ? wtot[w][3] : kmin;
                amin = wtot[w][4] < amin ? wtot[w][4] : amin;
            }
            bbase = sum ? atomicAdd(cnt, sum) : 0ull;
            if (fsum) {
                atomicAdd(far, fsum);
                atomicMin(fmin, kmin);
            }
            // a plain read first: most blocks hold no new minimum and skip the atomic
            if (kall && amin < __hip_atomic_load(kall, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(kall, amin);
        }
        __syncthreads();
        if (ti) {
            uint32_t bi = (uint32_t)(bbase >> 32), be = (uint32_t)bbase;
            for (uint32_t w = 0; w < wave; ++w) {
                bi += wtot[w][0];
                be += wtot[w][1];
            }
#pragma unroll
            for (int s = 0; s < kIdSteps; ++s)
                if (ni[s]) emit(id[s], bi + pi[s], be + pe[s], ni[s], ne[s], aux[s]);
        }
        __syncthreads();
        post();
    }
}

// Task lists of a compaction whose ids expand to several tasks each (task q
// of id c is the 64-bit word (q << 32) | c).  An id with one task has it
// written by the lane that holds it; an id with more is listed in LDS, and
// after each group of ids (post() of compact_flags) the whole block writes the
// listed tasks, each thread finding the id of its task by a binary search over
// the list's running task counts, so a hub's 10^5 tasks and many small ids
// are written at the same rate.  A full list falls back to the holding lane.
constexpr uint32_t kTaskListCap = 2048;
struct TaskList {
    uint32_t n;
    uint32_t id[kTaskListCap], first[kTaskListCap], cnt[kTaskListCap], pre[kTaskListCap];
    uint32_t wsum[kCompactWaves];
};

__device__ __forceinline__ void task_list_init(TaskList& tl) {
    if (threadIdx.x == 0) tl.n = 0;
    __syncthreads();
}

__device__ __forceinline__ void task_list_add(TaskList& tl, uint64_t* __restrict__ tasks, uint32_t c, uint32_t first,
                                              uint32_t items) {
    uint32_t k = kTaskListCap;
    if (items > 1) k = atomicAdd(&tl.n, 1u);
    if (k < kTaskListCap) {
        tl.id[k] = c;
        tl.first[k] = first;
        tl.cnt[k] = items;
    } else {
        for (uint32_t q = 0; q < items; ++q) tasks[first + q] = ((uint64_t)q << 32) | c;
    }
}

// Every thread of the block (kCompactBlock of them) calls it.
__device__ __forceinline__ void task_list_flush(TaskList& tl, uint64_t* __restrict__ tasks) {
    constexpr uint32_t kPer = kTaskListCap / kCompactBlock;
    const uint32_t nb = tl.n < kTaskListCap ? tl.n : kTaskListCap;
    if (nb) {
        const uint32_t lane = lane_id(), wave = threadIdx.x >> 6, k0 = threadIdx.x * kPer;
        uint32_t s = 0;
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j) s += k0 + j < nb ? tl.cnt[k0 + j] : 0u;
        const uint32_t incl = wave_incl_scan(s);
        if (lane == 63) tl.wsum[wave] = incl;
        __syncthreads();
        uint32_t off = incl - s, tot = 0;
        for (uint32_t w = 0; w < kCompactWaves; ++w) {
            off += w < wave ? tl.wsum[w] : 0u;
            tot += tl.wsum[w];
        }
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j)
            if (k0 + j < nb) {
                tl.pre[k0 + j] = off;
                off += tl.cnt[k0 + j];
            }
        __syncthreads();
        for (uint32_t t = threadIdx.x; t < tot; t += kCompactBlock) {
            uint32_t lo = 0, hi = nb;  // largest k with pre[k] <= t
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if (tl.pre[mid] <= t) lo = mid;
                else hi = mid;
            }
            const uint32_t q = t - tl.pre[lo];
            tasks[tl.first[lo] + q] = ((uint64_t)q << 32) | tl.id[lo];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) tl.n = 0;
}

// Host side: launch-ahead driver of a frontier loop.
class HostSlots {
  public:
    static constexpr uint32_t kSlots = 256;
    static constexpr uint32_t kMail = kSlots;  // three words of mail from one kernel: arrived, then two counts
    static constexpr uint32_t kWords = kSlots + 8;
    static constexpr unsigned long long kEmpty = ~0ull;  // no published word (slot_word never gives it)
    static HostSlots& get();  // one per host thread
    unsigned long long* host() const { return h_; }
    unsigned long long* dev() const { return d_; }
    // Slot numbering runs on across loops, so that the iterations a finished
    // loop issued past its end (still queued) never write a slot that the
    // next loop has just reset.
    uint64_t next = 0;

  private:
    HostSlots();
    unsigned long long* h_ = nullptr;
    unsigned long long* d_ = nullptr;
};

// Issues launches of an iteration (issue(it, parity, first)) ahead of the one
// whose published word it waits for (InFlight(depth) says how many); stops at
// the first that says the loop is done.  Returns the number of non-empty iterations and adds the
// published counts (items processed) to *items; f_parity is advanced past
// every issued launch.
template <typename IssueFn>
uint64_t drive_loop(IssueFn issue, int& f_parity, hipStream_t s, uint64_t max_iters, const char* what,
                    uint64_t* items = nullptr, uint64_t depth = 0);

void wait_slot(volatile unsigned long long* slot, hipStream_t s, const char* what);

// Iterations kept in flight by drive_loop: EVQ_LAUNCH_DEPTH (1..32), default 3.
uint64_t launch_depth();
// Polls of a team's waits (EVQ_TEAM_SPINS, default kTeamSpins) and its most
// members (EVQ_TEAM_BLOCKS, default and at most kTeamBlocks), read once.
TeamRules team_rules(uint32_t place);
// EVQ_TRACE_LOOPS=1: drive_loop prints each iteration's published count to stderr.
bool trace_loops();

// Iterations a launch ran, from its published word.
inline uint32_t iterations_of(unsigned long long w) { return (uint32_t)(w >> 32) & 0x3FFFFFFFu; }

// Launches a loop keeps in flight: launch_depth(), or the given depth where
// teams run the small iterations.  Such a loop goes to launch_depth() once
// kSteadyLaunches in a row have run one iteration each, and back with the next
// that runs more: a deep graph whose lists stay above the teams' limit has
// hundreds of such launches, where the next one's launch latency shows (BFS, 40000
// to 480000 edges a list, 100 to 400 iterations: 3-10% of the query), while the
// dense iterations of a power-law graph are fewer than that.
class InFlight {
  public:
    explicit InFlight(uint64_t depth) : few_(depth ? depth : launch_depth()), most_(depth ? launch_depth() : few_) {
        if (most_ < few_) most_ = few_;
    }
    uint64_t launches() const { return steady_ < kSteadyLaunches ? few_ : most_; }
    void took(unsigned long long w) { steady_ = iterations_of(w) == 1 ? steady_ + 1 : 0; }

  private:
    static constexpr uint64_t kSteadyLaunches = 16;
    uint64_t few_, most_, steady_ = 0;
};

// Counts a published word in; true when it says the loop is done.
inline bool loop_step(unsigned long long w, const char* what, uint64_t max_iters, uint64_t& consumed, uint64_t* items) {
    if (w & kSlotFailed) fail(EVQ_EDEVICE, std::string(what) + ": a team of blocks gave up waiting for its members");
    const uint32_t n = (uint32_t)w, it = iterations_of(w);
    if (trace_loops())
        fprintf(stderr, "[evq] %s iteration %llu: %u (%u iterations)\n", what, (unsigned long long)consumed, n, it);
    if (items) *items += n;
    consumed += it;
    if (consumed > max_iters) fail(EVQ_ENOCONV, std::string(what) + " exceeded its iteration cap");
    return (w & kSlotDone) != 0;
}

// Inside a no-allocation call: the published words go to the first bytes of
// the scratch array; each batch of launches (one more than in flight
// otherwise) is followed by one copy of its counts to host memory and a stream
// synchronisation.
template <typename IssueFn>
uint64_t drive_loop_sync(IssueFn issue, int& f_parity, hipStream_t s, uint64_t max_iters, const char* what,
                         uint64_t* items, uint64_t depth, NoAlloc& na) {
    static_assert(kNoAllocSlotBytes >= 33 * 8, "slots of one batch");
    unsigned long long* dslots = reinterpret_cast<unsigned long long*>(na.base);
    InFlight flight(depth);
    unsigned long long h[33];
    uint64_t issued = 0, consumed = 0;
    for (;;) {
        const uint64_t batch = flight.launches() + 1;
        for (uint64_t j = 0; j < batch; ++j, ++issued) {
            issue(issued, f_parity, issued == 0, dslots + j);
            f_parity ^= 1;
        }
        EVQ_HIP(hipMemcpyAsync(h, dslots, batch * 8, hipMemcpyDeviceToHost, s));
        EVQ_HIP(hipStreamSynchronize(s));
        for (uint64_t j = 0; j < batch; ++j) {
            if (loop_step(h[j], what, max_iters, consumed, items)) return consumed;
            flight.took(h[j]);
        }
    }
}

template <typename IssueFn>
uint64_t drive_loop(IssueFn issue, int& f_parity, hipStream_t s, uint64_t max_iters, const char* what,
                    uint64_t* items, uint64_t depth) {
    if (NoAlloc* na = noalloc_ctx()) return drive_loop_sync(issue, f_parity, s, max_iters, what, items, depth, *na);
    InFlight flight(depth);
    HostSlots& hs = HostSlots::get();
    uint64_t issued = 0, taken = 0, consumed = 0;
    const uint64_t base = hs.next;
    struct Advance {
        HostSlots& hs;
        const uint64_t& end;
        ~Advance() { hs.next = end; }
    };
    uint64_t end = base;
    Advance adv{hs, end};
    for (;;) {
        while (issued < taken + flight.launches()) {
            const uint32_t k = (uint32_t)((base + issued) % HostSlots::kSlots);
            __atomic_store_n(&hs.host()[k], HostSlots::kEmpty, __ATOMIC_RELEASE);
            issue(issued, f_parity, issued == 0, hs.dev() + k);
            f_parity ^= 1;
            ++issued;
            end = base + issued;
        }
        volatile unsigned long long* slot = hs.host() + ((base + taken) % HostSlots::kSlots);
        wait_slot(slot, s, what);
        ++taken;
        const unsigned long long w = *slot;
        if (loop_step(w, what, max_iters, consumed, items)) break;
        flight.took(w);
    }
    return consumed;
}

}  // namespace evq
