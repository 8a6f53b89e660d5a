// gfx950 kernels for push-relabel max-flow with dynamic capacity updates.
//
// Method: Kannappan, Kumar and Nasre, "Efficient Dynamic MaxFlow Computation
// on GPUs" (arXiv 2511.05895).  Static solve: Sec. 3, Alg. 1-3.  Dynamic
// repair: Sec. 4.1, Alg. 4-5.  Execution: data-driven worklists (Sec. 5.3) or
// topology-driven sweeps (Sec. 5.2) over a bi-directional CSR (Sec. 5.1).
//
// Design for CDNA4 (not the paper's CUDA design):
//  * One persistent kernel runs the whole solve loop (global relabel -> active
//    test -> push/relabel -> invalid-edge removal) with grid-wide barriers
//    between phases, so no host round trip happens inside a solve.  With one
//    workgroup the barrier is a plain workgroup barrier.
//  * The backward BFS expands frontier items of at most kChunk arcs with a
//    wavefront-wide load-balanced scan (prefix sum over item lengths, each lane
//    takes one arc), so a hub's arcs spread over many wavefronts and low-degree
//    frontiers still fill all 64 lanes.  The active worklist is built during the
//    same BFS (a discovered vertex with positive excess is active), with
//    ballot/mbcnt compaction and one atomic per wavefront, or per workgroup
//    (LDS staging) on large levels; small frontiers and short round lists stay
//    in the LDS of a team on one XCD, or of one workgroup (runs of levels
//    and rounds, see bfs_run and pr_rounds).
//  * Push/relabel gives a group of lanes to a vertex with at most kLightMaxDeg
//    arcs, a wavefront to a longer list and a workgroup to a huge one.  Every
//    counter or list that all workgroups share is updated once per workgroup
//    and round (LDS sums and staging): atomics on one address serialise, and a
//    round has thousands of wavefronts.
//  * Memory ordering: only the owner lowers c_f of its arcs and its own excess
//    during a sweep; others only raise them.  The first cycle of a visit takes
//    an arc's residual from the {head, residual} record it loads anyway (read
//    after the round's barrier, so at most stale-low); later cycles of the
//    same visit, and every excess, use device-scope atomic loads, so a push
//    never exceeds the latest residual or excess.  Heights may be stale, which
//    the method tolerates (Sec. 3: invalid edges are repaired by
//    RemoveInvalidEdges).
#include "mf_internal.h"

#include <mutex>

namespace mf {

// ---------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Scoped atomics.  The one-workgroup solve kernel works at workgroup scope
// (atomics resolve in the compute unit's own caches); the multi-workgroup
// kernel and the update kernels need device scope, because gfx950 spreads a
// grid over eight XCDs with separate L2 caches.
constexpr int kAgent = __HIP_MEMORY_SCOPE_AGENT;
constexpr int kGroup = __HIP_MEMORY_SCOPE_WORKGROUP;
// A team whose workgroups all run on one XCD (kXcd) shares that XCD's L2.  Its
// stores reach the L2 once the storing wave has waited for them, its atomics
// resolve there, and a load that skips the L1 (a relaxed agent-scope load)
// reads it, so the team needs no L2 write-back and no invalidation at its
// barriers.  Every load of data that the loop changes goes through get<SC>,
// which skips the L1 for such a team (the L1 of another compute unit may hold
// a stale line, and the only instruction that drops it drops the L2's lines
// too) and is a plain load for the others.
constexpr int kXcd = 100;
template <int SC>
constexpr int scope_of = SC == kXcd ? kAgent : SC;

template <int SC>
__device__ __forceinline__ int32_t ld(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, scope_of<SC>);
}
template <int SC>
__device__ __forceinline__ int64_t ld(const int64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, scope_of<SC>);
}
template <int SC>
__device__ __forceinline__ int32_t get(const int32_t *p) {
    if constexpr (SC == kXcd) return ld<SC>(p);
    else return *p;
}
template <int SC>
__device__ __forceinline__ int64_t get(const int64_t *p) {
    if constexpr (SC == kXcd) return ld<SC>(p);
    else return *p;
}
template <int SC>
__device__ __forceinline__ int2 get(const int2 *p) {
    if constexpr (SC == kXcd) {
        const int64_t x = ld<SC>(reinterpret_cast<const int64_t *>(p));
        return make_int2((int)(uint32_t)x, (int)((uint64_t)x >> 32));
    } else {
        return *p;
    }
}
template <int SC>
__device__ __forceinline__ void add(int32_t *p, int32_t v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, scope_of<SC>);
}
template <int SC>
__device__ __forceinline__ void add(int64_t *p, int64_t v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, scope_of<SC>);
}
template <int SC>
__device__ __forceinline__ int32_t fetch_add(int32_t *p, int32_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, scope_of<SC>);
}
template <int SC>
__device__ __forceinline__ int64_t fetch_add(int64_t *p, int64_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, scope_of<SC>);
}
template <int SC>
__device__ __forceinline__ int32_t xchg(int32_t *p, int32_t v) {
    return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, scope_of<SC>);
}
template <int SC>
__device__ __forceinline__ bool cas(int32_t *p, int32_t expected, int32_t desired) {
    return __hip_atomic_compare_exchange_strong(p, &expected, desired, __ATOMIC_RELAXED,
                                                __ATOMIC_RELAXED, scope_of<SC>);
}

// The value found (the swap happened when it is `expected`).
template <int SC>
__device__ __forceinline__ int32_t cas_seen(int32_t *p, int32_t expected, int32_t desired) {
    __hip_atomic_compare_exchange_strong(p, &expected, desired, __ATOMIC_RELAXED, __ATOMIC_RELAXED, scope_of<SC>);
    return expected;
}

// Workgroup barrier after which every wave may read what the others stored.
// With loads that skip the L1 (kXcd) each wave first waits until its own
// stores and atomics have reached the L2.
template <int SC>
__device__ __forceinline__ void block_sync() {
    if constexpr (SC == kXcd) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// residual capacity field of arc a
__device__ __forceinline__ int32_t *cf_ptr(int2 *arc, int32_t a) {
    return reinterpret_cast<int32_t *>(arc) + 2 * (int64_t)a + 1;
}

// Wavefront scans and reductions on the vector ALU's lane-shift paths (DPP):
// row shifts by 1, 2, 4, 8 inside rows of 16 lanes, then the last lane of one
// row added to the next row and of the first half to the second.  A step costs
// a few cycles, where a shuffle goes through the LDS unit and returns after
// about a hundred; a push/relabel or BFS step has dozens of them one after
// another.  Every lane of the wavefront must call them.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp(int identity, int x) {
    return __builtin_amdgcn_update_dpp(identity, x, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int64_t dpp(int64_t identity, int64_t x) {
    const uint32_t lo = (uint32_t)dpp<CTRL, ROWS>((int)(uint32_t)identity, (int)(uint32_t)x);
    const uint32_t hi = (uint32_t)dpp<CTRL, ROWS>((int)((uint64_t)identity >> 32), (int)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <typename T, typename OP>
__device__ __forceinline__ T wave_scan(T x, T identity, OP op) {
    x = op(x, dpp<0x111, 0xf>(identity, x));  // row_shr 1
    x = op(x, dpp<0x112, 0xf>(identity, x));
    x = op(x, dpp<0x114, 0xf>(identity, x));
    x = op(x, dpp<0x118, 0xf>(identity, x));
    x = op(x, dpp<0x142, 0xa>(identity, x));  // row_bcast 15 into rows 1 and 3
    x = op(x, dpp<0x143, 0xc>(identity, x));  // row_bcast 31 into rows 2 and 3
    return x;
}
// value of a lane known at compile time or alike in all lanes
__device__ __forceinline__ int lane_value(int x, int lane) { return __builtin_amdgcn_readlane(x, lane); }
__device__ __forceinline__ int64_t lane_value(int64_t x, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)((uint64_t)x >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int wave_incl_scan(int x) {
    return wave_scan(x, 0, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ int64_t wave_incl_scan64(int64_t x) {
    return wave_scan(x, (int64_t)0, [](int64_t a, int64_t b) { return a + b; });
}
__device__ __forceinline__ int64_t wave_sum(int64_t x) { return lane_value(wave_incl_scan64(x), 63); }
__device__ __forceinline__ int wave_sum(int x) { return lane_value(wave_incl_scan(x), 63); }
__device__ __forceinline__ int wave_min(int x) {
    return lane_value(wave_scan(x, INT32_MAX, [](int a, int b) { return min(a, b); }), 63);
}
__device__ __forceinline__ uint64_t wave_or(uint64_t x) {
    return (uint64_t)lane_value(wave_scan((int64_t)x, (int64_t)0, [](int64_t a, int64_t b) { return a | b; }), 63);
}
// Minimum over a group of 8 lanes (pairs, then quads, then the mirrored half
// row), for all of them; lanes outside a group may idle.
__device__ __forceinline__ int group8_min(int x) {
    x = min(x, dpp<0xb1, 0xf>(x, x));
    x = min(x, dpp<0x4e, 0xf>(x, x));
    return min(x, dpp<0x141, 0xf>(x, x));
}

__device__ __forceinline__ int mask_rank(uint64_t mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Reserve one slot per lane with pred; one atomic per wavefront.  Every lane
// of the wavefront must call it.  Returns the slot, or -1 without pred.
template <int SC>
__device__ __forceinline__ int wave_append1(int32_t *counter, bool pred) {
    uint64_t mask = __ballot(pred);
    if (mask == 0) return -1;
    int leader = __ffsll((unsigned long long)mask) - 1;
    int base = 0;
    if (lane_id() == leader) base = fetch_add<SC>(counter, __popcll(mask));
    base = lane_value(base, __builtin_amdgcn_readfirstlane(leader));
    return pred ? base + mask_rank(mask) : -1;
}

// A slot for each lane that is active here (all with the same counter), one
// atomic for them all: what the stages of a round have no room for comes by the
// million, onto one word.  (Left to the compiler, which finds neither the
// counter's address nor the lanes alike: solve of a star, s - 4 M vertices - t, half
// of them listed and relabelled at once, 42 ms; 10.2 ms so.)
template <int SC>
__device__ __forceinline__ int append_here(int32_t *counter) {
    const uint64_t mask = __ballot(true);
    const int leader = __ffsll((unsigned long long)mask) - 1;
    int base = 0;
    if (lane_id() == leader) base = fetch_add<SC>(counter, __popcll(mask));
    return lane_value(base, __builtin_amdgcn_readfirstlane(leader)) + mask_rank(mask);
}

// Reserve c slots per lane (c >= 0); one atomic per wavefront.  Every lane must
// call it.  Returns the first slot of this lane's range.
template <int SC>
__device__ __forceinline__ int wave_appendn(int32_t *counter, int c) {
    int incl = wave_incl_scan(c);
    const int total = lane_value(incl, 63);
    if (total == 0) return 0;
    int base = 0;
    if (lane_id() == 63) base = fetch_add<SC>(counter, total);
    base = lane_value(base, 63);
    return base + incl - c;
}

// One of a view's rotating buffers by a number known only at run time: picked by
// selects (an indexed read of the kernel's argument would put a copy of the
// whole view in scratch memory).
__device__ __forceinline__ int2 *frontier(const DevGraph &g, int L) { return (L & 1) ? g.q[1] : g.q[0]; }
__device__ __forceinline__ int32_t *round_list(const DevGraph &g, int k) {
    return k == 0 ? g.list[0] : k == 1 ? g.list[1] : g.list[2];
}
__device__ __forceinline__ int32_t *huge_list(const DevGraph &g, int k) {
    return k == 0 ? g.huge[0] : k == 1 ? g.huge[1] : g.huge[2];
}

__device__ __forceinline__ int n_items(int deg) { return (deg + kChunk - 1) / kChunk; }

// Appends of a round to the next round's list are staged per workgroup in
// LDS (up to kStageCap light and kStageCap long-list vertices) and reserved
// with one atomic per workgroup and list at the end of the round; beyond
// that, or without a stage, a lane appends on its own.  A vertex enters a
// list at most once (mark[]), so no list outgrows its |V| slots.
constexpr int kStageCap = 1024;

// A value every lane of the wavefront holds alike (read after a barrier),
// moved to a scalar register so it does not occupy a vector register.
__device__ __forceinline__ int32_t uniform(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform(int64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The workgroups that run one solve loop together: ranks 0..size-1.  Either
// the workgroups of a launch that joined (join_team), or a single workgroup of a batched
// launch (then every barrier is a workgroup barrier).
struct Team {
    int rank, size;
    __device__ int64_t tid() const { return (int64_t)rank * blockDim.x + threadIdx.x; }
    __device__ int64_t nthreads() const { return (int64_t)size * blockDim.x; }
    __device__ int64_t wave() const { return (int64_t)rank * (blockDim.x >> 6) + (threadIdx.x >> 6); }
    __device__ int64_t nwaves() const { return (int64_t)size * (blockDim.x >> 6); }
};

// Number of the XCD that runs this wave: hardware register XCC_ID (id 20), low
// four bits.
__device__ __forceinline__ int xcd_id() { return (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & (kXccIds - 1)); }

// Barrier of a team with a bounded wait.  Arrivals count up monotonic counters
// (cleared before every launch).  A team of one XCD has one counter and needs
// no cache maintenance.  A team all over the device arrives XCD by XCD: the
// workgroups of an XCD wait until their stores are in its L2 and count up the
// XCD's counter, and the last of them alone writes that L2 back (the release
// fence) and counts up the top counter, which every workgroup polls.  The
// write-back is what such a barrier costs; made by every workgroup
// such a barrier of 256 took 8.5 to 10.4 us, made once per XCD 3.9 to 5.2
// (solve of R-MAT 2^22 x 16: 8.67 -> 8.25 ms, 1000 x 1000 grid: 175 -> 162 ms).
// How many workgroups an XCD has in the team is counted at the first barrier
// (`epoch` 0), at which every workgroup writes back and arrives at bar_count.
// One acquire fence after the wait; the polls themselves are relaxed loads,
// so waiting does not keep invalidating the caches that the team's other
// workgroups are still working from.  Returns false when the wait ran out
// (wall clock, `limit` ticks) or another workgroup aborted; the caller must
// then leave the kernel, so every workgroup ends even if co-residency ever
// failed.  Every thread of every workgroup of the team calls it with the same
// epoch, which it advances.
template <int SC>
__device__ __forceinline__ bool grid_barrier(Ctrl *c, const Team &tm, uint32_t &epoch, int64_t limit) {
    if constexpr (SC == kAgent) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    block_sync<SC>();
    if (tm.size == 1) return true;
    __shared__ int s_ok;
    __shared__ uint32_t s_members, s_xcds;  // the team's workgroups on this XCD, its XCDs
    if (threadIdx.x == 0) {
        int ok = 1;
        uint32_t target;
        PaddedU32 *top = &c->bar_count;
        if (SC == kXcd || epoch == 0) {
            if constexpr (SC == kAgent) {
                __hip_atomic_fetch_add(&c->bar_members[xcd_id()].v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            }
            target = (epoch + 1u) * (uint32_t)tm.size;
            __hip_atomic_fetch_add(&top->v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            top = &c->bar_top;
            target = epoch * s_xcds;
            if (__hip_atomic_fetch_add(&c->bar_xcd[xcd_id()].v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u ==
                epoch * s_members) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                __hip_atomic_fetch_add(&top->v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        uint32_t spins = 0;
        uint64_t tw = 0;
        while ((int32_t)(__hip_atomic_load(&top->v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0) {
            if ((++spins & 255u) == 0) {
                if (tw == 0) tw = wall_clock64();
                if (__hip_atomic_load(&c->abort.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
                    (int64_t)(wall_clock64() - tw) > limit) {
                    __hip_atomic_store(&c->abort.v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ok = 0;
                    break;
                }
            }
        }
        if constexpr (SC == kAgent) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (epoch == 0) {
                uint32_t xcds = 0;
                for (int x = 0; x < kXccIds; ++x)
                    xcds += __hip_atomic_load(&c->bar_members[x].v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
                s_xcds = xcds;
                s_members = __hip_atomic_load(&c->bar_members[xcd_id()].v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        s_ok = ok;
    }
    ++epoch;
    __syncthreads();
    return s_ok != 0;
}

// LDS of a run: consecutive BFS levels or push/relabel rounds whose frontier or
// list stays in the workgroups' LDS (see bfs_run and rounds_run).
constexpr int kRunItems = 1024;
struct RunStage {
    // BFS: frontier items of two levels, kRunItems each; rounds: short lists
    // of two rounds, then long lists of two rounds, kStageCap each
    int32_t buf[4 * kRunItems];
    // BFS: active vertices found, rounds: vertices for RemoveInvalidEdges;
    // short lists, then long ones
    int32_t aux[2 * kStageCap];
    int32_t lcnt[2], hcnt[2], rcnt[2];
    // BFS, of the two levels in buf: frontier items (spilled ones too) and the
    // arcs of the vertices discovered (0 for those that the run starts with)
    int32_t found[2], larcs[2];
    uint64_t act;   // BFS: short (low half) and long active vertices found in this run
    int32_t spill;     // something did not fit and went to the global lists
    int32_t firsts;    // rounds: vertices relabelled for the first time in the phase
    int32_t relabels;  // of this round
    int32_t deliv;     // this round delivered excess
    int32_t base[4];
    int64_t acc[4];    // of the run: excess into t, relabels, pushes, deliveries into deficits
    int64_t arcs;      // arcs of the vertices that a BFS run discovered, its last level left out
    uint64_t total;    // sum of the last team_sum
    int32_t ok;
};
// The workgroup's one RunStage.  (Functions name it here instead of taking a
// pointer, so that every access is known to be LDS.)
__device__ __forceinline__ RunStage *run_stage() {
    __shared__ RunStage s;
    return &s;
}
static_assert(kStageCap == kRunItems, "the two views of RunStage::buf");

// Barrier of a run that also adds up one word per workgroup (thread 0's
// `mine`, below 2^56 in sum): a level or round ends with one atomic and its
// poll, and the poll brings the totals that the next decision needs.  The
// words rotate over four, each cleared by the leader two barriers before its
// next use.  Only for teams of one workgroup, or of one XCD (no cache
// maintenance; call block_sync first).  Every thread of the team calls it.
template <int SC>
__device__ __forceinline__ uint64_t team_sum(BarWords *c, const Team &tm, uint32_t &epoch, uint64_t mine, int64_t limit, bool *ok) {
    RunStage *rs = run_stage();
    if (threadIdx.x == 0) {
        int good = 1;
        uint64_t x = mine;
        if (tm.size > 1) {
            uint64_t *word = &c->sum[epoch & 3u].v;
            constexpr uint64_t one = 1ull << 56;
            x = __hip_atomic_fetch_add(word, mine + one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine + one;
            uint32_t spins = 0;
            uint64_t t0 = 0;
            while ((int)(x >> 56) != tm.size) {
                if ((++spins & 1023u) == 0) {
                    if (t0 == 0) t0 = wall_clock64();
                    if (__hip_atomic_load(&c->abort.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
                        (int64_t)(wall_clock64() - t0) > limit) {
                        __hip_atomic_store(&c->abort.v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        good = 0;
                        break;
                    }
                }
                x = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (tm.rank == 0) c->sum[(epoch + 2u) & 3u].v = 0;
            x &= one - 1;
        }
        rs->total = x;
        rs->ok = good;
    }
    ++epoch;
    __syncthreads();
    *ok = rs->ok != 0;
    return (uint64_t)uniform((int64_t)rs->total);
}

// Waits until `want` workgroups have registered in *joined or `limit` ticks have
// passed, closes it and publishes the team's size (the first of them calls it).
constexpr uint32_t kTeamClosed = 0x80000000u;
__device__ __forceinline__ uint32_t close_team(uint32_t *joined, uint32_t *size, int want, int64_t limit) {
    const uint64_t t0 = wall_clock64();
    while ((int)__hip_atomic_load(joined, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want &&
           (int64_t)(wall_clock64() - t0) < limit) {
    }
    const uint32_t n = __hip_atomic_fetch_or(joined, kTeamClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(size, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return n;
}

// The team of a launch forms itself: the workgroups that arrive register, the
// first of them closes the team once `want` have registered or `limit` ticks
// have passed, and whoever arrives later leaves the kernel.  A
// team is thus made of workgroups that are running already, whatever else
// occupies the device, so its barriers need no co-residency promise (and no
// cooperative launch, whose host call costs several times a plain one's).
//
// With kXcd the launch has `want` workgroups for every XCD.  Each registers on
// its own, and the first XCD to have them all is the team's; the others' leave.
// If none is complete after a quarter of `limit` (other work holds units of
// them all, perhaps another launch of this kind that waits in the same way), it
// is the one with the most, ties broken differently for different handles; what
// leaves the others then makes room for its rest.
//
// Returns size 0 to a workgroup that is not in the team.  Every thread calls it
// once, before any grid barrier, on a cleared control block.
template <int SC>
__device__ __forceinline__ Team join_team(Ctrl *c, int want, int64_t limit) {
    __shared__ int s_rank, s_size;
    if (threadIdx.x == 0) {
        uint32_t *joined = &c->join.v;
        const uint32_t me = (uint32_t)xcd_id() + 1u;
        if constexpr (SC == kXcd) joined = &c->bar_xcd[me - 1u].v;  // (such a team's barrier does not use it)
        const uint32_t rank = __hip_atomic_fetch_add(joined, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool in = rank < (uint32_t)want;
        if constexpr (SC == kXcd) {
            if (in) {
                uint32_t pick = 0, none = 0;
                if (rank + 1u == (uint32_t)want)
                    __hip_atomic_compare_exchange_strong(&c->xcd_pick.v, &none, me, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
                const uint64_t t0 = wall_clock64();
                while ((pick = __hip_atomic_load(&c->xcd_pick.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) {
                    __builtin_amdgcn_s_sleep(1);
                    if ((int64_t)(wall_clock64() - t0) < limit / 4) continue;
                    const uint32_t from = ((uint32_t)(reinterpret_cast<uint64_t>(c) >> 8) * 2654435761u) >> 29;
                    uint32_t most = 0, at = 0;
                    for (uint32_t k = 0; k < (uint32_t)kXccIds; ++k) {
                        const uint32_t x = (from + k) & (kXccIds - 1);
                        const uint32_t n = __hip_atomic_load(&c->bar_xcd[x].v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (n > most) {
                            most = n;
                            at = x + 1u;
                        }
                    }
                    none = 0;
                    __hip_atomic_compare_exchange_strong(&c->xcd_pick.v, &none, at, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
                }
                in = pick == me;
            }
        }
        uint32_t size = 0;
        if (in) {
            if (rank == 0) {
                size = close_team(joined, &c->team_size.v, want, limit);
            } else {
                while ((size = __hip_atomic_load(&c->team_size.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0)
                    __builtin_amdgcn_s_sleep(1);
            }
            if (SC == kXcd && size > (uint32_t)want) size = (uint32_t)want;
        }
        s_rank = (int)rank;
        s_size = (int)size;
    }
    __syncthreads();
    return Team{s_rank, s_size};
}

// Per-thread event counters (32-bit), summed into the 64-bit Ctrl::stat at the
// end of every loop round and of the kernel, then cleared.
struct Tally {
    uint32_t bfs_v = 0, bfs_a = 0, pr_cyc = 0, pr_a = 0, push = 0, relabel = 0, rie_a = 0, rie_sat = 0;
    int64_t deliv = 0;  // excess this lane delivered into deficient vertices (per round)
};

// Every thread of the workgroup must call it.
template <int SC>
__device__ __forceinline__ void flush_tally(Ctrl *c, Tally &t) {
    __shared__ int64_t s_acc[8];
    if (threadIdx.x < 8) s_acc[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t v[8] = {t.bfs_v, t.bfs_a, t.pr_cyc, t.pr_a, t.push, t.relabel, t.rie_a, t.rie_sat};
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int64_t w = wave_sum((int64_t)v[i]);
        if (lane_id() == 0 && w) atomicAdd((unsigned long long *)&s_acc[i], (unsigned long long)w);
    }
    __syncthreads();
    const int slot[8] = {kStBfsVertices, kStBfsArcs, kStPrCycles, kStPrArcs,
                         kStPushes,      kStRelabels, kStRieArcs, kStRieSat};
    if (threadIdx.x < 8 && s_acc[threadIdx.x]) add<SC>(&c->stat[slot[threadIdx.x]], s_acc[threadIdx.x]);
    t = Tally{};
}

// ---------------------------------------------------------------------------
// Global relabel (Alg. 4 height reset + BFS_Backward)
// ---------------------------------------------------------------------------

// Height reset: t and every deficient vertex other than s are roots (height
// 0); all others get |V|.  Roots become the level-0 frontier.  With part
// tags, only vertices of the wanted part can be roots, and with part_restrict
// the heights of the other vertices are left alone.  Returns the lane's share
// of the deficits, of all parts.
//
// One pass over e and h, bound by the latency of its loads where the team has
// fewer threads than the graph vertices: a wavefront then has U = 4 groups of
// 64 vertices in flight, and the work for roots, which are few, is left to the
// wavefronts that find one.  4.2 M vertices on 256 workgroups, this pass and a second one for
// the deficits after the last relabel: 100 us of solve kernel per update, 85 us
// with the groups and without the second pass.
template <int SC, int U>
__device__ __forceinline__ int64_t bfs_roots_by(const DevGraph &g, const Team &tm, bool counts, bool feats, bool track, Tally &tl) {
    const int lane = lane_id();
    int64_t deficit = 0;
    for (int64_t base = tm.wave() * 64 * U; base < g.n; base += tm.nwaves() * 64 * U) {
        bool root[U];
        bool any = false;
        int64_t ev[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t i = base + 64 * k + lane;
            ev[k] = i < g.n ? get<SC>(&g.e[i]) : 0;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t i = base + 64 * k + lane;
            const int v = (int)i;
            root[k] = false;
            if (i < g.n) {
                if (ev[k] < 0 && v != g.s && v != g.t) deficit += ev[k];
                const bool mine = !g.part || g.part[v] == g.part_want;
                if (mine || !g.part_restrict) {
                    root[k] = mine && (v == g.t || (v != g.s && ev[k] < 0));
                    g.h[v] = root[k] ? 0 : g.n;
                }
            }
            any |= root[k];
        }
        if (__ballot(any) == 0) continue;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int v = (int)(base + 64 * k + lane);
            const int nroot = __popcll(__ballot(root[k]));
            if (nroot == 0) continue;
            const int beg = root[k] ? g.row_ptr[v] : 0, end = root[k] ? g.row_ptr[v + 1] : 0;
            const int c = root[k] ? n_items(end - beg) : 0;
            if (counts && lane == 0) add<SC>(&g.hcount[0], nroot);
            if (feats && lane == 0) add<SC>(&g.ctrl->feat_reached, nroot);
            if (track) {
                const int64_t ra = wave_sum((int64_t)(end - beg));
                if (lane == 0) {
                    add<SC>(&g.ctrl->qverts[0], nroot);
                    add<SC>(&g.ctrl->qarcs[0], ra);
                }
            }
            const int at = wave_appendn<SC>(&g.ctrl->qcount[0], c);
            for (int j = 0; j < c; ++j)
                g.q[0][at + j] = make_int2(beg + j * kChunk, min(beg + (j + 1) * kChunk, end));
            tl.bfs_v += root[k];
        }
    }
    return deficit;
}
template <int SC>
__device__ __forceinline__ int64_t bfs_roots(const DevGraph &g, const Team &tm, bool counts, bool feats, bool track, Tally &tl) {
    return g.n > tm.nthreads() ? bfs_roots_by<SC, 4>(g, tm, counts, feats, track, tl)
                               : bfs_roots_by<SC, 1>(g, tm, counts, feats, track, tl);
}

// Features of the learned schedule: excess sum of the active vertices a BFS
// finds and their count per bin of floor(log2 e) / 4.  Wave-uniform calls.
template <int SC>
__device__ __forceinline__ void feature_tally(Ctrl *c, bool active, int64_t ev) {
    if (__ballot(active) == 0) return;
    const int64_t es = wave_sum(active ? ev : (int64_t)0);
    const int bin = active ? min(7, (63 - __clzll((unsigned long long)ev)) >> 2) : -1;
    if (lane_id() == 0) add<SC>(&c->feat_esum, es);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const int cb = __popcll(__ballot(bin == b));
        if (lane_id() == 0 && cb) add<SC>(&c->feat_hist[b], cb);
    }
}

// Per-workgroup staging of a large BFS level's output in LDS: frontier items
// and active-list entries are reserved in LDS first and the workgroup then
// reserves its whole share of each global list with one atomic, instead of
// every wavefront step hitting the same few global counters.  A reservation
// that does not fit goes to the global list directly, so nothing is lost and
// no slot stays unwritten.
constexpr int kBfsStageItems = 2048;
// frontier size (items) from which a level stages its output
constexpr int kBfsStageMin = 1024;
struct BfsStage {
    int2 items[kBfsStageItems];
    int32_t light[kStageCap], heavy[kStageCap];
    int32_t cnt[4];  // items, light, heavy, discovered vertices of this level
    int32_t res[6];  // the level's flush: global bases, then counts, of items, light, heavy
    int64_t arcs;    // arcs of the vertices this level discovered (direction rule)
    // the direction rule's tallies of a level that is not staged (vertices
    // and arcs discovered), added to the global counters once per workgroup:
    // per wavefront step they would queue behind the frontier reservations
    // on the same cache line
    int32_t tverts;
    int64_t tarcs;
};

// The workgroup's one BfsStage (teams of several workgroups only).
__device__ __forceinline__ BfsStage *bfs_stage() {
    __shared__ BfsStage s;
    return &s;
}

// Reserve k slots of an LDS counter if they fit under cap (no partial
// reservation); returns the first slot or -1.
__device__ __forceinline__ int stage_reserve(int32_t *ctr, int k, int cap) {
    int old = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    for (;;) {
        if (old + k > cap) return -1;
        if (__hip_atomic_compare_exchange_strong(ctr, &old, old + k, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
            return old;
    }
}

// Output of one 64-lane BFS step (every lane of the wavefront calls it): a
// lane that discovered v (disc; its arc range [vbeg, vend) and excess ev)
// appends v's frontier items for the next level and, when v is active (A of
// Alg. 1: e > 0 and h < |V|, t excluded), v to the active worklist.  The
// frontier items, both halves of the active list through one packed 64-bit
// counter {light, heavy}, and the level's vertex and arc tallies are reserved
// by one lane, back to back so their round trips overlap, or in the
// workgroup's stage (st).  counts: per-height vertex counts (gap heuristic);
// feats: the schedule's features; track: vertices and arcs discovered per
// level (the direction rule of the BFS), tallied in tst when the level is not
// staged (null: straight to the global counters).
template <int SC>
__device__ __forceinline__ void bfs_emit(const DevGraph &g, int L, bool disc, int v, int vbeg, int vend, int64_t ev,
                                         bool feats, bool counts, bool track, bool staged, int2 *qout,
                                         int32_t *qout_count, Tally &tl) {
    BfsStage *st = bfs_stage();
    const int lane = lane_id();
    const int n = g.n;
    bool active = false;
    if (disc) {
        active = (v != g.t) && ev > 0;
        tl.bfs_v++;
    } else {
        vbeg = vend = 0;
    }
    if (feats) feature_tally<SC>(g.ctrl, active, ev);
    const int vdeg = vend - vbeg;
    const int c = disc ? n_items(vdeg) : 0;
    const int cincl = wave_incl_scan(c);
    const int ctotal = lane_value(cincl, 63);
    const bool light = active && vdeg <= kLightMaxDeg;
    const bool heavy = active && vdeg > kLightMaxDeg && vdeg <= kHugeDeg;
    const bool huge = active && vdeg > kHugeDeg;
    const uint64_t lm = __ballot(light), hm = __ballot(heavy);
    const int ndisc = counts || feats || track ? __popcll(__ballot(disc)) : 0;
    const int64_t darcs = track ? (int64_t)wave_sum(vdeg) : 0;  // at most A < 2^31
    int qbase = 0, lsb = -1, hsb = -1, qsb = -1;
    int64_t lbase = 0;
    if (lane == 63) {
        const int nl = __popcll(lm), nh = __popcll(hm);
        if (SC != kGroup && staged) {
            if (ctotal) qsb = stage_reserve(&st->cnt[0], ctotal, kBfsStageItems);
            if (nl) lsb = stage_reserve(&st->cnt[1], nl, kStageCap);
            if (nh) hsb = stage_reserve(&st->cnt[2], nh, kStageCap);
            if (ndisc) atomicAdd(&st->cnt[3], ndisc);
            if (darcs) atomicAdd(reinterpret_cast<unsigned long long *>(&st->arcs), (unsigned long long)darcs);
        } else if (ndisc) {
            if (counts) add<SC>(&g.hcount[L + 1], ndisc);
            if (feats) add<SC>(&g.ctrl->feat_reached, ndisc);
            if (SC != kGroup && track) {
                atomicAdd(&st->tverts, ndisc);
                atomicAdd(reinterpret_cast<unsigned long long *>(&st->tarcs), (unsigned long long)darcs);
            }
        }
        if (ctotal && qsb < 0) qbase = fetch_add<SC>(qout_count, ctotal);
        const int gl = lsb < 0 ? nl : 0, gh = hsb < 0 ? nh : 0;
        if (gl | gh)
            lbase = fetch_add<SC>(reinterpret_cast<int64_t *>(&g.ctrl->lst[0]), ((int64_t)gh << 32) | (int64_t)gl);
    }
    qbase = lane_value(qbase, 63);
    lbase = lane_value(lbase, 63);
    qsb = lane_value(qsb, 63);
    lsb = lane_value(lsb, 63);
    hsb = lane_value(hsb, 63);
    const int qb = cincl - c;
    for (int k = 0; k < c; ++k) {
        const int2 item = make_int2(vbeg + k * kChunk, min(vbeg + (k + 1) * kChunk, vend));
        if (qsb < 0) qout[qbase + qb + k] = item;
        else st->items[qsb + qb + k] = item;
    }
    if (light) {
        if (lsb < 0) g.list[0][(int)(uint32_t)lbase + mask_rank(lm)] = v;
        else st->light[lsb + mask_rank(lm)] = v;
    }
    if (heavy) {
        if (hsb < 0) g.list[0][n - 1 - ((int)(lbase >> 32) + mask_rank(hm))] = v;
        else st->heavy[hsb + mask_rank(hm)] = v;
    }
    const int su = wave_append1<SC>(&g.ctrl->lst[0].huge, huge);  // rare: hubs only
    if (huge) g.huge[0][su] = v;
}

// End of a staged BFS level: one reservation per list for the workgroup's
// staged output, then a coalesced copy (the stage counters start from zero
// again).  Every thread of the workgroup calls it.
template <int SC>
__device__ __forceinline__ void bfs_flush(const DevGraph &g, int L, bool counts, bool feats, bool track, int2 *qout,
                          int32_t *qout_count) {
    BfsStage *st = bfs_stage();
    const int n = g.n;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nq = st->cnt[0], nl = st->cnt[1], nh = st->cnt[2], nd = st->cnt[3];
        int64_t lb = 0;
        st->res[0] = nq ? fetch_add<SC>(qout_count, nq) : 0;
        if (nl | nh)
            lb = fetch_add<SC>(reinterpret_cast<int64_t *>(&g.ctrl->lst[0]), ((int64_t)nh << 32) | (int64_t)nl);
        if (nd && counts) add<SC>(&g.hcount[L + 1], nd);
        if (nd && feats) add<SC>(&g.ctrl->feat_reached, nd);
        if (nd && track) {
            add<SC>(&g.ctrl->qverts[(L + 1) % 3], nd);
            add<SC>(&g.ctrl->qarcs[(L + 1) % 3], st->arcs);
        }
        st->res[1] = (int)(uint32_t)lb;
        st->res[2] = (int)(lb >> 32);
        st->res[3] = nq;
        st->res[4] = nl;
        st->res[5] = nh;
        st->cnt[0] = st->cnt[1] = st->cnt[2] = st->cnt[3] = 0;
        st->arcs = 0;
    }
    __syncthreads();
    const int nq = st->res[3], nl = st->res[4], nh = st->res[5];
    for (int i = threadIdx.x; i < nq; i += blockDim.x) qout[st->res[0] + i] = st->items[i];
    for (int i = threadIdx.x; i < nl; i += blockDim.x) g.list[0][st->res[1] + i] = st->light[i];
    for (int i = threadIdx.x; i < nh; i += blockDim.x) g.list[0][n - 1 - (st->res[2] + i)] = st->heavy[i];
}

// End of a level that was not staged: the workgroup's direction tallies go to
// the global counters, one atomic each (every thread of the workgroup calls
// it; the next use of the tallies comes after a barrier).
template <int SC>
__device__ __forceinline__ void bfs_tally_flush(const DevGraph &g, int L) {
    BfsStage *tst = bfs_stage();
    __syncthreads();
    if (threadIdx.x == 0 && tst->tverts) {
        add<SC>(&g.ctrl->qverts[(L + 1) % 3], tst->tverts);
        add<SC>(&g.ctrl->qarcs[(L + 1) % 3], tst->tarcs);
        tst->tverts = 0;
        tst->tarcs = 0;
    }
}

// One BFS level, top-down: for every arc (w -> v) of a frontier item, v joins
// level L+1 when it is unvisited (height |V|), is not s, and has residual
// capacity toward w (the twin arc v -> w).  Newly reached vertices become
// frontier items of the next level; those with positive excess go to the
// active worklist (A of Alg. 1: e > 0 and h < |V|, s and t excluded).
// With a stage (st), the level's output is staged per workgroup and flushed
// at its end; counts: keep the per-height vertex counts (gap heuristic);
// feats: tally the schedule's features.  Every thread of the workgroup calls
// it.
template <int SC>
__device__ __forceinline__ void bfs_level(const DevGraph &g, const Team &tm, int L, int cnt, bool feats, bool counts,
                          bool track, bool lazy, bool staged, Tally &tl) {
    const int2 *qin = frontier(g, L);
    int2 *qout = frontier(g, L + 1);
    int32_t *qout_count = &g.ctrl->qcount[(L + 1) % 3];
    const int lane = lane_id();
    const int64_t gwave = tm.wave();
    const int64_t nwaves = tm.nwaves();
    const int n = g.n;
    // items per wavefront: up to 64, fewer when the frontier is small, so
    // that every wavefront of the team takes part and each one expands as
    // few 64-arc steps one after another as possible
    const int64_t ipw = min((int64_t)64, max((int64_t)1, ((int64_t)cnt + nwaves - 1) / nwaves));
    // A frontier of fewer items than half the wavefronts (a hub's list, say) is
    // cut finer, down to 64 arcs, one step each, and dealt out workgroup by
    // workgroup: R-MAT 2^20, the sink's list and two short levels, 66 -> 51 us.
    const int parts = 4 * (int64_t)cnt <= nwaves ? 4 : 2 * (int64_t)cnt <= nwaves ? 2 : 1;
    const int64_t first = parts == 1 ? gwave : (int64_t)(threadIdx.x >> 6) * tm.size + tm.rank;
    for (int64_t base = first * ipw; base < (int64_t)cnt * parts; base += nwaves * ipw) {
        const int64_t idx = base + lane;
        int beg = 0, len = 0;
        if (lane < ipw && idx < (int64_t)cnt * parts) {
            const int2 it = get<SC>(&qin[idx / parts]);  // arc range {first, end} of one item
            beg = it.x + (int)(idx % parts) * (kChunk / parts);
            len = max(0, min(it.y - beg, kChunk / parts));
        }
        const int incl = wave_incl_scan(len);
        const int excl = incl - len;
        const int total = lane_value(incl, 63);
        for (int off = 0; off < total; off += 64) {
            const int j = off + lane;
            // the lane whose item holds arc j: items are never empty, so it is
            // the number of items that start at or before j, less one
            const bool here = len > 0 && excl >= off && excl < off + 64;
            const uint64_t starts = wave_or(here ? 1ull << (excl - off) : 0ull);
            const int before = __popcll(__ballot(len > 0 && excl < off));
            const int o = before + mask_rank(starts) + (int)((starts >> lane) & 1ull) - 1;
            const int obeg = __shfl(beg, o, 64);
            const int oexcl = __shfl(excl, o, 64);
            bool disc = false;
            int v = -1, vbeg = 0, vend = 0;
            int64_t ev = 0;
            if (j < total) {
                const int a = obeg + (j - oexcl);
                // the head and the twin index come in one step, the head's height
                // and the twin's residual in the next; on a large level the
                // twin's residual (a gather from anywhere in the arc array) is
                // read only for heads not reached yet
                const int2 rec = get<SC>(&g.arc[a]);
                const int tw = g.twin[a];
                v = rec.x;
                const int hv = get<SC>(&g.h[v]);
                const bool cand = v != g.s && hv == n;
                int cft = 1;
                if (!lazy || cand) cft = get<SC>(cf_ptr(g.arc, tw));
                tl.bfs_a++;
                if (cand && cft > 0 && (!g.part_restrict || g.part[v] == g.part_want)) {
                    // the candidate's row bounds and excess load alongside the
                    // compare-and-swap that decides the discovery
                    vbeg = g.row_ptr[v];
                    vend = g.row_ptr[v + 1];
                    ev = get<SC>(&g.e[v]);
                    disc = cas<SC>(&g.h[v], n, L + 1);
                }
            }
            bfs_emit<SC>(g, L, disc, v, vbeg, vend, ev, feats, counts, track, staged, qout, qout_count, tl);
        }
    }
    if constexpr (SC != kGroup) {
        if (staged) bfs_flush<SC>(g, L, counts, feats, track, qout, qout_count);
        else if (track) bfs_tally_flush<SC>(g, L);
    }
}

// One BFS level, bottom-up (the direction-optimising BFS): every vertex v
// not reached yet (height |V|, not s) looks through its own arcs (v -> w)
// for one with residual capacity whose head w is on level L, and joins level
// L+1 at the first it finds.  The same vertices join the level as in the
// top-down step, but only v's own arc records and the heads' heights are
// read (no gather of twin residuals), and a vertex stops at its first
// parent.  The team walks the static item list g.bu_items: a wavefront takes
// 64 items and runs through their remaining arcs 64 at a time (load-balanced
// scan), dropping an item as soon as its vertex has a parent.  Several items
// of one long list can find parents at once; the compare-and-swap on the
// height makes one of them the discovery.  Output as in the top-down step.
// Every thread of the workgroup calls it.
template <int SC>
__device__ __forceinline__ void bfs_bottom_up(const DevGraph &g, const Team &tm, int L, bool feats, bool counts, Tally &tl) {
    int2 *qout = frontier(g, L + 1);
    int32_t *qout_count = &g.ctrl->qcount[(L + 1) % 3];
    const int lane = lane_id();
    const int n = g.n;
    const int64_t nb = g.n_bu_items;
    const int64_t nwaves = tm.nwaves();
    for (int64_t base = tm.wave() * 64; base < nb; base += nwaves * 64) {
        const int64_t idx = base + lane;
        int v = -1, beg = 0, len = 0;
        if (idx < nb) {
            const int4 it = g.bu_items[idx];
            if (it.x != g.s && get<SC>(&g.h[it.x]) == n) {
                v = it.x;
                beg = it.y;
                len = it.z - it.y;
            }
        }
        bool disc = false;
        for (;;) {
            const int incl = wave_incl_scan(len);
            const int total = lane_value(incl, 63);
            if (total == 0) break;
            const int excl = incl - len;
            // largest lane o with excl[o] <= lane (that lane still has arcs)
            int o = 0;
#pragma unroll
            for (int step = 32; step >= 1; step >>= 1) {
                const int cand = o + step;
                const int ex = __shfl(excl, cand, 64);
                if (ex <= lane) o = cand;
            }
            const int obeg = __shfl(beg, o, 64);
            const int oexcl = __shfl(excl, o, 64);
            bool hit = false;
            if (lane < total) {
                const int2 r = get<SC>(&g.arc[obeg + (lane - oexcl)]);
                if (r.y > 0) hit = get<SC>(&g.h[r.x]) == L;
                tl.bfs_a++;
            }
            const uint64_t hm = __ballot(hit);
            // this lane's item owns the step's arcs [lo, hi)
            const int lo = min(excl, 64), hi = min(incl, 64);
            const int used = hi - lo;
            const bool found = used > 0 && ((hm >> lo) & (used == 64 ? ~0ull : ((1ull << used) - 1))) != 0;
            if (found) {
                len = 0;
                disc = cas<SC>(&g.h[v], n, L + 1);
            } else {
                beg += used;
                len -= used;
            }
        }
        int vbeg = 0, vend = 0;
        int64_t ev = 0;
        if (disc) {
            vbeg = g.row_ptr[v];
            vend = g.row_ptr[v + 1];
            ev = get<SC>(&g.e[v]);
        }
        bfs_emit<SC>(g, L, disc, v, vbeg, vend, ev, feats, counts, true, true, qout, qout_count, tl);
    }
    bfs_flush<SC>(g, L, counts, feats, true, qout, qout_count);
}

// A run of BFS levels, top-down, whose frontier stays in LDS: every workgroup
// of the team keeps the items of the vertices it discovered and expands them
// in the next level, so a level needs no reservation in a shared list, no
// reload of items or counters and only the barrier that also sums the next
// frontier's size.  What bounds such a level is its chain of dependent loads
// (arc and twin, head height and twin residual, compare-and-swap), not the
// work.  Starts with the `cnt` items of level L in the global frontier; ends
// when a level finds nothing, or with the next level's items back in the
// global frontier when they hold more than `most` arcs, when a workgroup's share
// outgrew its LDS or after a quarter of the barrier's wait limit.  Returns the
// level it ended at; *ok is false when a barrier wait ran out.  Measured on an
// XCD team of 32 workgroups, segmentation grids 256^2 / 512^2: 6.4 / 8.3 us a
// level through the global frontier, 3.8 / 5.2 us in a run; push/relabel rounds
// (pr_rounds, the same way) 8.4 / 14.8 us, in runs 5.3 / 10.0 us.
template <int SC>
__device__ __forceinline__ int bfs_run(const DevGraph &g, const Team &tm, const LoopParams &p, int L, int cnt, int64_t most, bool feats,
                       bool counts, bool dir, uint32_t &epoch, Tally &tl, bool *ok) {
    RunStage *rs = run_stage();
    const int t = threadIdx.x, lane = lane_id(), w = uniform(t >> 6), nw = blockDim.x >> 6;
    const int nw_bits = 31 - __clz(nw);  // a power of two
    const int n = g.n;
    Ctrl *c = g.ctrl;
    int2 *items = reinterpret_cast<int2 *>(rs->buf);
    {
        const int2 *q = frontier(g, L);
        const int mine = (cnt - tm.rank + tm.size - 1) / tm.size;
        for (int i = t; i < mine; i += blockDim.x) items[i] = get<SC>(&q[tm.rank + i * tm.size]);
        if (t == 0) {
            rs->found[0] = mine;
            rs->found[1] = 0;
            rs->larcs[0] = rs->larcs[1] = 0;
            rs->spill = 0;
            rs->act = 0;
            rs->arcs = 0;
        }
    }
    __syncthreads();
    const uint64_t ts = wall_clock64();
    constexpr int G = 8;  // lanes per item while every item of a wavefront's batch is short
    const int gl = lane & (G - 1);
    int cur = 0;
    bool dump = false;
    for (int it = 1;; ++it) {
        if (t == 0 && tm.rank == 0) {
            c->qcount[(L + 2) % 3] = 0;
            c->qverts[(L + 2) % 3] = 0;
            c->qarcs[(L + 2) % 3] = 0;
        }
        const int m = min(rs->found[cur], kRunItems), nxt = cur ^ 1;
        const int2 *in = items + cur * kRunItems;
        int found_arcs = 0;
        // a wavefront takes 8 items at a time: 8 lanes each when none is long,
        // otherwise all lanes over the items' arcs in turn.  Items that are long on
        // average (a hub's list), and those that the run starts with, are dealt out
        // one by one when there are not enough for all wavefronts; short ones are
        // not, a step of a wavefront costs the same with 8 as with 1.  (edge_flow of
        // a 40 x 40 grid, whose t has 1600 arcs: 308 us with 8 at a time, 195 us dealt
        // out; all items dealt out, solve of a 256 x 256 grid: 25.6 -> 31 ms.)
        const bool deal = it == 1 || rs->larcs[cur] > m * 4 * G;
        const int q = uniform(deal ? min(G, (m + nw - 1) >> nw_bits) : G);
        for (int base = w * q; base < m; base += nw * q) {
            int beg = 0, len = 0;
            if (lane / G < q && base + lane / G < m) {
                const int2 item = in[base + lane / G];
                beg = item.x;
                len = item.y - item.x;
            }
            const bool spread = __ballot(len > 4 * G) != 0;
            int excl = 0, total = 0;
            if (spread) {  // item k moves to lane k
                const int b = __shfl(beg, (lane * G) & 63, 64), l = __shfl(len, (lane * G) & 63, 64);
                beg = b;
                len = lane < G ? l : 0;
                const int incl = wave_incl_scan(len);
                excl = incl - len;
                total = lane_value(incl, 63);
            }
            for (int off = 0;; off += spread ? 64 : G) {
                int a = beg + off + gl;
                bool valid = off + gl < len;
                if (spread) {
                    if (off >= total) break;
                    const bool here = len > 0 && excl >= off && excl < off + 64;
                    const uint64_t starts = wave_or(here ? 1ull << (excl - off) : 0ull);
                    const int before = __popcll(__ballot(len > 0 && excl < off));
                    const int o = before + mask_rank(starts) + (int)((starts >> lane) & 1ull) - 1;
                    a = __shfl(beg, o, 64) + (off + lane - __shfl(excl, o, 64));
                    valid = off + lane < total;
                } else if (__ballot(valid) == 0) {
                    break;
                }
                // the compare-and-swap leaves first and its result is used after
                // the loads beside it have left too
                int v = -1, seen = -1, row0 = 0, row1 = 0;
                int64_t ev = 0;
                if (valid) {
                    const int2 rec = get<SC>(&g.arc[a]);
                    const int tw = g.twin[a];
                    v = rec.x;
                    const int hv = get<SC>(&g.h[v]);
                    const int cft = get<SC>(cf_ptr(g.arc, tw));
                    tl.bfs_a++;
                    if (v != g.s && hv == n && cft > 0 && (!g.part_restrict || g.part[v] == g.part_want)) {
                        seen = cas_seen<SC>(&g.h[v], n, L + 1);
                        row0 = g.row_ptr[v];
                        row1 = g.row_ptr[v + 1];
                        ev = get<SC>(&g.e[v]);
                    }
                }
                const bool disc = seen == n;
                const uint64_t dm = __ballot(disc);
                if (dm == 0) continue;
                const int vbeg = row0, vdeg = row1 - row0;
                // what the step found goes to the stage: frontier items, short
                // and long active vertices, one reservation for the three
                const int ni = disc ? n_items(vdeg) : 0;
                int slot = mask_rank(dm), ntot = __popcll(dm);
                if (__ballot(ni > 1) != 0) {
                    const int ii = wave_incl_scan(ni);
                    ntot = lane_value(ii, 63);
                    slot = ii - ni;
                }
                const bool active = disc && v != g.t && ev > 0;
                const bool light = active && vdeg <= kLightMaxDeg;
                const bool heavy = active && vdeg > kLightMaxDeg && vdeg <= kHugeDeg;
                const bool huge = active && vdeg > kHugeDeg;
                const uint64_t lm = __ballot(light), hm = __ballot(heavy);
                const int nl = __popcll(lm), nh = __popcll(hm);
                int ib = 0;
                uint64_t ab = 0;
                if (lane == 0) {
                    ib = atomicAdd(&rs->found[nxt], ntot);
                    if (nl | nh)
                        ab = atomicAdd(reinterpret_cast<unsigned long long *>(&rs->act),
                                       ((unsigned long long)nh << 32) | (unsigned long long)nl);
                }
                ib = lane_value(ib, 0);
                ab = (uint64_t)lane_value((int64_t)ab, 0);
                const int lb = (int)(uint32_t)ab, hb = (int)(ab >> 32);
                // what the stage has no room for goes straight to the global
                // lists: from their bases (ig, lg, hg) less the stage's size
                int ig = 0, lg = 0, hg = 0;
                const bool full = ib + ntot > kRunItems || lb + nl > kStageCap || hb + nh > kStageCap;
                if (full) {
                    const int io = max(ib, kRunItems), lo = max(lb, kStageCap), ho = max(hb, kStageCap);
                    if (lane == 0) {
                        if (ib + ntot > io) {
                            rs->spill = 1;
                            ig = fetch_add<SC>(&c->qcount[(L + 1) % 3], ib + ntot - io);
                        }
                        if (lb + nl > lo) lg = fetch_add<SC>(&c->lst[0].light, lb + nl - lo);
                        if (hb + nh > ho) hg = fetch_add<SC>(&c->lst[0].heavy, hb + nh - ho);
                    }
                    ig = lane_value(ig, 0) - io;
                    lg = lane_value(lg, 0) - lo;
                    hg = lane_value(hg, 0) - ho;
                }
                for (int k = 0; k < ni; ++k) {
                    const int2 item = make_int2(vbeg + k * kChunk, min(vbeg + (k + 1) * kChunk, vbeg + vdeg));
                    const int at = ib + slot + k;
                    if (at < kRunItems) items[nxt * kRunItems + at] = item;
                    else frontier(g, L + 1)[ig + at] = item;
                }
                if (light) {
                    const int at = lb + mask_rank(lm);
                    if (at < kStageCap) rs->aux[at] = v;
                    else g.list[0][lg + at] = v;
                }
                if (heavy) {
                    const int at = hb + mask_rank(hm);
                    if (at < kStageCap) rs->aux[kStageCap + at] = v;
                    else g.list[0][n - 1 - (hg + at)] = v;
                }
                const int su = wave_append1<SC>(&c->lst[0].huge, huge);  // rare: hubs only
                if (huge) g.huge[0][su] = v;
                if (counts && lane == 0) add<SC>(&g.hcount[L + 1], __popcll(dm));
                if (feats) {
                    if (lane == 0) add<SC>(&c->feat_reached, __popcll(dm));
                    feature_tally<SC>(c, active, ev);
                }
                if (disc) {
                    tl.bfs_v++;
                    found_arcs += vdeg;
                }
            }
        }
        if (w * q < m) {
            const int fa = wave_sum(found_arcs);  // below A < 2^31
            if (lane == 0 && fa) atomicAdd(&rs->larcs[nxt], fa);
        }
        block_sync<SC>();
        uint64_t mine = 0;
        if (t == 0) {
            const bool late = (it & 15) == 0 && (int64_t)(wall_clock64() - ts) > p.barrier_ticks / 4;
            mine = (uint64_t)rs->larcs[nxt] | ((uint64_t)(rs->spill || late) << 48);
            atomicAdd(reinterpret_cast<unsigned long long *>(&rs->arcs), (unsigned long long)rs->larcs[cur]);
            rs->found[cur] = rs->larcs[cur] = 0;
        }
        const uint64_t sum = team_sum<SC>(c, tm, epoch, mine, p.barrier_ticks, ok);
        if (!*ok) return L;
        ++L;
        cur = nxt;
        dump = (sum >> 48) != 0 || (int64_t)sum > most;
        if (dump || sum == 0) break;
    }
    // the active vertices found (and the items, when the run ends early) go
    // to the global lists, one reservation each
    const int nq = dump ? min(rs->found[cur], kRunItems) : 0;
    const int nl = min((int)(uint32_t)rs->act, kStageCap), nh = min((int)(rs->act >> 32), kStageCap);
    if (t == 0) {
        if (nq) {
            rs->base[0] = fetch_add<SC>(&c->qcount[L % 3], nq);
            if (dir) {  // the level's, spilled items too; the direction rule takes an item for a vertex here
                add<SC>(&c->qverts[L % 3], rs->found[cur]);
                add<SC>(&c->qarcs[L % 3], (int64_t)rs->larcs[cur]);
            }
        }
        if (nl | nh) {
            const int64_t b = fetch_add<SC>(reinterpret_cast<int64_t *>(&c->lst[0]), ((int64_t)nh << 32) | (int64_t)nl);
            rs->base[1] = (int)(uint32_t)b;
            rs->base[2] = (int)(b >> 32);
        }
    }
    __syncthreads();
    if (dir && t == 0 && rs->arcs) add<SC>(&c->run_arcs, rs->arcs);
    for (int i = t; i < nq; i += blockDim.x) frontier(g, L)[rs->base[0] + i] = items[cur * kRunItems + i];
    for (int i = t; i < nl; i += blockDim.x) g.list[0][rs->base[1] + i] = rs->aux[i];
    for (int i = t; i < nh; i += blockDim.x) g.list[0][n - 1 - (rs->base[2] + i)] = rs->aux[kStageCap + i];
    __syncthreads();  // the stage is free again
    return L;
}

// ---------------------------------------------------------------------------
// PushRelabel (Alg. 2), run in rounds
//
// A phase between two global relabels runs rounds.  Round r processes the
// vertices of list r; a vertex whose excess turns positive through a push, or
// that keeps excess after its visit, is added once (round-id stamp) to list
// r+1.  So excess can travel many arcs between global relabels instead of one
// arc per relabel.  A phase ends when a list is empty, or when the relabel
// budget or the round cap is spent; the next global relabel then restarts from
// exact heights.
//
// One cycle (KERNELCYCLES counts cycles) scans the arcs for the lowest residual
// neighbour height h^; if h(u) > h^ it pushes along the arcs at height h^ in
// arc order until the excess is gone (the paper's cycles pick the lowest arc,
// first in arc order, one push each; with the same h^ the next cycles would
// take exactly these arcs), otherwise it relabels h(u) = h^ + 1.
// ---------------------------------------------------------------------------

// Per-workgroup sums of a round's pushes by target vertex (LDS, direct
// mapped): a push into a vertex that holds a slot adds to the slot; the
// workgroup adds every slot to the target's excess with one atomic at the end
// of the round.  Pushes whose slot belongs to another vertex go straight to
// the excess.  Vertices of huge degree take pushes from thousands of others
// in one round, and this turns them into one atomic per workgroup.
constexpr int kCombineBits = 9;
constexpr int kCombine = 1 << kCombineBits;
struct Combine {
    int32_t key[kCombine];  // target vertex, or -1
    int64_t sum[kCombine];
};

// The workgroup's one Combine.
__device__ __forceinline__ Combine *combine_stage() {
    __shared__ Combine s;
    return &s;
}

// A round: appends to the next round's lists and first relabels are staged in
// the workgroup's RunStage, half `par` of its list buffers.
struct RoundCtx {
    int32_t *next;     // list of the next round
    int32_t *next_huge;  // its huge-vertex list
    ListCtr *next_ctr;
    int32_t next_id;   // round id stamped into mark[] for that list
    int32_t phase_id;  // stamped into rmark[] on a vertex's first relabel
    int32_t par;
    bool comb;         // add pushes up per target first (combine_stage)
    bool use_gap;      // gap heuristic on
    bool eager;        // a push lists its target whatever excess it had (see push_arc)
};

// Put v (of deg arcs) on the next round's list.
template <int SC>
__device__ __forceinline__ void list_append(const DevGraph &g, const RoundCtx &rc, int v, int deg) {
    RunStage *rs = run_stage();
    if (deg <= kLightMaxDeg) {
        const int k = atomicAdd(&rs->lcnt[rc.par], 1);
        if (k < kStageCap) {
            rs->buf[rc.par * kStageCap + k] = v;
            return;
        }
        const int slot = append_here<SC>(&rc.next_ctr->light);
        rc.next[slot] = v;
    } else if (deg <= kHugeDeg) {
        const int k = atomicAdd(&rs->hcnt[rc.par], 1);
        if (k < kStageCap) {
            rs->buf[(2 + rc.par) * kStageCap + k] = v;
            return;
        }
        const int slot = append_here<SC>(&rc.next_ctr->heavy);
        rc.next[g.n - 1 - slot] = v;
    } else {
        const int slot = append_here<SC>(&rc.next_ctr->huge);
        rc.next_huge[slot] = v;
    }
    rs->spill = 1;
}

// The same unless v is there already.
template <int SC>
__device__ __forceinline__ void list_add(const DevGraph &g, const RoundCtx &rc, int v, int deg) {
    if (xchg<SC>(&g.mark[v], rc.next_id) != rc.next_id) list_append<SC>(g, rc, v, deg);
}

// u was relabelled, `rose` above its height at the start of the visit.  Counts
// u once per phase, and remembers it for RemoveInvalidEdges when it rose by 3
// or more: only such a vertex can own a steep arc.  (A relabel leaves u at most
// one above every head it saw residual; heights never drop inside a phase.  So
// an arc (u, v) can be steep only if it turned residual after u's scan, by a
// push from v.  A push in a later round finds h(v) above u's new height; one in
// the same round found h(v) at least 1 above u's height at the start of the
// round, so h(v) + 2 <= h(u) asks for a rise of 3.)  With the gap heuristic,
// which lifts vertices without a scan, every relabelled vertex is remembered.
// Only the one lane (or group) visiting u in a round touches rmark[u]; `stamp`
// is its value as read at the start of the visit: twice the phase's id, plus one
// once u is remembered.
template <int SC>
__device__ __forceinline__ void note_relabel(const DevGraph &g, const RoundCtx &rc, int u, int deg, int rose,
                                             int32_t &stamp) {
    const int32_t once = (int32_t)(2u * (uint32_t)rc.phase_id);
    const bool first = (stamp & ~1) != once;
    const bool keep = (rose >= 3 || rc.use_gap) && (first || stamp == once);
    if (!first && !keep) return;
    stamp = once | (keep ? 1 : 0);
    g.rmark[u] = stamp;
    RunStage *rs = run_stage();
    if (first) atomicAdd(&rs->firsts, 1);
    if (!keep) return;
    const int far = deg > kLightMaxDeg;  // short lists from the front, long ones from the back
    const int k = atomicAdd(&rs->rcnt[far], 1);
    if (k < kStageCap) {
        rs->aux[far * kStageCap + k] = u;
    } else if (far) {
        g.relab[g.n - 1 - append_here<SC>(&g.ctrl->nrelab[1])] = u;
    } else {
        g.relab[append_here<SC>(&g.ctrl->nrelab[0])] = u;
    }
}

// Relabel u from height ho to hmin + 1 (Alg. 2), keeping the per-height
// counts of the gap heuristic: a height left empty by this move means every
// vertex above it has no residual path to a root under a valid labelling
// (heights drop by at most one per residual arc), so heights above the lowest
// such gap count as |V|.  A count that hits zero only transiently (racing
// relabels) just deactivates vertices that the next global relabel restores.
// Returns the new height.
template <int SC>
__device__ __forceinline__ int relabel_to(const DevGraph &g, int u, int ho, int hmin, bool use_gap) {
    int hn = hmin + 1;
    if (use_gap) {
        const int gap = ld<SC>(&g.ctrl->gap);
        if (hn > gap) hn = g.n;
        if (hn < g.n) add<SC>(&g.hcount[hn], 1);
        if (fetch_add<SC>(&g.hcount[ho], -1) == 1 && ho > 0)
            __hip_atomic_fetch_min(&g.ctrl->gap, ho, __ATOMIC_RELAXED, scope_of<SC>);
    }
    if (hn > g.n) hn = g.n;
    g.h[u] = hn;
    return hn;
}

// Take a push of d into v into the workgroup's push sums; false when its slot
// belongs to another vertex (or sums are off).
__device__ __forceinline__ bool combine_push(const RoundCtx &rc, int v, int32_t d) {
    if (!rc.comb) return false;
    Combine *comb = combine_stage();
    const int slot = (int)(((uint32_t)v * 2654435761u) >> (32 - kCombineBits));
    int k = comb->key[slot];
    if (k < 0) {
        k = atomicCAS(&comb->key[slot], -1, v);
        if (k < 0) k = v;
    }
    if (k != v) return false;
    atomicAdd(reinterpret_cast<unsigned long long *>(&comb->sum[slot]), (unsigned long long)d);
    return true;
}

// Push d from u along arc a to v = head(a).  Residual capacity moves to the
// twin; excess moves from u to v except that the excess taken from u is
// subtracted by the caller (one atomic per visit chunk).
template <int SC>
__device__ __forceinline__ void push_arc(const DevGraph &g, const RoundCtx &rc, int a, int tw, int v,
                                         int32_t d, int64_t &to_t, Tally &tl) {
    add<SC>(cf_ptr(g.arc, a), -d);
    add<SC>(cf_ptr(g.arc, tw), d);
    if (v == g.t) {
        to_t += d;
    } else if (!combine_push(rc, v, d)) {
        const int dv = g.row_ptr[v + 1] - g.row_ptr[v];  // read alongside the addition
        const int64_t old = fetch_add<SC>(&g.e[v], (int64_t)d);
        if (old < 0) tl.deliv += min((int64_t)d, -old);  // part of a deficit filled
        if (old <= 0 && old + d > 0 && v != g.s) list_add<SC>(g, rc, v, dv);
    }
}

// Lowest residual neighbour height over the arcs first, first + stride, ...
// below last, and the residual capacity of the arcs at that height; four
// arcs per lane in flight.
template <int SC>
__device__ __forceinline__ void scan_lowest(const DevGraph &g, int first, int last, int stride, int &hmin,
                                            int64_t &cmin) {
    int a = first;
    for (; a + 3 * stride < last; a += 4 * stride) {
        int2 r[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = get<SC>(&g.arc[a + k * stride]);
        int hv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) hv[k] = r[k].y > 0 ? get<SC>(&g.h[r[k].x]) : INT32_MAX;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (hv[k] < hmin) {
                hmin = hv[k];
                cmin = r[k].y;
            } else if (hv[k] == hmin) {
                cmin += r[k].y;
            }
        }
    }
    for (; a < last; a += stride) {
        const int2 r = get<SC>(&g.arc[a]);
        const int hv = r.y > 0 ? get<SC>(&g.h[r.x]) : INT32_MAX;
        if (hv < hmin) {
            hmin = hv;
            cmin = r.y;
        } else if (hv == hmin) {
            cmin += r.y;
        }
    }
}

// Inclusive scan over groups of 8 lanes, saturating at 2^32 - 1.  Row shifts
// cross from one group into the next of the same row of 16: those lanes take
// nothing.  Every lane of the wavefront must call it.
__device__ __forceinline__ uint32_t group8_incl_scan_sat(uint32_t x) {
    const int gl = lane_id() & 7;
    const uint32_t y1 = (uint32_t)dpp<0x111, 0xf>(0, (int)x);
    x = __builtin_elementwise_add_sat(x, gl >= 1 ? y1 : 0u);
    const uint32_t y2 = (uint32_t)dpp<0x112, 0xf>(0, (int)x);
    x = __builtin_elementwise_add_sat(x, gl >= 2 ? y2 : 0u);
    const uint32_t y4 = (uint32_t)dpp<0x114, 0xf>(0, (int)x);
    return __builtin_elementwise_add_sat(x, gl >= 4 ? y4 : 0u);
}

// A wavefront visits vertex u: the lanes scan its arcs 64 at a time for the
// lowest residual neighbour height, and the push pass hands the excess to the
// lowest arcs in arc order with a prefix sum of their residual capacities.
// u < 0: idle.  Returns relabels (on lane 0).
template <int SC>
__device__ __forceinline__ int discharge_wave(const DevGraph &g, int u, int kc, const RoundCtx &rc, Tally &tl, int64_t &to_t) {
    const int lane = lane_id();
    if (u < 0) return 0;
    const int n = g.n;
    const int beg = g.row_ptr[u], end = g.row_ptr[u + 1];
    int hu = get<SC>(&g.h[u]);
    int32_t stamp = get<SC>(&g.rmark[u]);
    const int h0 = hu;
    int relabels = 0;
    if (rc.use_gap && hu < n && hu > ld<SC>(&g.ctrl->gap)) {  // above a gap: cut off
        if (lane == 0) {
            add<SC>(&g.hcount[hu], -1);
            g.h[u] = n;
        }
        hu = n;
    }
    // excess of u as last seen: loaded once, then taken from the returning
    // subtraction of what u pushed (incoming pushes only ever add to it)
    int64_t eu = lane_value(ld<SC>(&g.e[u]), 0);
    for (int cyc = 0; cyc < kc && hu < n; ++cyc) {
        if (eu <= 0) break;
        if (lane == 0) tl.pr_cyc++;
        int hmin = INT32_MAX;
        int64_t cmin = 0;  // not needed here
        scan_lowest<SC>(g, beg + lane, end, 64, hmin, cmin);
        if (lane == 0) tl.pr_a += end - beg;
        hmin = wave_min(hmin);
        if (hmin == INT32_MAX) break;
        if (hu > hmin) {
            int64_t sent = 0, now = eu;
            for (int base = beg; base < end && sent < eu; base += 64) {
                const int a = base + lane;
                int64_t c = 0;
                int v = -1, tw = 0;
                if (a < end) {
                    const int2 r = get<SC>(&g.arc[a]);
                    tw = g.twin[a];
                    if (r.y > 0 && get<SC>(&g.h[r.x]) == hmin) {
                        c = cyc == 0 ? r.y : max(0, ld<SC>(cf_ptr(g.arc, a)));
                        v = r.x;
                    }
                }
                const int64_t incl = wave_incl_scan64(c);  // in arc order
                const int64_t room = eu - sent;
                const int64_t excl = incl - c;
                const int64_t d = (c > 0 && excl < room) ? min(c, room - excl) : 0;
                const int64_t tot = min(lane_value(incl, 63), room);
                // the total leaves u before the lanes push it on, so the
                // returning subtraction overlaps the pushes
                if (lane == 0 && tot > 0) now = fetch_add<SC>(&g.e[u], -tot) - tot;
                if (d > 0) {
                    push_arc<SC>(g, rc, a, tw, v, (int32_t)d, to_t, tl);
                    tl.push++;
                }
                sent += tot;
            }
            eu = lane_value(now, 0);
        } else {
            int hn = 0;
            if (lane == 0) {
                hn = relabel_to<SC>(g, u, hu, hmin, rc.use_gap);
                tl.relabel++;
                note_relabel<SC>(g, rc, u, end - beg, hn - h0, stamp);
            }
            hu = lane_value(hn, 0);
            relabels++;
        }
    }
    if (lane == 0 && hu < n && eu > 0) list_add<SC>(g, rc, u, end - beg);
    return lane == 0 ? relabels : 0;
}

// Groups of 8 lanes visit vertices of at most 8 * K arcs, one each (u < 0: the
// group idles): the cycle of discharge_wave with the arcs, twins and head
// heights held in registers between the scan and the pushes.  What bounds a
// visit in a short list is its chain of dependent steps: bounds and state
// (loaded by the caller), arcs, head heights, atomics.  So pushes and relabels
// of different groups issue their atomics before anyone waits for a result,
// and with rc.eager a push stamps its target's mark beside the addition to
// its excess instead of after it.  Then the target is listed whatever excess
// it had: one that empties in its own visit of this round, or is still in
// deficit, is visited in vain in the next.  The group's last lane acts for
// the group (a scan's total is already there).  Every lane of the wavefront
// calls it.  Returns relabels (on the groups' last lanes).
template <int SC, int K>
__device__ __forceinline__ int visit_light(const DevGraph &g, int u, int beg, int end, int hu, int64_t eu,
                                           int32_t stamp, int kc, const RoundCtx &rc, Tally &tl, int64_t &to_t) {
    constexpr int G = 8;
    const int gl = lane_id() & (G - 1);
    const bool lead = gl == G - 1;
    const int n = g.n;
    const int h0 = hu;
    int relabels = 0;
    bool spent = false;   // no residual arc left: the cycles end
    bool listed = false;  // already on the next list
    for (int cyc = 0; cyc < kc; ++cyc) {
        const bool act = hu < n && eu > 0 && !spent;  // alike in a group
        if (__ballot(act) == 0) break;
        int v[K], c[K], tw[K], hv[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int a = beg + k * G + gl;
            c[k] = v[k] = tw[k] = 0;
            if (act && a < end) {
                const int2 r = get<SC>(&g.arc[a]);
                tw[k] = g.twin[a];
                v[k] = r.x;
                c[k] = r.y;
                if (cyc > 0) c[k] = max(0, ld<SC>(cf_ptr(g.arc, a)));
            }
        }
        int hmin = INT32_MAX;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            hv[k] = c[k] > 0 ? get<SC>(&g.h[v[k]]) : INT32_MAX;
            hmin = min(hmin, hv[k]);
        }
        hmin = group8_min(hmin);
        const bool push = act && hmin < hu;
        const bool lift = act && !push && hmin != INT32_MAX;
        spent = act && hmin == INT32_MAX;
        if (act && lead) {
            tl.pr_cyc++;
            tl.pr_a += end - beg;
        }
        int64_t left = eu, now = eu;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (k > 0 && __ballot(push && beg + k * G < end) == 0) break;
            // shares in arc order; the scan saturates at 2^32 - 1, above any room
            const uint32_t room = (uint32_t)min(left, (int64_t)INT32_MAX);
            const uint32_t ck = push && hv[k] == hmin ? (uint32_t)c[k] : 0u;
            const uint32_t incl = group8_incl_scan_sat(ck);
            const uint32_t before = (uint32_t)dpp<0x111, 0xf>(0, (int)incl);
            const uint32_t excl = gl == 0 ? 0u : before;
            const uint32_t d = excl < room ? min(ck, room - excl) : 0u;
            const int64_t tot = (int64_t)min(incl, room);  // the group's on its last lane
            // all atomics leave before any result is used
            const bool out = d > 0, pay = lead && tot > 0, up = k == 0 && lift && lead;
            const bool side = out && v[k] != g.t && !combine_push(rc, v[k], (int32_t)d);
            int64_t had = 0, old = 1;
            int32_t seen = rc.next_id, seen_u = rc.next_id;
            int row0 = 0, row1 = 0;
            if (pay) had = fetch_add<SC>(&g.e[u], -tot);
            if (side) {
                old = fetch_add<SC>(&g.e[v[k]], (int64_t)d);
                if (rc.eager) seen = xchg<SC>(&g.mark[v[k]], rc.next_id);
                row0 = g.row_ptr[v[k]];
                row1 = g.row_ptr[v[k] + 1];
            }
            if (up) {
                hu = relabel_to<SC>(g, u, hu, hmin, rc.use_gap);
                // u keeps its excess, so after the last cycle it is listed
                if (cyc == kc - 1 && hu < n) seen_u = xchg<SC>(&g.mark[u], rc.next_id);
                tl.relabel++;
                relabels++;
                note_relabel<SC>(g, rc, u, end - beg, hu - h0, stamp);
            }
            if (out) {
                add<SC>(cf_ptr(g.arc, beg + k * G + gl), -(int32_t)d);
                add<SC>(cf_ptr(g.arc, tw[k]), (int32_t)d);
                tl.push++;
                if (v[k] == g.t) to_t += d;
            }
            if (side) {
                if (old < 0) tl.deliv += min((int64_t)d, -old);  // part of a deficit filled
                if (v[k] != g.s) {
                    if (rc.eager) {
                        if (seen != rc.next_id) list_append<SC>(g, rc, v[k], row1 - row0);
                    } else if (old <= 0 && old + d > 0) {
                        list_add<SC>(g, rc, v[k], row1 - row0);
                    }
                }
            }
            if (up && cyc == kc - 1) {
                if (seen_u != rc.next_id) list_append<SC>(g, rc, u, end - beg);
                listed = true;
            }
            if (pay) now = had - tot;
            if (K > 1) left -= __shfl(tot, G - 1, G);
        }
        eu = now;
        if (kc > 1) {
            eu = __shfl(eu, G - 1, G);
            hu = __shfl(hu, G - 1, G);
        }
    }
    if (lead && !listed && hu < n && eu > 0) list_add<SC>(g, rc, u, end - beg);
    return relabels;
}

// Groups of 8 lanes visit vertices of at most kLightMaxDeg arcs (u < 0: the
// group idles); a wavefront whose lists all hold at most 8 arcs takes the
// shorter code.  Every lane of the wavefront calls it.
template <int SC>
__device__ __forceinline__ int discharge_light(const DevGraph &g, int u, int kc, const RoundCtx &rc, Tally &tl,
                                               int64_t &to_t) {
    int beg = 0, end = 0, hu = g.n;
    int32_t stamp = 0;
    int64_t eu = 0;
    if (u >= 0) {
        beg = g.row_ptr[u];
        end = g.row_ptr[u + 1];
        hu = get<SC>(&g.h[u]);
        stamp = get<SC>(&g.rmark[u]);
        eu = ld<SC>(&g.e[u]);
        if (rc.use_gap && hu < g.n && hu > ld<SC>(&g.ctrl->gap)) {  // above a gap: cut off
            if ((lane_id() & 7) == 7) {
                add<SC>(&g.hcount[hu], -1);
                g.h[u] = g.n;
            }
            hu = g.n;
        }
    }
    if (__ballot(end - beg > 8) == 0) return visit_light<SC, 1>(g, u, beg, end, hu, eu, stamp, kc, rc, tl, to_t);
    return visit_light<SC, kLightMaxDeg / 8>(g, u, beg, end, hu, eu, stamp, kc, rc, tl, to_t);
}

// A wavefront visits vertex u by walking its arcs in arc order, 64 at a
// time: the residual arcs that go downhill (head below u) take the excess in
// arc order (prefix sum of their residual capacities over the wavefront) and
// the walk stops as soon as the excess is gone; only when it reaches the end
// of the list with excess left does u relabel, to one above the lowest head
// among the arcs still residual.  Under exact labels the downhill arcs are
// those at h(u) - 1, the lowest residual heights, so this is the push of
// Alg. 2 without the full scan for the minimum before it; a head that a racy
// relabel left steep is pushed to like any downhill head.  Every lane of the
// wavefront calls it with the same u (u < 0: idle).  Returns relabels (lane 0).
template <int SC>
__device__ __forceinline__ int discharge_walk(const DevGraph &g, int u, int kc, const RoundCtx &rc, Tally &tl, int64_t &to_t) {
    const int lane = lane_id();
    if (u < 0) return 0;
    const int n = g.n;
    const int beg = g.row_ptr[u], end = g.row_ptr[u + 1];
    int hu = get<SC>(&g.h[u]);
    int32_t stamp = get<SC>(&g.rmark[u]);
    const int h0 = hu;
    int relabels = 0;
    if (rc.use_gap && hu < n && hu > ld<SC>(&g.ctrl->gap)) {  // above a gap: cut off
        if (lane == 0) {
            add<SC>(&g.hcount[hu], -1);
            g.h[u] = n;
        }
        hu = n;
    }
    int64_t eu = lane_value(ld<SC>(&g.e[u]), 0);
    for (int cyc = 0; cyc < kc && hu < n; ++cyc) {
        if (eu <= 0) break;
        if (lane == 0) tl.pr_cyc++;
        const int64_t e0 = eu;  // what this walk hands out
        int64_t sent = 0, now = eu;
        int hrest = INT32_MAX;  // lowest head among the arcs left residual
        int walked = 0;
        for (int base = beg; base < end && sent < e0; base += 64) {
            const int a = base + lane;
            int64_t c = 0;
            int v = -1, hv = INT32_MAX;
            if (a < end) {
                const int2 r = get<SC>(&g.arc[a]);
                if (r.y > 0) {
                    hv = get<SC>(&g.h[r.x]);
                    if (hv < hu) {
                        c = cyc == 0 ? r.y : max(0, ld<SC>(cf_ptr(g.arc, a)));
                        v = r.x;
                    }
                }
            }
            walked += min(64, end - base);
            if (__ballot(c > 0) == 0) {  // nothing downhill in this step (the common case
                                         // of a walk that ends in a relabel)
                if (v < 0 && hv != INT32_MAX) hrest = min(hrest, hv);
                continue;
            }
            const int64_t incl = wave_incl_scan64(c);
            const int64_t room = e0 - sent;
            const int64_t excl = incl - c;
            const int64_t d = (c > 0 && excl < room) ? min(c, room - excl) : 0;
            const int64_t tot = min(lane_value(incl, 63), room);
            if (lane == 0 && tot > 0) now = fetch_add<SC>(&g.e[u], -tot) - tot;
            if (d > 0) {
                push_arc<SC>(g, rc, a, g.twin[a], v, (int32_t)d, to_t, tl);
                tl.push++;
            }
            if (d < c || (v < 0 && hv != INT32_MAX)) hrest = min(hrest, hv);
            sent += tot;
        }
        if (lane == 0) tl.pr_a += walked;
        eu = lane_value(now, 0);
        if (sent >= e0) continue;  // the excess went downhill
        // the walk reached the end of the list with excess left: relabel
        if (eu <= 0) break;
        hrest = wave_min(hrest);
        if (hrest == INT32_MAX) break;  // no residual arc left
        int hn = 0;
        if (lane == 0) {
            hn = relabel_to<SC>(g, u, hu, hrest, rc.use_gap);
            tl.relabel++;
            note_relabel<SC>(g, rc, u, end - beg, hn - h0, stamp);
        }
        hu = lane_value(hn, 0);
        relabels++;
    }
    if (lane == 0 && hu < n && eu > 0) list_add<SC>(g, rc, u, end - beg);
    return lane == 0 ? relabels : 0;
}

// A whole workgroup visits vertex u (more than kHugeDeg arcs).  Each
// wavefront owns a contiguous chunk of u's arcs and finds, in one pass, its
// lowest residual neighbour height and the residual capacity toward it; the
// chunks' capacities at the overall lowest height h^ split the excess in arc
// order, so every wavefront then pushes its share along its own chunk without
// workgroup barriers.  Without races this makes exactly the pushes of one
// pass over all arcs in arc order (the same as discharge_wave); a capacity
// or height that changed since the scan only leaves excess behind.  Every
// thread of the workgroup calls it with the same u; all decisions are
// uniform.
template <int SC>
__device__ __forceinline__ int discharge_block(const DevGraph &g, int u, int kc, const RoundCtx &rc, Tally &tl,
                               int64_t &to_t) {
    __shared__ int s_min[32];
    __shared__ int64_t s_sum[32];
    __shared__ int64_t s_now;
    __shared__ int s_h;
    const int t = threadIdx.x, lane = lane_id(), w = t >> 6, nw = blockDim.x >> 6;
    const int n = g.n;
    const int beg = g.row_ptr[u], end = g.row_ptr[u + 1];
    const int chunk = ((end - beg + nw - 1) / nw + 63) & ~63;
    const int cb = min(end, beg + w * chunk), ce = min(end, cb + chunk);
    int hu = get<SC>(&g.h[u]);
    int32_t stamp = get<SC>(&g.rmark[u]);
    const int h0 = hu;
    int relabels = 0;
    if (rc.use_gap && hu < n && hu > ld<SC>(&g.ctrl->gap)) {  // above a gap: cut off
        if (t == 0) {
            add<SC>(&g.hcount[hu], -1);
            g.h[u] = n;
        }
        hu = n;
    }
    if (t == 0) s_now = ld<SC>(&g.e[u]);
    __syncthreads();
    int64_t eu = s_now;
    for (int cyc = 0; cyc < kc && hu < n; ++cyc) {
        if (eu <= 0) break;
        if (t == 0) {
            tl.pr_cyc++;
            tl.pr_a += end - beg;
        }
        int hm = INT32_MAX;
        int64_t cm = 0;
        scan_lowest<SC>(g, cb + lane, ce, 64, hm, cm);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const int oh = __shfl_xor(hm, d, 64);
            const int64_t oc = __shfl_xor(cm, d, 64);
            if (oh < hm) {
                hm = oh;
                cm = oc;
            } else if (oh == hm) {
                cm += oc;
            }
        }
        if (lane == 0) {
            s_min[w] = hm;
            s_sum[w] = cm;
        }
        __syncthreads();
        int hmin = INT32_MAX;
        for (int k = 0; k < nw; ++k) hmin = min(hmin, s_min[k]);
        int64_t off = 0;  // capacity at h^ in the chunks before this one
        for (int k = 0; k < w; ++k)
            if (s_min[k] == hmin) off += s_sum[k];
        const int64_t mine = hm == hmin ? cm : 0;
        __syncthreads();
        if (hmin == INT32_MAX) break;
        if (hu > hmin) {
            // this chunk's part of [0, eu) in arc order
            const int64_t room = max((int64_t)0, min(mine, eu - off));
            int64_t sent = 0;
            for (int base = cb; base < ce && sent < room; base += 64) {
                const int a = base + lane;
                int64_t c = 0;
                int v = -1, tw = 0;
                if (a < ce) {
                    const int2 r = get<SC>(&g.arc[a]);
                    tw = g.twin[a];
                    if (r.y > 0 && get<SC>(&g.h[r.x]) == hmin) {
                        c = cyc == 0 ? r.y : max(0, ld<SC>(cf_ptr(g.arc, a)));
                        v = r.x;
                    }
                }
                const int64_t incl = wave_incl_scan64(c);
                const int64_t rem = room - sent;
                const int64_t excl = incl - c;
                const int64_t d = (c > 0 && excl < rem) ? min(c, rem - excl) : 0;
                if (d > 0) {
                    push_arc<SC>(g, rc, a, tw, v, (int32_t)d, to_t, tl);
                    tl.push++;
                }
                sent += min(lane_value(incl, 63), rem);
            }
            if (lane == 0 && sent > 0) add<SC>(&g.e[u], -sent);
            __syncthreads();
            if (t == 0) s_now = ld<SC>(&g.e[u]);
            __syncthreads();
            eu = s_now;
        } else {
            if (t == 0) {
                s_h = relabel_to<SC>(g, u, hu, hmin, rc.use_gap);
                tl.relabel++;
                note_relabel<SC>(g, rc, u, end - beg, s_h - h0, stamp);
            }
            __syncthreads();
            hu = s_h;
            __syncthreads();
            relabels++;
        }
    }
    if (t == 0 && hu < n && eu > 0) list_add<SC>(g, rc, u, end - beg);
    return t == 0 ? relabels : 0;
}

// The walk of discharge_walk done by a whole workgroup (vertices of more than
// kHugeDeg arcs): one step covers blockDim.x arcs, the downhill residual
// capacities are prefix-summed over the workgroup (wavefront scans, then the
// wavefront totals through LDS), and the walk stops at the step where the
// excess runs out.  Only a walk that reaches the end of the list relabels.
// Every thread of the workgroup calls it with the same u; all decisions are
// uniform.
template <int SC>
__device__ __forceinline__ int discharge_block_walk(const DevGraph &g, int u, int kc, const RoundCtx &rc, Tally &tl,
                                    int64_t &to_t) {
    __shared__ int64_t s_wsum[32];
    __shared__ int s_wmin[32];
    __shared__ int64_t s_now;
    __shared__ int s_h;
    const int t = threadIdx.x, lane = lane_id(), w = t >> 6, nw = blockDim.x >> 6;
    const int n = g.n;
    const int beg = g.row_ptr[u], end = g.row_ptr[u + 1];
    int hu = get<SC>(&g.h[u]);
    int32_t stamp = get<SC>(&g.rmark[u]);
    const int h0 = hu;
    int relabels = 0;
    if (rc.use_gap && hu < n && hu > ld<SC>(&g.ctrl->gap)) {  // above a gap: cut off
        if (t == 0) {
            add<SC>(&g.hcount[hu], -1);
            g.h[u] = n;
        }
        hu = n;
    }
    if (t == 0) s_now = ld<SC>(&g.e[u]);
    __syncthreads();
    int64_t eu = s_now;
    for (int cyc = 0; cyc < kc && hu < n; ++cyc) {
        if (eu <= 0) break;
        if (t == 0) tl.pr_cyc++;
        const int64_t e0 = eu;
        int64_t sent = 0;
        int hrest = INT32_MAX;
        int walked = 0;
        for (int base = beg; base < end && sent < e0; base += blockDim.x) {
            const int a = base + t;
            int64_t c = 0;
            int v = -1, hv = INT32_MAX;
            if (a < end) {
                const int2 r = get<SC>(&g.arc[a]);
                if (r.y > 0) {
                    hv = get<SC>(&g.h[r.x]);
                    if (hv < hu) {
                        c = cyc == 0 ? r.y : max(0, ld<SC>(cf_ptr(g.arc, a)));
                        v = r.x;
                    }
                }
            }
            walked += min((int)blockDim.x, end - base);
            if (!__syncthreads_or(c > 0)) {  // nothing downhill in this step of the workgroup
                if (v < 0 && hv != INT32_MAX) hrest = min(hrest, hv);
                continue;
            }
            const int64_t incl = wave_incl_scan64(c);
            if (lane == 63) s_wsum[w] = incl;
            __syncthreads();
            int64_t woff = 0, btot = 0;
            for (int k = 0; k < nw; ++k) {
                const int64_t x = s_wsum[k];
                if (k < w) woff += x;
                btot += x;
            }
            __syncthreads();
            const int64_t room = e0 - sent;
            const int64_t excl = woff + incl - c;
            const int64_t d = (c > 0 && excl < room) ? min(c, room - excl) : 0;
            if (d > 0) {
                push_arc<SC>(g, rc, a, g.twin[a], v, (int32_t)d, to_t, tl);
                tl.push++;
            }
            if (d < c || (v < 0 && hv != INT32_MAX)) hrest = min(hrest, hv);
            sent += min(btot, room);
        }
        if (t == 0) {
            tl.pr_a += walked;
            if (sent > 0) add<SC>(&g.e[u], -sent);
        }
        __syncthreads();
        if (t == 0) s_now = ld<SC>(&g.e[u]);
        __syncthreads();
        eu = s_now;
        if (sent >= e0) continue;  // the excess went downhill
        if (eu <= 0) break;
        hrest = wave_min(hrest);
        if (lane == 0) s_wmin[w] = hrest;
        __syncthreads();
        int hmin = INT32_MAX;
        for (int k = 0; k < nw; ++k) hmin = min(hmin, s_wmin[k]);
        __syncthreads();
        if (hmin == INT32_MAX) break;  // no residual arc left
        if (t == 0) {
            s_h = relabel_to<SC>(g, u, hu, hmin, rc.use_gap);
            tl.relabel++;
            note_relabel<SC>(g, rc, u, end - beg, s_h - h0, stamp);
        }
        __syncthreads();
        hu = s_h;
        __syncthreads();
        relabels++;
    }
    if (t == 0 && hu < n && eu > 0) list_add<SC>(g, rc, u, end - beg);
    return t == 0 ? relabels : 0;
}

// Copy the workgroup's staged appends (half rc.par) into the next round's list
// and the phase's relabelled list, one reservation per list and workgroup, and
// add the workgroup's counters (acc: excess into t, relabels, pushes,
// deliveries into deficits).  Every thread of the workgroup calls it.
template <int SC>
__device__ __forceinline__ void flush_stage(const DevGraph &g, const RoundCtx &rc) {
    RunStage *rs = run_stage();
    __syncthreads();
    const int nl = min(rs->lcnt[rc.par], kStageCap), nh = min(rs->hcnt[rc.par], kStageCap);
    const int nr = min(rs->rcnt[0], kStageCap), nf = min(rs->rcnt[1], kStageCap);
    if (threadIdx.x == 0) {
        rs->base[0] = nl ? fetch_add<SC>(&rc.next_ctr->light, nl) : 0;
        rs->base[1] = nh ? fetch_add<SC>(&rc.next_ctr->heavy, nh) : 0;
        Ctrl *c = g.ctrl;
        rs->base[2] = nr ? fetch_add<SC>(&c->nrelab[0], nr) : 0;
        rs->base[3] = nf ? fetch_add<SC>(&c->nrelab[1], nf) : 0;
        if (rs->firsts) add<SC>(&c->nfirsts, rs->firsts);
        const int64_t *acc = rs->acc;
        if (acc[0]) add<SC>(&g.e[g.t], acc[0]);
        if (acc[0] + acc[3]) add<SC>(&c->phase_deliv, acc[0] + acc[3]);
        if (acc[1]) add<SC>(&c->phase_relabels, acc[1]);
        if (acc[2]) add<SC>(&c->phase_pushes, acc[2]);
    }
    __syncthreads();
    const int32_t *light = rs->buf + rc.par * kStageCap, *heavy = rs->buf + (2 + rc.par) * kStageCap;
    for (int i = threadIdx.x; i < nl; i += blockDim.x) rc.next[rs->base[0] + i] = light[i];
    for (int i = threadIdx.x; i < nh; i += blockDim.x) rc.next[g.n - 1 - (rs->base[1] + i)] = heavy[i];
    for (int i = threadIdx.x; i < nr; i += blockDim.x) g.relab[rs->base[2] + i] = rs->aux[i];
    for (int i = threadIdx.x; i < nf; i += blockDim.x) g.relab[g.n - 1 - (rs->base[3] + i)] = rs->aux[kStageCap + i];
    __syncthreads();  // the stage is free again
}

// Add the workgroup's push sums to the targets' excess (every thread of the
// workgroup calls it); a target whose excess turns positive joins the next
// round's list, as after a single push.
template <int SC>
__device__ __forceinline__ void flush_combine(const DevGraph &g, const RoundCtx &rc, Tally &tl) {
    Combine *comb = combine_stage();
    __syncthreads();
    for (int i = threadIdx.x; i < kCombine; i += blockDim.x) {
        const int v = comb->key[i];
        if (v < 0) continue;
        const int64_t d = comb->sum[i];
        comb->key[i] = -1;
        comb->sum[i] = 0;
        const int64_t old = fetch_add<SC>(&g.e[v], d);
        if (old < 0) tl.deliv += min(d, -old);
        if (old <= 0 && old + d > 0 && v != g.s) list_add<SC>(g, rc, v, g.row_ptr[v + 1] - g.row_ptr[v]);
    }
}

// One round, or a run of rounds, of push/relabel.
//
// A round visits list r: a group of 8 lanes per short arc list, a workgroup
// per huge one, a wavefront per other long one, dealt out round-robin (no
// shared counter for thousands of wavefronts to contend on).  Topology-driven
// rounds visit every vertex instead (idle when inactive).
//
// A run (run = true; lists of round r, none huge) is consecutive rounds whose
// lists stay in LDS: every workgroup of the team keeps the vertices that its
// visits put on the next round's list and visits them in that round, and a
// round ends with the barrier that also sums list sizes, relabels and
// deliveries, with which the phase's limits are tested as between single
// rounds.  It ends with the phase (*done and its *reason), or with the next
// lists back in global memory when they hold more than `most` vertices, a huge
// one, more than a workgroup's LDS, or after a quarter of the barrier's wait
// limit.  The totals (excess into t, relabels, pushes, deliveries, relabelled
// vertices) are added at the end of the round or run.  Returns the number of
// the next round; *ok is false when a barrier wait ran out.
struct PhaseLimits {
    int64_t budget;
    int round_cap, stall;
};
template <int SC, bool WALK>
__device__ __forceinline__ int pr_rounds(const DevGraph &g, const Team &tm, const LoopParams &p, const PhaseLimits &lim, bool run,
                         int32_t rbase, int r, int nl, int nh, int nu, int64_t relabels, int most, int *reason,
                         bool *done, int *last_change, uint32_t &epoch, Tally &tl, bool *ok) {
    constexpr int G = 8;  // lanes per vertex with a short arc list
    const int t = threadIdx.x, lane = lane_id(), w = uniform(t >> 6), nw = blockDim.x >> 6;
    const bool topology = p.mode == 1;
    const bool comb = SC != kGroup && p.combine;
    Ctrl *c = g.ctrl;
    RunStage *rs = run_stage();
    {
        const int32_t *lst = round_list(g, r % 3);
        const int ml = run ? (nl - tm.rank + tm.size - 1) / tm.size : 0;
        const int mh = run ? (nh - tm.rank + tm.size - 1) / tm.size : 0;
        for (int i = t; i < ml; i += blockDim.x) rs->buf[i] = get<SC>(&lst[tm.rank + i * tm.size]);
        for (int i = t; i < mh; i += blockDim.x)
            rs->buf[2 * kStageCap + i] = get<SC>(&lst[g.n - 1 - (tm.rank + i * tm.size)]);
        if (t == 0) {
            rs->lcnt[0] = ml;
            rs->hcnt[0] = mh;
            rs->lcnt[1] = rs->hcnt[1] = rs->rcnt[0] = rs->rcnt[1] = rs->firsts = 0;
            rs->spill = rs->relabels = rs->deliv = 0;
        }
        if (t < 4) rs->acc[t] = 0;
    }
    __syncthreads();
    const uint64_t ts = run ? wall_clock64() : 0;
    const uint32_t push0 = tl.push;
    int64_t to_t = 0, all_deliv = 0, all_relabels = 0;
    int cur = 0;
    bool dump = true;
    for (int it = 1;; ++it) {
        if (t == 0 && tm.rank == 0) c->lst[(r + 2) % 3] = ListCtr{};
        const int nxt = cur ^ 1, wr = (r + 1) % 3;
        const RoundCtx rc{round_list(g, wr), huge_list(g, wr), &c->lst[wr], rbase + r + 1, rbase, nxt, comb, p.use_gap != 0,
                          run && !comb};
        const int32_t *lst = round_list(g, r % 3);
        int rl = 0;
        const int64_t to_t0 = to_t;
        {
            const int *light = rs->buf + cur * kStageCap;
            const int ml = run ? rs->lcnt[cur] : topology ? g.n : nl;
            const int64_t step = (run ? nw : tm.nwaves()) * (64 / G);
            for (int64_t base = (run ? w : tm.wave()) * (64 / G); base < ml; base += step) {
                const int i = (int)base + lane / G;
                int u = -1;
                if (i < ml) {
                    u = run ? light[i] : topology ? i : get<SC>(&lst[i]);
                    if (topology && (u == g.s || u == g.t || g.row_ptr[u + 1] - g.row_ptr[u] > kLightMaxDeg)) u = -1;
                }
                rl += discharge_light<SC>(g, u, p.kc, rc, tl, to_t);
            }
        }
        if (nu > 0 && !topology) {  // handed out by a counter (heavy_all holds them too)
            __shared__ int s_idx;
            const int32_t *hl = huge_list(g, r % 3);
            for (;;) {
                if (t == 0) s_idx = fetch_add<SC>(&c->lst[r % 3].hgrab, 1);
                __syncthreads();
                const int idx = s_idx;
                __syncthreads();
                if (idx >= nu) break;
                if constexpr (WALK) rl += discharge_block_walk<SC>(g, get<SC>(&hl[idx]), p.kc, rc, tl, to_t);
                else rl += discharge_block<SC>(g, get<SC>(&hl[idx]), p.kc, rc, tl, to_t);
            }
        }
        {
            const int *heavy = rs->buf + (2 + cur) * kStageCap;
            const int mh = run ? rs->hcnt[cur] : topology ? g.n_heavy_all : nh;
            const int64_t step = run ? nw : tm.nwaves();
            for (int64_t i = run ? w : tm.wave(); i < mh; i += step) {
                const int u = uniform(run ? heavy[i] : topology ? g.heavy_all[i] : get<SC>(&lst[g.n - 1 - i]));
                if constexpr (WALK) rl += discharge_walk<SC>(g, u, p.kc, rc, tl, to_t);
                else rl += discharge_wave<SC>(g, u, p.kc, rc, tl, to_t);
            }
        }
        if (comb) flush_combine<SC>(g, rc, tl);
        all_relabels += rl;
        all_deliv += tl.deliv;
        if (!run) {
            tl.deliv = 0;
            ++r;
            cur = nxt;
            break;
        }
        const int s = wave_sum(rl);
        if (lane == 0 && s) atomicAdd(&rs->relabels, s);
        if (__ballot(to_t != to_t0 || tl.deliv != 0) != 0 && lane == 0) rs->deliv = 1;
        tl.deliv = 0;
        block_sync<SC>();
        uint64_t mine = 0;
        if (t == 0) {
            const bool late = (it & 15) == 0 && (int64_t)(wall_clock64() - ts) > p.barrier_ticks / 4;
            const int list = min(rs->lcnt[nxt], kStageCap) + min(rs->hcnt[nxt], kStageCap);
            // relabels are capped so that a team's sum fits its 20 bits (only
            // the budget test reads them)
            mine = (uint64_t)min(rs->relabels, (1 << 20) / tm.size - 1) | ((uint64_t)list << 20) |
                   ((uint64_t)rs->deliv << 40) | ((uint64_t)(rs->spill || late) << 48);
            rs->lcnt[cur] = rs->hcnt[cur] = rs->relabels = rs->deliv = 0;
        }
        const uint64_t sum = team_sum<SC>(c, tm, epoch, mine, p.barrier_ticks, ok);
        if (!*ok) return r;
        ++r;
        cur = nxt;
        relabels += (int64_t)(sum & 0xfffffu);
        const int size = (int)((sum >> 20) & 0xfffffu);
        if ((sum >> 40) & 0xffu) *last_change = r;
        dump = (sum >> 48) != 0 || size > most;
        if (dump) break;
        // the phase's limits, in the order of the rounds outside a run
        if (size != 0) {
            if (r >= lim.round_cap) *reason = 1;
            else if (relabels > lim.budget) *reason = 2;
            else if (lim.stall > 0 && r - *last_change >= lim.stall) *reason = 3;
            else continue;
        }
        *done = true;
        break;
    }
    // the totals, and the lists when the phase goes on outside the run
    const int64_t v[4] = {wave_sum(to_t), wave_sum(all_relabels), (int64_t)wave_sum((int)(tl.push - push0)),
                          wave_sum(all_deliv)};
    if (lane == 0)
        for (int k = 0; k < 4; ++k)
            if (v[k]) atomicAdd(reinterpret_cast<unsigned long long *>(&rs->acc[k]), (unsigned long long)v[k]);
    if (!dump) {
        __syncthreads();
        if (t == 0) rs->lcnt[cur] = rs->hcnt[cur] = 0;
    }
    const RoundCtx rc{round_list(g, r % 3), nullptr, &c->lst[r % 3], 0, 0, cur, false, false, false};
    flush_stage<SC>(g, rc);
    return r;
}

// ---------------------------------------------------------------------------
// RemoveInvalidEdges (Alg. 3): saturate every residual arc (u, v) with
// h(u) > h(v) + 1.  Only vertices that rose by 3 or more in one visit can own
// such an arc (see note_relabel); the phase keeps them in a list, short arc
// lists from its front and long ones from its back.  Only u lowers c_f of its
// own arcs, so an exchange with 0 reads and clears the residual in one step.
// What bounded it was the scan itself and its uneven lists: with every
// relabelled vertex listed and a hub scanned by one wavefront, on R-MAT
// 2^22 x 16 a solve read 205 M arcs here (12.3 ms in all); now 9 k (8.7 ms).
// R-MAT 2^20: 6.3 -> 5.0 ms, 2^18: 2.5 -> 1.9 ms.
// ---------------------------------------------------------------------------

template <int SC>
__device__ __forceinline__ void rie_arc(const DevGraph &g, int u, int hu, int a, Tally &tl) {
    const int2 r = get<SC>(&g.arc[a]);
    if (r.y > 0 && hu > get<SC>(&g.h[r.x]) + 1) {
        const int32_t c = xchg<SC>(cf_ptr(g.arc, a), 0);
        if (c > 0) {
            add<SC>(cf_ptr(g.arc, g.twin[a]), c);
            add<SC>(&g.e[u], -(int64_t)c);
            add<SC>(&g.e[r.x], (int64_t)c);
            tl.rie_sat++;
        }
    }
}

// With the gap heuristic on, a vertex cut off at height |V| is skipped: its arcs
// look steep only because it was lifted deliberately, and saturating them
// would push flow out of the source side and create deficits (new roots)
// there, undoing the cut.
template <int SC>
__device__ __forceinline__ void remove_invalid(const DevGraph &g, const Team &tm, int nshort, int nlong, bool skip_cut,
                                               Tally &tl) {
    // a group of 8 lanes per short list
    constexpr int G = 8;
    const int lane = lane_id(), gl = lane & (G - 1);
    const int64_t ngrp = tm.nthreads() / G;
    for (int64_t i = tm.tid() / G; i < nshort; i += ngrp) {
        const int u = get<SC>(&g.relab[i]);
        const int hu = get<SC>(&g.h[u]);
        if (skip_cut && hu >= g.n) continue;
        const int beg = g.row_ptr[u], end = g.row_ptr[u + 1];
        for (int a = beg + gl; a < end; a += G) rie_arc<SC>(g, u, hu, a, tl);
        if (gl == 0) tl.rie_a += end - beg;
    }
    // a wavefront per long list, a workgroup per huge one: the workgroup takes
    // up to 64 vertices at a time, one lane each, and deals them out
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int per = min(64, max(1, (nlong + tm.size - 1) / tm.size));
    for (int64_t base = (int64_t)tm.rank * per; base < nlong; base += (int64_t)tm.size * per) {
        int u = -1, hu = 0, beg = 0, end = 0;
        if (lane < per && base + lane < nlong) {
            u = get<SC>(&g.relab[g.n - 1 - (base + lane)]);
            hu = get<SC>(&g.h[u]);
            if (!(skip_cut && hu >= g.n)) {
                beg = g.row_ptr[u];
                end = g.row_ptr[u + 1];
            }
        }
        for (uint64_t m = __ballot(end > beg); m; m &= m - 1) {
            const int l = __ffsll((unsigned long long)m) - 1;
            const int b = lane_value(beg, l), e = lane_value(end, l);
            const bool all = e - b > kHugeDeg;
            if (!all && l % nw != w) continue;
            const int v = lane_value(u, l), hv = lane_value(hu, l);
            const int step = all ? blockDim.x : 64;
            for (int a = b + (all ? (int)threadIdx.x : lane); a < e; a += step) rie_arc<SC>(g, v, hv, a, tl);
            if (lane == 0 && (!all || w == 0)) tl.rie_a += e - b;
        }
    }
}

// ---------------------------------------------------------------------------
// Learned phase schedule
//
// Right after a global relabel found active vertices, the schedule picks the
// limits of the coming phase among kPolK actions: relabel budget x b/4,
// rounds per BFS level x r/2, stall limit x l/2 (0: none).  Action 0 is the
// fixed rule.  Every action keeps the result exact: only the moment of the
// next global relabel changes.
// ---------------------------------------------------------------------------

__device__ __forceinline__ int act_budget(int a) { return a == 1 ? 1 : a == 2 ? 2 : a == 3 ? 8 : a == 4 ? 16 : 4; }
__device__ __forceinline__ int act_rpl(int a) { return a == 4 || a == 6 ? 4 : a == 5 ? 1 : 2; }
__device__ __forceinline__ int act_stall(int a) { return a == 6 ? 1 : a == 7 ? 0 : 2; }

// splitmix64 finaliser (Steele, Lea and Flood, 2014): counter-based draws of
// the exploration mode.
__device__ __forceinline__ uint64_t mix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

// Run by the 64 lanes of the leader's wavefront after the barrier that ends
// the BFS.  Features (every lane computes them), then the action: the
// network's lowest predicted cost
// when it beats action 0 by the margin (learned), a seeded draw (explore) or
// a fixed action (forced).  Lane 0 publishes the action in Ctrl; the features
// and the action go to the policy trace.
template <int SC>
__device__ __forceinline__ int policy_decide(const DevGraph &g, const LoopParams &p, Ctrl *c, int L, int64_t iter) {
    constexpr int F = kPolF, H = kPolH, K = kPolK;
    constexpr int oW1 = 0, ob1 = oW1 + H * F, oW2 = ob1 + H, ob2 = oW2 + H * H, oW3 = ob2 + H, ob3 = oW3 + K * H;
    const int lane = lane_id();
    const int64_t reached = ld<SC>(&c->feat_reached);
    const int cnt = ld<SC>(&c->lst[0].light) + ld<SC>(&c->lst[0].heavy) + ld<SC>(&c->lst[0].huge);
    const int64_t es = ld<SC>(&c->feat_esum);
    float x[F];
    x[0] = log2f((float)(1 + cnt)) / 24.f;
    x[1] = log2f((float)(1 + es)) / 40.f;
#pragma unroll
    for (int b = 0; b < 8; ++b) x[2 + b] = cnt ? (float)ld<SC>(&c->feat_hist[b]) / (float)cnt : 0.f;
    x[10] = log2f((float)(1 + L)) / 12.f;
    x[11] = (float)reached / (float)g.n;
    x[12] = log2f((float)(1 + ld<SC>(&c->prev_pushes))) / 32.f;
    x[13] = log2f((float)(1 + ld<SC>(&c->prev_relabels))) / 32.f;
    x[14] = log2f((float)(1 + iter)) / 8.f;
    x[15] = p.batch_fraction;
    int act = 0;
    if (p.policy_per_call && iter > 0) {
        act = ld<SC>(&c->action);  // the call's first decision holds
    } else if (p.policy_mode == kPolicyLearned) {
        const float *W = p.policy_w;
        const int j = lane & (H - 1);
        float z = W[ob1 + j];
#pragma unroll
        for (int i = 0; i < F; ++i) z = fmaf(W[oW1 + j * F + i], x[i], z);
        const float h1 = z > 0.f ? z : 0.f;
        float z2 = W[ob2 + j];
#pragma unroll
        for (int l = 0; l < H; ++l) z2 = fmaf(W[oW2 + j * H + l], __shfl(h1, l, 64), z2);
        const float h2 = z2 > 0.f ? z2 : 0.f;
        const int k = lane & (K - 1);
        float q = W[ob3 + k];
#pragma unroll
        for (int l = 0; l < H; ++l) q = fmaf(W[oW3 + k * H + l], __shfl(h2, l, 64), q);
        const float q0 = __shfl(q, 0, 64);
        float best = q0;
        int ba = 0;
#pragma unroll
        for (int kk = 1; kk < K; ++kk) {
            const float qk = __shfl(q, kk, 64);
            if (qk < best) {
                best = qk;
                ba = kk;
            }
        }
        act = (q0 - best > p.policy_margin) ? ba : 0;
    } else if (p.policy_mode == kPolicyExplore) {
        const uint64_t r = mix64(p.policy_seed ^ mix64(((uint64_t)(uint32_t)p.seq_base << 32) ^ (uint64_t)iter));
        const float u = (float)(r >> 40) * (1.0f / 16777216.0f);
        act = u < p.policy_explore ? (int)((r & 0xffffffffull) % (uint64_t)K) : 0;
    } else if (p.policy_mode == kPolicyForced) {
        act = p.policy_action;
    }
    const int rec = ld<SC>(&c->ntrace);
    if (g.ptrace && rec < kTraceCap) {
        float *pr = g.ptrace + (int64_t)rec * kPolRec;
#pragma unroll
        for (int f = 0; f < F; ++f)
            if (lane == f) pr[f] = x[f];
        if (lane == 0) pr[F] = (float)act;
    }
    if (lane == 0) c->action = act;
    return act;
}

// ---------------------------------------------------------------------------
// The persistent solve loop (Alg. 1 / Alg. 4 while-loop)
// ---------------------------------------------------------------------------

// Clear the LDS stages that start from zero (every thread of the workgroup).
__device__ __forceinline__ void init_stages() {
    BfsStage *st = bfs_stage();
    Combine *comb = combine_stage();
    if (threadIdx.x < 4) st->cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        st->arcs = 0;
        st->tverts = 0;
        st->tarcs = 0;
    }
    for (int i = threadIdx.x; i < kCombine; i += blockDim.x) {
        comb->key[i] = -1;
        comb->sum[i] = 0;
    }
    __syncthreads();
}

template <int SC, bool WALK>
__device__ __forceinline__ void solve_loop(const DevGraph &g, const Team &tm, const LoopParams &p, uint32_t &bar_epoch) {
    Ctrl *c = g.ctrl;
    if (ld<SC>(&c->err)) return;  // update batch rejected: leave the state alone
    Tally tl;
    const bool leader = tm.rank == 0 && threadIdx.x == 0;
    const bool topology = p.mode == 1;
    int64_t iter = 0;
    uint32_t sum_epoch = 0;  // summing barriers of the launch's runs
    // Runs (frontier or list in LDS) are made by the whole team when it is one
    // workgroup or shares an XCD, and by the first workgroup alone otherwise.
    const Team run_team = SC == kAgent ? Team{0, 1} : tm;
    const bool runner = SC != kAgent || tm.rank == 0;
    // Items or vertices up to which a run starts (a list's run ends above
    // twice that), and arcs above which a BFS run ends (it starts with up to half that):
    // a frontier that gives every lane of the run's workgroups more than an arc or
    // two is bound by throughput, which the whole team has more of, and the
    // direction rule applies to it.  One workgroup has no other choice.
    // (R-MAT 2^14, 2^15 static: 1.36, 1.96 ms without the arc limit, 1.09, 1.48 with it.)
    const bool apart = SC == kAgent && tm.size > 1;
    const int run_from = apart ? min(p.solo_items, kRunItems / 2) : tm.size * (kRunItems / 4);
    const int run_most = apart ? run_from : 2 * run_from;
    const int64_t run_arcs_most = apart ? 8 * kBlock : tm.size > 1 ? (int64_t)tm.size * 2 * kBlock : INT64_MAX;
    int64_t run_arcs = 0;  // arcs discovered in BFS runs so far
    const bool policy = p.policy_mode != kPolicyFixed;
    // vertices per height are counted only for the gap heuristic
    const bool counts = p.use_gap != 0;
    const uint64_t t0 = wall_clock64();
    // arcs of the vertices that the previous global relabel of this launch
    // reached (-1: none yet); the BFS direction rule takes the other arcs as
    // those a bottom-up level scans in full without finding a parent
    int64_t reach_prev = -1;
    __shared__ int64_t s_def[kBlock / 64];  // the wavefronts' shares of the deficits
    for (;;) {
        // time budget: the leader raised `stop` before the last barrier, so
        // every workgroup sees the same value here
        if (ld<SC>(&c->stop)) {
            if (leader) c->status = kDeadline;
            int64_t d = 0;  // the last rounds changed it
            for (int64_t v = tm.tid(); v < g.n; v += tm.nthreads()) {
                const int64_t ev = get<SC>(&g.e[v]);
                if (ev < 0 && v != g.s && v != g.t) d += ev;
            }
            d = wave_sum(d);
            if (lane_id() == 0) s_def[threadIdx.x >> 6] = d;
            break;
        }
        // --- global relabel ---
        if (leader) {
            for (int k = 0; k < 3; ++k) c->lst[k] = ListCtr{};
            c->prev_pushes = ld<SC>(&c->phase_pushes);
            c->prev_relabels = ld<SC>(&c->phase_relabels);
            c->feat_esum = 0;
            for (int b = 0; b < 8; ++b) c->feat_hist[b] = 0;
            c->nrelab[0] = c->nrelab[1] = c->nfirsts = 0;
            c->phase_relabels = 0;
            c->phase_pushes = 0;
            c->phase_deliv = 0;
            c->gap = g.n;
            add<SC>(&c->stat[kStGlobalRelabels], 1);
        }
        const uint64_t tb = wall_clock64();
        // the BFS tallies the schedule's features only where a decision uses
        // them: every phase, or the first phase of a call decided per call
        const bool feats = policy && !(p.policy_per_call && iter > 0);
        // direction rule of the BFS (direction-optimising BFS): a level runs
        // bottom-up when its frontier's arcs are a large share of the arcs
        // that a bottom-up pass would scan, and stays so while the frontier is
        // large; small and restricted BFS passes stay top-down.  A bottom-up
        // pass stops early only at vertices it discovers: the vertices that
        // no level will reach (estimated by those the previous global relabel
        // did not reach) have their whole arc lists scanned at every level
        const bool dir = p.bu_alpha > 0 && g.bu_items != nullptr && !g.part_restrict;
        {
            const int64_t d = wave_sum(bfs_roots<SC>(g, tm, counts, feats, dir, tl));
            if (lane_id() == 0) s_def[threadIdx.x >> 6] = d;
        }
        if (!grid_barrier<SC>(c, tm, bar_epoch, p.barrier_ticks)) return;
        int L = 0;
        bool bu = false;
        int64_t seen_arcs = 0;  // arcs of the vertices reached so far (a run's last level by qarcs)
        for (;;) {
            // the level's counters are loaded together: one round trip after
            // the barrier, not one per counter
            const int cnt = uniform(ld<SC>(&c->qcount[L % 3]));
            const int64_t fa = dir ? uniform(ld<SC>(&c->qarcs[L % 3])) : 0;
            const int fv = dir ? uniform(ld<SC>(&c->qverts[L % 3])) : 0;
            if (cnt == 0) break;
            if (dir) {
                seen_arcs += fa;
                const int64_t rest = (int64_t)g.A - seen_arcs;
                const int64_t dead = reach_prev < 0 ? 0 : min(rest, max((int64_t)0, (int64_t)g.A - reach_prev));
                bu = bu ? (int64_t)fv * p.bu_beta >= g.n : fa * p.bu_alpha > rest + (p.bu_alpha - 1) * dead;
            }
            // A small frontier is expanded in a run (bfs_run): by the first
            // workgroup alone, while the others wait at the next grid
            // barrier, or by the whole of a team that shares an XCD.
            if (!bu && cnt <= run_from && fa <= run_arcs_most / 2) {
                bool ok = true;
                if (runner) {
                    L = bfs_run<SC>(g, run_team, p, L, cnt, run_arcs_most, feats, counts, dir, sum_epoch, tl, &ok);
                    if (SC == kAgent && threadIdx.x == 0) c->solo_level = L;
                }
                if (!ok || !grid_barrier<SC>(c, tm, bar_epoch, p.barrier_ticks)) return;
                if (SC == kAgent) L = uniform(ld<SC>(&c->solo_level));
                if (dir) {
                    const int64_t ra = uniform(ld<SC>(&c->run_arcs));
                    seen_arcs += ra - run_arcs;
                    run_arcs = ra;
                }
                continue;
            }
            if (threadIdx.x == 0 && tm.rank == 0) {
                c->qcount[(L + 2) % 3] = 0;
                c->qverts[(L + 2) % 3] = 0;
                c->qarcs[(L + 2) % 3] = 0;
            }
            // large levels of a team stage their output per workgroup
            if (SC != kGroup && bu)
                bfs_bottom_up<SC>(g, tm, L, feats, counts, tl);
            else
                bfs_level<SC>(g, tm, L, cnt, feats, counts, dir, cnt >= p.lazy_items,
                              SC != kGroup && cnt >= kBfsStageMin, tl);
            if (!grid_barrier<SC>(c, tm, bar_epoch, p.barrier_ticks)) return;
            ++L;
        }
        if (dir) reach_prev = seen_arcs;
        const uint64_t tp = wall_clock64();
        if (leader) {
            add<SC>(&c->stat[kStLevels], (int64_t)L);
            add<SC>(&c->stat[kStBfsTicks], (int64_t)(tp - tb));
        }
        // --- termination test right after a fresh global relabel ---
        {
            const int nl = uniform(ld<SC>(&c->lst[0].light));
            const int nh = uniform(ld<SC>(&c->lst[0].heavy));
            const int nu = uniform(ld<SC>(&c->lst[0].huge));
            if (nl + nh + nu == 0) {
                if (leader) c->status = kSolved;
                break;
            }
        }
        if (p.max_iter >= 0 && iter >= p.max_iter) {
            if (leader) c->status = kIterLimit;
            break;
        }
        // --- limits of the coming phase (fixed rule, or the schedule's action) ---
        int act = 0;
        if (policy) {
            if (tm.rank == 0 && threadIdx.x < 64) policy_decide<SC>(g, p, c, L, iter);
            if (!grid_barrier<SC>(c, tm, bar_epoch, p.barrier_ticks)) return;
            act = uniform(ld<SC>(&c->action));
        }
        const int64_t budget = act == 0 ? p.relabel_budget : max((int64_t)64, p.relabel_budget * act_budget(act) / 4);
        const int rpl = act == 0 ? p.rounds_per_level : max(1, p.rounds_per_level * act_rpl(act) / 2);
        const int round_cap = p.rounds_per_level > 0 ? min(p.max_rounds, rpl * L + 16) : p.max_rounds;
        const int stall_lim = p.stall_rounds <= 0 ? 0
                              : act == 0      ? max(p.stall_rounds, L)
                                              : (act_stall(act) == 0 ? 0 : max(1, max(p.stall_rounds, L) * act_stall(act) / 2));
        // --- push/relabel rounds ---
        const int32_t rbase = p.seq_base + uniform(ld<SC>(&c->rounds));
        const int active0 =
            uniform(ld<SC>(&c->lst[0].light) + ld<SC>(&c->lst[0].heavy) + ld<SC>(&c->lst[0].huge));
        int r = 0, reason = 0;
        int64_t last_deliv = -1;
        int last_change = 0;
        for (;;) {
            const int rd = r % 3;
            // the round's control words, read together before any decision;
            // all were written before the last barrier, so every workgroup of
            // the team takes the same decisions
            const int64_t lh = uniform(ld<SC>(reinterpret_cast<const int64_t *>(&c->lst[rd])));
            const int nu = uniform(ld<SC>(&c->lst[rd].huge));
            const int64_t prl = uniform(ld<SC>(&c->phase_relabels));
            const int64_t dl = uniform(ld<SC>(&c->phase_deliv));
            const int nl = (int)(uint32_t)lh;
            const int nh = (int)((uint64_t)lh >> 32);
            if (nl + nh + nu == 0) break;
            if (dl != last_deliv) {
                last_deliv = dl;
                last_change = r;
            }
            if (r >= round_cap) {
                reason = 1;
                break;
            }
            if (prl > budget) {
                reason = 2;
                break;
            }
            if (stall_lim > 0 && r - last_change >= stall_lim) {
                reason = 3;
                break;
            }
            // A small round list without huge vertices is worked in a run of
            // rounds, like a small BFS frontier.
            const bool run = !topology && nu == 0 && nl + nh <= run_from;
            bool ok = true, done = false;
            if (!run || runner)
                r = pr_rounds<SC, WALK>(g, run ? run_team : tm, p, PhaseLimits{budget, round_cap, stall_lim}, run, rbase,
                                        r, nl, nh, nu, prl, run_most, &reason, &done, &last_change, sum_epoch, tl, &ok);
            if (SC == kAgent && run && runner && threadIdx.x == 0) {
                c->solo_r = r;
                c->solo_done = done ? 1 : 0;
                c->solo_reason = reason;
                c->solo_last_change = last_change;
            }
            if (!ok || !grid_barrier<SC>(c, tm, bar_epoch, p.barrier_ticks)) return;
            if (run) {
                if (SC == kAgent) {
                    r = uniform(ld<SC>(&c->solo_r));
                    reason = uniform(ld<SC>(&c->solo_reason));
                    last_change = uniform(ld<SC>(&c->solo_last_change));
                    done = uniform(ld<SC>(&c->solo_done)) != 0;
                }
                last_deliv = uniform(ld<SC>(&c->phase_deliv));
                if (done) break;
            }
        }
        // --- RemoveInvalidEdges over the vertices that relabelled ---
        const uint64_t tr = wall_clock64();
        const int nrel = uniform(ld<SC>(&c->nrelab[0])), nrel_long = uniform(ld<SC>(&c->nrelab[1]));
        if (!p.no_rie) remove_invalid<SC>(g, tm, nrel, nrel_long, p.use_gap != 0, tl);
        if (counts)
            for (int64_t i = tm.tid(); i <= g.n; i += tm.nthreads()) g.hcount[i] = 0;
        {
            if (leader && c->ntrace < kTraceCap) {
                int32_t *tr_rec = c->trace[c->ntrace];
                tr_rec[kTrLevels] = L;
                tr_rec[kTrActive] = active0;
                tr_rec[kTrRounds] = r;
                tr_rec[kTrReason] = reason;
                tr_rec[kTrRelabels] = (int32_t)min<int64_t>(ld<SC>(&c->phase_relabels), INT32_MAX);
                tr_rec[kTrRelabelled] = ld<SC>(&c->nfirsts);
                tr_rec[kTrPushes] = (int32_t)min<int64_t>(ld<SC>(&c->phase_pushes), INT32_MAX);
                tr_rec[kTrLastDeliv] = last_change;
                if (policy && g.ptrace)
                    g.ptrace[(int64_t)c->ntrace * kPolRec + kPolF + 1] = (float)(wall_clock64() - tb);
                c->ntrace++;
            }
        }
        if (leader) {
            add<SC>(&c->stat[kStPrTicks], (int64_t)(tr - tp));
            add<SC>(&c->stat[kStRieTicks], (int64_t)(wall_clock64() - tr));
            for (int k = 0; k < 3; ++k) {
                c->qcount[k] = 0;
                c->qverts[k] = 0;
                c->qarcs[k] = 0;
            }
            c->feat_reached = 0;  // counted from the next phase's roots on
            c->rounds += r + 1;
            add<SC>(&c->stat[kStIterations], 1);
            add<SC>(&c->stat[kStRounds], (int64_t)r);
            if ((int64_t)(wall_clock64() - t0) > p.deadline_ticks) c->stop = 1;
        }
        flush_tally<SC>(c, tl);
        if (!grid_barrier<SC>(c, tm, bar_epoch, p.barrier_ticks)) return;
        ++iter;
    }
    // --- value: e(t) plus the deficits of vertices other than s and t, which
    // nothing changed since the last global relabel read them ---
    // (every workgroup reaches this point after the same, uniform decision)
    {
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t sum = 0;
            for (int w = 0; w < (int)(blockDim.x >> 6); ++w) sum += s_def[w];
            if (sum) add<SC>(&c->deficit, sum);
        }
        if (leader) c->e_t = get<SC>(&g.e[g.t]);
    }
    flush_tally<SC>(c, tl);
}

// ---------------------------------------------------------------------------
// Source saturation and repair of a batch
// ---------------------------------------------------------------------------

// Saturate every residual arc out of s: c_f(s,u) -> 0, the twin gains it,
// e(u) += d, e(s) -= d (Alg. 1 third loop; Alg. 4 lines 3-8, where the
// remaining residual is pushed rather than e(u) overwritten).
template <int SC>
__device__ __forceinline__ void saturate_source(const DevGraph &g, const Team &tm) {
    if (ld<SC>(&g.ctrl->err)) return;
    __shared__ int64_t s_sum, s_cnt;
    if (threadIdx.x == 0) {
        s_sum = 0;
        s_cnt = 0;
    }
    __syncthreads();
    const int beg = g.row_ptr[g.s], end = g.row_ptr[g.s + 1];
    int64_t sum = 0, cnt = 0;
    for (int64_t a = beg + tm.tid(); a < end; a += tm.nthreads()) {
        const int2 r = get<SC>(&g.arc[a]);
        if (r.y > 0) {
            g.arc[a].y = 0;
            add<SC>(cf_ptr(g.arc, g.twin[a]), r.y);
            add<SC>(&g.e[r.x], (int64_t)r.y);
            sum += r.y;
            cnt++;
        }
    }
    sum = wave_sum(sum);
    cnt = wave_sum(cnt);
    if (lane_id() == 0 && sum) {
        atomicAdd((unsigned long long *)&s_sum, (unsigned long long)sum);
        atomicAdd((unsigned long long *)&s_cnt, (unsigned long long)cnt);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_sum) {
        add<SC>(&g.e[g.s], -s_sum);
        add<SC>(&g.ctrl->stat[kStSourcePushes], s_cnt);
    }
}

__global__ void k_saturate_source(DevGraph g) {
    saturate_source<kAgent>(g, Team{(int)blockIdx.x, (int)gridDim.x});
}

// Edges per thread of a batch that one workgroup repairs alone.
constexpr int kAloneEdges = kRepairMax / kBlock;

// Batch validation: ids in [0, m), capacities in [0, cap_limit], ids distinct
// (a batch is a set).  Sets Ctrl::err; the rest of the call then leaves the
// state alone.
__global__ void k_validate_updates(DevGraph g, Repair b) {
    const Team tm{(int)blockIdx.x, (int)gridDim.x};
    for (int64_t i = tm.tid(); i < b.k; i += tm.nthreads()) {
        const int64_t id = b.ids[i];
        const int32_t cv = b.caps[i];
        if (id < 0 || id >= g.m) {
            atomicOr(&g.ctrl->err, 1);
            continue;
        }
        if (cv < 0 || cv > b.cap_limit) atomicOr(&g.ctrl->err, 2);
        if (atomicExch(&g.stamp[id], b.epoch) == b.epoch) atomicOr(&g.ctrl->err, 4);
    }
}

// Alg. 5 first loop: c_f(u,v) += c' - c; the stored capacities follow.
__global__ void k_apply_delta(DevGraph g, Repair b) {
    if (ld<kAgent>(&g.ctrl->err)) return;
    const Team tm{(int)blockIdx.x, (int)gridDim.x};
    int64_t cnt = 0;
    for (int64_t i = tm.tid(); i < b.k; i += tm.nthreads()) {
        const int64_t id = b.ids[i];
        const int32_t cv = b.caps[i];
        const int32_t a = g.edge2arc[id];
        const int32_t d = cv - g.ecap[id];
        g.ecap[id] = cv;
        if (a >= 0 && d != 0) {
            add<kAgent>(&g.cap[a], d);
            add<kAgent>(cf_ptr(g.arc, a), d);
        }
        cnt++;
    }
    cnt = wave_sum(cnt);
    if (lane_id() == 0 && cnt) add<kAgent>(&g.ctrl->stat[kStUpdates], cnt);
}

// Alg. 5 second loop restricted to the updated arc pairs (only they can have
// gone negative), with the excess change booked at once: the flow clamped by
// o = -c_f(a) returns o units to the tail (e += o) and takes them from the
// head (e -= o).  At most one arc of a pair can be negative (their residuals
// sum to the pair's capacity); a compare-and-swap makes each clamp happen
// once even when several updates share a pair.
template <int SC>
__device__ __forceinline__ int clamp_arc(const DevGraph &g, int x, int y, int32_t cv, int tail, int head) {
    if (!cas<SC>(cf_ptr(g.arc, x), cv, 0)) return 0;
    const int32_t o = -cv;
    add<SC>(cf_ptr(g.arc, y), -o);
    add<SC>(&g.e[tail], (int64_t)o);
    add<SC>(&g.e[head], -(int64_t)o);
    return 1;
}
__global__ void k_clamp(DevGraph g, Repair b) {
    if (ld<kAgent>(&g.ctrl->err)) return;
    const Team tm{(int)blockIdx.x, (int)gridDim.x};
    int64_t cnt = 0;
    for (int64_t i = tm.tid(); i < b.k; i += tm.nthreads()) {
        const int32_t a0 = g.edge2arc[b.ids[i]];
        if (a0 < 0) continue;
        const int32_t a1 = g.twin[a0];
        const int32_t r0 = ld<kAgent>(cf_ptr(g.arc, a0)), r1 = ld<kAgent>(cf_ptr(g.arc, a1));
        if (r0 >= 0 && r1 >= 0) continue;
        const int head = get<kAgent>(&g.arc[a0]).x, tail = get<kAgent>(&g.arc[a1]).x;
        if (r0 < 0) cnt += clamp_arc<kAgent>(g, a0, a1, r0, tail, head);
        if (r1 < 0) cnt += clamp_arc<kAgent>(g, a1, a0, r1, head, tail);
    }
    cnt = wave_sum(cnt);
    if (lane_id() == 0 && cnt) add<kAgent>(&g.ctrl->stat[kStClamps], cnt);
}

// ---------------------------------------------------------------------------
// Local stage of a dynamic update, between the batch repair (Alg. 5) and the
// global loop: the updated arcs that now cross the last cut are saturated,
// and the deficits the batch left are filled from excess nearby (the ideas of
// Dynamic Push-Pull, Sec. 4.2 / Alg. 6 and 8, applied to the batch's own
// arcs).  Every step is a push along a residual arc, so the global loop that
// follows, with its unchanged termination test, still ends at a maximum flow;
// the stage only saves it the work of letting every vertex that holds excess
// on the source side chase a small deficit.
// ---------------------------------------------------------------------------

// Saturate every updated arc that is residual from the source side of the
// last cut (height |V|) to its sink side (height < |V|).  A solved state has
// no such arc, and only arcs whose capacity grew can have gained one: the
// clamp and the source re-saturation only lower residuals across it.  The
// flow moved becomes excess at the head and a deficit at the tail (Alg. 8,
// "remove S to T edges", on the batch).  Heights are those of the last
// global relabel.
template <int SC>
__device__ __forceinline__ void cut_arc_saturate(const DevGraph &g, int x, int y, int tail, int head) {
    if (ld<SC>(cf_ptr(g.arc, x)) <= 0) return;
    const int32_t c = xchg<SC>(cf_ptr(g.arc, x), 0);  // updates sharing the pair: one takes it
    if (c > 0) {
        add<SC>(cf_ptr(g.arc, y), c);
        add<SC>(&g.e[tail], -(int64_t)c);
        add<SC>(&g.e[head], (int64_t)c);
    }
}
__global__ void k_cut_saturate(DevGraph g, Repair b) {
    if (ld<kAgent>(&g.ctrl->err)) return;
    const Team tm{(int)blockIdx.x, (int)gridDim.x};
    for (int64_t i = tm.tid(); i < b.k; i += tm.nthreads()) {
        const int32_t a0 = g.edge2arc[b.ids[i]];
        if (a0 < 0) continue;
        const int32_t a1 = g.twin[a0];
        const int2 r0 = g.arc[a0], r1 = g.arc[a1];
        const bool h0 = g.h[r0.x] >= g.n, h1 = g.h[r1.x] >= g.n;  // head of a0, and its tail
        if (h1 && !h0) cut_arc_saturate<kAgent>(g, a0, a1, r1.x, r0.x);
        if (h0 && !h1) cut_arc_saturate<kAgent>(g, a1, a0, r0.x, r1.x);
    }
}

// One round of local pulls.  Every deficient vertex v of list `in` takes what
// it lacks from its in-neighbours w (residual arc w -> v) that hold excess,
// in arc order: d moves as a push from w to v (c_f(w,v) -= d, c_f(v,w) += d,
// e(w) -= d, e(v) += d), as Alg. 6 pulls, here without heights.  With `out`,
// what is still lacking is then taken from in-neighbours along their residual
// arcs whatever their excess, which hands the deficit on to them; a giver
// left with a deficit joins `out` (once, pmark tag).  s and t never give.  A
// wavefront per vertex; v's own excess is touched by its wavefront only.
// Each pass looks at no more than kPullScan arcs of v, the excess pass at the
// front of v's list and the hand-on pass at its back (from the last chunk
// backwards), so that a hub costs a bounded number of steps and the deficit
// is handed on to the neighbours at the end of the list (the low-degree ones
// when vertices are numbered by falling degree); what stays lacking is left
// to the global loop.
constexpr int kPullScan = 4096;
// The first round takes its vertices from the batch itself (ids, k: both
// ends of every updated arc pair, s and t left out, each deficient vertex
// claimed once with tag - 1); the later ones from the list `in` of the round
// before.  Marks only grow (pmark holds the largest tag given to a vertex,
// tags rise from call to call), so a claim or an append takes a vertex only
// if its mark is still below the tag: a vertex that round 0 already put on
// the next round's list (tag) is not claimed again as a batch end (tag - 1)
// while its first visit may still be running.  The list counters rotate over
// three words, cnt[r % 3] read and cnt[(r + 1) % 3] appended to by round r,
// which clears cnt[(r + 2) % 3] for round r + 1; they all start at zero with
// the call's control block.
//
// A wavefront looks its share of the batch up lane by lane and then visits the
// deficient ends it found, one after another: what bounds a large batch is the
// chain of lookups before a visit (the first round on 336 k ends of R-MAT 2^20:
// 82 us with a wavefront per end, 18.5 us so).
template <int SC>
__device__ __forceinline__ void pull_round(const DevGraph &g, const Team &tm, const Repair &b, const int32_t *in,
                                           int r, int32_t *out) {
    const int lane = lane_id();
    const int32_t tag = b.tag + r;
    int32_t *cnt = g.ctrl->pull_cnt;
    if (tm.rank == 0 && threadIdx.x == 0) cnt[(r + 2) % 3] = 0;
    int32_t *out_cnt = &cnt[(r + 1) % 3];
    const int64_t items = r == 0 ? 2 * b.k : (int64_t)ld<SC>(&cnt[r % 3]);
    const int64_t nwaves = tm.nwaves();
    const int share = (int)min((int64_t)64, (items + nwaves - 1) / nwaves);
    for (int64_t base = tm.wave() * share; base < items; base += nwaves * share) {
        const int64_t i = base + lane;
        int mine = -1;
        int64_t lacks = 0;
        if (lane < share && i < items) {
            int w;
            if (r == 0) {
                const int32_t a0 = g.edge2arc[b.ids[i >> 1]];
                w = a0 < 0 ? -1 : get<SC>(&g.arc[(i & 1) ? g.twin[a0] : a0]).x;
                if (w == g.s || w == g.t) w = -1;
                if (w >= 0) {
                    lacks = -ld<SC>(&g.e[w]);
                    if (lacks > 0 && __hip_atomic_fetch_max(&b.pmark[w], tag - 1, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT) < tag - 1)
                        mine = w;
                }
            } else {
                mine = get<SC>(&in[i]);
                lacks = -ld<SC>(&g.e[mine]);
            }
        }
        uint64_t todo = __ballot(mine >= 0 && lacks > 0);
        while (todo) {
            const int from = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const int v = lane_value(mine, from);
            const int64_t need = -uniform(ld<SC>(&g.e[v]));
            if (need <= 0) continue;
            const int beg = g.row_ptr[v], end = g.row_ptr[v + 1];
            int64_t got = 0;
            // chunks of 64 arcs aligned to the start of v's list in both passes,
            // so that an arc the first pass pushed along is read again by the
            // same lane (its own earlier atomic orders the read; another lane's
            // would not)
            const int nchunks = (end - beg + 63) / 64;
            for (int hand_on = 0; hand_on < (out ? 2 : 1) && got < need; ++hand_on) {
                const int lo = hand_on ? max(beg, end - kPullScan) : beg;
                const int hi = hand_on ? end : min(end, beg + kPullScan);
                const int c_first = hand_on ? nchunks - 1 : 0;
                const int c_last = hand_on ? (lo - beg) / 64 : (hi - beg + 63) / 64 - 1;
                for (int c = c_first; (hand_on ? c >= c_last : c <= c_last) && got < need; c += hand_on ? -1 : 1) {
                    const int a = beg + 64 * c + lane;
                    int64_t avail = 0;
                    int w = -1, tw = 0;
                    if (a >= lo && a < hi) {
                        w = get<SC>(&g.arc[a]).x;
                        tw = g.twin[a];
                        if (w != g.s && w != g.t) {
                            const int32_t r = ld<SC>(cf_ptr(g.arc, tw));
                            if (r > 0) {
                                if (hand_on) {
                                    avail = r;
                                } else {
                                    const int64_t ew = ld<SC>(&g.e[w]);
                                    if (ew > 0) avail = min((int64_t)r, ew);
                                }
                            }
                        }
                    }
                    const int64_t incl = wave_incl_scan64(avail);
                    const int64_t excl = incl - avail;
                    const int64_t room = need - got;
                    const int64_t d = (avail > 0 && excl < room) ? min(avail, room - excl) : 0;
                    int64_t moved = 0;
                    if (d > 0) {
                        // The excess pass claims its share of w's excess first and
                        // gives back what w no longer holds (other deficits may pull
                        // from the same giver at once), so that it never overdraws a
                        // giver: an overdrawn giver left after the last round is a
                        // deficit that the global loop would reach from the whole
                        // source side.  The hand-on pass takes along the residual
                        // whatever w holds, and lists a giver it leaves in deficit.
                        const int64_t old = fetch_add<SC>(&g.e[w], -d);
                        moved = d;
                        if (!hand_on) {
                            moved = old >= d ? d : (old > 0 ? old : 0);
                            if (moved < d) add<SC>(&g.e[w], d - moved);
                        }
                        if (moved > 0) {
                            add<SC>(cf_ptr(g.arc, tw), -(int32_t)moved);
                            add<SC>(cf_ptr(g.arc, a), (int32_t)moved);
                        }
                        if (out && hand_on && old - d < 0 &&
                            __hip_atomic_fetch_max(&b.pmark[w], tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < tag)
                            out[fetch_add<SC>(out_cnt, 1)] = w;
                    }
                    got += wave_sum(moved);
                }
            }
            if (lane == 0 && got > 0) add<SC>(&g.e[v], got);
        }
    }
}

__global__ void k_pull_round(DevGraph g, Repair b, const int32_t *in, int r, int32_t *out) {
    if (ld<kAgent>(&g.ctrl->err)) return;
    pull_round<kAgent>(g, Team{(int)blockIdx.x, (int)gridDim.x}, b, in, r, out);
}

// Repair of a batch of at most kRepairMax edges by one workgroup, up to the
// pulls; the source only with `source`.  Everything that the steps look up
// (ids, arcs, twins, ends, heights) is loaded once, at the validation, and
// kept; a step then waits for its own atomics only.  Works as a team of one
// XCD does, so that no stale line is left in the L1.
__device__ __forceinline__ void repair_alone(const DevGraph &g, const Repair &b, bool source) {
    constexpr int SC = kXcd, U = kAloneEdges;
    int64_t id[U];
    int32_t cv[U], a0[U], a1[U], d[U], head[U], tail[U];
    bool mine[U], up[U], down[U];  // on the source side: tail only (of a0), head only
    int bad = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t i = threadIdx.x + (int64_t)u * kBlock;
        mine[u] = i < b.k;
        id[u] = mine[u] ? b.ids[i] : 0;
        cv[u] = mine[u] ? b.caps[i] : 0;
        if (mine[u] && (cv[u] < 0 || cv[u] > b.cap_limit)) bad |= 2;
        if (mine[u] && (id[u] < 0 || id[u] >= g.m)) {
            bad |= 1;
            mine[u] = false;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        a0[u] = mine[u] ? g.edge2arc[id[u]] : -1;
        d[u] = mine[u] ? cv[u] - g.ecap[id[u]] : 0;
        if (mine[u] && atomicExch(&g.stamp[id[u]], b.epoch) == b.epoch) bad |= 4;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) a1[u] = a0[u] >= 0 ? g.twin[a0[u]] : 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        head[u] = a0[u] >= 0 ? get<SC>(&g.arc[a0[u]]).x : 0;
        tail[u] = a0[u] >= 0 ? get<SC>(&g.arc[a1[u]]).x : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool hs = g.h[head[u]] >= g.n, ts = g.h[tail[u]] >= g.n;
        up[u] = ts && !hs;
        down[u] = hs && !ts;
    }
    if (bad) atomicOr(&g.ctrl->err, bad);
    if (__syncthreads_or(bad)) return;
    int cnt = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (!mine[u]) continue;
        g.ecap[id[u]] = cv[u];
        if (a0[u] >= 0 && d[u] != 0) {
            add<SC>(&g.cap[a0[u]], d[u]);
            add<SC>(cf_ptr(g.arc, a0[u]), d[u]);
        }
        cnt++;
    }
    cnt = wave_sum(cnt);
    if (lane_id() == 0 && cnt) add<SC>(&g.ctrl->stat[kStUpdates], (int64_t)cnt);
    block_sync<SC>();
    cnt = 0;
    int32_t r0[U], r1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        r0[u] = a0[u] >= 0 ? ld<SC>(cf_ptr(g.arc, a0[u])) : 0;
        r1[u] = a0[u] >= 0 ? ld<SC>(cf_ptr(g.arc, a1[u])) : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (r0[u] < 0) cnt += clamp_arc<SC>(g, a0[u], a1[u], r0[u], tail[u], head[u]);
        if (r1[u] < 0) cnt += clamp_arc<SC>(g, a1[u], a0[u], r1[u], head[u], tail[u]);
    }
    cnt = wave_sum(cnt);
    if (lane_id() == 0 && cnt) add<SC>(&g.ctrl->stat[kStClamps], (int64_t)cnt);
    block_sync<SC>();
    // (the arcs out of s are the source saturation's, now or later)
    if (b.pulls) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (a0[u] >= 0 && up[u] && tail[u] != g.s) cut_arc_saturate<SC>(g, a0[u], a1[u], tail[u], head[u]);
            if (a0[u] >= 0 && down[u] && head[u] != g.s) cut_arc_saturate<SC>(g, a1[u], a0[u], head[u], tail[u]);
        }
    }
    if (source) saturate_source<SC>(g, Team{0, 1});
}

// The repair of a dynamic update at the head of its solve kernel: validation,
// capacity changes and clamps (Alg. 5), the source saturated again, and the
// local stage.  As kernels of their own these were ten launches of 2 to 4 us
// with 4 to 8 us between them; here a step of the team ends with its barrier
// (1 us on one XCD, 4 to 5 all over the device), and the batch itself is the
// first workgroup's alone (repair_alone), which has still cheaper barriers, as
// is the source when its list is as short as a batch.  The pulls are made by the
// whole team and stop at the first round that hands nothing on.  Returns false
// when a barrier failed.  A whole update, kernels of their own against this:
// 1 k vertices, 100 edges 95 -> 52 us; 20 k vertices, 1000 edges 112 -> 75;
// R-MAT 2^20, 1000 edges 180 -> 140.
template <int SC>
__device__ __forceinline__ bool repair(const DevGraph &g, const Team &tm, const LoopParams &p, const Repair &b,
                                       uint32_t &epoch) {
    constexpr int PS = SC == kGroup ? kXcd : SC;  // scope of the pulls
    const bool source_alone = SC == kGroup || g.row_ptr[g.s + 1] - g.row_ptr[g.s] <= kRepairMax;
    if (tm.rank == 0) repair_alone(g, b, source_alone);
    block_sync<PS>();
    if (!grid_barrier<SC>(g.ctrl, tm, epoch, p.barrier_ticks)) return false;
    if (ld<PS>(&g.ctrl->err)) return true;
    if constexpr (SC != kGroup) {
        if (!source_alone) {
            saturate_source<SC>(g, tm);
            if (!grid_barrier<SC>(g.ctrl, tm, epoch, p.barrier_ticks)) return false;
        }
    }
    for (int r = 0; r < b.pulls; ++r) {
        const bool last = r == b.pulls - 1;
        pull_round<PS>(g, tm, b, (r & 1) ? g.list[2] : g.list[1], r, last ? nullptr : (r & 1) ? g.list[1] : g.list[2]);
        block_sync<PS>();
        if (!grid_barrier<SC>(g.ctrl, tm, epoch, p.barrier_ticks)) return false;
        if (last || uniform(ld<PS>(&g.ctrl->pull_cnt[(r + 1) % 3])) == 0) break;
    }
    return true;
}

// The whole grid is one team (see join_team), or a single workgroup.
// WALK: long arc lists are visited by the downhill walk (else scan first);
// the two are separate instances, since both inlined side by side would spill.
template <int BLOCK, int SC, bool WALK>
__global__ void __launch_bounds__(BLOCK) k_loop(DevGraph g, LoopParams p, Repair b) {
    Team tm{0, 1};
    uint32_t epoch = 0;  // barriers this launch has passed
    if constexpr (SC != kGroup) {
        tm = join_team<SC>(g.ctrl, p.team_want, p.join_ticks);
        if (tm.size == 0) return;
        init_stages();
    }
    if (b.on && !repair<SC>(g, tm, p, b, epoch)) return;
    solve_loop<SC, WALK>(g, tm, p, epoch);
    // the control block to the host, which saves a copy's dispatch
    block_sync<SC == kGroup ? kXcd : SC>();
    if (!grid_barrier<SC>(g.ctrl, tm, epoch, p.barrier_ticks)) return;
    if (b.host && tm.rank == 0) {
        constexpr int from = (int)(offsetof(Ctrl, qcount) / sizeof(int)), words = (int)(sizeof(Ctrl) / sizeof(int));
        const int *w = reinterpret_cast<const int *>(g.ctrl);
        int *out = reinterpret_cast<int *>(b.host);
        for (int i = from + threadIdx.x; i < words; i += BLOCK) out[i] = ld<SC == kGroup ? kXcd : SC>(&w[i]);
    }
}

// A view read from a device table, its pointers read as pointers to global
// memory.  Read as they are they would be generic addresses, and every access
// through them a flat one, which also waits on the LDS counter.
template <typename T>
__device__ __forceinline__ T *as_global(T *const &field) {
    using Global = __attribute__((address_space(1))) T;
    return (T *)*reinterpret_cast<Global *const *>(&field);
}
__device__ __forceinline__ DevGraph global_view(const DevGraph &v) {
    DevGraph g;
    g.n = v.n;
    g.s = v.s;
    g.t = v.t;
    g.A = v.A;
    g.m = v.m;
    g.qcap = v.qcap;
    g.n_heavy_all = v.n_heavy_all;
    g.n_bu_items = v.n_bu_items;
    g.part_want = v.part_want;
    g.part_restrict = v.part_restrict;
    g.row_ptr = as_global(v.row_ptr);
    g.arc = as_global(v.arc);
    g.twin = as_global(v.twin);
    g.cap = as_global(v.cap);
    g.edge2arc = as_global(v.edge2arc);
    g.ecap = as_global(v.ecap);
    g.stamp = as_global(v.stamp);
    g.e = as_global(v.e);
    g.h = as_global(v.h);
    g.q[0] = as_global(v.q[0]);
    g.q[1] = as_global(v.q[1]);
    g.list[0] = as_global(v.list[0]);
    g.list[1] = as_global(v.list[1]);
    g.list[2] = as_global(v.list[2]);
    g.huge[0] = as_global(v.huge[0]);
    g.huge[1] = as_global(v.huge[1]);
    g.huge[2] = as_global(v.huge[2]);
    g.mark = as_global(v.mark);
    g.rmark = as_global(v.rmark);
    g.relab = as_global(v.relab);
    g.hcount = as_global(v.hcount);
    g.heavy_all = as_global(v.heavy_all);
    g.bu_items = as_global(v.bu_items);
    g.ptrace = as_global(v.ptrace);
    g.ctrl = as_global(v.ctrl);
    g.part = as_global(v.part);
    return g;
}

// Two teams in one cooperative launch: workgroups [0, split) run the solve
// loop on view a, the others on view b, each view with its own state and
// control block (its own barrier).  The views must touch disjoint arc pairs
// and vertices (the S and T sides of a cut with no residual arc from S to
// T).  split follows the arc counts work[0] (view a) and work[1] (view b),
// at least one workgroup each.
template <int BLOCK, bool WALK>
__global__ void __launch_bounds__(BLOCK)
    k_teams(const DevGraph *__restrict__ views, const LoopParams *__restrict__ params, const int64_t *work) {
    init_stages();
    const int G = (int)gridDim.x;
    const int64_t wa = work[0], wb = work[1];
    int64_t sp = (wa + wb) > 0 ? ((int64_t)G * wa + (wa + wb) / 2) / (wa + wb) : G / 2;
    const int split = (int)min((int64_t)G - 1, max((int64_t)1, sp));
    const int side = (int)blockIdx.x < split ? 0 : 1;
    const Team tm = side == 0 ? Team{(int)blockIdx.x, split} : Team{(int)blockIdx.x - split, G - split};
    const LoopParams &p = params[side];
    uint32_t epoch = 0;
    solve_loop<kAgent, WALK>(global_view(views[side]), tm, p, epoch);
}

// ---------------------------------------------------------------------------
// Part tags and views of the residual state (Dynamic Push-Pull, Sec. 4.2 /
// Alg. 8; returning excess to s and filling deficits from t, Sec. 3.1 and the
// proof of Sec. 4.1.1)
// ---------------------------------------------------------------------------

// part[v] = T when the last global relabel reached v (h < |V|: v reaches t or
// a deficient vertex in the residual graph), S otherwise (Alg. 8 first loop).
// work[0] / work[1] receive the arcs of the S / T vertices (cleared before).
__global__ void k_part_from_heights(DevGraph g, uint8_t *part, int64_t *work) {
    int64_t ws = 0, wt = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < g.n;
         v += (int64_t)gridDim.x * blockDim.x) {
        const bool tside = g.h[v] < g.n;
        part[v] = tside ? kPartT : kPartS;
        const int64_t d = g.row_ptr[v + 1] - g.row_ptr[v];
        if (tside) wt += d;
        else ws += d;
    }
    ws = wave_sum(ws);
    wt = wave_sum(wt);
    if (lane_id() == 0) {
        if (ws) add<kAgent>(&work[0], ws);
        if (wt) add<kAgent>(&work[1], wt);
    }
}

// After the two teams of a push-pull update: vertices that neither the
// backward BFS (heights h, from t and the deficient vertices of T) nor the
// forward BFS (heights hv, from s and the overflowing vertices of S) reached
// form P (Alg. 8, the localized stage); the others keep their side.
__global__ void k_part_localized(DevGraph g, const int32_t *hv, uint8_t *part) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < g.n;
         v += (int64_t)gridDim.x * blockDim.x)
        if (g.h[v] >= g.n && hv[v] >= g.n) part[v] = kPartP;
}

// Saturate every residual arc from S to T (Alg. 8, "remove S to T edges"),
// booking the moved flow as excess at the head and deficit at the tail (the
// paper recomputes every excess afterwards; the change is the same).
__global__ void k_saturate_cut(DevGraph g, const uint8_t *part) {
    for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < g.A;
         a += (int64_t)gridDim.x * blockDim.x) {
        const int2 r = g.arc[a];
        if (r.y <= 0 || part[r.x] != kPartT) continue;
        const int32_t tw = g.twin[a];
        const int u = g.arc[tw].x;  // tail of a
        if (part[u] != kPartS) continue;
        g.arc[a].y = 0;  // only this thread touches the pair: its twin runs T -> S
        add<kAgent>(cf_ptr(g.arc, tw), r.y);
        add<kAgent>(&g.e[u], -(int64_t)r.y);
        add<kAgent>(&g.e[r.x], (int64_t)r.y);
    }
}

// Build a view of the state: rev = 0 copies arcs and excesses; rev = 1 gives
// arc a = (u, v) the residual of its twin (v, u) and every excess the
// opposite sign.  In the reversed view, pulling d into u along (v, u)
// (Alg. 6: c_f(v, u) -= d, c_f(u, v) += d, e(u) += d, e(v) -= d) is pushing d
// from u to v; the forward BFS of h_- is the backward BFS of the view, and
// the invalid-edge rule of Alg. 7 is that of Alg. 3 in the view.
__global__ void k_view_make(DevGraph g, int2 *varc, int64_t *ve, int rev) {
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t a = gtid; a < g.A; a += stride) {
        const int2 r = g.arc[a];
        varc[a] = rev ? make_int2(r.x, g.arc[g.twin[a]].y) : r;
    }
    for (int64_t v = gtid; v < g.n; v += stride) ve[v] = rev ? -g.e[v] : g.e[v];
}

// Write back a view's arcs between two vertices tagged `want`, and their
// excesses (rev: the view is reversed).
__global__ void k_view_merge(DevGraph g, const int2 *varc, const int64_t *ve, const uint8_t *part,
                             uint8_t want, int rev) {
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t a = gtid; a < g.A; a += stride) {
        const int32_t tw = g.twin[a];
        const int head = g.arc[a].x, tail = g.arc[tw].x;
        if (part[head] == want && part[tail] == want) g.arc[a].y = rev ? varc[tw].y : varc[a].y;
    }
    for (int64_t v = gtid; v < g.n; v += stride)
        if (part[v] == want) g.e[v] = rev ? -ve[v] : ve[v];
}

// Per-edge flow from the pair flows of a valid flow.  The flow on arc a is
// f(a) = cap(a) - c_f(a) where positive; it is shared out among the input
// edges merged into a, each taking min(its capacity, what is left), so that
// 0 <= flow <= capacity for every edge and the edges of a carry f(a).  rem
// (int32[A]) holds what is left per arc; edges of one arc draw from it with a
// compare-and-swap (in no fixed order among duplicates).
__global__ void k_arc_flow(DevGraph g, const int2 *carc, int32_t *rem) {
    for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < g.A;
         a += (int64_t)gridDim.x * blockDim.x)
        rem[a] = max(0, g.cap[a] - carc[a].y);
}

__global__ void k_edge_flow(DevGraph g, int32_t *rem, int32_t *flow) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < g.m;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t a = g.edge2arc[i];
        const int32_t c = g.ecap[i];
        int32_t give = 0;
        if (a >= 0 && c > 0) {
            int32_t old = ld<kAgent>(&rem[a]);
            for (;;) {
                give = min(c, old);
                if (give == 0) break;
                if (__hip_atomic_compare_exchange_strong(&rem[a], &old, old - give, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, kAgent))
                    break;
            }
        }
        flow[i] = give;
    }
}

// ---------------------------------------------------------------------------
// Initialisation, source saturation and update repair
// ---------------------------------------------------------------------------

// Start of a call: the control block is cleared, and a batch that waits in
// pinned host memory is fetched (`words` words; read over the bus by the
// kernel, which saves the copy's own dispatch).
__global__ void k_begin(Ctrl *c, const int32_t *src, int32_t *dst, int64_t words) {
    if (blockIdx.x == 0) {
        int *w = reinterpret_cast<int *>(c);
        for (int i = threadIdx.x; i < (int)(sizeof(Ctrl) / sizeof(int)); i += blockDim.x) w[i] = 0;
    }
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) dst[i] = src[i];
}

// Alg. 1 first loops: e = 0, h = 0, c_f = c.
__global__ void k_init_state(DevGraph g) {
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t a = gtid; a < g.A; a += stride) g.arc[a].y = g.cap[a];
    for (int64_t v = gtid; v < g.n; v += stride) {
        g.e[v] = 0;
        g.h[v] = 0;
    }
}

// Certificate: side of the caller's vertex v (internal number new_of_old[v], or
// v) = 1 when h(v) >= |V|; cut = sum of cap over arcs from the source side to
// the sink side, taken from the sink side's lists (the twins of its arcs whose
// head is on the source side).  The sink side is usually the smaller one by
// far, and a list of it is read in order with one height gather per arc; only
// a crossing arc reads its twin and that arc's capacity.  If some list has more
// than kChunk arcs, those of more than kCutList go to k_cut_items in items: hubs
// are split over the device, and vertices of many arcs, which are neighbours in
// the degree order, do not end up with one wavefront (up to 64 x 256 arcs, one
// step after another).  A small graph's vertices go to more wavefronts for the
// same reason.  With the cut at s, all lists of the sink side: R-MAT 2^14 142 us,
// 43 so, 2^16 177 and 84, 2^18 245 and 132; 100 vertices of 180 arcs 61 and 19.
// Bound by the read of the heights when the sink side is small.  R-MAT 2^22 x
// 16: 5.1 ms (scanning the source side, the numbering undone on the host) ->
// 0.36 ms; 2^20: 1.12 -> 0.11 ms; a 512 x 512 grid: 175 -> 112 us; 20 k vertices:
// 62 -> 17 us, one launch (without lists to split) and no copy.
__device__ __forceinline__ int64_t cut_arc(const DevGraph &g, int a) {
    return g.h[g.arc[a].x] >= g.n ? (int64_t)g.cap[g.twin[a]] : 0;
}

// The last workgroup of the launch hands the sum out and leaves the words at
// zero for the next cut.  Every thread calls it.
__device__ __forceinline__ void cut_finish(Ctrl *c, int64_t *cut) {
    block_sync<kXcd>();  // the workgroup's additions have been made
    if (threadIdx.x != 0) return;
    const int last = (int)gridDim.x - 1;
    if (__hip_atomic_fetch_add(&c->cut_done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != last) return;
    *cut = __hip_atomic_exchange(&c->cut, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    c->cut_items = 0;
    c->cut_done = 0;
}

// cut: where the sum goes, or null if k_cut_items follows.  per: vertices of a
// wavefront at a time.
constexpr int kCutList = 16;  // arcs of a list that its wavefront reads itself
__global__ void k_cut_side(DevGraph g, const int32_t *new_of_old, uint8_t *side, int64_t *cut, int per) {
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if (side) {  // four vertices a word (side is allocated in whole words)
        for (int64_t w = gtid; 4 * w < g.n; w += stride) {
            uint32_t bits = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t v = 4 * w + k;
                if (v < g.n && g.h[new_of_old ? new_of_old[v] : v] >= g.n) bits |= 1u << (8 * k);
            }
            reinterpret_cast<uint32_t *>(side)[w] = bits;
        }
    }
    const int lane = lane_id();
    const int longest = cut ? INT32_MAX : kCutList;
    int64_t part = 0;
    for (int64_t base = (gtid >> 6) * per; base < g.n; base += (stride >> 6) * per) {
        const int64_t v = base + lane;
        int beg = 0, len = 0;
        if (lane < per && v < g.n && g.h[v] < g.n) {
            beg = g.row_ptr[v];
            len = g.row_ptr[v + 1] - beg;
        }
        if (__ballot(len > 0) == 0) continue;
        const int ni = len > longest ? n_items(len) : 0;
        const int slot = wave_appendn<kAgent>(&g.ctrl->cut_items, ni);
        for (int k = 0; k < ni; ++k)
            g.q[0][slot + k] = make_int2(beg + k * kChunk, min(beg + (k + 1) * kChunk, beg + len));
        if (ni) len = 0;
        const int incl = wave_incl_scan(len);
        const int excl = incl - len, total = lane_value(incl, 63);
        const uint64_t full = __ballot(len > 0);
        for (int off = 0; off < total; off += 64) {
            // the lane whose list holds arc off + lane: the last of those that
            // start there or before (empty lists start where the next one does)
            int o = 0;
#pragma unroll
            for (int step = 32; step >= 1; step >>= 1) {
                const int ex = __shfl(excl, o + step, 64);
                if (ex <= off + lane) o += step;
            }
            const int a = __shfl(beg, o, 64) + (off + lane - __shfl(excl, o, 64));
            if (off + lane < total && ((full >> o) & 1)) part += cut_arc(g, a);
        }
    }
    part = wave_sum(part);
    if (lane == 0 && part) add<kAgent>(&g.ctrl->cut, part);
    if (cut) cut_finish(g.ctrl, cut);
}

__global__ void k_cut_items(DevGraph g, int64_t *cut) {
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int cnt = g.ctrl->cut_items;
    int64_t part = 0;
    for (int64_t i = wave; i < cnt; i += nwaves) {
        const int2 it = g.q[0][i];
        for (int a = it.x + lane; a < it.y; a += 64) part += cut_arc(g, a);
    }
    part = wave_sum(part);
    if (lane == 0 && part) add<kAgent>(&g.ctrl->cut, part);
    cut_finish(g.ctrl, cut);
}

__global__ void k_fill_i32(int32_t *p, int64_t count, int32_t value) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

static int grid_for(int64_t work, int block, int cap = 8192);

// Invariants of a residual state (the debug check after a solving call).
__global__ void k_check_state(DevGraph g, int solved) {
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int32_t f = 0;
    for (int64_t a = gtid; a < g.A; a += stride) {
        const int2 r = g.arc[a];
        const int32_t tw = g.twin[a];
        const int2 q = g.arc[tw];
        if (r.y < 0) f |= 1;
        if ((int64_t)r.y + q.y != (int64_t)g.cap[a] + g.cap[tw]) f |= 2;
        if (solved && r.y > 0 && g.h[q.x] >= g.n && g.h[r.x] < g.n) f |= 16;  // q.x: tail of a
    }
    for (int64_t v = gtid; v < g.n; v += stride) {
        int64_t x = 0;
        for (int a = g.row_ptr[v]; a < g.row_ptr[v + 1]; ++a) x += (int64_t)g.arc[a].y - g.cap[a];
        if (x != g.e[v]) f |= 4;
        if (solved && v != g.s && v != g.t && g.e[v] > 0 && g.h[v] < g.n) f |= 8;
    }
    if (f) atomicOr(&g.ctrl->check, f);
}

hipError_t launch_check_state(const DevGraph &g, int solved, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, &g.ctrl->check, (int64_t)1, 0);
    const int64_t work = g.A > g.n ? g.A : g.n;
    hipLaunchKernelGGL(k_check_state, dim3(grid_for(work, 256, 4096)), dim3(256), 0, st, g, solved);
    return hipGetLastError();
}


// ---------------------------------------------------------------------------
// Batched solve: one workgroup per instance, or a team of one XCD
// ---------------------------------------------------------------------------

// order[blockIdx.x] names the instance.  Its workgroup clears the control
// block, stamps and per-height counts, initialises the state (c_f = c,
// e = h = 0), saturates the source and runs the solve loop to the end, all
// separated by workgroup barriers only; res[i] receives the value and the
// loop status.  Workgroups never wait for each other.
//
// Workgroups of 256 threads get three wavefronts to a SIMD, so 168 registers (it
// would take 196, and two wavefronts): batches of many small instances are bound
// by how many run at once.  4000 grids of side 10 to 39: 24.0 ms with two, 17.4
// with three; 4000 random graphs of 50 to 1050 vertices 3.84 and 2.91 ms.
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK, BLOCK == 256 ? 3 : BLOCK / 256)
    k_batch(const DevGraph *__restrict__ graphs, const int32_t *__restrict__ order, LoopParams p,
            const int32_t *__restrict__ kc, BatchResult *__restrict__ res) {
    const int i = order[blockIdx.x];
    const DevGraph g = global_view(graphs[i]);
    const Team tm{0, 1};
    {
        int *w = reinterpret_cast<int *>(g.ctrl);
        const int words = (int)(sizeof(Ctrl) / sizeof(int));
        for (int j = threadIdx.x; j < words; j += BLOCK) w[j] = 0;
    }
    for (int v = threadIdx.x; v < g.n; v += BLOCK) {
        g.mark[v] = 0;
        g.rmark[v] = 0;
        g.e[v] = 0;
        g.h[v] = 0;
    }
    for (int v = threadIdx.x; v <= g.n; v += BLOCK) g.hcount[v] = 0;
    for (int a = threadIdx.x; a < g.A; a += BLOCK) g.arc[a].y = g.cap[a];
    __syncthreads();
    saturate_source<kGroup>(g, tm);
    __syncthreads();
    LoopParams q = p;
    q.kc = kc[i];
    if (q.relabel_budget <= 0) q.relabel_budget = max((int64_t)1024, (int64_t)g.n / 16);
    uint32_t epoch = 0;
    solve_loop<kGroup, false>(g, tm, q, epoch);
    __syncthreads();
    if (threadIdx.x == 0) {
        BatchResult r;
        r.value = g.ctrl->e_t + g.ctrl->deficit;
        r.status = g.ctrl->status;
        r.pad = 0;
        res[i] = r;
    }
}

// A team under three quarters of the size that was meant.
__device__ __forceinline__ bool team_is_short(int members, int want) { return 4 * members < 3 * want; }

// Join the team that is forming on this XCD (one thread calls it).  *open holds
// its number times 256 plus its members so far; whoever completes it opens the
// next one, so workgroups that get a compute unit late, behind other classes or
// tenants, still make teams.  A team's first member closes it short after `limit`
// ticks if it has half its members, and after ten times that with any number (a
// member or two would hold up the batch with a large instance).  sizes[team] is
// set once the team is closed.  *team is -1 beyond kBatchTeams.
// Batches beside a class of small instances, with one pool per XCD that closed
// after `limit` against this: 1000 grids of side 10 to 69, 62 against 23 ms; 600
// of side 10 to 39 and four of 250, 76 against 35; 256 instances of up to 524 k
// arcs 35 against 33.
__device__ __forceinline__ void join_batch_team(PaddedU32 *open, uint32_t *sizes, int want, int64_t limit, int *team,
                                                int *rank, int *size) {
    uint32_t seen = __hip_atomic_load(&open->v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), next;
    do {
        if ((seen >> 8) >= (uint32_t)kBatchTeams) {
            *team = -1;
            return;
        }
        next = (int)(seen & 255u) + 1 == want ? (seen & ~255u) + 256u : seen + 1u;
    } while (!__hip_atomic_compare_exchange_strong(&open->v, &seen, next, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT));
    const uint32_t id = seen >> 8;
    uint32_t n = 0;
    if ((next >> 8) != id) {
        n = (uint32_t)want;
        __hip_atomic_store(&sizes[id], n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        const uint64_t t0 = wall_clock64();
        while ((n = __hip_atomic_load(&sizes[id], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) {
            __builtin_amdgcn_s_sleep(1);
            const int64_t waited = (int64_t)(wall_clock64() - t0);
            if ((seen & 255u) != 0 || waited < limit) continue;
            uint32_t now = __hip_atomic_load(&open->v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t members = now & 255u;
            if ((now >> 8) != id ||  // complete: its last member is about to set the size
                (team_is_short((int)members, want) && waited < 10 * limit) ||
                !__hip_atomic_compare_exchange_strong(&open->v, &now, (id + 1u) << 8, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT))
                continue;
            __hip_atomic_store(&sizes[id], members, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    *team = (int)id;
    *rank = (int)(seen & 255u);
    *size = (int)n;
}

// The larger instances of a batch: a workgroup alone is bound by what one
// compute unit issues and gathers, and the batch ends with its largest
// instance.  So the workgroups of each XCD form teams of `team` (as they get
// compute units, see join_batch_team), and the teams take instances from the
// order, largest first.  A team never waits for another.
// Measured, 64 grids and random graphs of up to 524 k arcs: 72 ms with one
// workgroup each, 24 ms by teams (the largest alone: 21.4 ms).
__global__ void __launch_bounds__(kBlock)
    k_batch_teams(const DevGraph *__restrict__ graphs, const int32_t *__restrict__ order, int count, LoopParams p,
                  const int32_t *__restrict__ kc, BatchResult *__restrict__ res, BatchCtl *ctl, int team) {
    __shared__ int s_team, s_rank, s_size;
    const int xcc = xcd_id();
    if (threadIdx.x == 0)
        join_batch_team(&ctl->open[xcc], ctl->size[xcc], team, p.join_ticks, &s_team, &s_rank, &s_size);
    __syncthreads();
    if (s_team < 0) return;
    const Team tm{s_rank, s_size};
    BarWords *bar = &ctl->team[xcc * kBatchTeams + s_team];
    init_stages();
    uint32_t epoch = 0;
    bool ok = true;
    const bool back = team_is_short(tm.size, team);
    for (;;) {
        uint64_t mine = 0;
        if (threadIdx.x == 0 && tm.rank == 0) {
            const uint64_t taken = __hip_atomic_fetch_add(&ctl->next.v, back ? 1ull << 32 : 1ull, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT);
            const int front = (int)(uint32_t)taken, behind = (int)(taken >> 32);
            mine = 1u + (uint32_t)(front + behind >= count ? count : back ? count - 1 - behind : front);
        }
        block_sync<kXcd>();
        const int idx = (int)team_sum<kXcd>(bar, tm, epoch, mine, p.barrier_ticks, &ok) - 1;
        if (!ok || idx >= count) return;
        const int i = order[idx];
        const DevGraph g = global_view(graphs[i]);
        if (tm.rank == 0) {
            int *w = reinterpret_cast<int *>(g.ctrl);
            const int words = (int)(sizeof(Ctrl) / sizeof(int));
            for (int j = threadIdx.x; j < words; j += kBlock) w[j] = 0;
        }
        const int64_t stride = tm.nthreads();
        for (int64_t v = tm.tid(); v <= g.n; v += stride) {
            g.hcount[v] = 0;
            if (v == g.n) break;
            g.mark[v] = 0;
            g.rmark[v] = 0;
            g.e[v] = 0;
            g.h[v] = 0;
        }
        for (int64_t a = tm.tid(); a < g.A; a += stride) g.arc[a].y = g.cap[a];
        block_sync<kXcd>();
        (void)team_sum<kXcd>(bar, tm, epoch, 0, p.barrier_ticks, &ok);
        if (!ok) return;
        saturate_source<kXcd>(g, tm);
        block_sync<kXcd>();
        (void)team_sum<kXcd>(bar, tm, epoch, 0, p.barrier_ticks, &ok);
        if (!ok) return;
        LoopParams q = p;
        q.kc = kc[i];
        if (q.relabel_budget <= 0) q.relabel_budget = max((int64_t)1024, (int64_t)g.n / 16);
        uint32_t loop_epoch = 0;
        solve_loop<kXcd, false>(g, tm, q, loop_epoch);
        block_sync<kXcd>();
        (void)team_sum<kXcd>(bar, tm, epoch, 0, p.barrier_ticks, &ok);
        if (!ok) return;
        if (threadIdx.x == 0 && tm.rank == 0) {
            BatchResult r;
            r.value = ld<kXcd>(&g.ctrl->e_t) + ld<kXcd>(&g.ctrl->deficit);
            r.status = ld<kXcd>(&g.ctrl->status);
            r.pad = 0;
            res[i] = r;
        }
    }
}

__global__ void k_batch_reset(BatchCtl *ctl, int nctl, BatchResult *res, int count) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    int *w = reinterpret_cast<int *>(ctl);
    for (int j = t; j < nctl * (int)(sizeof(BatchCtl) / sizeof(int)); j += stride) w[j] = 0;
    for (int i = t; i < count; i += stride) res[i].status = kRunning;
}

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------

static int grid_for(int64_t work, int block, int cap) {
    int64_t b = (work + block - 1) / block;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (int)b;
}

hipError_t launch_begin(const DevGraph &g, const void *src, void *dst, int64_t words, hipStream_t st) {
    hipLaunchKernelGGL(k_begin, dim3(grid_for(words, 256, 512)), dim3(256), 0, st, g.ctrl,
                       static_cast<const int32_t *>(src), static_cast<int32_t *>(dst), words);
    return hipGetLastError();
}

hipError_t launch_init_state(const DevGraph &g, hipStream_t st) {
    const int64_t work = g.A > g.n ? g.A : g.n;
    hipLaunchKernelGGL(k_init_state, dim3(grid_for(work, 256)), dim3(256), 0, st, g);
    return hipGetLastError();
}

hipError_t launch_saturate_source(const DevGraph &g, hipStream_t st) {
    // the degree of s is only known on the host side of the handle; a fixed
    // grid with grid-stride loops covers any degree
    hipLaunchKernelGGL(k_saturate_source, dim3(256), dim3(256), 0, st, g);
    return hipGetLastError();
}

hipError_t launch_validate_updates(const DevGraph &g, const Repair &b, hipStream_t st) {
    if (b.k <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_validate_updates, dim3(grid_for(b.k, 256)), dim3(256), 0, st, g, b);
    return hipGetLastError();
}

hipError_t launch_apply_delta(const DevGraph &g, const Repair &b, hipStream_t st) {
    if (b.k <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_apply_delta, dim3(grid_for(b.k, 256)), dim3(256), 0, st, g, b);
    return hipGetLastError();
}

hipError_t launch_clamp(const DevGraph &g, const Repair &b, hipStream_t st) {
    if (b.k <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_clamp, dim3(grid_for(b.k, 256)), dim3(256), 0, st, g, b);
    return hipGetLastError();
}

hipError_t loop_max_coresident(int device, int *blocks) {
    int per_cu = 0, per_cu2 = 0, cus = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void *>(k_loop<kBlock, kAgent, true>), kBlock, 0);
    if (e != hipSuccess) return e;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu2, reinterpret_cast<const void *>(k_loop<kBlock, kAgent, false>), kBlock, 0);
    if (e != hipSuccess) return e;
    per_cu = min(per_cu, per_cu2);
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    *blocks = per_cu * cus;
    return hipSuccess;
}

hipError_t launch_local_stage(const DevGraph &g, const Repair &b, hipStream_t st) {
    if (b.k <= 0 || b.pulls == 0) return hipSuccess;
    hipLaunchKernelGGL(k_cut_saturate, dim3(grid_for(b.k, 256)), dim3(256), 0, st, g, b);
    // at most 2k deficits in any list, a wavefront each
    const dim3 blocks(grid_for(2 * b.k * 64, 256, 4096));
    for (int r = 0; r < b.pulls; ++r)
        hipLaunchKernelGGL(k_pull_round, blocks, dim3(256), 0, st, g, b, (r & 1) ? g.list[2] : g.list[1], r,
                           r == b.pulls - 1 ? nullptr : (r & 1) ? g.list[1] : g.list[2]);
    return hipGetLastError();
}

hipError_t launch_loop(const DevGraph &g, const LoopParams &p, const Repair &b, int grid, hipStream_t st) {
    if (grid <= 1) {
        if (p.walk) hipLaunchKernelGGL((k_loop<kBlock, kGroup, true>), dim3(1), dim3(kBlock), 0, st, g, p, b);
        else hipLaunchKernelGGL((k_loop<kBlock, kGroup, false>), dim3(1), dim3(kBlock), 0, st, g, p, b);
        return hipGetLastError();
    }
    LoopParams pa = p;
    pa.team_want = grid;
    if (p.xcd) {  // `grid` for every XCD, one of which is the team
        const dim3 blocks(grid * kXcds);
        if (p.walk) hipLaunchKernelGGL((k_loop<kBlock, kXcd, true>), blocks, dim3(kBlock), 0, st, g, pa, b);
        else hipLaunchKernelGGL((k_loop<kBlock, kXcd, false>), blocks, dim3(kBlock), 0, st, g, pa, b);
    } else {
        if (p.walk) hipLaunchKernelGGL((k_loop<kBlock, kAgent, true>), dim3(grid), dim3(kBlock), 0, st, g, pa, b);
        else hipLaunchKernelGGL((k_loop<kBlock, kAgent, false>), dim3(grid), dim3(kBlock), 0, st, g, pa, b);
    }
    return hipGetLastError();
}

hipError_t launch_batch(const DevGraph *graphs, const int32_t *order, int count, const LoopParams &p,
                        const int32_t *kc, BatchResult *res, int block, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    switch (block) {
    case 256:
        hipLaunchKernelGGL((k_batch<256>), dim3(count), dim3(256), 0, st, graphs, order, p, kc, res);
        break;
    case 512:
        hipLaunchKernelGGL((k_batch<512>), dim3(count), dim3(512), 0, st, graphs, order, p, kc, res);
        break;
    case 1024:
        hipLaunchKernelGGL((k_batch<1024>), dim3(count), dim3(1024), 0, st, graphs, order, p, kc, res);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_batch_teams(const DevGraph *graphs, const int32_t *order, int count, const LoopParams &p,
                              const int32_t *kc, BatchResult *res, BatchCtl *ctl, int team, int blocks,
                              hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_teams, dim3(blocks), dim3(kBlock), 0, st, graphs, order, count, p, kc, res, ctl, team);
    return hipGetLastError();
}

hipError_t launch_batch_reset(BatchCtl *ctl, int nctl, BatchResult *res, int count, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_reset, dim3(64), dim3(256), 0, st, ctl, nctl, res, count);
    return hipGetLastError();
}

hipError_t launch_teams(const DevGraph *d_views, const LoopParams *d_params, bool walk, const int64_t *work,
                        int grid, hipStream_t st) {
    if (grid < 2) return hipErrorInvalidValue;
    const DevGraph *v = d_views;
    const LoopParams *q = d_params;
    const int64_t *w = work;
    void *args[] = {&v, &q, &w};
    const void *fn = walk ? reinterpret_cast<const void *>(k_teams<kBlock, true>)
                          : reinterpret_cast<const void *>(k_teams<kBlock, false>);
    return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kBlock), args, 0, st);
}

hipError_t teams_max_coresident(int device, int *blocks) {
    int per_cu = 0, per_cu2 = 0, cus = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void *>(k_teams<kBlock, true>), kBlock, 0);
    if (e != hipSuccess) return e;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu2, reinterpret_cast<const void *>(k_teams<kBlock, false>), kBlock, 0);
    if (e != hipSuccess) return e;
    per_cu = min(per_cu, per_cu2);
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    *blocks = per_cu * cus;
    return hipSuccess;
}

hipError_t launch_part_from_heights(const DevGraph &g, uint8_t *part, int64_t *work, hipStream_t st) {
    hipLaunchKernelGGL(k_part_from_heights, dim3(grid_for(g.n, 256, 2048)), dim3(256), 0, st, g, part, work);
    return hipGetLastError();
}

hipError_t launch_part_localized(const DevGraph &g, const int32_t *hv, uint8_t *part, hipStream_t st) {
    hipLaunchKernelGGL(k_part_localized, dim3(grid_for(g.n, 256, 2048)), dim3(256), 0, st, g, hv, part);
    return hipGetLastError();
}

hipError_t launch_saturate_cut(const DevGraph &g, const uint8_t *part, hipStream_t st) {
    hipLaunchKernelGGL(k_saturate_cut, dim3(grid_for(g.A, 256)), dim3(256), 0, st, g, part);
    return hipGetLastError();
}

hipError_t launch_view_make(const DevGraph &g, int2 *varc, int64_t *ve, int rev, hipStream_t st) {
    const int64_t work = g.A > g.n ? g.A : g.n;
    hipLaunchKernelGGL(k_view_make, dim3(grid_for(work, 256)), dim3(256), 0, st, g, varc, ve, rev);
    return hipGetLastError();
}

hipError_t launch_view_merge(const DevGraph &g, const int2 *varc, const int64_t *ve, const uint8_t *part,
                             uint8_t want, int rev, hipStream_t st) {
    const int64_t work = g.A > g.n ? g.A : g.n;
    hipLaunchKernelGGL(k_view_merge, dim3(grid_for(work, 256)), dim3(256), 0, st, g, varc, ve, part, want, rev);
    return hipGetLastError();
}

hipError_t launch_edge_flow(const DevGraph &g, const int2 *carc, int32_t *rem, int32_t *flow, hipStream_t st) {
    if (g.A > 0) hipLaunchKernelGGL(k_arc_flow, dim3(grid_for(g.A, 256)), dim3(256), 0, st, g, carc, rem);
    if (g.m > 0) hipLaunchKernelGGL(k_edge_flow, dim3(grid_for(g.m, 256)), dim3(256), 0, st, g, rem, flow);
    return hipGetLastError();
}

hipError_t launch_min_cut(const DevGraph &g, const int32_t *new_of_old, uint8_t *side, bool long_lists, int64_t *cut,
                          hipStream_t st) {
    const int per = max(4, min(64, g.n / 512));  // up to 32 k vertices, about 512 wavefronts
    hipLaunchKernelGGL(k_cut_side, dim3(grid_for(((int64_t)g.n + per - 1) / per, 4, 2048)), dim3(256), 0, st, g,
                       new_of_old, side, long_lists ? nullptr : cut, per);
    if (long_lists)
        hipLaunchKernelGGL(k_cut_items, dim3(grid_for(g.A / kChunk, 4, 1024)), dim3(256), 0, st, g, cut);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int64_t count, int32_t value, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(count, 256)), dim3(256), 0, st, p, count, value);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batch staging of the allocation-free update call: one array per GPU, held
// until the process ends.  Host code never hands the array's name to a
// kernel (in host code it is only a stand-in for the symbol); its device
// address comes from hipGetSymbolAddress, once per device with that device
// current, and the kernels take that address like any other batch pointer.
// ---------------------------------------------------------------------------

static __device__ __align__(256) uint8_t scratch[kNoAllocIdsBytes + kNoAllocCapsBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_setup(int device) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    int cur = 0;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = ptr;
    return hipSuccess;
}

void *noalloc_scratch(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return g_scratch_ptr[device];
}

}  // namespace mf
