// Device build of the merged arc-pair layout (the bi-directional CSR of
// Sec. 5.1), run once per mf_create.  Every unordered vertex pair {u, v}
// (u != v) joined by at least one input edge gets one arc u->v in u's list
// and one arc v->u in v's list, twins of each other; parallel and antiparallel
// input edges share the pair (the residual of Sec. 2.3 is per vertex pair),
// cap[u->v] is the sum of the capacities of the input edges u->v, arcs of a
// vertex are sorted by neighbour id and self-loops get no arc.
//
// Steps (all on the device):
//  1. tail of every input edge (binary search in the input row pointers);
//  2. two half-edges per edge that is not a self-loop, one owned by each end,
//     keyed (owner, neighbour), compacted;
//  3. a stable least-significant-digit radix sort of the keys (8-bit digits:
//     per-tile digit counts, one exclusive scan over all tiles, a stable
//     scatter that ranks each item within its tile);
//  4. runs of equal keys are arcs: arc index by a scan of the run starts,
//     capacity sums, edge -> arc map, twins, multiplicity, row pointers.
#include "mf_internal.h"

namespace mf {
namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;  // 2048 values per workgroup
constexpr int kSortThreads = 256;
constexpr int kSortItems = 16;  // 4096 items per tile
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kDigitBits = 8;
constexpr int kDigits = 1 << kDigitBits;

__device__ __forceinline__ int lane_of() { return (int)__lane_id(); }

// Exclusive scan of one value per thread over the workgroup; returns this
// thread's prefix and sets *total.  Every thread calls it.
template <int T>
__device__ __forceinline__ int64_t block_excl_scan(int64_t x, int64_t *total) {
    __shared__ int64_t s_w[T / 64];
    const int lane = lane_of(), w = threadIdx.x >> 6;
    int64_t incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int64_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
    if (lane == 63) s_w[w] = incl;
    __syncthreads();
    int64_t off = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < T / 64; ++k) {
        const int64_t v = s_w[k];
        if (k < w) off += v;
        tot += v;
    }
    __syncthreads();
    *total = tot;
    return off + incl - x;
}

// --- exclusive scan of int64 data in place (recursive over block sums) ---

__global__ void __launch_bounds__(kScanThreads) k_scan_local(int64_t *data, int64_t n, int64_t *sums) {
    const int64_t base = ((int64_t)blockIdx.x * kScanThreads + threadIdx.x) * kScanItems;
    int64_t v[kScanItems];
    int64_t t = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        v[j] = base + j < n ? data[base + j] : 0;
        t += v[j];
    }
    int64_t tot = 0;
    int64_t run = block_excl_scan<kScanThreads>(t, &tot);
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        if (base + j < n) data[base + j] = run;
        run += v[j];
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_add(int64_t *data, int64_t n, const int64_t *offs) {
    const int64_t base = ((int64_t)blockIdx.x * kScanThreads + threadIdx.x) * kScanItems;
    const int64_t o = offs[blockIdx.x];
#pragma unroll
    for (int j = 0; j < kScanItems; ++j)
        if (base + j < n) data[base + j] += o;
}

constexpr int64_t kScanBlockSpan = (int64_t)kScanThreads * kScanItems;

int64_t scan_tmp_count(int64_t n) {
    int64_t t = 0;
    while (n > 1) {
        n = (n + kScanBlockSpan - 1) / kScanBlockSpan;
        t += n + 1;
    }
    return t + 1;
}

hipError_t scan_exclusive(int64_t *data, int64_t n, int64_t *tmp, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int64_t nb = (n + kScanBlockSpan - 1) / kScanBlockSpan;
    hipLaunchKernelGGL(k_scan_local, dim3((unsigned)nb), dim3(kScanThreads), 0, st, data, n, tmp);
    if (nb > 1) {
        hipError_t e = scan_exclusive(tmp, nb, tmp + nb + 1, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(kScanThreads), 0, st, data, n, tmp);
    }
    return hipGetLastError();
}

// --- stable LSD radix sort of (uint64 key, uint32 value) pairs ---

// Digit counts of every tile: hist[d * tiles + tile].
__global__ void __launch_bounds__(kSortThreads) k_rs_hist(const uint64_t *keys, int64_t n, int shift,
                                                          int64_t *hist, int64_t tiles) {
    __shared__ int s_cnt[kDigits];
    static_assert(kDigits == kSortThreads, "a thread per digit");
    s_cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
    uint64_t k[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const int64_t i = base + j * kSortThreads + threadIdx.x;
        k[j] = i < n ? keys[i] : 0;
    }
#pragma unroll
    for (int j = 0; j < kSortItems; ++j)
        if (base + j * kSortThreads + threadIdx.x < n) atomicAdd(&s_cnt[(int)((k[j] >> shift) & (kDigits - 1))], 1);
    __syncthreads();
    hist[(int64_t)threadIdx.x * tiles + blockIdx.x] = s_cnt[threadIdx.x];
}

// Stable scatter of one tile.  Wavefront w holds the items [1024 w, 1024 w +
// 1024) of the tile, 64 consecutive ones per step.  An item's rank among those
// of its digit: the lanes before it with the same digit (eight ballots find
// them), the wavefront's earlier steps (a count per wavefront and digit in
// LDS), then the earlier wavefronts and, for its place in the tile, the smaller
// digits.  The tile is laid out in that order in LDS and stored from there, so
// that a digit's items leave in runs of consecutive lanes.
// Bound by the memory it moves, 24 bytes an item there and back: of 8 M items a
// pass of 8 bits takes 60 us; one of 4 bits that ranked by thread and stored
// from registers took 190.
__global__ void __launch_bounds__(kSortThreads)
    k_rs_scatter(const uint64_t *keys, const uint32_t *vals, int64_t n, int shift, const int64_t *offs,
                 int64_t tiles, uint64_t *keys_out, uint32_t *vals_out) {
    constexpr int kWaves = kSortThreads / 64;
    __shared__ int s_cnt[kWaves][kDigits];
    __shared__ int64_t s_to[kDigits];  // global position of a digit's first item, less its place in the tile
    __shared__ uint64_t s_key[kSortTile];
    __shared__ uint32_t s_val[kSortTile];
    const int t = threadIdx.x, lane = lane_of(), w = t >> 6;
    const int64_t tile0 = (int64_t)blockIdx.x * kSortTile;
    const int here = (int)min((int64_t)kSortTile, n - tile0);
    const int at0 = w * (kSortTile / kWaves) + lane;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) s_cnt[k][t] = 0;
    uint64_t k[kSortItems];
    uint32_t v[kSortItems];
    int rank[kSortItems];
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const bool ok = at0 + 64 * j < here;
        k[j] = ok ? keys[tile0 + at0 + 64 * j] : 0;
        v[j] = ok ? vals[tile0 + at0 + 64 * j] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const bool ok = at0 + 64 * j < here;
        const int d = (int)((k[j] >> shift) & (kDigits - 1));
        uint64_t same = __ballot(ok);
#pragma unroll
        for (int bit = 0; bit < kDigitBits; ++bit) {
            const uint64_t ones = __ballot((d >> bit) & 1);
            same &= ((d >> bit) & 1) ? ones : ~ones;
        }
        const int before = __popcll(same & ((1ull << lane) - 1));
        const int base = ok ? s_cnt[w][d] : 0;
        rank[j] = base + before;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (ok && before == 0) s_cnt[w][d] = base + __popcll(same);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    // thread t: digit t's items in the tile, and per wavefront where they begin
    int64_t tot = 0;
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) sum += s_cnt[k][t];
    int run = (int)block_excl_scan<kSortThreads>((int64_t)sum, &tot);
    s_to[t] = offs[(int64_t)t * tiles + blockIdx.x] - run;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        const int c = s_cnt[k][t];
        s_cnt[k][t] = run;
        run += c;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        if (at0 + 64 * j >= here) continue;
        const int p = s_cnt[w][(int)((k[j] >> shift) & (kDigits - 1))] + rank[j];
        s_key[p] = k[j];
        s_val[p] = v[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
        const int i = j * kSortThreads + t;
        if (i >= here) continue;
        const uint64_t key = s_key[i];
        const int64_t p = s_to[(int)((key >> shift) & (kDigits - 1))] + i;
        if (p < 0 || p >= n) continue;  // only on a broken scan: never write out of bounds
        keys_out[p] = key;
        vals_out[p] = s_val[i];
    }
}

// --- the layout ---

// Tail of every input edge: the row v with row_ptr[v] <= i < row_ptr[v+1].
__global__ void k_tails(const int64_t *rp, int32_t n, int64_t m, int32_t *tail) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        int32_t lo = 0, hi = n - 1;  // largest v with rp[v] <= i
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo + 1) / 2;
            if (rp[mid] <= i) lo = mid;
            else hi = mid - 1;
        }
        tail[i] = lo;
    }
}

// 1 for an edge that is not a self-loop.
__global__ void k_nonloop(const int32_t *tail, const int32_t *col, int64_t m, int64_t *flag) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x)
        flag[i] = tail[i] != col[i] ? 1 : 0;
}

// The two half-edges of every edge that is not a self-loop, at 2 * pos[i]:
// key (owner << b) | neighbour, value (edge << 1) | reverse.  With perm, the
// ends are the vertices' numbers in the handle's order (perm[caller's id]).
__global__ void k_half_edges(const int32_t *tail, const int32_t *col, int64_t m, const int64_t *pos, int b,
                             const int32_t *perm, uint64_t *keys, uint32_t *vals) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        int32_t u = tail[i], v = col[i];
        if (u == v) continue;
        if (perm) {
            u = perm[u];
            v = perm[v];
        }
        const int64_t p = 2 * pos[i];
        keys[p] = ((uint64_t)u << b) | (uint64_t)v;
        vals[p] = (uint32_t)((uint64_t)i << 1);
        keys[p + 1] = ((uint64_t)v << b) | (uint64_t)u;
        vals[p + 1] = (uint32_t)(((uint64_t)i << 1) | 1u);
    }
}

// 1 where a run of equal keys (one arc) starts.
__global__ void k_run_starts(const uint64_t *keys, int64_t nh, int64_t *flag) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nh; k += (int64_t)gridDim.x * blockDim.x)
        flag[k] = (k == 0 || keys[k] != keys[k - 1]) ? 1 : 0;
}

// Per half-edge k (sorted): its arc a = idx[k] + start(k) - 1 (idx: the
// exclusive scan of the run starts).  A run start records the arc's neighbour, owner and first
// position; a forward half-edge adds its capacity and fixes edge2arc, a
// reverse one the arc of the reverse direction.
__global__ void k_arcs(const uint64_t *keys, const uint32_t *vals, const int64_t *idx, int64_t nh, int64_t A, int b,
                       const int32_t *cap, int32_t *col_out, int32_t *owner, int64_t *start, int64_t *capsum,
                       int32_t *edge2arc, int32_t *rev_arc) {
    const uint64_t mask = (1ull << b) - 1;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nh; k += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t key = keys[k];
        const bool first = k == 0 || keys[k - 1] != key;
        const int64_t a = idx[k] + (first ? 0 : -1);
        if (a < 0 || a >= A) continue;  // only on a broken scan
        if (first) {
            col_out[a] = (int32_t)(key & mask);
            owner[a] = (int32_t)(key >> b);
            start[a] = k;
        }
        const uint32_t code = vals[k];
        const int64_t i = (int64_t)(code >> 1);
        if (code & 1u) {
            rev_arc[i] = (int32_t)a;
        } else {
            edge2arc[i] = (int32_t)a;
            atomicAdd((unsigned long long *)&capsum[a], (unsigned long long)cap[i]);
        }
    }
}

// Arc records, capacities, the largest multiplicity (half-edges per arc) and
// a flag for a capacity sum above int32.  (One maximum into the common word per
// thread was what it spent its time on: 750 us for 8 M arcs, 75 us with one per
// workgroup.)
__global__ void __launch_bounds__(256) k_arc_records(const int32_t *col, const int64_t *capsum, const int64_t *start, int64_t A, int64_t nh,
                              int2 *arc, int32_t *cap, int32_t *maxmult, int32_t *overflow) {
    int32_t mm = 0;
    for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < A; a += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = capsum[a];
        if (c > INT32_MAX) atomicOr(overflow, 1);
        const int32_t cc = (int32_t)min(c, (int64_t)INT32_MAX);
        cap[a] = cc;
        arc[a] = make_int2(col[a], cc);
        const int64_t len = (a + 1 < A ? start[a + 1] : nh) - start[a];
        mm = max(mm, (int32_t)min(len, (int64_t)INT32_MAX));
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) mm = max(mm, __shfl_xor(mm, d, 64));
    __shared__ int s_mm[256 / 64];
    if (lane_of() == 0) s_mm[threadIdx.x >> 6] = mm;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < 256 / 64; ++k) mm = max(mm, s_mm[k]);
    if (mm > *maxmult) atomicMax(maxmult, mm);
}

// row_ptr[v] = first arc owned by a vertex >= v (arcs are sorted by owner).
__global__ void k_row_ptr(const int32_t *owner, int64_t A, int32_t n, int32_t *row_ptr) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v <= n; v += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = A;
        while (lo < hi) {
            const int64_t mid = (lo + hi) / 2;
            if (owner[mid] < v) lo = mid + 1;
            else hi = mid;
        }
        row_ptr[v] = (int32_t)lo;
    }
}

__global__ void k_twins(const int32_t *edge2arc, const int32_t *rev_arc, int64_t m, int64_t A, int32_t *twin) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t a = edge2arc[i];
        const int32_t r = rev_arc[i];
        if (a < 0 || r < 0 || a >= A || r >= A) continue;
        twin[a] = r;
        twin[r] = a;
    }
}

// Edges at every vertex (either end; self-loops left out).  Bound by the
// additions to a hub's count, which follow one another: a workgroup adds up the
// vertices that come first to their slot of a table in LDS, hubs among them,
// and only the others go to memory at once.  (R-MAT 2^18, 4 M
// edges: 1055 us with two additions to memory per edge, 254 us so.)
constexpr int kDegThreads = 1024;
constexpr int kDegSlotBits = 12;
__global__ void __launch_bounds__(kDegThreads) k_degree(const int32_t *tail, const int32_t *col, int64_t m, int32_t *deg) {
    __shared__ int s_tag[1 << kDegSlotBits], s_sum[1 << kDegSlotBits];
    for (int i = threadIdx.x; i < (1 << kDegSlotBits); i += kDegThreads) {
        s_tag[i] = -1;
        s_sum[i] = 0;
    }
    __syncthreads();
    auto count = [&](int32_t v) {
        const int slot = (int)(((uint32_t)v * 2654435769u) >> (32 - kDegSlotBits));
        int tag = s_tag[slot];
        if (tag == -1) tag = atomicCAS(&s_tag[slot], -1, v);
        if (tag == -1 || tag == v) atomicAdd(&s_sum[slot], 1);
        else atomicAdd(&deg[v], 1);
    };
    for (int64_t i = (int64_t)blockIdx.x * kDegThreads + threadIdx.x; i < m; i += (int64_t)gridDim.x * kDegThreads) {
        const int32_t u = tail[i], v = col[i];
        if (u == v) continue;
        count(u);
        count(v);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < (1 << kDegSlotBits); i += kDegThreads)
        if (s_sum[i]) atomicAdd(&deg[s_tag[i]], s_sum[i]);
}

// Sort keys of the vertices for falling degree, ties by id:
// ((kDegMax - min(deg, kDegMax)) << b) | v.
constexpr int kDegBits = 24;
constexpr int32_t kDegMax = (1 << kDegBits) - 1;
__global__ void k_vertex_keys(const int32_t *deg, int32_t n, int b, uint64_t *keys, uint32_t *vals) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int32_t d = deg[v] < kDegMax ? deg[v] : kDegMax;
        keys[v] = ((uint64_t)(kDegMax - d) << b) | (uint64_t)v;
        vals[v] = (uint32_t)v;
    }
}

// perm[v] = position of v in the sorted order.
__global__ void k_rank_of(const uint32_t *sorted_vals, int64_t n, int32_t *perm) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        perm[sorted_vals[i]] = (int32_t)i;
}

// Key of every arc in the caller's numbering: (owner << b) | head, through
// old_of_new (the tail of arc a is the head of its twin).
__global__ void k_caller_arc_keys(const int2 *arc, const int32_t *twin, int64_t A, const int32_t *old_of_new, int b,
                                  uint64_t *keys, uint32_t *vals) {
    for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < A; a += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t u = (uint64_t)old_of_new[arc[twin[a]].x], v = (uint64_t)old_of_new[arc[a].x];
        keys[a] = (u << b) | v;
        vals[a] = (uint32_t)a;
    }
}

__global__ void k_fill32(int32_t *p, int64_t count, int32_t value) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

int grid_of(int64_t work) {
    int64_t b = (work + 255) / 256;
    return (int)(b < 1 ? 1 : (b > 16384 ? 16384 : b));
}

// Stable LSD sort of n (key, value) pairs on their low `bits` key bits, 8 bits
// a pass, between the buffer pairs (k0, v0) and (k1, v1); the sorted pairs end
// in (*k0, *v0) (the pointers are swapped as the passes go).  hist and scan:
// kDigits * tiles and scan_tmp_count(kDigits * tiles) entries.
hipError_t radix_sort(uint64_t **k0, uint32_t **v0, uint64_t **k1, uint32_t **v1, int64_t n, int bits,
                      int64_t *hist, int64_t *scan, hipStream_t st) {
    const int64_t tiles = (n + kSortTile - 1) / kSortTile;
    if (n <= 1) return hipSuccess;
    hipError_t e = hipSuccess;
    for (int shift = 0; shift < bits; shift += kDigitBits) {
        hipLaunchKernelGGL(k_rs_hist, dim3((unsigned)tiles), dim3(kSortThreads), 0, st, *k0, n, shift, hist, tiles);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = scan_exclusive(hist, kDigits * tiles, scan, st)) != hipSuccess) return e;
        hipLaunchKernelGGL(k_rs_scatter, dim3((unsigned)tiles), dim3(kSortThreads), 0, st, *k0, *v0, n, shift, hist,
                           tiles, *k1, *v1);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        std::swap(*k0, *k1);
        std::swap(*v0, *v1);
    }
    return hipSuccess;
}

int id_bits(int64_t n) {
    int b = 1;
    while ((1ll << b) < n) ++b;
    return b;
}

}  // namespace

hipError_t build_layout_device(int32_t n, int64_t m, const int64_t *h_row_ptr, const int32_t *h_col,
                               const int32_t *h_cap, bool renumber, const BuildAlloc &mem, hipStream_t st,
                               DeviceLayout *out, std::vector<int32_t> *h_row_ptr_out,
                               std::vector<int32_t> *h_new_of_old, std::string *err) {
    std::vector<void *> tmp;
    auto cleanup = [&]() {
        (void)hipStreamSynchronize(st);
        for (void *p : tmp) mem.release(p);
        tmp.clear();
    };
#define BTRY(expr)                                                    \
    do {                                                              \
        hipError_t e_ = (expr);                                       \
        if (e_ != hipSuccess) {                                       \
            *err = std::string(#expr) + ": " + hipGetErrorString(e_); \
            cleanup();                                                \
            return e_;                                                \
        }                                                             \
    } while (0)
    int64_t *d_rp = nullptr, *d_flag = nullptr, *d_scan = nullptr, *d_hist = nullptr;
    int32_t *d_tail = nullptr, *d_col = nullptr, *d_ecap = nullptr, *d_info = nullptr;
    int32_t *d_perm = nullptr;
    const int64_t mm = m > 0 ? m : 1;
    BTRY(mem.alloc({want(&d_rp, (int64_t)n + 1), want(&d_col, m), want(&d_tail, m), want(&d_info, 4),
                    want(&d_flag, mm + 1), want(&d_scan, scan_tmp_count(2 * mm + 1))},
                   &tmp));
    // the edge capacities stay with the handle (ecap), and so does the numbering
    if (renumber && n > 0) BTRY(mem.keep({want(&d_ecap, m), want(&d_perm, n)}));
    else BTRY(mem.keep({want(&d_ecap, m)}));
    BTRY(hipMemcpyAsync(d_rp, h_row_ptr, sizeof(int64_t) * (n + 1), hipMemcpyHostToDevice, st));
    if (m > 0) {
        BTRY(hipMemcpyAsync(d_col, h_col, sizeof(int32_t) * m, hipMemcpyHostToDevice, st));
        BTRY(hipMemcpyAsync(d_ecap, h_cap, sizeof(int32_t) * m, hipMemcpyHostToDevice, st));
    }
    // 1-2: tails, non-loop positions, half-edges
    int64_t nonloop = 0;
    if (m > 0) {
        hipLaunchKernelGGL(k_tails, dim3(grid_of(m)), dim3(256), 0, st, d_rp, n, m, d_tail);
        hipLaunchKernelGGL(k_nonloop, dim3(grid_of(m)), dim3(256), 0, st, d_tail, d_col, m, d_flag);
        BTRY(hipGetLastError());
        int64_t last_flag = 0;
        BTRY(hipMemcpyAsync(&last_flag, d_flag + m - 1, sizeof(int64_t), hipMemcpyDeviceToHost, st));
        BTRY(hipStreamSynchronize(st));
        BTRY(scan_exclusive(d_flag, m, d_scan, st));
        int64_t last_pos = 0;
        BTRY(hipMemcpyAsync(&last_pos, d_flag + m - 1, sizeof(int64_t), hipMemcpyDeviceToHost, st));
        BTRY(hipStreamSynchronize(st));
        nonloop = last_pos + last_flag;
    }
    const int64_t nh = 2 * nonloop;
    if (nh / 2 > INT32_MAX / 2) {
        *err = "too many arcs for int32 arc indices";
        cleanup();
        return hipErrorInvalidValue;
    }
    const int b = id_bits(n);  // bits of a vertex id
    uint64_t *d_k0 = nullptr, *d_k1 = nullptr;
    uint32_t *d_v0 = nullptr, *d_v1 = nullptr;
    const int64_t nhh = std::max<int64_t>(nh > 0 ? nh : 1, renumber ? n : 1);
    const int64_t tiles = (nhh + kSortTile - 1) / kSortTile;
    int64_t *d_scan2 = nullptr, *d_idx = nullptr;
    BTRY(mem.alloc({want(&d_k0, nhh), want(&d_k1, nhh), want(&d_v0, nhh), want(&d_v1, nhh),
                    want(&d_hist, kDigits * tiles), want(&d_scan2, scan_tmp_count(kDigits * tiles)),
                    want(&d_idx, nhh + 1)},
                   &tmp));
    // 2b: the handle's vertex order: falling degree (ties by id), so that the
    // hubs' heights, excesses and row bounds share a few cache lines and
    // every arc list starts with its hub neighbours
    if (renumber && n > 0) {
        out->new_of_old = d_perm;
        BTRY(hipMemsetAsync(d_perm, 0, sizeof(int32_t) * n, st));
        if (m > 0)
            hipLaunchKernelGGL(k_degree, dim3(std::min(512, grid_of(m))), dim3(kDegThreads), 0, st, d_tail, d_col, m,
                               d_perm);
        hipLaunchKernelGGL(k_vertex_keys, dim3(grid_of(n)), dim3(256), 0, st, d_perm, n, b, d_k0, d_v0);
        BTRY(hipGetLastError());
        BTRY(radix_sort(&d_k0, &d_v0, &d_k1, &d_v1, n, b + kDegBits, d_hist, d_scan2, st));
        hipLaunchKernelGGL(k_rank_of, dim3(grid_of(n)), dim3(256), 0, st, d_v0, (int64_t)n, d_perm);
        BTRY(hipGetLastError());
        h_new_of_old->assign((size_t)n, 0);
        BTRY(hipMemcpyAsync(h_new_of_old->data(), d_perm, sizeof(int32_t) * n, hipMemcpyDeviceToHost, st));
    } else {
        h_new_of_old->clear();
    }
    if (m > 0) {
        hipLaunchKernelGGL(k_half_edges, dim3(grid_of(m)), dim3(256), 0, st, d_tail, d_col, m, d_flag, b, d_perm,
                           d_k0, d_v0);
        BTRY(hipGetLastError());
    }
    // 3: sort by (owner, neighbour)
    BTRY(radix_sort(&d_k0, &d_v0, &d_k1, &d_v1, nh, 2 * b, d_hist, d_scan2, st));
    // 4: arcs
    int64_t A = 0;
    if (nh > 0) {
        hipLaunchKernelGGL(k_run_starts, dim3(grid_of(nh)), dim3(256), 0, st, d_k0, nh, d_idx);
        BTRY(hipGetLastError());
        int64_t last_flag = 0, last_idx = 0;
        BTRY(hipMemcpyAsync(&last_flag, d_idx + nh - 1, sizeof(int64_t), hipMemcpyDeviceToHost, st));
        BTRY(hipStreamSynchronize(st));
        BTRY(scan_exclusive(d_idx, nh, d_scan, st));
        BTRY(hipMemcpyAsync(&last_idx, d_idx + nh - 1, sizeof(int64_t), hipMemcpyDeviceToHost, st));
        BTRY(hipStreamSynchronize(st));
        A = last_idx + last_flag;
    }
    if (A > INT32_MAX) {
        *err = "too many arcs for int32 arc indices";
        cleanup();
        return hipErrorInvalidValue;
    }
    const int64_t AA = A > 0 ? A : 1;
    int32_t *d_colA = nullptr, *d_owner = nullptr, *d_rev = nullptr;
    int64_t *d_start = nullptr, *d_capsum = nullptr;
    BTRY(mem.alloc({want(&d_colA, AA), want(&d_owner, AA), want(&d_start, AA), want(&d_capsum, AA), want(&d_rev, mm)},
                   &tmp));
    // the handle's arrays
    BTRY(mem.keep({want(&out->row_ptr, (int64_t)n + 1), want(&out->arc, AA), want(&out->twin, AA),
                   want(&out->cap, AA), want(&out->edge2arc, mm)}));
    out->ecap = d_ecap;
    BTRY(hipMemsetAsync(d_capsum, 0, sizeof(int64_t) * AA, st));
    BTRY(hipMemsetAsync(d_info, 0, sizeof(int32_t) * 4, st));
    hipLaunchKernelGGL(k_fill32, dim3(grid_of(mm)), dim3(256), 0, st, out->edge2arc, mm, -1);
    hipLaunchKernelGGL(k_fill32, dim3(grid_of(mm)), dim3(256), 0, st, d_rev, mm, -1);
    if (nh > 0)
        hipLaunchKernelGGL(k_arcs, dim3(grid_of(nh)), dim3(256), 0, st, d_k0, d_v0, d_idx, nh, A, b, d_ecap, d_colA,
                           d_owner, d_start, d_capsum, out->edge2arc, d_rev);
    if (A > 0)
        hipLaunchKernelGGL(k_arc_records, dim3(grid_of(A)), dim3(256), 0, st, d_colA, d_capsum, d_start, A, nh,
                           out->arc, out->cap, d_info, d_info + 1);
    hipLaunchKernelGGL(k_row_ptr, dim3(grid_of((int64_t)n + 1)), dim3(256), 0, st, d_owner, A, n, out->row_ptr);
    if (m > 0) hipLaunchKernelGGL(k_twins, dim3(grid_of(m)), dim3(256), 0, st, out->edge2arc, d_rev, m, A, out->twin);
    BTRY(hipGetLastError());
    int32_t info[4] = {0, 0, 0, 0};
    BTRY(hipMemcpyAsync(info, d_info, sizeof(info), hipMemcpyDeviceToHost, st));
    h_row_ptr_out->assign((size_t)n + 1, 0);
    BTRY(hipMemcpyAsync(h_row_ptr_out->data(), out->row_ptr, sizeof(int32_t) * (n + 1), hipMemcpyDeviceToHost, st));
    BTRY(hipStreamSynchronize(st));
    cleanup();
#undef BTRY
    if (info[1]) {
        *err = "summed capacity of one arc exceeds int32";
        return hipErrorInvalidValue;
    }
    out->A = (int32_t)A;
    out->max_pair_mult = info[0] > 0 ? info[0] : 1;
    return hipSuccess;
}

hipError_t caller_arc_order(int32_t n, int64_t A, const int2 *arc, const int32_t *twin,
                            const std::vector<int32_t> &old_of_new, const BuildAlloc &mem, hipStream_t st,
                            std::vector<int32_t> *h_caller_of_arc) {
    std::vector<void *> tmp;
    hipError_t e = hipSuccess;
    auto done = [&](hipError_t r) {
        (void)hipStreamSynchronize(st);
        for (void *p : tmp) mem.release(p);
        return r;
    };
    const int64_t AA = A > 0 ? A : 1;
    const int64_t tiles = (AA + kSortTile - 1) / kSortTile;
    uint64_t *k0 = nullptr, *k1 = nullptr;
    uint32_t *v0 = nullptr, *v1 = nullptr;
    int32_t *d_old = nullptr, *d_rank = nullptr;
    int64_t *hist = nullptr, *scan = nullptr;
    e = mem.alloc({want(&k0, AA), want(&k1, AA), want(&v0, AA), want(&v1, AA), want(&d_old, n), want(&d_rank, AA),
                   want(&hist, kDigits * tiles), want(&scan, scan_tmp_count(kDigits * tiles))},
                  &tmp);
    if (e != hipSuccess) return done(e);
    if (n > 0 && (e = hipMemcpyAsync(d_old, old_of_new.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, st)) !=
                     hipSuccess)
        return done(e);
    const int b = id_bits(n);
    if (A > 0) {
        hipLaunchKernelGGL(k_caller_arc_keys, dim3(grid_of(A)), dim3(256), 0, st, arc, twin, A, d_old, b, k0, v0);
        if ((e = hipGetLastError()) != hipSuccess) return done(e);
        if ((e = radix_sort(&k0, &v0, &k1, &v1, A, 2 * b, hist, scan, st)) != hipSuccess) return done(e);
        hipLaunchKernelGGL(k_rank_of, dim3(grid_of(A)), dim3(256), 0, st, v0, A, d_rank);
        if ((e = hipGetLastError()) != hipSuccess) return done(e);
    }
    h_caller_of_arc->assign((size_t)A, 0);
    if (A > 0 && (e = hipMemcpyAsync(h_caller_of_arc->data(), d_rank, sizeof(int32_t) * A, hipMemcpyDeviceToHost,
                                     st)) != hipSuccess)
        return done(e);
    return done(hipSuccess);
}

}  // namespace mf
