// Small levels (gfx950): degree classes, renumbering and aggregation of a
// level in a dozen launches and two host waits.
//
// A level of a few thousand entries takes its sorts, scans, per-class
// summations and read-backs at 2-10 us apiece, whatever it holds: some 80
// launches and eight host round trips a level, 0.5 ms, where the sweeps take
// 0.3 ms.  Here the class lists are placed by counters instead of a sort, scans
// are single launches (decoupled look-back), the coarse graph is summed in one
// hash table instead of member lists, segments and per-class tables, sizes
// that the next kernel needs stay on the device, and what the host needs is
// posted to pinned memory by the kernel that finds it.
//
// The order of a class's rows and of a coarse row's columns depends on timing;
// nothing computed from them does (sums of integers, and a best candidate with
// ties broken by id).
#include <algorithm>

#include "lv_device.h"

namespace lv {

using namespace dev;

namespace {

constexpr int SBS = 1024;

// ------------------------------------------------------------------ single-pass scan
// Exclusive prefix of this tile's sum `agg` over the tiles before it, by
// decoupled look-back; called by one whole wavefront of every tile's
// workgroup.  st[t]: 0 = nothing yet, else (1 = the tile's own sum, 2 = its
// inclusive prefix) in the high word and the value in the low one, written
// and read as one 64-bit word.  A tile waits only for tiles with smaller
// numbers, and numbers are handed out by a counter as workgroups start, so
// the smallest unfinished tile never waits and every wait ends.
__device__ __forceinline__ uint32_t lookback(unsigned long long* st, uint32_t tile, uint32_t agg)
{
    const int lane = (int)lane_id();
    if (lane == 0)
        __hip_atomic_store(&st[tile], ((unsigned long long)(tile == 0 ? 2u : 1u) << 32) | agg, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    uint32_t before = 0;
    for (int64_t top = (int64_t)tile - 1; top >= 0;) {
        const int64_t t = top - lane;
        unsigned long long v = 2ull << 32;  // before the first tile: prefix 0
        if (t >= 0) v = __hip_atomic_load(&st[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t f = (uint32_t)(v >> 32);
        const uint64_t none = __ballot(f == 0), pre = __ballot(f == 2);
        const int upto = pre ? __ffsll((unsigned long long)pre) - 1 : WAVE - 1;  // nearest tile with a prefix
        if (none & (upto == 63 ? ~0ull : ((1ull << (upto + 1)) - 1ull))) {
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        uint32_t x = lane <= upto ? (uint32_t)v : 0u;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d);
        before += x;
        if (pre) break;
        top -= WAVE;
    }
    if (lane == 0 && tile > 0)
        __hip_atomic_store(&st[tile], (2ull << 32) | (before + agg), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return before;
}

// Exclusive scan of val(i), i < n, over tiles of SCAN_TILE consecutive
// elements, each thread SCAN_PER of them; out(i, prefix, value) for each, and
// the total to *total by the last tile.  Every thread of the workgroup calls
// it; tiles numbered by *ticket.
template <typename V, typename F>
__device__ __forceinline__ void scan_tiles(int64_t n, uint32_t* ticket, unsigned long long* st, int32_t* total, V&& val,
                                           F&& out)
{
    constexpr int PER = SMALL_SCAN_TILE / SBS;
    __shared__ uint32_t s_tile, s_before;
    __shared__ uint32_t s_wave[SBS / WAVE];
    if (threadIdx.x == 0) s_tile = atomicAdd(ticket, 1u);
    __syncthreads();
    const uint32_t tile = s_tile;
    const int64_t t0 = (int64_t)tile * SMALL_SCAN_TILE;
    if (t0 >= n && tile > 0) return;
    const int64_t i0 = t0 + (int64_t)threadIdx.x * PER;
    uint32_t v[PER], sum = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        v[u] = i0 + u < n ? (uint32_t)val(i0 + u) : 0u;
        sum += v[u];
    }
    uint32_t x = sum;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        const uint32_t y = __shfl_up(x, d);
        if ((int)lane_id() >= d) x += y;
    }
    const int wid = (int)(threadIdx.x / WAVE);
    if (lane_id() == WAVE - 1) s_wave[wid] = x;
    __syncthreads();
    uint32_t wbase = 0, all = 0;
    for (int w = 0; w < SBS / WAVE; ++w) {
        if (w < wid) wbase += s_wave[w];
        all += s_wave[w];
    }
    if (wid == 0) {
        const uint32_t b = lookback(st, tile, all);
        if (lane_id() == 0) s_before = b;
    }
    __syncthreads();
    uint32_t at = s_before + wbase + x - sum;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (i0 + u < n) out(i0 + u, (int32_t)at, (int32_t)v[u]);
        at += v[u];
    }
    if (threadIdx.x == 0 && t0 + SMALL_SCAN_TILE >= n) *total = (int32_t)(s_before + all);
}

// ------------------------------------------------------------------ level start
__device__ __forceinline__ int row_class(const SmallLevel& a, int32_t L)
{
    if (L <= 0) return CLS_NONE;
    for (int q = CLS_L4; q < CLS_HUB; ++q)
        if (L <= a.bounds[q]) return q;
    return CLS_HUB;
}

// This workgroup's share of the n positions (the same in both passes below).
__device__ __forceinline__ void small_share(int32_t n, int64_t& lo, int64_t& hi)
{
    lo = (int64_t)n * blockIdx.x / gridDim.x;
    hi = (int64_t)n * (blockIdx.x + 1) / gridDim.x;
}

// Singleton communities (label, volume, smallest member: isolated vertices
// have theirs now), the level's sweep control, and the number of rows per
// degree class; the last workgroup turns these into the class bounds, on the
// device and in the mail.
__global__ __launch_bounds__(SBS) void k_level_init(SmallLevel a, SweepEnd p, const int32_t* gactive)
{
    __shared__ int32_t h[NUM_CLS];
    __shared__ int32_t s_last;
    static_assert(NUM_CLS <= WAVE, "the first wavefront adds the class counts");
    if (threadIdx.x < NUM_CLS) h[threadIdx.x] = 0;
    __syncthreads();
    int64_t lo, hi;
    small_share(a.n, lo, hi);
    for (int64_t i = lo + threadIdx.x; i < hi; i += SBS) {
        const int c = row_class(a, a.off[i + 1] - a.off[i]);
        const int32_t id = a.orig ? a.orig[i] : (int32_t)i;
        a.comm[i] = id;
        a.sigma[id] = a.k[i];
        a.minv[id] = c == CLS_NONE ? id : INT32_MAX;
        if (c != CLS_NONE) atomicAdd(&h[c], 1);
    }
    const int64_t t0 = (int64_t)blockIdx.x * SBS + threadIdx.x, stride = (int64_t)gridDim.x * SBS;
    for (int64_t t = t0; t < (int64_t)p.G * p.max_sweeps; t += stride) p.gmoves[t] = 0;
    for (int64_t g = t0; g < p.G; g += stride) {
        p.gdone[g] = gactive && !gactive[g] ? 1 : 0;
        p.gsweeps[g] = 0;
        a.st_sums[g] = 0;
        a.st_sums[p.G + g] = 0;
    }
    if (t0 < CTR_WAYS) {
        p.ctr->way[t0].chg = 0;
        p.ctr->way[t0].moves = 0;
        p.ctr->way[t0].ticket = 0;
    }
    if (t0 == 0) {
        p.ctr->ways_done = 0;
        *p.ctl = SweepCtl{};
    }
    __syncthreads();
    if (threadIdx.x < WAVE) {
        if (threadIdx.x < NUM_CLS && h[threadIdx.x]) atomicAdd(&a.st->cls_cnt[threadIdx.x], h[threadIdx.x]);
        __builtin_amdgcn_s_waitcnt(0);  // the counts before the ticket
        if (threadIdx.x == 0) s_last = atomicAdd(&a.st->init_ticket, 1u) + 1u == gridDim.x;
    }
    __syncthreads();
    if (!s_last || threadIdx.x != 0) return;
    int32_t cnt[NUM_CLS], active = 0;
    for (int c = CLS_L4; c < NUM_CLS; ++c) active += cnt[c] = atomicAdd(&a.st->cls_cnt[c], 0);
    int32_t at = a.n - active;
    a.st->active0 = at;
    a.mail->start[CLS_NONE] = 0;
    for (int c = CLS_L4; c < NUM_CLS; ++c) {
        a.st->cls_cur[c] = at;
        a.mail->start[c] = at;
        at += cnt[c];
    }
    a.mail->start[NUM_CLS] = a.n;
    __threadfence_system();
    __hip_atomic_store(&a.mail->ready, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The rows with entries, listed by class, with their descriptors; and their
// vertices' pairs.
__global__ __launch_bounds__(SBS) void k_level_rows(SmallLevel a)
{
    __shared__ int32_t h[NUM_CLS], base[NUM_CLS];
    if (threadIdx.x < NUM_CLS) h[threadIdx.x] = 0;
    __syncthreads();
    int64_t lo, hi;
    small_share(a.n, lo, hi);
    for (int64_t i = lo + threadIdx.x; i < hi; i += SBS) {
        const int c = row_class(a, a.off[i + 1] - a.off[i]);
        if (c != CLS_NONE) atomicAdd(&h[c], 1);
    }
    __syncthreads();
    if (threadIdx.x < NUM_CLS) {
        base[threadIdx.x] = h[threadIdx.x] ? atomicAdd(&a.st->cls_cur[threadIdx.x], h[threadIdx.x]) : 0;
        h[threadIdx.x] = 0;
    }
    __syncthreads();
    const int32_t active0 = a.st->active0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += SBS) {
        const int32_t b = a.off[i], e = a.off[i + 1];
        const int c = row_class(a, e - b);
        if (c == CLS_NONE) continue;
        const int32_t t = base[c] + atomicAdd(&h[c], 1);
        const int32_t kv = a.k[i];
        a.vert[t] = (int32_t)i;
        a.rows[t - active0] = make_int4((int32_t)i, b, e, kv);
        a.cs[i] = make_int2(a.comm[i], kv);
    }
}

// ------------------------------------------------------------------ renumbering
// Smallest member of every community with entries (isolated vertices have
// theirs since the level's start).
__global__ __launch_bounds__(256) void k_small_minv(SmallLevel a, int32_t active)
{
    for (int64_t b = (int64_t)blockIdx.x * 256; b < active; b += (int64_t)gridDim.x * 256) {
        const int64_t t = b + threadIdx.x;
        const bool ok = t < active;
        const int32_t v = ok ? a.rows[t].x : 0;
        const int32_t c = ok ? a.comm[v] : 0;
        const int32_t id = ok ? (a.orig ? a.orig[v] : v) : INT32_MAX;
        min_by_community(a.minv, c, id, ok);
    }
}
__global__ void k_small_flag(SmallLevel a)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t id = a.orig[i];
        a.flag[id] = a.minv[a.comm[i]] == id ? 1 : 0;
    }
}
// pos[id] = communities whose smallest member is below id; pos[n] = their number
template <bool BY_ID>  // positions are ids: the flag is computed here
__global__ __launch_bounds__(SBS) void k_small_rank(SmallLevel a)
{
    scan_tiles(
        a.n, &a.st->rank_ticket, a.scan_rank, &a.st->n2,
        [&](int64_t i) { return BY_ID ? (a.minv[a.comm[i]] == (int32_t)i ? 1 : 0) : a.flag[i]; },
        [&](int64_t i, int32_t at, int32_t) { a.pos[i] = at; });
}
// Labels by position (and by id where they differ); per community: its
// volume, its graph, an empty row; per graph: the volumes' squares.
__global__ __launch_bounds__(256) void k_small_labels(SmallLevel a, SmallCoarse c)
{
    int64_t cur = -1;
    unsigned long long s = 0;
    unsigned long long* sq = (unsigned long long*)(a.st_sums + a.G);
    const int64_t lo = (int64_t)a.n * blockIdx.x / gridDim.x, hi = (int64_t)a.n * (blockIdx.x + 1) / gridDim.x;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
        const int32_t cm = a.comm[i], m = a.minv[cm], P = a.pos[m];
        const int32_t id = a.orig ? a.orig[i] : (int32_t)i;
        a.labels[i] = P;
        if (a.orig && a.labels_id) a.labels_id[id] = P;
        if (m != id || !c.k2) continue;
        const int32_t vol = a.sigma[cm];
        c.k2[P] = vol;
        c.cnt[P] = 0;
        const int32_t g = a.gid ? a.gid[i] : 0;
        if (c.gid2) c.gid2[P] = g;
        if (g != cur) {
            if (cur >= 0 && s) atomicAdd(&sq[cur], s);
            cur = g;
            s = 0;
        }
        s += (unsigned long long)((int64_t)vol * vol);
    }
    if (c.k2) block_flush_sums<256, unsigned long long>(sq, cur, s);
}

// ------------------------------------------------------------------ aggregation by hashing
// Sum the weights of equal (label(i), label(j)): a workgroup takes 1024
// merge-path items, sums its entries in an LDS table that always has room
// (at most 1024 keys in 2048 slots), and adds its distinct keys to a table
// in device memory of at least two slots per entry of the level; whoever
// claims a slot there counts it for its coarse row.  The weight inside
// communities goes to its graph's Sigma_in.
constexpr int AH_BS = 256, AH_IT = 4, AH_T = AH_BS * AH_IT, AH_SLOTS = 2 * AH_T;

__device__ __forceinline__ uint32_t hash_pair(uint64_t k)
{
    k *= 0x9E3779B97F4A7C15ull;
    return (uint32_t)(k >> 32) ^ (uint32_t)(k >> 11);
}

__global__ __launch_bounds__(AH_BS) void k_agg_hash(SmallLevel a, SmallCoarse c)
{
    __shared__ unsigned long long h_key[AH_SLOTS];
    __shared__ int32_t h_val[AH_SLOTS];
    for (int t = threadIdx.x; t < AH_SLOTS; t += AH_BS) { h_key[t] = HASH_EMPTY; h_val[t] = 0; }
    int64_t cur = -1;
    unsigned long long s = 0;
    unsigned long long* sin = (unsigned long long*)a.st_sums;
    for_tile_entries_at<AH_BS, AH_IT>((int64_t)blockIdx.x, a.off, a.n, a.nnz, [&](int32_t r, int64_t e) {
        const int32_t P = a.labels[r], Q = a.labels[a.idx[e]];
        const int32_t w = a.w ? a.w[e] : 1;
        const unsigned long long key = ((unsigned long long)(uint32_t)P << 32) | (uint32_t)Q;
        uint32_t h = hash_pair(key) & (AH_SLOTS - 1);
        for (;;) {
            const unsigned long long prev = atomicCAS(&h_key[h], HASH_EMPTY, key);
            if (prev == HASH_EMPTY || prev == key) break;
            h = (h + 1) & (AH_SLOTS - 1);
        }
        atomicAdd(&h_val[h], w);
        if (P == Q) {
            const int64_t g = a.gid ? a.gid[r] : 0;
            if (g != cur) {
                if (cur >= 0 && s) atomicAdd(&sin[cur], s);
                cur = g;
                s = 0;
            }
            s += (unsigned long long)w;
        }
    });
    __syncthreads();
    for (int t = threadIdx.x; t < AH_SLOTS; t += AH_BS) {
        const unsigned long long key = h_key[t];
        if (key == HASH_EMPTY) continue;
        uint32_t h = hash_pair(key) & c.mask;
        unsigned long long prev;
        for (;;) {
            prev = atomicCAS(&c.keys[h], HASH_EMPTY, key);
            if (prev == HASH_EMPTY || prev == key) break;
            h = (h + 1) & c.mask;
        }
        atomicAdd(&c.vals[h], h_val[t]);
        if (prev == HASH_EMPTY) atomicAdd(&c.cnt[(uint32_t)(key >> 32)], 1);
    }
    block_flush_sums<AH_BS, unsigned long long>(sin, cur, s);
}

// coarse row offsets (the row counts become the rows' write positions)
__global__ __launch_bounds__(SBS) void k_small_offsets(SmallLevel a, SmallCoarse c)
{
    const int32_t n2 = a.st->n2;
    scan_tiles(
        n2, &a.st->row_ticket, a.scan_rows, &a.st->e2, [&](int64_t i) { return c.cnt[i]; },
        [&](int64_t i, int32_t at, int32_t v) {
            c.off2[i] = at;
            c.cnt[i] = at;
            if (i == n2 - 1) c.off2[n2] = at + v;
        });
}

// the table's pairs to their rows; the table is left empty
__global__ void k_table_rows(SmallCoarse c)
{
    const int64_t slots = (int64_t)c.mask + 1;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < slots; t += (int64_t)gridDim.x * blockDim.x) {
        const unsigned long long key = c.keys[t];
        if (key == HASH_EMPTY) continue;
        const int32_t p = atomicAdd(&c.cnt[(uint32_t)(key >> 32)], 1);
        c.idx2[p] = (int32_t)(uint32_t)key;
        c.w2[p] = c.vals[t];
        c.keys[t] = HASH_EMPTY;
        c.vals[t] = 0;
    }
}

__global__ void k_hash_clear(unsigned long long* keys, int32_t* vals, int64_t slots)
{
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < slots; t += (int64_t)gridDim.x * blockDim.x) {
        keys[t] = HASH_EMPTY;
        vals[t] = 0;
    }
}

// What the host needs of the coarsened level, to pinned memory: the number of
// communities and coarse entries, and per graph c its first community, its
// first entry (with off2), Sigma_in and the sum of its squared volumes.
__global__ __launch_bounds__(256) void k_small_report(SmallLevel a, SmallCoarse c, const int32_t* voff, SmallReport r)
{
    const int32_t n2 = a.st->n2;
    for (int32_t g = threadIdx.x; g <= a.G; g += 256) {
        const int32_t at = voff ? voff[g] : (g == 0 ? 0 : a.n);
        const int32_t v = at < a.n ? a.pos[at] : n2;
        r.voff2[g] = v;
        if (c.off2) r.eoff2[g] = n2 > 0 ? c.off2[v] : 0;
        if (g < a.G) {
            r.sums[g] = a.st_sums[g];
            r.sums[a.G + g] = a.st_sums[a.G + g];
        }
    }
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(&a.mail->reported, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

unsigned small_grid(int32_t n)
{
    return (unsigned)std::min<int64_t>(256, std::max<int64_t>(1, ((int64_t)n + 2 * SBS - 1) / (2 * SBS)));
}

}  // namespace

hipError_t launch_level_start(const SmallLevel& a, const SweepEnd& end, const int32_t* gactive, hipStream_t s)
{
    k_level_init<<<small_grid(a.n), SBS, 0, s>>>(a, end, gactive);
    k_level_rows<<<small_grid(a.n), SBS, 0, s>>>(a);
    return hipGetLastError();
}
hipError_t launch_small_renumber(const SmallLevel& a, int32_t active, const SmallCoarse& c, hipStream_t s)
{
    if (active > 0) k_small_minv<<<grid_for(active, 256, 4096), 256, 0, s>>>(a, active);
    const unsigned tiles = (unsigned)(((int64_t)a.n + SMALL_SCAN_TILE - 1) / SMALL_SCAN_TILE);
    if (a.orig) {
        k_small_flag<<<grid_for(a.n, 256, 65536), 256, 0, s>>>(a);
        k_small_rank<false><<<tiles, SBS, 0, s>>>(a);
    } else {
        k_small_rank<true><<<tiles, SBS, 0, s>>>(a);
    }
    k_small_labels<<<grid_for(a.n, 1024, 512), 256, 0, s>>>(a, c);
    return hipGetLastError();
}
hipError_t launch_small_aggregate(const SmallLevel& a, const SmallCoarse& c, hipStream_t s)
{
    const int64_t items = (int64_t)a.n + a.nnz;
    k_agg_hash<<<(unsigned)((items + AH_T - 1) / AH_T), AH_BS, 0, s>>>(a, c);
    const unsigned tiles = (unsigned)(((int64_t)a.n + SMALL_SCAN_TILE - 1) / SMALL_SCAN_TILE);
    k_small_offsets<<<tiles, SBS, 0, s>>>(a, c);
    k_table_rows<<<grid_for((int64_t)c.mask + 1, 256, 8192), 256, 0, s>>>(c);
    return hipGetLastError();
}
hipError_t launch_hash_clear(unsigned long long* keys, int32_t* vals, int64_t slots, hipStream_t s)
{
    if (slots > 0) k_hash_clear<<<LV_GRID(slots)>>>(keys, vals, slots);
    return hipGetLastError();
}
hipError_t launch_small_report(const SmallLevel& a, const SmallCoarse& c, const int32_t* voff, const SmallReport& r,
                               hipStream_t s)
{
    k_small_report<<<1, 256, 0, s>>>(a, c, voff, r);
    return hipGetLastError();
}

}  // namespace lv
