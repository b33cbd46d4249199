// Graph preparation, validation and modularity kernels (gfx950).
//
// Graph model of the paper's Section II-A: undirected, integer weights, a loop
// counts twice in the weighted degree (stored as A_vv = 2w).  Modularity of
// Section II-C in integer form: Q_int = M * Sigma_in - sum_C Sigma_tot(C)^2.
#include "lv_device.h"

namespace lv {

using namespace dev;

namespace {

// err bits: 1 offsets, 2 indices, 4 weights, 8 asymmetric, 16 overflow
__global__ void k_check_offsets(int32_t n, const int32_t* off, int64_t nnz, int32_t* err)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += (int64_t)gridDim.x * blockDim.x) {
        bool bad = false;
        if (i == 0) bad = off[0] != 0;
        if (i == n) bad = bad || (int64_t)off[n] != nnz;
        if (i < n) bad = bad || off[i] > off[i + 1];
        if (bad) atomicOr(err, 1);
    }
}

__global__ __launch_bounds__(TILE_BS) void k_check_entries(int32_t n, const int32_t* off, const int32_t* idx,
                                                            const int32_t* w, int64_t nnz, int32_t* err)
{
    for_tile_entries<TILE_BS, TILE_IT>(off, n, nnz, [&](int32_t r, int64_t e) {
        const int32_t j = idx[e];
        if (j < 0 || j >= n) atomicOr(err, 2);
        else if (e > off[r] && idx[e - 1] >= j) atomicOr(err, 2);
        if (w && w[e] < 1) atomicOr(err, 4);
    });
}

// diag_pos[i] = entry of the loop (i, i), or -1
__global__ void k_diag_scan(int32_t n, const int32_t* off, const int32_t* idx, int32_t* diag_pos, int32_t* any)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = off[i], hi = off[i + 1];
        while (lo < hi) {
            const int64_t mid = (lo + hi) / 2;
            if (idx[mid] < i) lo = mid + 1; else hi = mid;
        }
        const bool has = lo < off[i + 1] && idx[lo] == i;
        diag_pos[i] = has ? (int32_t)lo : -1;
        if (has) atomicOr(any, 1);
    }
}

// A = caller weights (or 1); each loop entry doubled
__global__ void k_adjacency_copy(const int32_t* w_in, int64_t nnz, int32_t* w_out)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * blockDim.x)
        w_out[e] = w_in ? w_in[e] : 1;
}
__global__ void k_adjacency_double(int32_t n, const int32_t* diag_pos, int32_t* w_out, int32_t* err)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t p = diag_pos[i];
        if (p < 0) continue;
        const int64_t v = 2 * (int64_t)w_out[p];
        if (v > INT32_MAX) atomicOr(err, 16);
        else w_out[p] = (int32_t)v;
    }
}

// k64[r] += row sums: per-thread runs of one row, one atomic per run
__global__ __launch_bounds__(TILE_BS) void k_row_sums(int32_t n, const int32_t* off, const int32_t* w, int64_t nnz,
                                                       unsigned long long* k64)
{
    int32_t cur = -1;
    int64_t acc = 0;
    for_tile_entries<TILE_BS, TILE_IT>(off, n, nnz, [&](int32_t r, int64_t e) {
        if (r != cur) {
            if (cur >= 0) atomicAdd(&k64[cur], (unsigned long long)acc);
            cur = r;
            acc = 0;
        }
        acc += w[e];
    });
    if (cur >= 0) atomicAdd(&k64[cur], (unsigned long long)acc);
}

__global__ __launch_bounds__(256) void k_narrow_sum(int32_t n, const unsigned long long* k64, int32_t* k,
                                                     unsigned long long* total)
{
    __shared__ unsigned long long red[4];
    unsigned long long s = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const unsigned long long v = k64[i];
        k[i] = v > (unsigned long long)INT32_MAX ? INT32_MAX : (int32_t)v;
        s += v;
    }
    s = block_sum<256>(s, red);
    if (threadIdx.x == 0) atomicAdd(total, s);
}

__global__ void k_degree_unit(int32_t n, const int32_t* off, int32_t* k)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        k[i] = off[i + 1] - off[i];
}

// Per-thread running sum for one graph, flushed when the graph changes and at
// the end (one atomic per graph per wavefront in the common case).
struct GraphAcc {
    int32_t g = -1;
    unsigned long long s = 0;
    __device__ void add(unsigned long long* out, int32_t gg, unsigned long long x)
    {
        if (gg != g) {
            if (g >= 0 && s) atomicAdd(&out[g], s);
            g = gg;
            s = 0;
        }
        s += x;
    }
    // all threads of a 256-thread workgroup must call it
    __device__ void flush_block(unsigned long long* out) { block_flush_sums<256, unsigned long long>(out, g, s); }
};

// Merge-path tiles visited by each workgroup of a grid of at most this many
// (fewer workgroups, fewer atomics on the per-graph sums)
constexpr unsigned SUM_GRID = 1024;
// Workgroups of the per-vertex sums: each ends in one atomic on one address,
// and those are served one after another (about 13 ns each: 4096 workgroups
// took 52 us over 2 M vertices).
constexpr int64_t VSUM_GRID = 512;

// out[g] += sum of v_i^2 (or v_i) over the vertices of graph g (gid null: one graph)
template <bool SQUARE>
__global__ __launch_bounds__(256) void k_sum_sq(int64_t n, const int32_t* v, const int32_t* gid,
                                                unsigned long long* out)
{
    // contiguous shares: a thread's running sum rarely changes graph
    GraphAcc acc;
    const int64_t end = n * (blockIdx.x + 1) / gridDim.x;
    for (int64_t i = n * blockIdx.x / gridDim.x + threadIdx.x; i < end; i += 256) {
        const int64_t x = (int64_t)v[i];
        acc.add(out, gid ? gid[i] : 0, (unsigned long long)(SQUARE ? x * x : x));
    }
    acc.flush_block(out);
}

// gid[v] = graph of vertex v: the last g with voff[g] <= v
__global__ void k_fill_gid(const int32_t* voff, int32_t G, int32_t n, int32_t* gid)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        int32_t lo = 0, hi = G;
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) / 2;
            if (voff[mid] <= v) lo = mid; else hi = mid;
        }
        gid[v] = lo;
    }
}

// out[g] += trace (sum of diagonal entries) of graph g
__global__ __launch_bounds__(TILE_BS) void k_trace(int32_t n, const int32_t* off, const int32_t* idx, const int32_t* w,
                                                    int64_t nnz, const int32_t* gid, unsigned long long* out)
{
    GraphAcc acc;
    const int64_t tiles = ((int64_t)n + nnz + TILE - 1) / TILE;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x)
        for_tile_entries_co_at<TILE_BS, TILE_IT>(t, off, n, nnz, [&](int32_t r, int64_t e) {
            if (idx[e] == r) acc.add(out, gid ? gid[r] : 0, (unsigned long long)(w ? w[e] : 1));
        });
    acc.flush_block(out);
}

// out[g] += Sigma_in of graph g: entries whose endpoints share a label
__global__ __launch_bounds__(TILE_BS) void k_sigma_in(int32_t n, const int32_t* off, const int32_t* idx, const int32_t* w,
                                                       int64_t nnz, const int32_t* labels, const int32_t* gid,
                                                       unsigned long long* out)
{
    GraphAcc acc;
    const int64_t tiles = ((int64_t)n + nnz + TILE - 1) / TILE;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x)
        for_tile_entries_co_at<TILE_BS, TILE_IT>(t, off, n, nnz, [&](int32_t r, int64_t e) {
            if (labels[idx[e]] == labels[r]) acc.add(out, gid ? gid[r] : 0, (unsigned long long)(w ? w[e] : 1));
        });
    acc.flush_block(out);
}

// Sigma_in without gathers: the neighbour's label of every entry is read
// from the entry cache, in entry order (loop entries, EMPTY_KEY there, are
// left to the caller).
__global__ __launch_bounds__(TILE_BS) void k_sigma_in_cached(int32_t n, const int32_t* off, const int2* ce,
                                                              const int32_t* w, int64_t nnz, const int32_t* labels,
                                                              unsigned long long* out)
{
    GraphAcc acc;
    const int64_t tiles = ((int64_t)n + nnz + TILE - 1) / TILE;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x)
        for_tile_entries_co_at<TILE_BS, TILE_IT>(t, off, n, nnz, [&](int32_t r, int64_t e) {
            if (__builtin_nontemporal_load(&ce[e].x) == labels[r])
                acc.add(out, 0, (unsigned long long)(w ? w[e] : 1));
        });
    acc.flush_block(out);
}

// The sum of squared volumes, added to out->sums[1]; the last workgroup posts
// all three results to pinned memory (mail null: not), in the launch that
// finds them.
__global__ __launch_bounds__(256) void k_mod_finish(const int64_t* vol, int64_t n, ModSums* out, ModMail* mail)
{
    __shared__ unsigned long long red[4];
    unsigned long long s = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        s += (unsigned long long)(vol[i] * vol[i]);
    s = block_sum<256>(s, red);
    if (threadIdx.x != 0) return;
    if (s) atomicAdd((unsigned long long*)&out->sums[1], s);
    if (!mail) return;
    __builtin_amdgcn_s_waitcnt(0);  // the sum before the ticket
    if (atomicAdd(&out->ticket, 1u) + 1u != gridDim.x) return;
    mail->sums[0] = out->sums[0];  // of the launch before this one
    mail->sums[1] = (int64_t)atomicAdd((unsigned long long*)&out->sums[1], 0ull);
    mail->err = out->err;
    __threadfence_system();
    __hip_atomic_store(&mail->ready, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---- storage order by descending degree
// key of position v: graph id above (maxdeg - degree), so that a stable sort
// keeps each packed graph's segment in place and puts its high-degree
// vertices first (ties keep their order)
__global__ void k_degree_keys(int32_t n, const int32_t* off, const int32_t* gid, int32_t maxdeg, int db, uint64_t* keys,
                              int32_t* vals)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t g = gid ? (uint64_t)gid[v] : 0ull;
        keys[v] = (g << db) | (uint64_t)(maxdeg - (off[v + 1] - off[v]));
        vals[v] = (int32_t)v;
    }
}
__global__ __launch_bounds__(256) void k_max_degree(int32_t n, const int32_t* off, int32_t* out)
{
    __shared__ int32_t red[256 / WAVE];
    int32_t m = 0;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < n; v += (int64_t)gridDim.x * 256)
        m = max(m, off[v + 1] - off[v]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, __shfl_xor(m, d));
    if (lane_id() == 0) red[threadIdx.x / WAVE] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / WAVE; ++w) m = max(m, red[w]);
        atomicMax(out, m);
    }
}
__global__ void k_inverse(const int32_t* perm, int32_t n, int32_t* inv)
{
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        inv[perm[q]] = (int32_t)q;
}
__global__ void k_perm_lengths(const int32_t* perm, int32_t n, const int32_t* off, int32_t* len)
{
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = perm[q];
        len[q] = off[v + 1] - off[v];
    }
}
// place[v] = (new position, new row start) of old row v: one gather an entry
// where the reverse entries are mapped too
__global__ void k_perm_places(const int32_t* perm, int32_t n, const int32_t* off_new, int2* place)
{
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        place[perm[q]] = make_int2((int32_t)q, off_new[q]);
}
// new row q = old row perm[q], its column positions mapped through inv, or
// through place with the reverse entries
template <bool REV>
__global__ __launch_bounds__(TILE_BS) void k_perm_rows(int32_t n, const int32_t* off_new, int64_t nnz,
                                                        const int32_t* perm, const int32_t* off, const int32_t* idx,
                                                        const int32_t* w, const int32_t* inv, const int2* place,
                                                        int32_t* idx_new, int32_t* w_new, const int32_t* rank,
                                                        int32_t* rev_new)
{
    for_tile_entries_co_at<TILE_BS, TILE_IT>((int64_t)blockIdx.x, off_new, n, nnz, [&](int32_t q, int64_t e) {
        const int64_t src = (int64_t)off[perm[q]] + (e - off_new[q]);
        if constexpr (REV) {  // the reverse entry keeps its rank within its (moved) row
            const int2 to = place[idx[src]];
            idx_new[e] = to.x;
            rev_new[e] = to.y + rank[src];
        } else {
            idx_new[e] = inv[idx[src]];
        }
        if (w) w_new[e] = w[src];
    });
}

// A stored CSR in vertex-id order and the caller's convention: row q of the
// result is the stored row at position inv[q] (null: q), a column the id
// orig[position] (null: the position).  Storing a graph by degree permutes its
// rows and keeps each row's entries in order, so the columns come out
// ascending.  Loops are stored doubled.  w_out null: no weights wanted.
__global__ __launch_bounds__(TILE_BS) void k_export_rows(int32_t n, const int32_t* off_out, int64_t nnz,
                                                          const int32_t* inv, const int32_t* orig, const int32_t* off,
                                                          const int32_t* idx, const int32_t* w, int32_t* idx_out,
                                                          int32_t* w_out)
{
    for_tile_entries_co_at<TILE_BS, TILE_IT>((int64_t)blockIdx.x, off_out, n, nnz, [&](int32_t q, int64_t e) {
        const int64_t src = (int64_t)off[inv ? inv[q] : q] + (e - off_out[q]);
        const int32_t p = idx[src];
        const int32_t id = orig ? orig[p] : p;
        idx_out[e] = id;
        if (w_out) {
            const int32_t x = w ? w[src] : 1;
            w_out[e] = w && id == q ? x / 2 : x;
        }
    });
}

// Symmetry and reverse entries of a CSR with sorted rows, from the stable
// order of its entries by column: entries are listed row by row, so those of
// column j come out in the order of their rows, and the t-th of them is the
// reverse of row j's t-th entry.  rev[e] = the listed entry and col[e] its
// column, as sorted: the entry is checked to lie in row idx[e], to point back,
// and (w not null) to have the same weight; rank[e] (null, or rev itself, too) = its
// position in that row.  Structural mismatches set structural_bits in err,
// weight mismatches weight_bits.  Three sorting passes and one gather per entry
// replace a binary search for each of them (twice: once to validate, once for
// the map).  54 M entries take 0.80 ms; with the column gathered from idx, 1.34.
__global__ __launch_bounds__(TILE_BS) void k_reverse_check(int32_t n, const int32_t* off, const int32_t* idx,
                                                            const int32_t* w, int64_t nnz, const int32_t* rev,
                                                            const int32_t* col, int32_t* rank, int32_t structural_bits,
                                                            int32_t weight_bits, int32_t* err)
{
    int32_t bad = 0;
    for_tile_entries_co_at<TILE_BS, TILE_IT>((int64_t)blockIdx.x, off, n, nnz, [&](int32_t r, int64_t e) {
        const int32_t c = idx[e], x = rev[e];
        const int32_t cb = off[c], ce = off[c + 1];
        if (x < cb || x >= ce || col[e] != r) bad |= structural_bits;
        else if (w && w[x] != w[e]) bad |= weight_bits;
        if (rank) rank[e] = x - cb;
    });
    if (bad) atomicOr(err, bad);
}

__global__ void k_reverse_from_rank(const int32_t* off, const int32_t* idx, int64_t nnz, const int32_t* rank,
                                    int32_t* rev)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * blockDim.x)
        rev[e] = off[idx[e]] + rank[e];
}
__global__ void k_scatter_i32(const int32_t* src, const int32_t* idx, int32_t m, int32_t* dst)
{
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < m; t += (int64_t)gridDim.x * blockDim.x)
        dst[idx[t]] = src[t];
}

}  // namespace

hipError_t launch_degree_keys(int32_t n, const int32_t* off, const int32_t* gid, int32_t maxdeg, int db, uint64_t* keys,
                              int32_t* vals, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_degree_keys<<<LV_GRID(n)>>>(n, off, gid, maxdeg, db, keys, vals);
    return hipGetLastError();
}
hipError_t launch_max_degree(int32_t n, const int32_t* off, int32_t* out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_max_degree<<<grid_for(n, 256, VSUM_GRID), 256, 0, s>>>(n, off, out);
    return hipGetLastError();
}
hipError_t launch_inverse(const int32_t* perm, int32_t n, int32_t* inv, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_inverse<<<LV_GRID(n)>>>(perm, n, inv);
    return hipGetLastError();
}
hipError_t launch_perm_lengths(const int32_t* perm, int32_t n, const int32_t* off, int32_t* len, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_perm_lengths<<<LV_GRID(n)>>>(perm, n, off, len);
    return hipGetLastError();
}
hipError_t launch_perm_rows(int32_t n, const int32_t* off_new, int64_t nnz, const int32_t* perm, const int32_t* off,
                            const int32_t* idx, const int32_t* w, const int32_t* inv, int32_t* idx_new, int32_t* w_new,
                            const int32_t* rank, int32_t* rev_new, void* place, hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    if (rank) {
        k_perm_places<<<LV_GRID(n)>>>(perm, n, off_new, (int2*)place);
        k_perm_rows<true><<<tiles_for(n, nnz), TILE_BS, 0, s>>>(n, off_new, nnz, perm, off, idx, w, nullptr,
                                                                (const int2*)place, idx_new, w_new, rank, rev_new);
    } else {
        k_perm_rows<false><<<tiles_for(n, nnz), TILE_BS, 0, s>>>(n, off_new, nnz, perm, off, idx, w, inv, nullptr,
                                                                 idx_new, w_new, nullptr, nullptr);
    }
    return hipGetLastError();
}
hipError_t launch_export_rows(int32_t n, const int32_t* off_out, int64_t nnz, const int32_t* inv, const int32_t* orig,
                              const int32_t* off, const int32_t* idx, const int32_t* w, int32_t* idx_out,
                              int32_t* w_out, hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    k_export_rows<<<tiles_for(n, nnz), TILE_BS, 0, s>>>(n, off_out, nnz, inv, orig, off, idx, w, idx_out, w_out);
    return hipGetLastError();
}
hipError_t launch_reverse_check(int32_t n, const int32_t* off, const int32_t* idx, const int32_t* w, int64_t nnz,
                                const int32_t* rev, const int32_t* col, int32_t* rank, int32_t structural_bits,
                                int32_t weight_bits, int32_t* err, hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    k_reverse_check<<<tiles_for(n, nnz), TILE_BS, 0, s>>>(n, off, idx, w, nnz, rev, col, rank, structural_bits,
                                                          weight_bits, err);
    return hipGetLastError();
}
hipError_t launch_reverse_from_rank(int32_t n, const int32_t* off, const int32_t* idx, int64_t nnz,
                                    const int32_t* rank, int32_t* rev, hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    (void)n;
    k_reverse_from_rank<<<LV_GRID(nnz)>>>(off, idx, nnz, rank, rev);
    return hipGetLastError();
}
hipError_t launch_scatter_i32(const int32_t* src, const int32_t* idx, int32_t m, int32_t* dst, hipStream_t s)
{
    if (m <= 0) return hipSuccess;
    k_scatter_i32<<<LV_GRID(m)>>>(src, idx, m, dst);
    return hipGetLastError();
}

hipError_t launch_check_offsets(int32_t n, const int32_t* off, int64_t nnz, int32_t* err, hipStream_t s)
{
    k_check_offsets<<<LV_GRID((int64_t)n + 1)>>>(n, off, nnz, err);
    return hipGetLastError();
}
hipError_t launch_check_entries(int32_t n, const int32_t* off, const int32_t* idx, const int32_t* w, int64_t nnz,
                                int32_t* err, hipStream_t s)
{
    if (nnz <= 0) return hipSuccess;
    k_check_entries<<<tiles_for(n, nnz), TILE_BS, 0, s>>>(n, off, idx, w, nnz, err);
    return hipGetLastError();
}
hipError_t launch_diag_scan(int32_t n, const int32_t* off, const int32_t* idx, int32_t* diag_pos, int32_t* any,
                            hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_diag_scan<<<LV_GRID(n)>>>(n, off, idx, diag_pos, any);
    return hipGetLastError();
}
hipError_t launch_adjacency_weights(int32_t n, const int32_t* w_in, const int32_t* diag_pos, int64_t nnz,
                                    int32_t* w_out, int32_t* err, hipStream_t s)
{
    if (nnz > 0) k_adjacency_copy<<<LV_GRID(nnz)>>>(w_in, nnz, w_out);
    if (n > 0) k_adjacency_double<<<LV_GRID(n)>>>(n, diag_pos, w_out, err);
    return hipGetLastError();
}
hipError_t launch_row_sums(int32_t n, const int32_t* off, const int32_t* w, int64_t nnz, int32_t* k, int64_t* k64,
                           int64_t* total, hipStream_t s)
{
    hipError_t e = hipMemsetAsync(k64, 0, sizeof(int64_t) * (size_t)(n > 0 ? n : 1), s);
    if (e != hipSuccess) return e;
    if (nnz > 0) k_row_sums<<<tiles_for(n, nnz), TILE_BS, 0, s>>>(n, off, w, nnz, (unsigned long long*)k64);
    if (n > 0)
        k_narrow_sum<<<grid_for(n, 256, VSUM_GRID), 256, 0, s>>>(n, (const unsigned long long*)k64, k,
                                                            (unsigned long long*)total);
    return hipGetLastError();
}
hipError_t launch_degree_unit(int32_t n, const int32_t* off, int32_t* k, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_degree_unit<<<LV_GRID(n)>>>(n, off, k);
    return hipGetLastError();
}
hipError_t launch_sum_sq(const int32_t* v, int64_t n, const int32_t* gid, int64_t* out, hipStream_t s)
{
    if (n > 0) k_sum_sq<true><<<grid_for(n, 256, VSUM_GRID), 256, 0, s>>>(n, v, gid, (unsigned long long*)out);
    return hipGetLastError();
}
hipError_t launch_seg_sum(const int32_t* v, int64_t n, const int32_t* gid, int64_t* out, hipStream_t s)
{
    if (n > 0) k_sum_sq<false><<<grid_for(n, 256, VSUM_GRID), 256, 0, s>>>(n, v, gid, (unsigned long long*)out);
    return hipGetLastError();
}
hipError_t launch_fill_gid(const int32_t* voff, int32_t G, int32_t n, int32_t* gid, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_fill_gid<<<LV_GRID(n)>>>(voff, G, n, gid);
    return hipGetLastError();
}
hipError_t launch_trace(int32_t n, const int32_t* off, const int32_t* idx, const int32_t* w, int64_t nnz,
                        const int32_t* gid, int64_t* out, hipStream_t s)
{
    if (nnz > 0) k_trace<<<std::min(tiles_for(n, nnz), SUM_GRID), TILE_BS, 0, s>>>(n, off, idx, w, nnz, gid, (unsigned long long*)out);
    return hipGetLastError();
}
hipError_t launch_sigma_in(int32_t n, const int32_t* off, const int32_t* idx, const int32_t* w, int64_t nnz,
                           const int32_t* labels, const int32_t* gid, int64_t* out, hipStream_t s)
{
    if (nnz > 0)
        k_sigma_in<<<std::min(tiles_for(n, nnz), SUM_GRID), TILE_BS, 0, s>>>(n, off, idx, w, nnz, labels, gid, (unsigned long long*)out);
    return hipGetLastError();
}
hipError_t launch_sigma_in_cached(int32_t n, const int32_t* off, const int2* ce, const int32_t* w, int64_t nnz,
                                  const int32_t* labels, int64_t* out, hipStream_t s)
{
    if (nnz > 0)
        k_sigma_in_cached<<<std::min(tiles_for(n, nnz), SUM_GRID), TILE_BS, 0, s>>>(n, off, ce, w, nnz, labels,
                                                                                     (unsigned long long*)out);
    return hipGetLastError();
}
hipError_t launch_modularity(int32_t n, const int32_t* off, const int32_t* idx, const int32_t* w, int64_t nnz,
                             const int32_t* k, const int32_t* labels, const int32_t* orig, int32_t* pos, int64_t* vol,
                             ModSums* out, ModMail* mail, hipStream_t s)
{
    hipError_t e = launch_mod_volumes(n, k, labels, orig, pos, vol, &out->err, s);
    if (e != hipSuccess) return e;
    if (nnz > 0)
        k_sigma_in<<<std::min(tiles_for(n, nnz), SUM_GRID), TILE_BS, 0, s>>>(n, off, idx, w, nnz, orig ? pos : labels,
                                                         nullptr, (unsigned long long*)&out->sums[0]);
    k_mod_finish<<<grid_for(n, 1024, VSUM_GRID), 256, 0, s>>>(vol, n, out, mail);
    return hipGetLastError();
}

}  // namespace lv
