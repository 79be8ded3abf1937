// HIP kernels (gfx950) that build the sparse permutohedral lattice of a
// point set (Joutard et al. 2019, Section 2: operator E of eq. 6 and the
// vertex set its simplices touch), and the simplex-sorted point order the
// filter kernels work in:
//   range      per point: rounded remainder-0 quotients -> per-coordinate
//              min/max (sizes the packed key)
//   layout     one thread: bit layout of the 63-bit packed key
//   insert     per tile of consecutive points: the distinct vertex-0 keys
//              into a hash table of buckets, and each point's place within
//              its bucket
//   scan       per bucket: its start in the order sorted by vertex 0
//   scatter    per point: its index written to its place in that order
//   tiles      per tile of the sorted order: simplices, weights and vertex
//              keys of its points; distinct keys as rows, inserted into the
//              vertex hash table; contributions sorted by row, segments,
//              work order
//   compact    per table slot: dense vertex ids
//   resolve    per tile row: its vertex id; per vertex and direction the
//              neighbour table, ids of key -/+ u_j (further blocks)
// Only a point's vertex 0 is needed to sort the points, and a tile of the
// sorted order has far fewer distinct vertices than one of consecutive
// points (128^3 volume, d = 5: about 65 against 290; 2 x 160x160x96, d = 8:
// about 330 against 940), so the d+1 keys of a point are deduplicated and
// inserted once, in the sorted order.
#include "pam_device.h"

#include <algorithm>

namespace pam {

// Per block: the min and max of the rounded quotients of its points, to
// part[c * kRangeBlocks + block] and part[(D + c) * kRangeBlocks + block],
// and whether one of them is not finite or too large, to
// part[2D * kRangeBlocks + block]; k_layout reduces the blocks.  The grid
// also empties the bucket table for the insert.
constexpr int kRangeUnroll = 4;

template <int D>
__global__ __launch_bounds__(kBlock) void k_range(const float *__restrict__ feat, int64_t n, Elev E,
                                                  int32_t *__restrict__ part, uint64_t *__restrict__ bkeys,
                                                  int32_t *__restrict__ bcount, uint64_t bcap)
{
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < bcap; i += (uint64_t)gridDim.x * kBlock) {
        bkeys[i] = kEmptyKey;
        bcount[i] = 0;
    }
    __shared__ int smin[kBlock / 64][D];
    __shared__ int smax[kBlock / 64][D];
    int qmin[D], qmax[D];
#pragma unroll
    for (int c = 0; c < D; ++c) {
        qmin[c] = INT_MAX;
        qmax[c] = INT_MIN;
    }
    bool bad = false;
    // kRangeUnroll points per thread and trip, their features requested
    // together before any is elevated
    constexpr int U = kRangeUnroll;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x; i0 < n; i0 += U * stride) {
        float pl[U][D];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + u * stride;
#pragma unroll
            for (int j = 0; j < D; ++j)
                pl[u][j] = i < n ? feat[i * D + j] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + u * stride >= n)
                break;
            float x[D + 1];
            const bool ok = elevate<D>(pl[u], E, x);
            bad |= !ok;
            // rounded quotients before the remainder-0 fix-up; the fix-up and
            // the vertex offsets move them by at most -2..+1
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const int q = ok ? (int)__builtin_rintf(x[c] * E.inv) : 0;
                qmin[c] = min(qmin[c], q);
                qmax[c] = max(qmax[c], q);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < D; ++c) {
        for (int off = 32; off > 0; off >>= 1) {
            qmin[c] = min(qmin[c], __shfl_xor(qmin[c], off));
            qmax[c] = max(qmax[c], __shfl_xor(qmax[c], off));
        }
    }
    int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < D; ++c) {
            smin[wave][c] = qmin[c];
            smax[wave][c] = qmax[c];
        }
    }
    __shared__ int bad_s;
    if (threadIdx.x == 0)
        bad_s = 0;
    __syncthreads();
    if (__ballot(bad) != 0 && lane == 0)
        bad_s = 1;
    __syncthreads();
    if (threadIdx.x == 0)
        part[2 * D * kRangeBlocks + blockIdx.x] = bad_s;
    if (threadIdx.x < D) {
        int c = threadIdx.x, lo = INT_MAX, hi = INT_MIN;
        for (int w = 0; w < kBlock / 64; ++w) {
            lo = min(lo, smin[w][c]);
            hi = max(hi, smax[w][c]);
        }
        part[c * kRangeBlocks + blockIdx.x] = lo;
        part[(D + c) * kRangeBlocks + blockIdx.x] = hi;
    }
}

// One block of 1024 threads: reduces the per-block ranges of k_range (all
// 2d+1 partial rows requested at once), resets the control block, and one
// thread lays out the packed key.
constexpr int kLayoutThreads = 1024;
static_assert(kRangeBlocks == 2 * kLayoutThreads, "two partials per layout thread");

template <int D>
__global__ __launch_bounds__(kLayoutThreads) void k_layout(Ctl *ctl, const int32_t *__restrict__ part, int nblocks,
                                                           int gbits)
{
    constexpr int d = D;
    constexpr int NW = kLayoutThreads / 64;
    __shared__ int sred[2 * D + 1][NW];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const bool on0 = t < nblocks, on1 = t + kLayoutThreads < nblocks;
    int v[2 * D + 1];
#pragma unroll
    for (int r = 0; r <= 2 * D; ++r) {
        const int id = r < D ? INT_MAX : (r < 2 * D ? INT_MIN : 0);
        const int a = on0 ? part[r * kRangeBlocks + t] : id;
        const int b = on1 ? part[r * kRangeBlocks + t + kLayoutThreads] : id;
        v[r] = r < D ? min(a, b) : (r < 2 * D ? max(a, b) : (a | b));
    }
#pragma unroll
    for (int r = 0; r <= 2 * D; ++r) {
        for (int off = 32; off > 0; off >>= 1) {
            const int o = __shfl_xor(v[r], off);
            v[r] = r < D ? min(v[r], o) : (r < 2 * D ? max(v[r], o) : (v[r] | o));
        }
        if (lane == 0)
            sred[r][wave] = v[r];
    }
    __syncthreads();
    if (t != 0)
        return;
    int bad = 0;
    for (int w = 0; w < NW; ++w)
        bad |= sred[2 * D][w];
    ctl->flags = bad ? kFlagBadFeature : 0u;
    ctl->count = 0;
    ctl->nvert = 0;
    ctl->nbucket = 0;
    ctl->nsorted = 0;
    for (int c = 0; c < d; ++c) {
        int lo = INT_MAX, hi = INT_MIN;
        for (int w = 0; w < NW; ++w) {
            lo = min(lo, sred[c][w]);
            hi = max(hi, sred[D + c][w]);
        }
        ctl->qmin[c] = lo;
        ctl->qmax[c] = hi;
    }
    KeyLayout &lay = ctl->lay;
    int kbits = 32 - __clz(d);  // bits for 0..d
    int shift = kbits;
    bool fits = true;
    for (int c = 0; c < d; ++c) {
        // vertex quotients lie in [qmin - 2, qmax + 1]; a neighbour outside
        // that range cannot be a vertex and packs as absent
        int64_t lo = (int64_t)ctl->qmin[c] - 2;
        int64_t width = (int64_t)ctl->qmax[c] - (int64_t)ctl->qmin[c] + 4;
        int bits = 64 - __clzll((unsigned long long)(width - 1));
        lay.lo[c] = (int32_t)lo;
        lay.shift[c] = shift;
        lay.bits[c] = bits;
        shift += bits;
        if (bits > 31 || shift > 63)
            fits = false;
    }
    lay.kbits = kbits;
    lay.gshift = shift;
    lay.gbits = gbits;
    shift += gbits;
    if (shift > 63)
        fits = false;
    lay.total_bits = shift;
    if (!fits)
        ctl->flags |= kFlagKeyRange;
}

__global__ void k_fill_f32(float *p, float value, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = value;
}

// Insert key into the open-addressing table (linear probing).  Plain loads
// may see a stale empty slot; the compare-and-swap decides.  Keys are only
// ever written once (empty -> key), so a stale read is either empty or the
// final key.  Most keys of a tile are already in the table (the tiles
// around it share them), and the plain load finds those in the caches,
// where a compare-and-swap would go to the L2 every time.  Counts new keys
// in `added`; sets `full` after kMaxProbe slots (or the whole table), a run
// that linear probing does not reach at the loads the build accepts (up to
// one half), so that a table far too small is given up at once.  Returns the
// key's slot (all ones when the table is full).
constexpr uint64_t kMaxProbe = 512;
// STRIDE: 64-bit words per slot, the key first.
template <int STRIDE>
__device__ __forceinline__ uint64_t table_insert(uint64_t *tkeys, uint64_t mask, uint64_t key, uint32_t &added,
                                                 bool &full)
{
    uint64_t h = mix64(key) & mask;
    for (uint64_t probe = 0; probe <= mask && probe < kMaxProbe; ++probe) {
        const uint64_t cur = tkeys[h * STRIDE];
        if (cur == key)
            return h;
        if (cur == kEmptyKey) {
            const uint64_t prev = atomicCAS((unsigned long long *)&tkeys[h * STRIDE], (unsigned long long)kEmptyKey,
                                            (unsigned long long)key);
            if (prev == kEmptyKey) {
                ++added;
                return h;
            }
            if (prev == key)
                return h;
        }
        h = (h + 1) & mask;
    }
    full = true;
    return ~0ull;
}

// Dense ids for the occupied slots: each block counts its PER * kBlock
// slots, scans the counts, and takes its id range with one update of a
// single counter (updates of one address serialise, so large tables take
// more slots per block).  The first thread publishes the build's outcome:
// to the control block for the resolve (whose further blocks zero the
// counters) and to the host (pinned memory), which waits for nothing more,
// so that the caller goes on while the compaction and the resolve run.  Ids
// from vcap on are not stored: the host then grows its buffers and launches
// again.
constexpr uint64_t kCompactWideCap = 1ull << 20;  // tables from this size take 16 slots per thread, else 4

template <int PER>
__global__ __launch_bounds__(kBlock) void k_compact(Slot *__restrict__ table,
                                                    uint64_t *vkeys, uint32_t vcap, uint64_t cap, Ctl *ctl,
                                                    HostResult *result, uint32_t attempt)
{
    constexpr int kCompactPer = PER;
    __shared__ int cs[kBlock];
    __shared__ int wsum[kBlock / 64 + 1];
    __shared__ uint32_t base_s;
    const uint32_t count = ctl->count;
    uint32_t flags = ctl->flags;
    if ((uint64_t)count > cap / 2)
        flags |= kFlagTableFull;  // load factor above one half: regrow as for a full table
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const BuildResult r = {flags, count, ctl->nbucket, 0u};
        ctl->result = r;
        const uint64_t tag = (uint64_t)attempt << 32;
        __hip_atomic_store(&result->flags, tag | r.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&result->count, tag | r.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&result->nbucket, tag | r.nbucket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    if (flags)
        return;
    const uint64_t b0 = (uint64_t)blockIdx.x * kBlock * kCompactPer + threadIdx.x;
    uint64_t key[kCompactPer];
    int c = 0;
#pragma unroll
    for (int j = 0; j < kCompactPer; ++j) {
        const uint64_t s = b0 + (uint64_t)j * kBlock;
        key[j] = s < cap ? table[s].key : kEmptyKey;
        c += key[j] != kEmptyKey ? 1 : 0;
    }
    cs[threadIdx.x] = c;
    __syncthreads();
    const int total = block_exclusive_scan(cs, kBlock, wsum);
    if (threadIdx.x == 0)
        base_s = total ? atomicAdd(&ctl->nvert, (uint32_t)total) : 0u;
    __syncthreads();
    uint32_t id = base_s + (uint32_t)cs[threadIdx.x];
#pragma unroll
    for (int j = 0; j < kCompactPer; ++j) {
        const uint64_t s = b0 + (uint64_t)j * kBlock;
        if (key[j] != kEmptyKey) {
            table[s].id = (int32_t)id;
            if (id < vcap)
                vkeys[id] = key[j];
            ++id;
        }
    }
}

__device__ __forceinline__ Slot load_slot(const Slot *__restrict__ table, uint64_t h)
{
    const ulonglong2 v = reinterpret_cast<const ulonglong2 *>(table)[h];
    return {v.x, (int32_t)(uint32_t)v.y, 0};
}

__device__ __forceinline__ int32_t probe_id(const Slot *__restrict__ table, uint64_t mask, uint64_t key)
{
    uint64_t h = mix64(key) & mask;
    for (uint64_t probe = 0; probe <= mask; ++probe) {
        const Slot cur = load_slot(table, h);
        if (cur.key == key)
            return cur.id;
        if (cur.key == kEmptyKey)
            return -1;
        h = (h + 1) & mask;
    }
    return -1;
}

__device__ __forceinline__ void unpack_key(uint64_t key, int d, const KeyLayout &lay, int *coord)
{
    int k = (int)(key & ((1ull << lay.kbits) - 1));
    for (int c = 0; c < d; ++c) {
        int t = (int)((key >> lay.shift[c]) & ((1ull << lay.bits[c]) - 1)) + lay.lo[c];
        coord[c] = k + (d + 1) * t;
    }
}

// Entry nbr_entry(j, m, M) of the neighbour table: the ids of key_m -/+ u_j
// (-1 if absent), u_j = (d+1) e_j - 1.  nbr is direction-major:
// nbr[(j * M + m) * 2 + 0] = id(key_m - u_j), nbr[(j * M + m) * 2 + 1] = id(key_m + u_j).
// On the packed key (remainder k, quotients t_c): adding u_j lowers every
// coordinate by one and raises coordinate j by d+1, so k becomes k - 1 with
// t_j + 1, or, from k = 0, k becomes d with every other t_c - 1; subtracting
// u_j is the reverse.  A quotient that would leave its field has no vertex.
template <int D>
__device__ __forceinline__ void neighbour_item(const uint64_t *__restrict__ vkeys, uint32_t M, const KeyLayout &lay,
                                               const Slot *__restrict__ table, uint64_t mask,
                                               int32_t *__restrict__ nbr, int j, int64_t m)
{
    const uint64_t key_m = vkeys[m];
    const int k = (int)(key_m & ((1ull << lay.kbits) - 1));
    uint64_t one_j = 0, others = 0;  // 1 in field j; 1 in every other field
    bool j_min = false, j_max = false, o_min = false, o_max = false;  // a field at its lowest / highest value
#pragma unroll
    for (int c = 0; c < D; ++c) {
        const uint64_t top = (1ull << lay.bits[c]) - 1;
        const uint64_t off = (key_m >> lay.shift[c]) & top;
        if (c == j) {
            one_j = 1ull << lay.shift[c];
            j_min = off == 0;
            j_max = off == top;
        } else {
            others |= 1ull << lay.shift[c];
            o_min |= off == 0;
            o_max |= off == top;
        }
    }
    uint64_t key[2];
    bool ok[2];
    if (k < D) {  // - u_j
        key[0] = key_m + 1 - one_j;
        ok[0] = !j_min;
    } else {
        key[0] = key_m - D + others;
        ok[0] = !o_max;
    }
    if (k > 0) {  // + u_j
        key[1] = key_m - 1 + one_j;
        ok[1] = !j_max;
    } else {
        key[1] = key_m + D - others;
        ok[1] = !o_min;
    }
    // both probes side by side: their first slots are requested together
    uint64_t h[2];
    Slot cur[2];
    int32_t id[2];
    for (int sgn = 0; sgn < 2; ++sgn) {
        h[sgn] = mix64(key[sgn]) & mask;
        cur[sgn] = ok[sgn] ? load_slot(table, h[sgn]) : Slot{kEmptyKey, -1, 0};
    }
    for (int sgn = 0; sgn < 2; ++sgn) {
        id[sgn] = -1;
        for (uint64_t probe = 0; ok[sgn] && probe <= mask; ++probe) {
            if (cur[sgn].key == key[sgn]) {
                id[sgn] = cur[sgn].id;
                break;
            }
            if (cur[sgn].key == kEmptyKey)
                break;
            h[sgn] = (h[sgn] + 1) & mask;
            cur[sgn] = load_slot(table, h[sgn]);
        }
    }
    reinterpret_cast<int2 *>(nbr)[nbr_entry(j, m, M)] = make_int2(id[0], id[1]);
}

__global__ void k_vertex_groups(const uint64_t *__restrict__ vkeys, int64_t M, const Ctl *ctl, int32_t *vgroup)
{
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M)
        return;
    const KeyLayout &lay = ctl->lay;
    vgroup[m] = lay.gbits ? (int32_t)((vkeys[m] >> lay.gshift) & ((1ull << lay.gbits) - 1)) : 0;
}

__global__ void k_unpack_keys(int d, const uint64_t *__restrict__ vkeys, int64_t M, const Ctl *ctl,
                              int32_t *keys)
{
    int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M)
        return;
    int coord[kMaxD];
    unpack_key(vkeys[m], d, ctl->lay, coord);
    for (int c = 0; c < d; ++c)
        keys[m * d + c] = coord[c];
}

// Per sorted position s: the point's vertex ids and barycentric weights as
// the filter kernels read them (the sorted records and the tile's rows),
// written back at the point's original index perm[s].
__global__ void k_export_points(int d, const uint8_t *__restrict__ pts, const uint8_t *__restrict__ tiles,
                                const int32_t *__restrict__ perm, int64_t n, int32_t *vert, float *bary)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n)
        return;
    const int64_t i = perm[s];
    const float *w = reinterpret_cast<const float *>(pts + s * point_bytes(d));
    const TileRec rec(d);
    const int64_t tile = s / rec.T;
    const int p = (int)(s - tile * rec.T);
    const uint8_t *R = tiles + (size_t)tile * rec.bytes;
    const int32_t *rowid = reinterpret_cast<const int32_t *>(R + rec.rowid);
    const uint16_t *lrow = reinterpret_cast<const uint16_t *>(R + rec.lrow);
    for (int k = 0; k <= d; ++k) {
        bary[i * (d + 1) + k] = w[k];
        vert[i * (d + 1) + k] = rowid[lrow[p * (d + 1) + k]];
    }
}

// The points' buckets, a tile of consecutive points at a time: a point's
// bucket is its vertex 0.  The tile's vertex-0 keys are deduplicated in an
// LDS hash (64-bit compare-and-swap; it holds twice the tile's points, so it
// never fills), the tile's points are counted per distinct key, and each
// distinct key takes its slot of the bucket table and, with one global
// atomic, its range of the bucket (same-address atomics per point would
// serialise).  Neighbouring points often share their vertex 0: only the
// first lane of a run of equal keys in a wave probes the LDS table.
// Per point: the bucket's slot and the point's place in the bucket.
// The grid's blocks past the last tile empty the vertex hash table (cap
// slots), which the tiles launch fills.
constexpr int kInsertPoints = 512;  // points (= threads) per tile
constexpr int kInsertHash = 2 * kInsertPoints;

template <int D>
__global__ __launch_bounds__(kInsertPoints) void k_insert(const float *__restrict__ feat, int64_t n, Elev E,
                                                          Groups64 grp, Ctl *ctl, KeyLayout fixed, int use_fixed,
                                                          uint64_t *bkeys, uint64_t bmask, int32_t *bcount,
                                                          int2 *__restrict__ place, Slot *__restrict__ table,
                                                          uint64_t cap)
{
    constexpr int T = kInsertPoints;
    constexpr int H = kInsertHash;
    __shared__ uint64_t hkey[H];
    __shared__ int hcnt[H];   // points of the key, then its base in the bucket
    __shared__ int hslot[H];  // its slot of the bucket table
    __shared__ int miss_s, full_s;
    __shared__ uint32_t added_s;
    const int t = threadIdx.x;
    const int64_t ntiles = (n + T - 1) / T;
    if ((int64_t)blockIdx.x >= ntiles) {  // block-uniform
        const uint64_t stride = (uint64_t)(gridDim.x - ntiles) * T;
        for (uint64_t e = (uint64_t)((int64_t)blockIdx.x - ntiles) * T + t; e < cap; e += stride)
            reinterpret_cast<ulonglong2 *>(table)[e] = make_ulonglong2(kEmptyKey, 0);
        return;
    }
    if (!use_fixed && (ctl->flags & (kFlagKeyRange | kFlagBadFeature)))
        return;
    const KeyLayout lay = use_fixed ? fixed : ctl->lay;
    if (use_fixed && blockIdx.x == 0 && t == 0)
        ctl->lay = fixed;  // for the later kernels of the build (identical in every block)
    const int64_t base = insert_tile(ntiles) * T;
    const int nt = (int)min((int64_t)T, n - base);
    for (int e = t; e < H; e += T) {
        hkey[e] = kEmptyKey;
        hcnt[e] = 0;
    }
    if (t == 0) {
        miss_s = 0;
        full_s = 0;
        added_s = 0;
    }
    __syncthreads();
    const int lane = t & 63;
    const bool valid = t < nt;
    uint64_t key = kEmptyKey;
    if (valid) {
        Simplex<D> s;
        const bool ok = embed<D>(feat + (base + t) * D, E, s);
        if (use_fixed) {
            // every vertex quotient of the point is q_c or q_c - 1: both must
            // fit the fixed layout's field (else the build takes the range pass)
            bool fits = ok;
#pragma unroll
            for (int c = 0; c < D; ++c)
                fits = fits && s.q[c] - 1 - lay.lo[c] >= 0 && s.q[c] - lay.lo[c] < (1 << lay.bits[c]);
            if (!ok)
                atomicOr(&ctl->flags, kFlagBadFeature);
            if (!fits)
                miss_s = 1;
        }
        key = pack_vertex<D>(s, 0, lay, group_field(grp, lay, base + t));
    }
    const LaneRun run = lane_run(key, valid);
    int found = 0, lpos = 0;
    if (valid && run.lead == lane) {
        uint32_t h = (uint32_t)(mix64(key) >> 32) & (H - 1);
        for (;;) {  // at most T of the H slots are ever taken: ends at the key or an empty slot
            const uint64_t prev = atomicCAS((unsigned long long *)&hkey[h], (unsigned long long)kEmptyKey,
                                            (unsigned long long)key);
            if (prev == kEmptyKey || prev == key)
                break;
            h = (h + 1) & (H - 1);
        }
        found = (int)h;
        lpos = atomicAdd(&hcnt[h], run.len);
    }
    found = __shfl(found, run.lead);
    lpos = __shfl(lpos, run.lead) + (lane - run.lead);
    __syncthreads();
    if (miss_s) {  // block-uniform: the keys are not valid in this layout
        if (t == 0)
            atomicOr(&ctl->flags, kFlagLayoutMiss);
        return;
    }
    uint32_t added = 0;
    bool full = false;
    for (int e = t; e < H; e += T) {
        if (hkey[e] != kEmptyKey) {
            const uint64_t slot = table_insert<1>(bkeys, bmask, hkey[e], added, full);
            if (!full) {
                hslot[e] = (int)slot;  // the bucket table has at most 2^31 slots
                hcnt[e] = atomicAdd(&bcount[slot], hcnt[e]);
            }
        }
    }
    if (added)
        atomicAdd(&added_s, added);
    if (full)
        full_s = 1;
    __syncthreads();
    if (t == 0) {
        // no result is needed here, so the adds do not return
        if (added_s)
            atomicAdd(&ctl->nbucket, added_s);
        if (full_s)
            atomicOr(&ctl->flags, kFlagBucketsFull);
    }
    if (valid && !full_s)
        place[base + t] = make_int2(hslot[found], hcnt[found] + lpos);
}

// Bucket counts to bucket starts in the sorted order, in place: each block
// scans its PER * kBlock slots and takes its range of the order with one
// update of a single counter.  The order of the buckets is arbitrary (it is
// the order of a hash), so no scan across blocks is needed.
template <int PER>
__global__ __launch_bounds__(kBlock) void k_starts(int32_t *__restrict__ bcount, uint64_t bcap, Ctl *ctl)
{
    __shared__ int cs[kBlock];
    __shared__ int wsum[kBlock / 64 + 1];
    __shared__ uint32_t base_s;
    if (ctl->flags)
        return;
    const uint64_t b0 = (uint64_t)blockIdx.x * kBlock * PER + threadIdx.x;
    int v[PER], c = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint64_t s = b0 + (uint64_t)j * kBlock;
        v[j] = s < bcap ? bcount[s] : 0;
        c += v[j];
    }
    cs[threadIdx.x] = c;
    __syncthreads();
    const int total = block_exclusive_scan(cs, kBlock, wsum);
    if (threadIdx.x == 0)
        base_s = total ? atomicAdd(&ctl->nsorted, (uint32_t)total) : 0u;
    __syncthreads();
    int start = (int)base_s + cs[threadIdx.x];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint64_t s = b0 + (uint64_t)j * kBlock;
        if (s < bcap)
            bcount[s] = start;
        start += v[j];
    }
}

// Every point's index to its place in the simplex-sorted order: points are
// grouped by their vertex 0 (bucket starts from k_starts), within a group in
// the order in which they took their places.
__global__ __launch_bounds__(kBlock) void k_scatter(const int2 *__restrict__ place,
                                                    const int32_t *__restrict__ start, int64_t n,
                                                    const Ctl *ctl, int32_t *__restrict__ perm)
{
    if (ctl->flags)
        return;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n)
        return;
    const int2 sp = place[i];
    perm[start[sp.x] + sp.y] = (int32_t)i;
}

// Per tile of the sorted order (one thread per point): the point's simplex
// and barycentric weights from its features; the record of weights and ranks
// the filter kernels read; the tile's distinct vertices become dense rows
// (LDS hash) whose keys are inserted into the vertex hash table, their slots
// kept in the tile record for the resolve; the tile's (point, vertex)
// contributions are counting-sorted by row (integer LDS atomics give each its
// position within its row); each row's contributions are cut evenly into
// segments of at most kSegLen, and the rows are counting-sorted by the length
// of their segments, longest first, the order in which the splat hands the
// segments out.
//
// A point's vertices are told apart within the tile by the bucket the point
// belongs to (its vertex 0; a bucket's points are consecutive) and the set of
// coordinates that vertex k has stepped down: a local key of 32 bits.  Only
// the distinct local keys are turned into packed keys (a vertex that two
// buckets share becomes two rows with one id; in dense tiles that is rare, and
// tiles of scattered points have room for the rows).  Keys of 32 bits are for
// LDS: a table of 64-bit packed keys that every tile fits would take 59 KB at
// d = 5 instead of 37, two blocks per CU instead of four.  They hardly change
// the time (128^3, d = 5: 1000 vector instructions per wave and 93 us; packed
// keys in a table of 2048 slots 1090 and 94), which vector instructions (they
// fill two thirds of the SIMDs' cycles) and memory (356 MB, 3.8 TB/s, where a
// copy reaches 5.9) share.
//
// Sorted points share vertices in runs: only the first lane of a run of
// equal keys in a wave probes the LDS table and later counts the whole run,
// the others take its results.
template <int D>
__global__ __launch_bounds__(tile_points(D)) void k_sorted_tiles(const float *__restrict__ feat, int64_t n, Elev E,
                                                                 Groups64 grp, Ctl *ctl,
                                                                 const int32_t *__restrict__ perm,
                                                                 uint8_t *__restrict__ psort, Slot *table,
                                                                 uint64_t mask, uint8_t *__restrict__ tiles)
{
    constexpr int T = tile_points(D), NW = T / 64;
    constexpr int NC = T * (D + 1);
    constexpr int PW = point_bytes(D) / 4;
    static_assert(NC < (1 << 13), "segment start and row must fit their 13-bit fields");
    constexpr int H = tile_slots(D);
    static_assert(H > NC, "a free slot whatever the keys: every probe ends");
    // two uses of one piece of LDS.  Until every contribution has its row:
    // the buckets' keys, the local keys in row order, and the hash (local
    // keys, their rows).  Then per row the count, then first entry (cnt), and
    // the first segment (nsg); and the weights and the sorted entries, on
    // their way to coalesced stores.
    constexpr int kCntBytes = (NC + 4) * 4, kNsgBytes = (NC + 8) * 2;
    constexpr int kHashBytes = T * 8 + NC * 4 + H * 4 + H * 2;
    constexpr int kEntryBytes = kCntBytes + kNsgBytes + NC * 4 + NC * 2;
    __shared__ __attribute__((aligned(16))) uint8_t pool[kHashBytes > kEntryBytes ? kHashBytes : kEntryBytes];
    uint64_t *bkey = reinterpret_cast<uint64_t *>(pool);
    uint32_t *rkey = reinterpret_cast<uint32_t *>(pool + T * 8);
    uint32_t *hkey = rkey + NC;
    uint16_t *hrow = reinterpret_cast<uint16_t *>(hkey + H);
    int *cnt = reinterpret_cast<int *>(pool);
    uint16_t *nsg = reinterpret_cast<uint16_t *>(pool + kCntBytes);
    float *sw = reinterpret_cast<float *>(pool + kCntBytes + kNsgBytes);
    uint16_t *slist = reinterpret_cast<uint16_t *>(sw + NC);
    __shared__ int hist[kSegLen + 1];
    __shared__ int wsum[2 * (T / 64 + 1)];
    __shared__ uint64_t last_s[NW];
    __shared__ int starts_s[NW];
    __shared__ int nrows_s, full_s;
    __shared__ uint32_t added_s;
    if (ctl->flags & ~kFlagTableFull)  // set by other blocks of this launch: TableFull only
        return;
    const KeyLayout lay = ctl->lay;
    const TileRec rec(D);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * T;
    const int nt = (int)min((int64_t)T, n - base);
    const int nc = nt * (D + 1);
    uint8_t *R = tiles + (size_t)blockIdx.x * rec.bytes;
    uint32_t *hdr = reinterpret_cast<uint32_t *>(R);
    int32_t *rowid = reinterpret_cast<int32_t *>(R + rec.rowid);
    uint64_t *rowkey = reinterpret_cast<uint64_t *>(R + rec.rowkey);
    uint16_t *sfirst = reinterpret_cast<uint16_t *>(R + rec.sfirst);
    uint32_t *seg = reinterpret_cast<uint32_t *>(R + rec.seg);
    uint16_t *order = reinterpret_cast<uint16_t *>(R + rec.order);
    uint16_t *lrow = reinterpret_cast<uint16_t *>(R + rec.lrow);
    uint32_t *wseg = reinterpret_cast<uint32_t *>(R + rec.wseg);
    float *weight = reinterpret_cast<float *>(R + rec.weight);
    uint16_t *point = reinterpret_cast<uint16_t *>(R + rec.point);
    const bool valid = t < nt;
    const int64_t i = valid ? perm[base + t] : 0;
    for (int e = t; e < H; e += T)
        hkey[e] = ~0u;
    for (int e = t; e <= kSegLen; e += T)
        hist[e] = 0;
    if (t == 0) {
        nrows_s = 0;
        full_s = 0;
        added_s = 0;
    }
    Simplex<D> s;
    float b[D + 1];
    uint64_t key0 = kEmptyKey;
    if (valid) {
        embed<D>(feat + i * D, E, s);
        key0 = pack_vertex<D>(s, 0, lay, group_field(grp, lay, i));
        barycentric<D>(s, feat + i * D, E, b);
        uint32_t w[PW];
#pragma unroll
        for (int u = 0; u < PW; ++u)
            w[u] = 0u;
#pragma unroll
        for (int k = 0; k <= D; ++k)
            w[k] = __float_as_uint(b[k]);
#pragma unroll
        for (int c = 0; c <= D; ++c)
            w[D + 1 + c / 4] |= (uint32_t)(s.rank[c] & 0xff) << (8 * (c % 4));
        uint4 *prec = reinterpret_cast<uint4 *>(psort + (base + t) * (PW * 4));
#pragma unroll
        for (int u = 0; u < PW / 4; ++u)
            prec[u] = make_uint4(w[4 * u], w[4 * u + 1], w[4 * u + 2], w[4 * u + 3]);
    }
    // the point's bucket within the tile: how many of the tile's points up to
    // it have another vertex 0 than the point before them
    if (lane == 63)
        last_s[wave] = key0;
    __syncthreads();
    const uint32_t plo = __shfl_up((uint32_t)key0, 1), phi = __shfl_up((uint32_t)(key0 >> 32), 1);
    const uint64_t prev = lane > 0 ? ((uint64_t)phi << 32) | plo : (wave > 0 ? last_s[wave - 1] : kEmptyKey);
    const bool first = valid && key0 != prev;  // the tile's first point has no point before it
    const uint64_t firsts = __ballot(first);
    if (lane == 0)
        starts_s[wave] = __popcll(firsts);
    __syncthreads();
    int bl = __popcll(firsts & (lane == 63 ? ~0ull : ((2ull << lane) - 1))) - 1;
    for (int w = 0; w < wave; ++w)
        bl += starts_s[w];
    if (first)
        bkey[bl] = key0;
    // the coordinate of each rank, 4 bits each (d = 16: 5)
    constexpr int CB = D < 16 ? 4 : 5;
    uint64_t by_rank[2] = {0, 0};  // ranks 0 .. 11 and 12 .. 16
    if (valid) {
#pragma unroll
        for (int c = 0; c <= D; ++c) {
            if constexpr (D < 12) {
                by_rank[0] |= (uint64_t)c << (CB * s.rank[c]);
            } else {
                const bool high = s.rank[c] >= 12;
                const uint64_t v = (uint64_t)c << (CB * (high ? s.rank[c] - 12 : s.rank[c]));
                by_rank[0] |= high ? 0 : v;
                by_rank[1] |= high ? v : 0;
            }
        }
    }
    // The loops over k are wave-uniform (cross-lane operations).
    int slot[D + 1];
    LaneRun run[D + 1];
    uint32_t lkey = (uint32_t)bl << (D + 1);  // vertex k steps down the coordinates of rank > d - k
#pragma unroll
    for (int k = 0; k <= D; ++k) {
        if (k > 0) {
            const int r = D + 1 - k;  // 1 .. D
            const uint32_t c = (uint32_t)(by_rank[r >= 12] >> (CB * (r >= 12 ? r - 12 : r))) & ((1u << CB) - 1);
            lkey |= 1u << c;
        }
        run[k] = lane_run32(lkey, valid);
        uint32_t h = 0;
        if (valid && run[k].lead == lane) {
            h = tile_hash(lkey, H);
            for (;;) {  // at most NC of the H slots are ever taken: ends at the key or an empty slot
                const uint32_t was = atomicCAS(&hkey[h], ~0u, lkey);
                if (was == ~0u) {
                    const int r = atomicAdd(&nrows_s, 1);
                    hrow[h] = (uint16_t)r;
                    rkey[r] = lkey;
                    break;
                }
                if (was == lkey)
                    break;
                h = h + 1 < (uint32_t)H ? h + 1 : 0;
            }
        }
        slot[k] = __shfl((int)h, run[k].lead);
    }
    __syncthreads();
    const int nrows = nrows_s;
    uint32_t added = 0;
    bool full = false;
    // each distinct key's slot, for the resolve; -1 when it does not fit an
    // int32 (the resolve then looks the key up)
    for (int r = t; r < nrows; r += T) {
        const uint32_t lk = rkey[r];
        // vertex k: the bucket's vertex 0 plus k, minus 1 in the field of
        // every stepped-down coordinate (coordinate d has no field)
        uint64_t kr = bkey[lk >> (D + 1)] + (uint32_t)__popc(lk & ((2u << D) - 1));
#pragma unroll
        for (int c = 0; c < D; ++c)
            kr -= (uint64_t)((lk >> c) & 1) << lay.shift[c];
        const uint64_t h = table_insert<2>(reinterpret_cast<uint64_t *>(table), mask, kr, added, full);
        rowkey[r] = kr;
        rowid[r] = h <= 0x7fffffffull ? (int32_t)h : -1;
    }
    int q[D + 1], pos[D + 1];
#pragma unroll
    for (int k = 0; k <= D; ++k)
        q[k] = valid ? (int)hrow[slot[k]] : 0;
    if (added)
        atomicAdd(&added_s, added);
    if (full)
        full_s = 1;
    __syncthreads();  // the keys and the hash are dead from here: their LDS takes the counters and entries
    if (t == 0) {
        // the count's result is not needed here (the compaction compares the
        // final count with the load limit), so the add does not return
        if (added_s)
            atomicAdd(&ctl->count, added_s);
        if (full_s)
            atomicOr(&ctl->flags, kFlagTableFull);
    }
    for (int e = t; e < nrows; e += T)
        cnt[e] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k <= D; ++k) {
        int first_pos = 0;
        if (valid && run[k].lead == lane)
            first_pos = atomicAdd(&cnt[q[k]], run[k].len);
        pos[k] = __shfl(first_pos, run[k].lead) + (lane - run[k].lead);
    }
    if (valid) {
        if constexpr ((D + 1) % 2 == 0) {
            uint32_t *lr = reinterpret_cast<uint32_t *>(lrow + t * (D + 1));
#pragma unroll
            for (int k = 0; k <= D; k += 2)
                lr[k / 2] = (uint32_t)q[k] | ((uint32_t)q[k + 1] << 16);
        } else {
#pragma unroll
            for (int k = 0; k <= D; ++k)
                lrow[t * (D + 1) + k] = (uint16_t)q[k];
        }
    }
    __syncthreads();
    // cnt[r]: first entry of row r; nsg[r]: its first segment
    const int nseg = block_exclusive_scan_ceil(cnt, nsg, nrows, kSegLen, wsum);
    if (valid) {
#pragma unroll
        for (int k = 0; k <= D; ++k) {
            sw[t * (D + 1) + k] = b[k];
            slist[cnt[q[k]] + pos[k]] = (uint16_t)((t << 5) | k);
        }
    }
    // segments in row order, and a histogram of their lengths (a row's last
    // segment counted with its others)
    for (int r = t; r < nrows; r += T) {
        const int e0 = cnt[r], e1 = (r + 1 < nrows) ? cnt[r + 1] : nc;
        const int ns = (e1 - e0 + kSegLen - 1) / kSegLen, len = (e1 - e0 + ns - 1) / ns;
        sfirst[r] = (uint16_t)nsg[r];
        for (int j = 0, e = e0; j < ns; ++j, e += len)
            seg[nsg[r] + j] = seg_encode(e, min(len, e1 - e), r);
        atomicAdd(&hist[kSegLen - len], ns);  // longest first
    }
    __syncthreads();
    for (int e = t; e < nc; e += T) {
        const int pk = slist[e];
        weight[e] = sw[(pk >> 5) * (D + 1) + (pk & 31)];
        point[e] = (uint16_t)pk;
    }
    if (t < 64) {
        // bucket starts (then used as cursors): an exclusive scan of the
        // histogram by the first wave, each lane over NBL consecutive buckets
        constexpr int NB = kSegLen + 1, NBL = (NB + 63) / 64;
        int v[NBL], sum = 0;
#pragma unroll
        for (int u = 0; u < NBL; ++u) {
            const int b = t * NBL + u;
            v[u] = b < NB ? hist[b] : 0;
            sum += v[u];
        }
        int incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(incl, off);
            if (t >= off)
                incl += y;
        }
        int first = incl - sum;
#pragma unroll
        for (int u = 0; u < NBL; ++u) {
            const int b = t * NBL + u;
            if (b < NB)
                hist[b] = first;
            first += v[u];
        }
    }
    if (t == 0) {
        sfirst[nrows] = (uint16_t)nseg;
        hdr[0] = (uint32_t)nrows;
        hdr[1] = 0;
        hdr[2] = (uint32_t)nc;
        hdr[3] = (uint32_t)nseg;
    }
    __syncthreads();
    // work order: rows of longest segments first, a row's segments together
    for (int r = t; r < nrows; r += T) {
        const int e0 = cnt[r], e1 = (r + 1 < nrows) ? cnt[r + 1] : nc;
        const int ns = (e1 - e0 + kSegLen - 1) / kSegLen, len = (e1 - e0 + ns - 1) / ns;
        const int at = atomicAdd(&hist[kSegLen - len], ns);
        for (int j = 0, e = e0; j < ns; ++j, e += len) {
            order[at + j] = (uint16_t)(nsg[r] + j);
            wseg[at + j] = seg_encode(e, min(len, e1 - e), r);
        }
    }
}

// The build's last launch, with three kinds of blocks:
// * tiles, resolve_waves(D) waves each (one up to d = 8, whose tiles have at
//   most a few hundred rows; four above, where a tile has thousands and one
//   wave's trips became the launch's tail: 40x36x28 points, d = 12, launch
//   181 us with one wave per tile): the slot of each row's key becomes its
//   vertex id (kResolveRows rows per lane requested together: slots, then
//   ids);
// * the neighbour table, one vertex of one direction per thread and trip;
// * clears: the first M * zld floats of z0 and z1 (the lattice buffers the
//   next filter calls splat into, zcap floats each, so that those calls
//   need no clearing launch of their own), the bucket table, and the
//   control block's counters, for the next build's insert.
// Reads the outcome the compaction published; does nothing when the build
// failed or its vertices do not fit vcap (the buffers of vkeys and nbr).
constexpr int kResolveRows = 4;
static_assert(kBlock == kGridBlock, "the neighbour blocks' arithmetic");
__host__ __device__ constexpr int resolve_waves(int d) { return d <= 8 ? 1 : 4; }

template <int D>
__global__ __launch_bounds__(kBlock) void k_resolve(int64_t n, Ctl *ctl, const Slot *__restrict__ table,
                                                    uint64_t mask, uint8_t *__restrict__ tiles,
                                                    const uint64_t *__restrict__ vkeys, uint32_t vcap,
                                                    int32_t *__restrict__ nbr, unsigned tile_blocks,
                                                    unsigned nbr_blocks, float *__restrict__ z0,
                                                    float *__restrict__ z1, int32_t zld, int64_t zcap,
                                                    uint64_t *__restrict__ bkeys, int32_t *__restrict__ bcount,
                                                    uint64_t bcap)
{
    constexpr int T = tile_points(D);
    const uint32_t M = ctl->result.count;
    if (ctl->result.flags || M > vcap)
        return;
    const KeyLayout lay = ctl->lay;
    if (blockIdx.x < tile_blocks) {
        const TileRec rec(D);
        const int lane = threadIdx.x & 63;
        constexpr int W = resolve_waves(D);
        const int64_t wave = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
        const int64_t tile = wave / W;
        const int part = (int)(wave % W) * 64 + lane;
        if (tile * T >= n)
            return;
        uint8_t *R = tiles + (size_t)tile * rec.bytes;
        const uint32_t *hdr = reinterpret_cast<const uint32_t *>(R);
        int32_t *rowid = reinterpret_cast<int32_t *>(R + rec.rowid);
        const uint64_t *rowkey = reinterpret_cast<const uint64_t *>(R + rec.rowkey);
        const int nrows = (int)hdr[0];
        constexpr int J = kResolveRows;
        for (int r0 = part; r0 < nrows; r0 += 64 * W * J) {
            int32_t hs[J], ids[J];
#pragma unroll
            for (int j = 0; j < J; ++j)
                hs[j] = r0 + j * 64 * W < nrows ? rowid[r0 + j * 64 * W] : 0;
#pragma unroll
            for (int j = 0; j < J; ++j)
                ids[j] = hs[j] >= 0 ? table[hs[j]].id : 0;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int r = r0 + j * 64 * W;
                if (r < nrows)
                    rowid[r] = hs[j] >= 0 ? ids[j] : max(probe_id(table, mask, rowkey[r]), 0);
            }
        }
        return;
    }
    const unsigned b = blockIdx.x - tile_blocks;
    if (b < nbr_blocks) {
        const unsigned per_dir = nbr_blocks / (D + 1);
        const int j = nbr_dir(b, per_dir);
        for (int64_t m = nbr_first(b, per_dir, (int)threadIdx.x); m < (int64_t)M; m += nbr_stride(per_dir))
            neighbour_item<D>(vkeys, M, lay, table, mask, nbr, j, m);
        return;
    }
    const uint64_t first = (uint64_t)(b - nbr_blocks) * kBlock + threadIdx.x;
    const uint64_t stride = (uint64_t)(gridDim.x - tile_blocks - nbr_blocks) * kBlock;
    const int64_t zelems = (int64_t)M * zld;  // a multiple of 4
    if (zelems <= zcap) {
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        for (uint64_t e = first; (int64_t)(4 * e) < zelems; e += stride) {
            reinterpret_cast<float4 *>(z0)[e] = z;
            reinterpret_cast<float4 *>(z1)[e] = z;
        }
    }
    for (uint64_t e = first; 2 * e < bcap; e += stride) {  // bcap is a power of two >= 64
        reinterpret_cast<ulonglong2 *>(bkeys)[e] = make_ulonglong2(kEmptyKey, kEmptyKey);
        reinterpret_cast<int2 *>(bcount)[e] = make_int2(0, 0);
    }
    if (first == 0) {
        ctl->flags = 0;
        ctl->count = 0;
        ctl->nvert = 0;
        ctl->nbucket = 0;
        ctl->nsorted = 0;
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

static unsigned range_blocks(int64_t n)
{
    const unsigned grid = blocks_for(n);
    return grid > kRangeBlocks ? kRangeBlocks : (grid == 0 ? 1 : grid);
}

size_t tile_record_bytes_build(int d) { return TileRec(d).bytes; }

hipError_t launch_range(int d, const float *feat, int64_t n, const Elev &E, int32_t *part, uint64_t *bkeys,
                        int32_t *bcount, uint64_t bcap, hipStream_t s)
{
    PAM_DISPATCH_D(d, hipLaunchKernelGGL(k_range<D>, dim3(range_blocks(n)), dim3(kBlock), 0, s, feat, n, E, part,
                                         bkeys, bcount, bcap));
    return hipGetLastError();
}

hipError_t launch_layout(int d, int64_t n, int gbits, Ctl *ctl, const int32_t *part, hipStream_t s)
{
    PAM_DISPATCH_D(d, hipLaunchKernelGGL(k_layout<D>, dim3(1), dim3(kLayoutThreads), 0, s, ctl, part,
                                         (int)range_blocks(n), gbits));
    return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, float value, int64_t count, hipStream_t s)
{
    if (count <= 0)
        return hipSuccess;
    unsigned grid = blocks_for(count);
    grid = grid > 4096 ? 4096 : grid;
    hipLaunchKernelGGL(k_fill_f32, dim3(grid), dim3(kBlock), 0, s, p, value, count);
    return hipGetLastError();
}

hipError_t launch_insert(int d, const float *feat, int64_t n, const Elev &E, const Groups64 &grp, Ctl *ctl,
                         const KeyLayout *fixed, uint64_t *bkeys, int32_t *bcount, uint64_t bcap, int2 *place,
                         Slot *table, uint64_t cap, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    if (bcap < 64 || (bcap & (bcap - 1)) != 0 || bcap > ((uint64_t)1 << 31) || cap < 64 || (cap & (cap - 1)) != 0)
        return hipErrorInvalidValue;
    const uint64_t T = kInsertPoints;
    const uint64_t grid = ((uint64_t)n + T - 1) / T + table_clear_blocks(cap, kInsertPoints);
    const KeyLayout lay = fixed ? *fixed : KeyLayout{};
    const int use_fixed = fixed ? 1 : 0;
    PAM_DISPATCH_D(d, hipLaunchKernelGGL(k_insert<D>, dim3((unsigned)grid), dim3(kInsertPoints), 0, s, feat, n, E,
                                         grp, ctl, lay, use_fixed, bkeys, bcap - 1, bcount, place, table, cap));
    return hipGetLastError();
}

bool fixed_layout(int d, int gbits, KeyLayout *lay)
{
    if (d < 1 || d > kMaxD)
        return false;
    int kbits = 0;
    while ((1 << kbits) <= d)
        ++kbits;  // bits for 0..d
    const int bits = (63 - kbits - gbits) / d;
    if (bits < 6)
        return false;
    KeyLayout L{};
    int shift = kbits;
    for (int c = 0; c < d; ++c) {
        L.lo[c] = -(1 << (bits - 1));
        L.bits[c] = bits;
        L.shift[c] = shift;
        shift += bits;
    }
    L.kbits = kbits;
    L.gshift = shift;
    L.gbits = gbits;
    L.total_bits = shift + gbits;
    *lay = L;
    return true;
}

hipError_t launch_starts(int32_t *bcount, uint64_t bcap, Ctl *ctl, hipStream_t s)
{
    if (bcap >= kCompactWideCap) {  // as in launch_compact
        const uint64_t per_block = (uint64_t)kBlock * 16;
        hipLaunchKernelGGL(k_starts<16>, dim3((unsigned)((bcap + per_block - 1) / per_block)), dim3(kBlock), 0, s,
                           bcount, bcap, ctl);
    } else {
        const uint64_t per_block = (uint64_t)kBlock * 4;
        hipLaunchKernelGGL(k_starts<4>, dim3((unsigned)((bcap + per_block - 1) / per_block)), dim3(kBlock), 0, s,
                           bcount, bcap, ctl);
    }
    return hipGetLastError();
}

hipError_t launch_scatter(const int2 *place, const int32_t *start, int64_t n, const Ctl *ctl, int32_t *perm,
                          hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_scatter, dim3(blocks_for(n)), dim3(kBlock), 0, s, place, start, n, ctl, perm);
    return hipGetLastError();
}

hipError_t launch_sorted_tiles(int d, const float *feat, int64_t n, const Elev &E, const Groups64 &grp, Ctl *ctl,
                               const int32_t *perm, uint8_t *psort, Slot *table, uint64_t cap, uint8_t *tiles,
                               hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    if (cap < 64 || (cap & (cap - 1)) != 0)
        return hipErrorInvalidValue;
    const int T = tile_points(d);
    PAM_DISPATCH_D(d, hipLaunchKernelGGL(k_sorted_tiles<D>, dim3((unsigned)((n + T - 1) / T)), dim3(T), 0, s, feat, n,
                                         E, grp, ctl, perm, psort, table, cap - 1, tiles));
    return hipGetLastError();
}

hipError_t launch_compact(Slot *table, uint64_t *vkeys, uint32_t vcap, uint64_t cap,
                          Ctl *ctl, HostResult *result, uint32_t attempt, hipStream_t s)
{
    if (cap >= kCompactWideCap) {
        const uint64_t per_block = (uint64_t)kBlock * 16;
        hipLaunchKernelGGL(k_compact<16>, dim3((unsigned)((cap + per_block - 1) / per_block)), dim3(kBlock), 0, s,
                           table, vkeys, vcap, cap, ctl, result, attempt);
    } else {
        const uint64_t per_block = (uint64_t)kBlock * 4;
        hipLaunchKernelGGL(k_compact<4>, dim3((unsigned)((cap + per_block - 1) / per_block)), dim3(kBlock), 0, s,
                           table, vkeys, vcap, cap, ctl, result, attempt);
    }
    return hipGetLastError();
}

hipError_t launch_resolve(int d, int64_t n, Ctl *ctl, const Slot *table, uint64_t cap, uint8_t *tiles,
                          const uint64_t *vkeys, uint32_t vcap, int64_t M_estimate,
                          int32_t *nbr, float *z0, float *z1, int32_t zld, int64_t zcap, uint64_t *bkeys,
                          int32_t *bcount, uint64_t bcap, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    if (zld % 4 != 0 || (zcap > 0 && (!z0 || !z1)) || (bcap & (bcap - 1)) != 0)
        return hipErrorInvalidValue;
    const int64_t ntiles = (n + tile_points(d) - 1) / tile_points(d);
    const int64_t tile_blocks = (ntiles * resolve_waves(d) + kBlock / 64 - 1) / (kBlock / 64);
    // the item and clear loops stride over whatever their extents turn out
    // to be; the estimate only sizes the launch
    const int64_t nbr_blocks = (int64_t)nbr_blocks_per_dir(M_estimate) * (d + 1);
    const int64_t pieces = std::max<int64_t>(M_estimate * zld / 4, (int64_t)(bcap / 2));
    const int64_t clear_blocks = std::min<int64_t>((pieces + kBlock - 1) / kBlock, 4096);
    PAM_DISPATCH_D(d, hipLaunchKernelGGL(k_resolve<D>, dim3((unsigned)(tile_blocks + nbr_blocks + clear_blocks)),
                                         dim3(kBlock), 0, s, n, ctl, table, cap - 1, tiles, vkeys, vcap, nbr, (unsigned)tile_blocks, (unsigned)nbr_blocks, z0, z1,
                                         zld, zcap, bkeys, bcount, bcap));
    return hipGetLastError();
}

hipError_t launch_export_points(int d, const uint8_t *pts, const uint8_t *tiles, const int32_t *perm, int64_t n,
                                int32_t *vert, float *bary, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_export_points, dim3(blocks_for(n)), dim3(kBlock), 0, s, d, pts, tiles, perm, n, vert, bary);
    return hipGetLastError();
}

hipError_t launch_vertex_groups(const uint64_t *vkeys, int64_t M, const Ctl *ctl, int32_t *vgroup, hipStream_t s)
{
    if (M <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_vertex_groups, dim3(blocks_for(M)), dim3(kBlock), 0, s, vkeys, M, ctl, vgroup);
    return hipGetLastError();
}

hipError_t launch_unpack_keys(int d, const uint64_t *vkeys, int64_t M, const Ctl *ctl, int32_t *keys,
                              hipStream_t s)
{
    if (M <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_unpack_keys, dim3(blocks_for(M)), dim3(kBlock), 0, s, d, vkeys, M, ctl, keys);
    return hipGetLastError();
}

}  // namespace pam
