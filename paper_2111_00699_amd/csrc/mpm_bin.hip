// Rebuild-mapping and particle sorting on gfx950.
//
// Paper, "Material Point Method on a Single GPU": particle codes interleave
// the 3-D cell index with the block code in the high bits and the cell code
// in the low bits; the blocks holding particles (gblocks) and their 3x3x3
// neighbours (pblocks) are recorded; particles are sorted to cell
// granularity.  "Rebuild-Mapping": particle blocks are shifted by -dx/2 so a
// particle block with its 3x3x3 neighbours covers a (10 dx)^3 free zone.
//
// MI355X design: the block table is a dense array over the padded domain
// (288 GB of HBM make a dense (n/4+2)^3 table trivial), so no hash is needed
// and block activation is a mark + compaction, deterministic and in block
// order.  Sorting is a stable LSD radix sort with 8-bit digits, ranks taken
// inside each wave64 from eight ballots (no atomics), so the permutation is
// exactly a stable sort by particle code.  A batched context puts the scene's
// rank above the Morton bits, so one sort orders every scene, scene by
// scene, and every later list (blocks, chunks, physical blocks) comes out
// rank-major; the per-rank ends of those lists let a substep run a prefix of
// the ranks.
#include "mpm_internal.h"

namespace mpm {

namespace {

// Radix tiles: 4096 keys, or 2048 up to RS_DIRECT_TILES of those.  Few tiles
// leave most CUs idle, and the smaller ones halve the rounds of a tile; up to
// that count a scatter workgroup also adds up the tiles' histograms itself
// (one coalesced row of 256 counts per tile, all loads in flight) instead of
// reading them scanned, which saves the scan's two launches per pass.  With
// 143K particles a pass takes 14 us that way and 29 us with 4096-key tiles and
// the scan; with 1M the rows would be 512, read by 512 workgroups.
constexpr int RS_LARGE = 16, RS_SMALL = 8;  // keys per thread
constexpr int RS_DIRECT_TILES = 128;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = WG * SCAN_ITEMS;  // 2048 entries per scan tile

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ int wave_incl_scan(int v) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(v, d, 64);
        if (lane_id() >= d) v += t;
    }
    return v;
}

// Exclusive scan over the 256 threads of a workgroup; *total gets the sum.
__device__ __forceinline__ int block_excl_scan(int v, int* total) {
    __shared__ int wsum[WG / 64];
    const int w = threadIdx.x >> 6;
    const int inc = wave_incl_scan(v);
    if (lane_id() == 63) wsum[w] = inc;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < WG / 64; ++i) {
        off += (i < w) ? wsum[i] : 0;
        tot += wsum[i];
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// ------------------------------------------------------------ particle code
// c = floor(x/dx + 1/2) = floor(x n - 1/2) + 1 per axis.  For power-of-two
// n, x*n is exact in FP32 and x*n - 1/2 is exact wherever it matters, so the
// code is bit-identical to one computed in FP64 from the same FP32 x.  The
// scene's rank goes above the Morton bits.
// A workgroup takes one radix tile and also counts the digits of the first pass.
template <int ITEMS, bool DIRECT>
__global__ __launch_bounds__(WG) void k_keys(const float* __restrict__ S, int64_t cap, int N, Scenes T,
                                             uint32_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                             int* __restrict__ ctl, int tiles, int* __restrict__ hist) {
    __shared__ int h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int first = blockIdx.x * (WG * ITEMS) + threadIdx.x;
    float id[ITEMS], x[ITEMS][3];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int j = min(first + r * WG, N - 1);
        id[r] = S[sidx(FSID, j, cap)];
#pragma unroll
        for (int a = 0; a < 3; ++a) x[r][a] = S[sidx(FX + a, j, cap)];
    }
    unsigned err = 0;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int j = first + r * WG;
        if (j >= N) break;
        const Scene& sc = T.scene[T.S == 1 ? 0 : fsid_scene(id[r])];
        const float fn = sc.P.fn;
        const int n = sc.P.n;
        uint32_t code = (uint32_t)sc.rank << T.shift;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float b = floorf(x[r][a] * fn - 0.5f);
            int c;
            if (!(b == b)) {
                err |= MPM_ERR_NONFINITE;
                c = 0;
            } else {
                if (!(b >= 0.0f && b <= (float)(n - 2))) err |= MPM_ERR_DOMAIN;
                c = (int)fminf(fmaxf(b + 1.0f, 0.0f), (float)(n - 1));
            }
            code |= spread3((uint32_t)c) << a;
        }
        keys[j] = code;
        vals[j] = (uint32_t)j;
        atomicAdd(&h[code & 255u], 1);
    }
    if (err) atomicOr(&ctl[CTL_ERROR], (int)err);
    __syncthreads();
    hist[DIRECT ? blockIdx.x * 256 + threadIdx.x : threadIdx.x * tiles + blockIdx.x] = h[threadIdx.x];
}

// --------------------------------------------------------------- radix sort
// Digit counts of each tile: DIRECT [tile][digit], else [digit][tile] (for the scan).
template <int ITEMS, bool DIRECT>
__global__ __launch_bounds__(WG) void k_rs_hist(const uint32_t* __restrict__ keys, int N, int shift, int tiles,
                                                int* __restrict__ hist) {
    __shared__ int h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int base = blockIdx.x * (WG * ITEMS);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = base + r * WG + threadIdx.x;
        if (i < N) atomicAdd(&h[(keys[i] >> shift) & 255u], 1);
    }
    __syncthreads();
    hist[DIRECT ? blockIdx.x * 256 + threadIdx.x : threadIdx.x * tiles + blockIdx.x] = h[threadIdx.x];
}

// Stable scatter: keys of the tile are taken in order, 256 at a time; inside
// a wave the rank among lanes with the same digit comes from eight ballots,
// across the four waves from per-wave digit counts in LDS.  The tile's keys
// are loaded before the first round (a load per round made the kernel wait
// for memory 16 times).  offs: the scanned histogram, or (DIRECT) the plain one.
template <int ITEMS, bool DIRECT>
__global__ __launch_bounds__(WG) void k_rs_scatter(const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                                   uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, int N,
                                                   int shift, int tiles, const int* __restrict__ offs) {
    __shared__ int base[256];
    __shared__ int wcnt[WG / 64][256];
    const int tid = threadIdx.x, w = tid >> 6, lane = lane_id();
    const int first = blockIdx.x * (WG * ITEMS) + tid;
    uint32_t key[ITEMS], val[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = min(first + r * WG, N - 1);
        key[r] = kin[i];
        val[r] = vin[i];
    }
    if constexpr (DIRECT) {
        int all = 0, before = 0;
#pragma unroll 16
        for (int t = 0; t < tiles; ++t) {
            const int v = offs[t * 256 + tid];
            all += v;
            before += t < (int)blockIdx.x ? v : 0;
        }
        int total;
        base[tid] = block_excl_scan(all, &total) + before;
    } else {
        base[tid] = offs[tid * tiles + blockIdx.x];
    }
#pragma unroll
    for (int i = 0; i < WG / 64; ++i) wcnt[i][tid] = 0;
    __syncthreads();
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool valid = first + r * WG < N;
        const uint32_t d = (key[r] >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const int rank = __popcll(peers & below);
        if (valid && rank == 0) wcnt[w][d] = __popcll(peers);
        __syncthreads();
        if (valid) {
            int off = base[d] + rank;
#pragma unroll
            for (int k = 0; k < WG / 64; ++k) off += (k < w) ? wcnt[k][d] : 0;
            kout[off] = key[r];
            vout[off] = val[r];
        }
        __syncthreads();
        int add = 0;
#pragma unroll
        for (int k = 0; k < WG / 64; ++k) {
            add += wcnt[k][tid];
            wcnt[k][tid] = 0;
        }
        base[tid] += add;
        __syncthreads();
    }
}

// --------------------------------------------------------- generic scan
// Per-tile totals, then a per-tile exclusive scan that hands each element its
// output offset.  Up to SCAN_DIRECT_TILES tiles a workgroup of the second adds
// up the totals of the tiles before its own (read coalesced), which saves a
// launch; those reads grow with the square of the tiles, so above that a launch
// between the two scans the totals first (SCANNED).  The particles' block scan
// that way and the other: 59.6 and 61.0 us at 12M particles (5.9K tiles), 80.5
// and 79.8 at 16.7M, 970 and 531 at 130M; a rebuild of 500M takes 76.3 and 67.9
// ms.
// op.limit(n): entries from there on count nothing (workgroups past it leave at
// once).
constexpr int SCAN_DIRECT_TILES = 8192;
template <int ITEMS, class Op>
__global__ __launch_bounds__(WG) void k_scan_count(Op op, int n, int* __restrict__ tile_sums) {
    const int first = blockIdx.x * (WG * ITEMS) + threadIdx.x * ITEMS;
    n = op.limit(n);
    if ((int)blockIdx.x * (WG * ITEMS) >= n) return;
    int s = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (first + i < n) s += op.count(first + i);
    int tot;
    block_excl_scan(s, &tot);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

// Sum of a[0 .. n) over the workgroup's threads.
__device__ __forceinline__ int block_sum(const int* __restrict__ a, int n) {
    int s = 0;
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += WG) s += a[i];
    int tot;
    block_excl_scan(s, &tot);
    return tot;
}

// a[0 .. n) to its exclusive sums, in place, by one workgroup.
__device__ __forceinline__ void scan_in_place(int* __restrict__ a, int n) {
    constexpr int PER = 8;
    int carry = 0;
    for (int base = 0; base < n; base += WG * PER) {
        const int first = base + threadIdx.x * PER;
        int v[PER], s = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            v[i] = first + i < n ? a[first + i] : 0;
            s += v[i];
        }
        int tot;
        int off = carry + block_excl_scan(s, &tot);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (first + i < n) a[first + i] = off;
            off += v[i];
        }
        carry += tot;
    }
}

template <int ITEMS, class Op>
__global__ __launch_bounds__(WG) void k_scan_top(Op op, int n, int* __restrict__ tile_sums) {
    scan_in_place(tile_sums, (op.limit(n) + WG * ITEMS - 1) / (WG * ITEMS));
}

template <int ITEMS, bool SCANNED, class Op>
__global__ __launch_bounds__(WG) void k_scan_emit(Op op, int n, const int* __restrict__ tile_sums,
                                                  int* __restrict__ total) {
    const int first = blockIdx.x * (WG * ITEMS) + threadIdx.x * ITEMS;
    n = op.limit(n);
    const int last = n > 0 ? (n - 1) / (WG * ITEMS) : 0;  // the workgroup that ends the scan
    if ((int)blockIdx.x > last) return;
    int c[ITEMS];
    int s = 0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        c[i] = (first + i < n) ? op.count(first + i) : 0;
        s += c[i];
    }
    const int before = SCANNED ? (n > 0 ? tile_sums[blockIdx.x] : 0) : block_sum(tile_sums, blockIdx.x);
    int tot;
    int off = before + block_excl_scan(s, &tot);
    if ((int)blockIdx.x == last && threadIdx.x == 0) *total = before + tot;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (c[i] > 0) op.emit(first + i, off, c[i]);
        off += c[i];
    }
}

template <int ITEMS = SCAN_ITEMS, class Op>
void device_scan(hipStream_t st, const Op& op, int n, int* tile_sums, int* total) {
    const int tiles = cdiv(n > 0 ? n : 1, WG * ITEMS);
    hipLaunchKernelGGL((k_scan_count<ITEMS, Op>), dim3(tiles), dim3(WG), 0, st, op, n, tile_sums);
    if (tiles > SCAN_DIRECT_TILES) {
        hipLaunchKernelGGL((k_scan_top<ITEMS, Op>), dim3(1), dim3(WG), 0, st, op, n, tile_sums);
        hipLaunchKernelGGL((k_scan_emit<ITEMS, true, Op>), dim3(tiles), dim3(WG), 0, st, op, n, tile_sums, total);
    } else {
        hipLaunchKernelGGL((k_scan_emit<ITEMS, false, Op>), dim3(tiles), dim3(WG), 0, st, op, n, tile_sums, total);
    }
}

struct OpHistScan {  // exclusive scan of the radix histogram in place
    int* h;
    __device__ int limit(int n) const { return n; }
    __device__ int count(int i) const { return h[i]; }
    __device__ void emit(int i, int off, int) const { h[i] = off; }
};

// Geometric blocks: positions where the block code (code >> 6) changes, and
// merge groups: runs of geometric blocks of one 2x2x1 slab of blocks (equal
// code >> 8; the rank bits make groups never cross scenes; without `pack`
// every block is a group of its own).  Both in one scan over the sorted codes.
__device__ __forceinline__ void block_heads(const uint32_t* keys, int j, int N, int pack, int& gb, int& gr) {
    gb = gr = 0;
    if (j >= N) return;
    const uint32_t k = keys[j], p = j > 0 ? keys[j - 1] : ~k;
    gb = (k >> 6) != (p >> 6) || j == 0 ? 1 : 0;
    gr = pack ? ((k >> 8) != (p >> 8) || j == 0 ? 1 : 0) : gb;
}

__global__ __launch_bounds__(WG) void k_blocks_count(const uint32_t* __restrict__ keys, int N, int pack, int tiles,
                                                     int* __restrict__ sums) {
    const int first = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
    int s0 = 0, s1 = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        int gb, gr;
        block_heads(keys, first + i, N, pack, gb, gr);
        s0 += gb;
        s1 += gr;
    }
    int t0, t1;
    block_excl_scan(s0, &t0);
    block_excl_scan(s1, &t1);
    if (threadIdx.x == 0) {
        sums[blockIdx.x] = t0;
        sums[tiles + blockIdx.x] = t1;
    }
}

// (a workgroup for the blocks' totals, one for the groups')
__global__ __launch_bounds__(WG) void k_blocks_top(int tiles, int* __restrict__ sums) {
    scan_in_place(sums + (int64_t)blockIdx.x * tiles, tiles);
}

template <bool SCANNED>
__global__ __launch_bounds__(WG) void k_blocks_emit(const uint32_t* __restrict__ keys, int N, int pack, int tiles,
                                                    const int* __restrict__ sums, int* __restrict__ gstart,
                                                    uint32_t* __restrict__ gcode, int* __restrict__ group_start,
                                                    int* __restrict__ ctl) {
    const int first = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
    int gb[SCAN_ITEMS], gr[SCAN_ITEMS], s0 = 0, s1 = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        block_heads(keys, first + i, N, pack, gb[i], gr[i]);
        s0 += gb[i];
        s1 += gr[i];
    }
    const int b0 = SCANNED ? sums[blockIdx.x] : block_sum(sums, blockIdx.x);
    const int b1 = SCANNED ? sums[tiles + blockIdx.x] : block_sum(sums + tiles, blockIdx.x);
    int t0, t1;
    int o0 = b0 + block_excl_scan(s0, &t0), o1 = b1 + block_excl_scan(s1, &t1);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        ctl[CTL_NGB] = b0 + t0;
        ctl[CTL_NGROUP] = b1 + t1;
    }
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        if (gb[i]) {
            gstart[o0] = first + i;
            gcode[o0] = keys[first + i] >> 6;
        }
        if (gr[i]) group_start[o1] = o0;
        o0 += gb[i];
        o1 += gr[i];
    }
}

// Work chunks, per merge group: consecutive blocks are packed into one chunk
// while the total stays within `chunk` particles; a block larger than that
// is cut into runs of `chunk`.  (Sparse regions then still fill the
// workgroups; a chunk's tile box stays within a 2x2x1 slab of blocks.)
// One group per thread: the walk over a group's blocks is a chain of
// dependent loads, which a thread with eight groups walked eight times (46 us
// at 143K particles; 4 us so).
struct OpChunks {
    const int* gstart;
    const uint32_t* gcode;
    const int* group_start;
    const int* ctl;
    int N, chunk;
    Chunk* out;
    Scenes T;
    // walk the group's blocks, calling put(start, count) for each chunk
    template <class Put>
    __device__ int walk(int s, Put put) const {
        const int ngb = ctl[CTL_NGB], g0 = group_start[s];
        const int g1 = s + 1 < ctl[CTL_NGROUP] ? group_start[s + 1] : ngb;
        int st[5];  // a group has at most four blocks: their starts and the end
#pragma unroll
        for (int i = 0; i < 5; ++i) st[i] = g0 + i < ngb ? gstart[g0 + i] : N;
        int k = 0, run0 = 0, runn = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (g0 + i >= g1) break;
            const int l = st[i + 1] - st[i];
            if (l > chunk) {
                if (runn) put(k++, run0, runn);
                runn = 0;
                for (int j = 0; j < l; j += chunk) put(k++, st[i] + j, min(chunk, l - j));
            } else {
                if (runn && runn + l > chunk) {
                    put(k++, run0, runn);
                    runn = 0;
                }
                if (!runn) run0 = st[i];
                runn += l;
            }
        }
        if (runn) put(k++, run0, runn);
        return k;
    }
    __device__ int limit(int n) const { return min(n, ctl[CTL_NGROUP]); }
    __device__ int count(int s) const {
        return walk(s, [](int, int, int) {});
    }
    __device__ void emit(int s, int off, int) const {
        const int scene = T.rank_scene[gcode[group_start[s]] >> (T.shift - 6)];  // a group is of one scene
        walk(s, [&](int k, int start, int n) {
            Chunk c;
            c.start = start;
            c.count = n;
            c.tile = 1;
            c.scene = scene;
            out[off + k] = c;
        });
    }
};

// Physical blocks in padded linear order; a block's state then names its
// position in the active list (3 + i), under which the rebuild lists the
// chunks whose tiles can reach it.
struct OpActive {
    int* state;
    int* active;
    __device__ int limit(int n) const { return n; }
    __device__ int count(int b) const { return state[b] != 0 ? 1 : 0; }
    __device__ void emit(int b, int off, int) const {
        active[off] = b;
        state[b] = 3 + off;
    }
};

// ------------------------------------------------------------ data movement
// Slot of rank r when a chunk's `count` particles are dealt over its 16-lane
// passes (pass k = slots 16k .. 16k+15; the last pass holds the remainder):
// rank r goes to place q = r / P of pass r mod P in the order 0, 2, 4, ...,
// 1, 3, 5, ... (P passes; places of the short last pass run out first), so
// consecutive ranks land in different passes, mostly two passes (32 lanes)
// apart.
__device__ __forceinline__ int dealt_slot(int count, int r) {
    const int P = (count + 15) >> 4, last = count - 16 * (P - 1), E = (P + 1) >> 1;
    int q, i, evens = E;
    if (r < last * P) {
        q = r / P;
        i = r - q * P;
    } else {
        const int r2 = r - last * P, Pm = P - 1;
        q = last + r2 / Pm;
        i = r2 - (q - last) * Pm;
        if (P & 1) evens = E - 1;  // the last pass is the last even one: drop it
    }
    const int pass = i < evens ? 2 * i : 2 * (i - evens) + 1;
    return pass * 16 + q;
}

// Gather the whole particle state into sorted order, one chunk per
// workgroup.  A chunk holds one to four blocks (segments of its sorted run).
// Unless `spread` is 0 (plain sorted order), the chunk's particles are
// ranked by the LDS bank pair of their cell in the P2G tile -- (x + 12 y +
// 8 z) mod 16 for cell (x, y, z), the tile's layout with a row pitch of 12
// (mod 16) and a plane pitch of 8 (mod 16) -- then by cell, and dealt over
// the 16-lane passes of the P2G scatter: a pass then meets each bank pair
// about as often as the chunk's cells allow, and particles of one cell sit in
// different passes.  Each particle's field FSID gets its block (its free
// zone).  Also records the insertion ids in plain sorted order for the
// binning view.
constexpr int PERMUTE_MAX = 512;  // the largest chunk
__global__ __launch_bounds__(WG) void k_permute_chunks(const float* __restrict__ Sin, float* __restrict__ Sout,
                                                       const int* __restrict__ idin, int* __restrict__ idout,
                                                       int* __restrict__ sorted_ids, const uint32_t* __restrict__ src,
                                                       const uint32_t* __restrict__ keys,
                                                       const Chunk* __restrict__ chunks, const int* __restrict__ ctl,
                                                       int64_t cap, int spread, int shift) {
    constexpr int NRK = 4096;  // ranking keys: 4-bit bank pair, 8-bit segment and cell
    __shared__ int rk[PERMUTE_MAX];
    __shared__ int below[NRK];  // per ranking key: how many of the chunk's particles rank lower
    const int nch = ctl[CTL_NCHUNK];
    const uint32_t mmask = (1u << shift) - 1u;
    int begin, end, stride;
    xcd_split(nch, begin, end, stride);
    for (int c = begin; c < end; c += stride) {
        const Chunk ch = chunks[c];
        const bool deal = spread && ch.count <= PERMUTE_MAX;  // workgroup-uniform
        // this thread's particle (the first pass) is loaded while the chunk is ranked
        float q[NF];
        int id = 0;
        auto load = [&](int t) {
            const int k = (int)src[ch.start + t];  // its position before the sort
#pragma unroll
            for (int f = 0; f < NF; ++f) q[f] = Sin[sidx(f, k, cap)];
            id = idin[k];
        };
        if ((int)threadIdx.x < ch.count) load(threadIdx.x);
        if (deal) {
            // a counting sort of the ranking keys: histogram, then its exclusive prefix sums
            for (int t = threadIdx.x; t < NRK; t += WG) below[t] = 0;
            __syncthreads();
            for (int t = threadIdx.x; t < ch.count; t += WG) {
                const uint32_t key = keys[ch.start + t] & mmask;
                const uint32_t bcode = key >> 6, cell = key & 63u;
                const int x = 4 * (int)compact3(bcode) + (int)compact3(cell);
                const int y = 4 * (int)compact3(bcode >> 1) + (int)compact3(cell >> 1);
                const int z = 4 * (int)compact3(bcode >> 2) + (int)compact3(cell >> 2);
                rk[t] = (((x + 12 * y + 8 * z) & 15) << 8) | (int)(key & 255u);  // bank, segment, cell
                atomicAdd(&below[rk[t]], 1);
            }
            __syncthreads();
            constexpr int PER = NRK / WG;
            int h[PER], sum = 0;
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                h[k] = below[threadIdx.x * PER + k];
                sum += h[k];
            }
            int total;
            int run = block_excl_scan(sum, &total);
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                below[threadIdx.x * PER + k] = run;
                run += h[k];
            }
            __syncthreads();
        }
        auto place = [&](int t) {  // the slot of sorted position t, and its free-zone block into q
            const uint32_t bcode = (keys[ch.start + t] & mmask) >> 6;
            q[FSID] = __int_as_float(fsid_scene(q[FSID]) | (int)(compact3(bcode) << 8) |
                                     (int)(compact3(bcode >> 1) << 16) | (int)(compact3(bcode >> 2) << 24));
            sorted_ids[ch.start + t] = id;
            if (!deal) return t;
            // rank = the particles with a lower ranking key + those before it with the same one.
            // Within a chunk (blocks of one 2x2x1 slab) the segment and cell bits identify the
            // particle code, so equal ranking keys are a run of equal codes, consecutive in
            // sorted order.
            const int mine = rk[t];
            int first = t;
            while (first > 0 && rk[first - 1] == mine) --first;
            return dealt_slot(ch.count, below[mine] + (t - first));
        };
        if (deal && ch.count <= WG) {
            // through LDS, 16 fields a round, so that a wave stores runs: dealt slots scatter its 64 lanes
            // over the chunk, four times the requests (298 -> 262 us at 3.1M particles, 20.3 -> 17.1 at 143K)
            const int t = threadIdx.x;
            const bool have = t < ch.count;
            const int slot = have ? place(t) : 0;
            float* row = reinterpret_cast<float*>(below);
            constexpr int FIELDS = NRK / WG;  // fields a round
#pragma unroll
            for (int f0 = 0; f0 <= NF; f0 += FIELDS) {  // (field NF: the insertion id)
                __syncthreads();
                if (have) {
#pragma unroll
                    for (int f = f0; f < f0 + FIELDS && f <= NF; ++f)
                        row[(f - f0) * WG + slot] = f < NF ? q[f] : __int_as_float(id);
                }
                __syncthreads();
                if (have) {
#pragma unroll
                    for (int f = f0; f < f0 + FIELDS && f <= NF; ++f) {
                        const float v = row[(f - f0) * WG + t];
                        if (f < NF)
                            Sout[sidx(f, ch.start + t, cap)] = v;
                        else
                            idout[ch.start + t] = __float_as_int(v);
                    }
                }
            }
            __syncthreads();
            continue;
        }
        for (int t = threadIdx.x; t < ch.count; t += WG) {
            if (t >= WG) load(t);
            const int dst = ch.start + place(t);
#pragma unroll
            for (int f = 0; f < NF; ++f) Sout[sidx(f, dst, cap)] = q[f];
            idout[dst] = id;
        }
        if (deal) __syncthreads();
    }
}

__global__ __launch_bounds__(WG) void k_copy_codes(uint32_t* __restrict__ dst, const uint32_t* __restrict__ src,
                                                   int n, uint32_t mask) {
    const int i = blockIdx.x * WG + threadIdx.x;
    if (i < n) dst[i] = src[i] & mask;
}

__global__ __launch_bounds__(WG) void k_clear2(int* __restrict__ p, int* __restrict__ q, int n) {
    const int i = blockIdx.x * WG + threadIdx.x;
    if (i < n) p[i] = q[i] = 0;
}

// Mark the 3x3x3 neighbourhood of every geometric block as physical, in
// the block grid of the block's scene.
__global__ __launch_bounds__(WG) void k_dilate(const uint32_t* __restrict__ gcode, const int* __restrict__ ctl,
                                               Scenes T, int* __restrict__ state) {
    const int total = ctl[CTL_NGB] * 27;
    const int bshift = T.shift - 6;
    for (int t = blockIdx.x * WG + threadIdx.x; t < total; t += gridDim.x * WG) {
        const int g = t / 27, o = t % 27;
        const uint32_t code = gcode[g] & ((1u << bshift) - 1u);
        const Scene& sc = T.scene[T.rank_scene[gcode[g] >> bshift]];
        const int NB = sc.P.NB;
        const int B0 = (int)compact3(code), B1 = (int)compact3(code >> 1), B2 = (int)compact3(code >> 2);
        const int bx = B0 + (o % 3);  // (B - 1) + o + 1 in padded coordinates
        const int by = B1 + (o / 3) % 3;
        const int bz = B2 + o / 9;
        state[sc.brick_base + (bz * NB + by) * NB + bx] = 1;
    }
}

// Per-rank ends of the sorted particles, geometric blocks, chunks and
// physical blocks (binary searches over the rank-major lists, one per thread;
// the last rank ends where its list does).  The rebuild also starts the
// overflow lists and fallback counts afresh.
__global__ __launch_bounds__(WG) void k_rank_ends(const uint32_t* __restrict__ keys, int N,
                                                  const uint32_t* __restrict__ gcode, const Chunk* __restrict__ chunks,
                                                  const int* __restrict__ active, int* __restrict__ ctl, Scenes T) {
    if (threadIdx.x == 0) {
        ctl[CTL_REBUILD] = 0;
        ctl[CTL_OVF] = ctl[CTL_OVF + 1] = 0;
        ctl[CTL_FB] = ctl[CTL_FB + 1] = 0;
    }
    for (int t = threadIdx.x; t < 4 * T.S; t += WG) {
        const int kind = t / T.S, r = t - kind * T.S;
        const int n = kind == RE_PART ? N : ctl[kind == RE_GBLOCK ? CTL_NGB : kind == RE_CHUNK ? CTL_NCHUNK : CTL_NACTIVE];
        int lo = 0, hi = n;
        if (r == T.S - 1) lo = n;
        while (lo < hi) {  // first index whose rank exceeds r
            const int mid = (lo + hi) >> 1;
            const int rank = kind == RE_PART     ? (int)(keys[mid] >> T.shift)
                             : kind == RE_GBLOCK ? (int)(gcode[mid] >> (T.shift - 6))
                             : kind == RE_CHUNK  ? T.scene[chunks[mid].scene].rank
                                                 : (active[mid] >= T.rank_brick[r + 1] ? r + 1 : r);
            if (rank <= r)
                lo = mid + 1;
            else
                hi = mid;
        }
        T.rank_end[t] = lo;
    }
}

// Tile registrations, one wave per chunk: the chunk's particle blocks (the
// blocks of its sorted range, at most the four of one 2x2x1 slab) reach
// padded blocks B .. B+2 per axis with in-zone stencils; the chunk is listed
// with each physical block of that region.  A full list clears the chunk's
// `tile` flag.
__global__ __launch_bounds__(WG) void k_register(Chunk* __restrict__ chunks, const uint32_t* __restrict__ keys,
                                                 const int* __restrict__ ctl, const int* __restrict__ state,
                                                 int* __restrict__ reg_n, int* __restrict__ reg, Scenes T) {
    const int nch = ctl[CTL_NCHUNK];
    const int lane = threadIdx.x & 63;
    const uint32_t mmask = (1u << T.shift) - 1u;
    for (int c = blockIdx.x * (WG / 64) + (threadIdx.x >> 6); c < nch; c += gridDim.x * (WG / 64)) {
        const Chunk ch = chunks[c];
        const Scene& sc = T.scene[ch.scene];
        const int NB = sc.P.NB;
        const uint32_t b0 = (keys[ch.start] & mmask) >> 6, b1 = (keys[ch.start + ch.count - 1] & mmask) >> 6;
        int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {INT_MIN, INT_MIN, INT_MIN};
        for (uint32_t b = b0; b <= b1; ++b) {  // Morton codes of one slab: at most four
            const int q[3] = {(int)compact3(b), (int)compact3(b >> 1), (int)compact3(b >> 2)};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                lo[a] = min(lo[a], q[a]);
                hi[a] = max(hi[a], q[a] + 2);
            }
        }
        const int n0 = hi[0] - lo[0] + 1, n1 = hi[1] - lo[1] + 1, n2 = hi[2] - lo[2] + 1;
        bool fail = false;
        for (int k = lane; k < n0 * n1 * n2; k += 64) {
            const int bx = lo[0] + k % n0, by = lo[1] + (k / n0) % n1, bz = lo[2] + k / (n0 * n1);
            const int s = state[sc.brick_base + (bz * NB + by) * NB + bx];
            if (s >= 3) {
                const int slot = atomicAdd(&reg_n[s - 3], 1);
                if (slot < REG_MAX)
                    reg[(int64_t)(s - 3) * REG_MAX + slot] = c;
                else
                    fail = true;
            }
        }
        if (__ballot(fail) != 0ull && lane == 0) chunks[c].tile = 0;
    }
}

// Each physical block's registration list in ascending chunk order (one wave
// per block; a lane's rank is the count of smaller entries), so the grid
// update sums the tiles in a fixed order.
__global__ __launch_bounds__(WG) void k_sort_registrations(const int* __restrict__ ctl, const int* __restrict__ reg_n,
                                                           int* __restrict__ reg) {
    __shared__ int buf[WG / 64][REG_MAX];
    const int nact = ctl[CTL_NACTIVE];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int i = blockIdx.x * (WG / 64) + wv; i < nact; i += gridDim.x * (WG / 64)) {
        const int m = min(__builtin_amdgcn_readfirstlane(reg_n[i]), REG_MAX);
        int* list = reg + (int64_t)i * REG_MAX;
        for (int k = lane; k < m; k += 64) buf[wv][k] = list[k];
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        int v[REG_MAX / 64], r[REG_MAX / 64];
#pragma unroll
        for (int u = 0; u < REG_MAX / 64; ++u) {
            const int k = lane + 64 * u;
            v[u] = k < m ? buf[wv][k] : 0;
            r[u] = 0;
        }
        for (int j = 0; j < m; ++j) {  // entries are distinct chunk indices
            const int e = buf[wv][j];
#pragma unroll
            for (int u = 0; u < REG_MAX / 64; ++u) r[u] += e < v[u] ? 1 : 0;
        }
#pragma unroll
        for (int u = 0; u < REG_MAX / 64; ++u)
            if (lane + 64 * u < m) list[r[u]] = v[u];
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

}  // namespace

// The overflow-block and tile-fallback counts of both substep parities
// cleared between substeps, as a rebuild leaves them (a graph frame without
// a rebuild starts with this).
__global__ void k_clear_overflow(int* ctl) {
    ctl[CTL_OVF] = ctl[CTL_OVF + 1] = 0;
    ctl[CTL_FB] = ctl[CTL_FB + 1] = 0;
}

void enqueue_clear_overflow(hipStream_t st, int* ctl) {
    hipLaunchKernelGGL(k_clear_overflow, dim3(1), dim3(1), 0, st, ctl);
}

void enqueue_copy_codes(hipStream_t st, uint32_t* dst, const uint32_t* src, int count, uint32_t mask) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_copy_codes, dim3(cdiv(count, WG)), dim3(WG), 0, st, dst, src, count, mask);
}

void enqueue_rebuild(hipStream_t st, const Scenes& T, float* S_cur, float* S_alt, int* id_cur, int* id_alt,
                     int64_t cap, int N, int chunk, int spread, int pack, BinBuffers& B, int* ctl, int nbricks,
                     int key_bits,
                     int* reg_n, int* reg) {
    const int n1 = N > 0 ? N : 1;
    const bool direct = cdiv(n1, WG * RS_SMALL) <= RS_DIRECT_TILES;
    const int tiles = cdiv(n1, WG * (direct ? RS_SMALL : RS_LARGE));
    // 1. particle codes, 2. stable radix sort of (code, position)
    if (N > 0) {
        if (direct)
            hipLaunchKernelGGL((k_keys<RS_SMALL, true>), dim3(tiles), dim3(WG), 0, st, S_cur, cap, N, T, B.keys[0],
                               B.vals[0], ctl, tiles, B.hist);
        else
            hipLaunchKernelGGL((k_keys<RS_LARGE, false>), dim3(tiles), dim3(WG), 0, st, S_cur, cap, N, T, B.keys[0],
                               B.vals[0], ctl, tiles, B.hist);
    }
    const int passes = N > 0 ? (key_bits + 7) / 8 : 0;
    int cur = 0;
    for (int p = 0; p < passes; ++p) {
        if (direct) {
            if (p > 0)
                hipLaunchKernelGGL((k_rs_hist<RS_SMALL, true>), dim3(tiles), dim3(WG), 0, st, B.keys[cur], N, 8 * p, tiles,
                                   B.hist);
            hipLaunchKernelGGL((k_rs_scatter<RS_SMALL, true>), dim3(tiles), dim3(WG), 0, st, B.keys[cur], B.vals[cur],
                               B.keys[cur ^ 1], B.vals[cur ^ 1], N, 8 * p, tiles, B.hist);
        } else {
            if (p > 0)
                hipLaunchKernelGGL((k_rs_hist<RS_LARGE, false>), dim3(tiles), dim3(WG), 0, st, B.keys[cur], N, 8 * p,
                                   tiles, B.hist);
            device_scan(st, OpHistScan{B.hist}, 256 * tiles, B.scan_tiles, ctl + CTL_SCAN);
            hipLaunchKernelGGL((k_rs_scatter<RS_LARGE, false>), dim3(tiles), dim3(WG), 0, st, B.keys[cur], B.vals[cur],
                               B.keys[cur ^ 1], B.vals[cur ^ 1], N, 8 * p, tiles, B.hist);
        }
        cur ^= 1;
    }
    B.sorted = cur;  // slot holding the sorted codes and their source positions
    // 3. geometric blocks with their merge groups, and work chunks
    const int stiles = cdiv(n1, SCAN_TILE);
    hipLaunchKernelGGL(k_blocks_count, dim3(stiles), dim3(WG), 0, st, B.keys[cur], N, pack, stiles, B.scan_tiles);
    if (stiles > SCAN_DIRECT_TILES) {
        hipLaunchKernelGGL(k_blocks_top, dim3(2), dim3(WG), 0, st, stiles, B.scan_tiles);
        hipLaunchKernelGGL(k_blocks_emit<true>, dim3(stiles), dim3(WG), 0, st, B.keys[cur], N, pack, stiles, B.scan_tiles,
                           B.gstart, B.gcode, B.group_start, ctl);
    } else {
        hipLaunchKernelGGL(k_blocks_emit<false>, dim3(stiles), dim3(WG), 0, st, B.keys[cur], N, pack, stiles, B.scan_tiles,
                           B.gstart, B.gcode, B.group_start, ctl);
    }
    // (no more groups than particles, nor than slabs, or single blocks, of the padded dense grids)
    const int slabs = pack ? nbricks / 4 + 1 : nbricks;
    device_scan<1>(st, OpChunks{B.gstart, B.gcode, B.group_start, ctl, N, chunk, B.chunks, T}, N < slabs ? N : slabs,
                   B.scan_tiles, ctl + CTL_NCHUNK);
    // 4. gather the whole particle state into (chunk-spread) sorted order
    hipLaunchKernelGGL(k_permute_chunks, dim3(2048), dim3(WG), 0, st, S_cur, S_alt, id_cur, id_alt, B.sorted_ids,
                       B.vals[cur], B.keys[cur], B.chunks, ctl, cap, spread, T.shift);
    // 5. physical blocks: 3x3x3 dilation, compacted in padded linear order
    hipLaunchKernelGGL(k_clear2, dim3(cdiv(nbricks, WG)), dim3(WG), 0, st, B.brick_state, reg_n, nbricks);
    hipLaunchKernelGGL(k_dilate, dim3(512), dim3(WG), 0, st, B.gcode, ctl, T, B.brick_state);
    device_scan(st, OpActive{B.brick_state, B.active}, nbricks, B.scan_tiles, ctl + CTL_NACTIVE);
    // 6. tile registrations of the chunks with the physical blocks
    hipLaunchKernelGGL(k_register, dim3(1024), dim3(WG), 0, st, B.chunks, B.keys[cur], ctl, B.brick_state, reg_n, reg,
                       T);
    hipLaunchKernelGGL(k_sort_registrations, dim3(1024), dim3(WG), 0, st, ctl, reg_n, reg);
    hipLaunchKernelGGL(k_rank_ends, dim3(1), dim3(WG), 0, st, B.keys[cur], N, B.gcode, B.chunks, B.active, ctl, T);
}

}  // namespace mpm
