// Binning and ordering of (tile, Gaussian) instances on gfx950 (Sec. 3.1:
// only Gaussians that intersect a tile take part in that tile, in depth
// order).
//
// Two equivalent orderings are provided:
//  - the literal one: duplicated 64-bit keys (tile << 32 | depth bits) with
//    value = record id, sorted by a stable LSD radix sort over all
//    significant bits (stage entry points mgs_duplicate / mgs_sort);
//  - the one the whole path uses: records are first sorted by their 32-bit
//    depth key (V*N elements), instances are then emitted in that order with
//    32-bit tile ids, and a stable LSD sort over the tile bits alone (one or
//    two passes) yields the same (tile, depth, record) order with a fraction
//    of the memory traffic, since K is often 100x the record count.
//
// The sort is reduce-then-scan (per-block digit histograms, a scan of each
// digit's row of them, then a stable scatter); it has no inter-block spin
// waits, so it needs no forward-progress guarantee between workgroups.
#include <mutex>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace mgs {
namespace {

// Scratch of the allocation-free scan (mgs_scan_noalloc): file-scope device
// memory, one copy per GPU, held until the process ends.  Host code never
// uses this name as an address: the per-device address comes from
// hipGetSymbolAddress (scan_noalloc_init) and is passed to the kernels.
static __device__ __align__(256) unsigned char scratch[SCAN_NOALLOC_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[MAX_DEVICES] = {};

constexpr int NT = 256;
constexpr int IPT = 16;
constexpr int TILE = NT * IPT;  // 4096 elements per block
constexpr int RADIX = 256;
static_assert(NT == RADIX, "one thread per digit in the histogram and scatter steps");
constexpr int64_t SORT_BLOCKS = 2048;  // 8 workgroups per CU on a 256-CU device

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
    const int lane = lane_id();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    return x;
}

// Exclusive scan over a 256-thread block; *total gets the block sum.
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T* sh, T* total) {
    const T inc = wave_inclusive_scan(v);
    const int w = threadIdx.x >> 6;
    if (lane_id() == 63) sh[w] = inc;
    __syncthreads();
    T wo = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        if (i < w) wo += sh[i];
        tot += sh[i];
    }
    *total = tot;
    __syncthreads();
    return wo + inc - v;
}

// The same over a block of NTH threads (a multiple of 64).
template <typename T, int NTH>
__device__ __forceinline__ T block_exclusive_scan_n(T v, T* sh, T* total) {
    const T inc = wave_inclusive_scan(v);
    const int w = threadIdx.x >> 6;
    if (lane_id() == 63) sh[w] = inc;
    __syncthreads();
    T wo = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NTH / 64; ++i) {
        if (i < w) wo += sh[i];
        tot += sh[i];
    }
    *total = tot;
    __syncthreads();
    return wo + inc - v;
}

__host__ __device__ inline int64_t nblocks(int64_t n) { return (n + TILE - 1) / TILE; }

// Items per thread of the sort's tiles: 8 for 64-bit keys (with 16, the
// keys, values and ranks a thread holds take 188 registers, two waves per
// SIMD), 16 for 32-bit keys.
template <typename KeyT>
constexpr int sort_ipt() {
    return sizeof(KeyT) == 8 ? 8 : 16;
}
template <typename KeyT>
constexpr int sort_tile() {
    return NT * sort_ipt<KeyT>();
}
constexpr int SORT_TILE_MIN = NT * 8;  // the smallest sort tile (sizes the histograms)
constexpr int64_t MAX_SORT_SEGMENTS = 16;  // segments of a segmented sort (one per view)
constexpr int64_t SHORT_MAX = 16384;       // longest segment sorted in one workgroup's LDS
// Segments of up to this many blocks need no row scan: 98 blocks, a pass's
// launches 16.7 us with their own sums, 18.7 with a row scan; 160 blocks 17 and
// 17, 366 blocks 28 and 24 us.
constexpr int64_t OWN_SCAN_BLOCKS = 128;

// Keys per workgroup of the sort: the host's chunk for a known count; with a
// device-side live count, the live keys are spread evenly over the nb
// workgroups the grid was sized for.
template <typename KeyT>
__device__ __forceinline__ int64_t sort_chunk(int64_t K, const uint64_t* K_dev, int64_t nb, int64_t chunk) {
    if (!K_dev) return chunk;
    constexpr int64_t ST = sort_tile<KeyT>();
    return (((K + ST - 1) / ST + nb - 1) / nb) * ST;
}

// ---------------------------------------------------------------------------
// scan of u32 counts (reduce, scan of block sums, downsweep)
// ---------------------------------------------------------------------------

__global__ void __launch_bounds__(NT) scan_reduce_kernel(const uint32_t* __restrict__ in, int64_t n,
                                                          uint64_t* __restrict__ partial) {
    __shared__ uint64_t sh[NT / 64];
    const int64_t base = (int64_t)blockIdx.x * TILE;
    uint64_t s = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const int64_t i = base + j * NT + threadIdx.x;
        if (i < n) s += in[i];
    }
    s = wave_inclusive_scan(s);
    if (lane_id() == 63) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int i = 0; i < NT / 64; ++i) t += sh[i];
        partial[blockIdx.x] = t;
    }
}

__global__ void __launch_bounds__(NT) scan_partials_kernel(uint64_t* __restrict__ partial, int64_t nb,
                                                            uint64_t* __restrict__ total_dev) {
    __shared__ uint64_t sh[NT / 64];
    uint64_t carry = 0;
    for (int64_t base = 0; base < nb; base += NT) {
        const int64_t i = base + threadIdx.x;
        const uint64_t v = i < nb ? partial[i] : 0;
        uint64_t tot;
        const uint64_t ex = block_exclusive_scan(v, sh, &tot);
        if (i < nb) partial[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0 && total_dev) *total_dev = carry;
}

__global__ void __launch_bounds__(NT) scan_down_kernel(const uint32_t* __restrict__ in, int64_t n,
                                                        const uint64_t* __restrict__ partial,
                                                        uint32_t* __restrict__ out) {
    __shared__ uint32_t tile[TILE];
    __shared__ uint32_t sh[NT / 64];
    const int64_t base = (int64_t)blockIdx.x * TILE;
    // coalesced load, then each thread takes 16 consecutive elements
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const int64_t i = base + j * NT + threadIdx.x;
        tile[j * NT + threadIdx.x] = i < n ? in[i] : 0u;
    }
    __syncthreads();
    uint32_t v[IPT];
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        v[j] = tile[threadIdx.x * IPT + j];
        s += v[j];
    }
    uint32_t tot;
    uint32_t run = block_exclusive_scan(s, sh, &tot) + (uint32_t)partial[blockIdx.x];
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        tile[threadIdx.x * IPT + j] = run;
        run += v[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const int64_t i = base + j * NT + threadIdx.x;
        if (i < n) out[i] = tile[j * NT + threadIdx.x];
    }
}

// ---------------------------------------------------------------------------
// literal key duplication (stage API): one thread per record
// ---------------------------------------------------------------------------

__global__ void __launch_bounds__(256) duplicate_kernel(
    const float4* __restrict__ rec, const float* __restrict__ radius, const float* __restrict__ depth,
    const uint32_t* __restrict__ tiles, const uint32_t* __restrict__ offsets, int64_t n_records, int64_t n_per_view,
    ViewSet views, DevSettings st, uint64_t* __restrict__ keys, uint32_t* __restrict__ vals, int64_t capacity,
    uint32_t* __restrict__ flags) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_records) return;
    const uint32_t cnt = tiles[r];
    if (cnt == 0) return;
    const int vi = (int)(r / n_per_view);
    const DevView& cam = views.v[vi];
    const Rect q = record_rect(rec, radius, r, cam, st);
    const uint64_t dbits = (uint64_t)__float_as_uint(depth[r]);
    int64_t off = offsets[r];
    bool overflow = false;
    for (int ty = q.y0; ty <= q.y1; ++ty) {
        const uint64_t row = (uint64_t)cam.tile_off + (uint64_t)ty * cam.grid_w;
        for (int tx = q.x0; tx <= q.x1; ++tx) {
            if (off < capacity) {
                keys[off] = ((row + tx) << 32) | dbits;
                vals[off] = (uint32_t)r;
            } else {
                overflow = true;
            }
            ++off;
        }
    }
    if (overflow) atomicOr(flags, FLAG_CAPACITY);
}

// ---------------------------------------------------------------------------
// LSD radix sort, 8 bits per pass, 16-, 32- or 64-bit keys with u32 values
// ---------------------------------------------------------------------------

__device__ __forceinline__ int64_t live_count(int64_t K, const uint64_t* K_dev) {
    if (!K_dev) return K;
    const uint64_t k = *K_dev;
    return (int64_t)(k < (uint64_t)K ? k : (uint64_t)K);
}

// Keys in registers (16-bit ones take a whole one).
template <typename KeyT>
using KeyReg = std::conditional_t<sizeof(KeyT) == 2, uint32_t, KeyT>;

template <typename KeyT>
__device__ __forceinline__ uint32_t digit_of(KeyT k, int shift) {
    return (uint32_t)(k >> shift) & (RADIX - 1);
}

// Number of the mask's lanes below this one.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Lanes of the wave with this lane's digit.  Per bit one extraction (0 or all
// ones), one comparison, and per half of the mask one three-operand operation
// that collects the lanes that differ: with the ranks by lane counts 54 vector
// instructions per 64 keys instead of 79 (selecting the mask or its complement,
// the first lane by a bit search).  Scatter of 20.2 M keys 106 and 84 -> 95 and
// 70 us, of 8 M 33 -> 25 to 26 us, of 300 k 10.3 -> 9.6 us.
__device__ __forceinline__ uint64_t digit_peers(uint32_t d) {
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const int m = (int)(d << (31 - b)) >> 31;
        const uint64_t bal = ballot(m != 0);
        lo |= (uint32_t)bal ^ (uint32_t)m;
        hi |= (uint32_t)(bal >> 32) ^ (uint32_t)m;
    }
    return ~((uint64_t)hi << 32 | lo);
}

// Segments: the keys may form consecutive segments of seg_len keys each
// (the last one shorter), sorted each on its own: block b works in segment
// b / nbs, on the (b % nbs)-th chunk of it, and the histograms are laid out
// (segment, digit, block).  A block's output position for digit d is the
// segment's start (seg * seg_len), plus the segment's counts of the digits
// below d, plus the counts of d in the segment's earlier blocks: the
// row scan gives the last term and the row totals, the scatter adds the
// rest.  With one segment (seg_len >= K, nbs = nb) the layout is the plain
// digit-major hist[d * nb + block].
//
// The depth sort's values are the keys' indices: its first pass reads none.
// Above DROP_MIN keys that pass also drops the dead ones (all ones: records
// without tiles): it counts and scatters the others only, writes their number
// per segment into live[seg], and places the dead keys' values behind them in
// the final value buffer, in order; the later passes end at live[seg].  A third
// of the keys dead (views inside their scene), the four passes with / without:
// 0.3 to 3.6 M keys 1.05 to 1.02 of the time (77 / 73 us, 216 / 212), where a
// pass takes as long for fewer keys and the first one longer; 4 M in four views
// 229 / 224, in eight 227 / 237; 5 M 270 / 269, 6.4 M 320 / 332, 8 M 372 / 387.
constexpr int64_t DROP_MIN = 4000000;
enum FirstPass { LATER = 0, INDEX = 1, INDEX_DROP = 2 };
struct SortSeg {
    int64_t seg, bl, beg, end;  // segment, block within it, chunk [beg, end)
};

// Logical block of this workgroup.  Workgroups are dealt to the 8 XCDs in
// turn (workgroup i to XCD i mod 8); the mapping gives every XCD one run of
// consecutive logical blocks, so the digit runs that neighbouring blocks
// scatter next to each other are written through the same L2.
__device__ __forceinline__ int64_t sort_block(int64_t nb) {
    const int64_t i = (int64_t)blockIdx.x;
    const int64_t q = nb >> 3, r = nb & 7, x = i & 7;
    return x * q + (x < r ? x : r) + (i >> 3);
}

__device__ __forceinline__ SortSeg sort_seg(int64_t K, int64_t seg_len, int64_t nbs, int64_t chunk, int64_t nb,
                                            const uint32_t* live) {
    SortSeg s;
    const int64_t b = sort_block(nb);
    s.seg = b / nbs;
    s.bl = b - s.seg * nbs;
    const int64_t sbeg = s.seg * seg_len;
    const int64_t send = live ? sbeg + live[s.seg] : min(sbeg + seg_len, K);
    s.beg = sbeg + s.bl * chunk;
    s.end = min(s.beg + chunk, send);
    return s;
}

// Per-block digit histograms, written (segment, digit, block)-major.
// Loads are vectorised and coalesced; each lane counts runs of equal digits
// in registers before touching LDS, so keys clustered by digit (neighbouring
// tiles of one splat) do not serialise on one LDS counter.
// Each block owns a contiguous chunk of `chunk` keys (a multiple of the sort tile),
// so a couple of thousand blocks cover any K and the digit-major histogram
// stays small.
// COPIES histograms per wave (lane mod COPIES picks one), so that lanes of
// a wave with equal digits rarely hit one LDS counter: 4 for the list
// entries' cell keys (digits clustered in the second pass), 1 for the
// depth keys
// BLOCKMAJOR: hist[(segment nbs + block) RADIX + digit] instead, for a scatter
// that adds up its segment's rows itself (radix_downsweep_kernel<.., true>)
template <typename KeyT, int COPIES, bool BLOCKMAJOR, int FIRST>
__global__ void __launch_bounds__(NT) radix_upsweep_kernel(const KeyT* __restrict__ keys, int64_t Kcap,
                                                            const uint64_t* __restrict__ K_dev, int shift,
                                                            uint32_t* __restrict__ hist, int64_t nb, int64_t chunk,
                                                            int64_t seg_len, int64_t nbs,
                                                            const uint32_t* __restrict__ live) {
    constexpr bool DROP = FIRST == INDEX_DROP;
    constexpr int VEC = 16 / sizeof(KeyT);  // keys per 16-byte load
    constexpr int SIPT = sort_ipt<KeyT>(), STILE = sort_tile<KeyT>();
    __shared__ uint32_t h[(NT / 64) * COPIES][RADIX];
    const int w = (threadIdx.x >> 6) * COPIES + (lane_id() & (COPIES - 1));
    for (int i = threadIdx.x; i < (NT / 64) * COPIES * RADIX; i += NT) (&h[0][0])[i] = 0u;
    __syncthreads();
    const int64_t K = live_count(Kcap, K_dev);
    chunk = sort_chunk<KeyT>(K, K_dev, nb, chunk);
    const SortSeg sg = sort_seg(K, seg_len, nbs, chunk, nb, DROP ? nullptr : live);
    const int64_t cbeg = sg.beg, cend = sg.end;
    for (int64_t base = cbeg; base < cend; base += STILE)
#pragma unroll
    for (int j = 0; j < SIPT / VEC; ++j) {
        const int64_t i0 = base + ((int64_t)j * NT + threadIdx.x) * VEC;
        KeyT k[VEC];
        int nv = 0;
        if (i0 + VEC <= cend) {
            if constexpr (VEC == 8) {
                const uint4 q = *reinterpret_cast<const uint4*>(keys + i0);
                const uint32_t qs[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                for (int v = 0; v < VEC; ++v) k[v] = (KeyT)(qs[v / 2] >> (16 * (v & 1)));
            } else if constexpr (VEC == 4) {
                const uint4 q = *reinterpret_cast<const uint4*>(keys + i0);
                k[0] = q.x; k[1] = q.y; k[2] = q.z; k[3] = q.w;
            } else {
                const ulonglong2 q = *reinterpret_cast<const ulonglong2*>(keys + i0);
                k[0] = q.x; k[1] = q.y;
            }
            nv = VEC;
        } else {
            for (int v = 0; v < VEC; ++v)
                if (i0 + v < cend) { k[v] = keys[i0 + v]; nv = v + 1; }
        }
        if constexpr (DROP) {
            for (int v = 0; v < nv; ++v)
                if (k[v] != ~(KeyT)0) atomicAdd(&h[w][digit_of(k[v], shift)], 1u);
        } else if (nv > 0) {
            uint32_t cur = digit_of(k[0], shift), run = 1;
            for (int v = 1; v < nv; ++v) {
                const uint32_t d = digit_of(k[v], shift);
                if (d == cur) {
                    ++run;
                } else {
                    atomicAdd(&h[w][cur], run);
                    cur = d;
                    run = 1;
                }
            }
            atomicAdd(&h[w][cur], run);
        }
    }
    __syncthreads();
    const int d = threadIdx.x;  // NT == RADIX
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < (NT / 64) * COPIES; ++i) s += h[i][d];
    if constexpr (BLOCKMAJOR) hist[(sg.seg * nbs + sg.bl) * RADIX + d] = s;
    else hist[(sg.seg * RADIX + d) * nbs + sg.bl] = s;
}

// Exclusive prefix of every (segment, digit) row of the block histograms
// over the row's blocks, and the row's total: one workgroup per row, each
// thread over a run of at most SORT_BLOCKS / NT consecutive blocks.
constexpr int ROW_PER_THREAD = (int)(SORT_BLOCKS / NT);
__global__ void __launch_bounds__(NT) radix_rowscan_kernel(const uint32_t* __restrict__ hist, int64_t nbs,
                                                            uint32_t* __restrict__ row_pre,
                                                            uint32_t* __restrict__ row_tot) {
    __shared__ uint32_t sh[NT / 64];
    const int64_t row = blockIdx.x;
    const uint32_t* h = hist + row * nbs;
    uint32_t* p = row_pre + row * nbs;
    const int per = (int)((nbs + NT - 1) / NT);
    const int64_t b0 = (int64_t)threadIdx.x * per;
    uint32_t v[ROW_PER_THREAD];
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < ROW_PER_THREAD; ++j) {
        v[j] = (j < per && b0 + j < nbs) ? h[b0 + j] : 0u;
        s += v[j];
    }
    uint32_t tot;
    uint32_t run = block_exclusive_scan(s, sh, &tot);
#pragma unroll
    for (int j = 0; j < ROW_PER_THREAD; ++j) {
        if (j < per && b0 + j < nbs) p[b0 + j] = run;
        run += v[j];
    }
    if (threadIdx.x == 0) row_tot[row] = tot;
}

// Threads of a scatter workgroup: 512 for 32-bit keys (8 per thread, so
// that twice the waves of a 256-thread workgroup share the tile's LDS), 256
// for 64-bit keys.
template <typename KeyT>
constexpr int sort_dt() {
    return sizeof(KeyT) == 8 ? 256 : 512;
}

// Threads t < RADIX own digit t in the digit steps; the per-wave digit
// counts (at most 64 x 8 per wave, prefixes at most the tile) fit 16 bits.
// OWN_SCAN: no row scan ran; row_pre holds the block-major histogram, and each
// workgroup adds up its segment's counts (two threads per digit), which costs
// less than a launch while a segment has few blocks.
// FIRST: see SortSeg (vals_in is not read; INDEX_DROP: dead values go to
// dead_out).
template <typename KeyT, bool OWN_SCAN, int FIRST>
__global__ void __launch_bounds__(sort_dt<KeyT>()) __attribute__((amdgpu_waves_per_eu(sizeof(KeyT) == 8 ? 1 : 6)))
radix_downsweep_kernel(
    const KeyT* __restrict__ keys_in, const uint32_t* __restrict__ vals_in, KeyT* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, int64_t Kcap, const uint64_t* __restrict__ K_dev, int shift,
    const uint32_t* __restrict__ row_pre, const uint32_t* __restrict__ row_tot, int64_t nb, int64_t chunk,
    int64_t seg_len, int64_t nbs, uint32_t* __restrict__ live, uint32_t* __restrict__ dead_out) {
    constexpr bool DROP = FIRST == INDEX_DROP;
    constexpr int DT = sort_dt<KeyT>();
    constexpr int STILE = sort_tile<KeyT>(), SIPT = STILE / DT;
    static_assert(SIPT * 64 <= 65535 && STILE <= 65535, "16-bit digit counts");
    __shared__ KeyT sk[STILE];
    __shared__ uint32_t sv[STILE];
    __shared__ uint16_t wcnt[DT / 64][RADIX];
    __shared__ uint32_t dstart[RADIX];
    __shared__ uint32_t gstart[RADIX];
    __shared__ uint32_t scan_sh[DT / 64];
    __shared__ uint32_t wdead_sh[DROP ? DT / 64 : 1];

    const int64_t K = live_count(Kcap, K_dev);
    chunk = sort_chunk<KeyT>(K, K_dev, nb, chunk);
    const SortSeg sg = sort_seg(K, seg_len, nbs, chunk, nb, DROP ? nullptr : live);
    const int64_t cbeg = sg.beg, cend = sg.end;
    if (cbeg >= cend) return;  // uniform over the block
    int64_t dead = 0;          // DROP: where the chunk's next dead value goes
    const int w = threadIdx.x >> 6, lane = lane_id();
    // global start of each digit for this chunk, advanced after every sub-tile
    const bool dig = threadIdx.x < RADIX;
    {
        const int64_t row = sg.seg * RADIX + (dig ? threadIdx.x : 0);
        uint32_t tot, pre, own;
        if constexpr (OWN_SCAN) {
            constexpr int PER = DT / RADIX;  // threads per digit, over every PER-th block
            const uint32_t* h = row_pre + sg.seg * nbs * RADIX + threadIdx.x % RADIX;
            const int64_t b0 = threadIdx.x / RADIX;
            pre = own = 0;
            constexpr uint32_t ROUND = 8;  // loads in flight
            const uint32_t n = (uint32_t)nbs, bl = (uint32_t)sg.bl;
            uint32_t b = (uint32_t)b0;
            for (; b + PER * (ROUND - 1) < n; b += PER * ROUND) {
                uint32_t c[ROUND];
#pragma unroll
                for (uint32_t j = 0; j < ROUND; ++j) c[j] = h[(b + PER * j) * RADIX];
#pragma unroll
                for (uint32_t j = 0; j < ROUND; ++j) {
                    own += c[j];
                    pre += b + PER * j < bl ? c[j] : 0u;
                }
            }
            if (b < n) {
                uint32_t c[ROUND];
#pragma unroll
                for (uint32_t j = 0; j < ROUND; ++j) c[j] = b + PER * j < n ? h[(b + PER * j) * RADIX] : 0u;
#pragma unroll
                for (uint32_t j = 0; j < ROUND; ++j) {
                    own += c[j];
                    pre += b + PER * j < bl ? c[j] : 0u;
                }
            }
            if constexpr (PER > 1) {
                static_assert(PER == 2, "one partner per digit");
                if (!dig) {
                    dstart[threadIdx.x - RADIX] = pre;
                    gstart[threadIdx.x - RADIX] = own;
                }
                __syncthreads();
                if (dig) {
                    pre += dstart[threadIdx.x];
                    own += gstart[threadIdx.x];
                }
            }
        } else {
            pre = dig ? row_pre[row * nbs + sg.bl] : 0u;
            own = row_tot[row];
        }
        const uint32_t below = block_exclusive_scan_n<uint32_t, DT>(dig ? own : 0u, scan_sh, &tot);
        if (dig) gstart[threadIdx.x] = (uint32_t)(sg.seg * seg_len) + below + pre;
        if constexpr (DROP) {
            // tot: the segment's live keys; those before this chunk
            uint32_t before;
            block_exclusive_scan_n<uint32_t, DT>(dig ? pre : 0u, scan_sh, &before);
            dead = cbeg + tot - before;
            if (sg.bl == 0 && threadIdx.x == 0) live[sg.seg] = tot;
        }
    }
    for (int64_t base = cbeg; base < cend; base += STILE) {
    const int nvalid = (int)min((int64_t)STILE, cend - base);
    for (int i = threadIdx.x; i < (DT / 64) * RADIX; i += DT) (&wcnt[0][0])[i] = 0u;
    __syncthreads();

    // wave w owns the contiguous span [w * 64 SIPT, (w + 1) * 64 SIPT) of the tile;
    // round j covers 64 consecutive items, lane l the (j * 64 + l)-th
    KeyReg<KeyT> key[SIPT];
    uint32_t val[SIPT];
    uint32_t rank[SIPT];
    // one address per array: the rounds are constant offsets from it
    const int l0 = w * (SIPT * 64) + lane;
    const KeyT* kp = keys_in + base + l0;
    const uint32_t* vp = vals_in + base + l0;
#pragma unroll
    for (int j = 0; j < SIPT; ++j) {
        if (l0 + j * 64 < nvalid) {
            key[j] = kp[j * 64];
            if constexpr (FIRST == LATER) val[j] = vp[j * 64];
        } else {
            key[j] = ~(KeyReg<KeyT>)0;  // digit 255 at every shift, ranked after every valid item
            val[j] = 0u;
        }
    }
    uint32_t wdead = 0;  // DROP: the wave's dead keys
#pragma unroll
    for (int j = 0; j < SIPT; ++j) {
        const uint32_t d = digit_of(key[j], shift);
        const bool lv = !DROP || key[j] != ~(KeyReg<KeyT>)0;
        const uint64_t peers = digit_peers(d) & (DROP ? ballot(lv) : ~0ull);
        const uint32_t before = wcnt[w][d], below = lanes_below(peers);
        rank[j] = before + below;
        if constexpr (DROP) {
            const uint64_t db = ballot(!lv && l0 + j * 64 < nvalid);
            if (!lv) rank[j] = wdead + lanes_below(db);
            wdead += (uint32_t)__popcll(db);
        }
        // the first lane of the digit (a dead one is never it)
        if (below == 0 && lv) wcnt[w][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
    }
    // the keys pass through an empty asm statement, so that the scatter below
    // derives each item's digit again instead of keeping its counter address
    // live (in registers) across the digit scan
#pragma unroll
    for (int j = 0; j < SIPT; ++j) asm volatile("" : "+v"(key[j]));
    __syncthreads();
    // per digit: offsets of each wave, block total, then block-wide digit starts
    uint32_t digit_total = 0;
    int nlive = nvalid;
    if constexpr (DROP) {
        if (lane == 0) wdead_sh[w] = wdead;
    }
    {
        const int d = threadIdx.x;
        uint32_t run = 0;
        if (dig) {
#pragma unroll
            for (int i = 0; i < DT / 64; ++i) {
                const uint32_t c = wcnt[i][d];
                wcnt[i][d] = (uint16_t)run;
                run += c;
            }
        }
        uint32_t tot;
        const uint32_t ds = block_exclusive_scan_n<uint32_t, DT>(run, scan_sh, &tot);
        if (dig) dstart[d] = ds;
        digit_total = run;
        if constexpr (DROP) nlive = (int)tot;
    }
    __syncthreads();
    // (FIRST: the items' indices)
    uint32_t i0 = (uint32_t)base + (uint32_t)l0;
    if constexpr (FIRST != LATER) asm volatile("" : "+v"(i0));
#pragma unroll
    for (int j = 0; j < SIPT; ++j) {
        if (DROP && key[j] == ~(KeyReg<KeyT>)0) {
            if (l0 + j * 64 >= nvalid) continue;
            int64_t o = dead + rank[j];
            for (int i = 0; i < w; ++i) o += wdead_sh[i];
            dead_out[o] = i0 + j * 64;
            continue;
        }
        const uint32_t d = digit_of(key[j], shift);
        const uint32_t pos = dstart[d] + wcnt[w][d] + rank[j];
        sk[pos] = (KeyT)key[j];
        sv[pos] = FIRST != LATER ? i0 + j * 64 : val[j];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nlive; i += DT) {
        const KeyT k = sk[i];
        const uint32_t d = digit_of(k, shift);
        const uint32_t o = gstart[d] + (uint32_t)i - dstart[d];
        keys_out[o] = k;
        vals_out[o] = sv[i];
    }
    __syncthreads();
    // padded items all carry digit 255 and sit past nvalid; they are not counted
    const uint32_t pad = !DROP && threadIdx.x == RADIX - 1 ? (uint32_t)(STILE - nvalid) : 0u;
    if (dig) gstart[threadIdx.x] += digit_total - pad;
    dead += nvalid - nlive;
    __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// short 32-bit sorts: one workgroup per segment, all passes in LDS
// ---------------------------------------------------------------------------

// At most 1024 IPW keys per segment.  The multi-block sort takes three
// launches of 3 to 7 us per pass whatever the size; this one holds keys and
// values in LDS and takes 3 to 5 us per pass (4096 keys, four passes: 59 ->
// 17.3 us).  Ranking as in radix_downsweep_kernel; keys past the live count are
// all ones and stay behind every valid key.  The loops over a thread's keys are
// unrolled: those of 8 with a break (4096 keys, 26.2 -> 25.5 us), those of 16,
// which the compiler then leaves as loops, without (16,384 keys, 64.5 -> 61.5
// us; stage times).  ranges (optional, cleared; one
// segment): [start, end) of every key below nbins, as tile_ranges_kernel.
// index_vals: the values are the keys' indices (vals is not read).
constexpr int SHORT_DT = 1024;
template <int IPW>
__global__ void __launch_bounds__(SHORT_DT) radix_short_kernel(uint32_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                                                int64_t Kcap, const uint64_t* __restrict__ K_dev,
                                                                int begin_bit, int end_bit, int64_t seg_len,
                                                                uint2* __restrict__ ranges, uint32_t nbins,
                                                                bool index_vals) {
    constexpr int NW = SHORT_DT / 64;
    __shared__ uint32_t sk[SHORT_DT * IPW];
    __shared__ uint32_t sv[SHORT_DT * IPW];
    __shared__ uint16_t wcnt[NW][RADIX];
    __shared__ uint32_t dstart[RADIX];
    __shared__ uint32_t scan_sh[NW];
    const int64_t K = live_count(Kcap, K_dev);
    const int64_t beg = (int64_t)blockIdx.x * seg_len;
    const int n = (int)min(seg_len, K - beg);
    if (n <= 0) return;  // uniform
    const int t = threadIdx.x, w = t >> 6, lane = lane_id();
    const bool dig = t < RADIX;
    // wave w owns the span [64 w rounds, 64 (w + 1) rounds) of the segment
    const int rounds = (n + SHORT_DT - 1) / SHORT_DT;
    const int l0 = w * rounds * 64 + lane;
    uint32_t key[IPW], val[IPW], rank[IPW];
#pragma unroll
    for (int j = 0; j < IPW; ++j) {
        const int i = l0 + j * 64;
        const bool in = j < rounds && i < n;
        key[j] = in ? keys[beg + i] : 0xffffffffu;
        val[j] = index_vals ? (uint32_t)(beg + i) : (in ? vals[beg + i] : 0u);
    }
    for (int shift = begin_bit; shift < end_bit; shift += 8) {
        for (int i = t; i < NW * RADIX; i += SHORT_DT) (&wcnt[0][0])[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPW; ++j) {
            if (j >= rounds) {
                if constexpr (IPW <= 8) break;
                else continue;
            }
            const uint32_t d = digit_of(key[j], shift);
            const uint64_t peers = digit_peers(d);
            const uint32_t before = wcnt[w][d], below = lanes_below(peers);
            rank[j] = before + below;
            if (below == 0) wcnt[w][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
        }
        __syncthreads();
        uint32_t run = 0;
        if (dig) {
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const uint32_t c = wcnt[i][t];
                wcnt[i][t] = (uint16_t)run;
                run += c;
            }
        }
        uint32_t tot;
        const uint32_t ds = block_exclusive_scan_n<uint32_t, SHORT_DT>(run, scan_sh, &tot);
        if (dig) dstart[t] = ds;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPW; ++j) {
            if (j >= rounds) {
                if constexpr (IPW <= 8) break;
                else continue;
            }
            const uint32_t d = digit_of(key[j], shift);
            const uint32_t pos = dstart[d] + wcnt[w][d] + rank[j];
            sk[pos] = key[j];
            sv[pos] = val[j];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < IPW; ++j) {
            if (j >= rounds) {
                if constexpr (IPW <= 8) break;
                else continue;
            }
            key[j] = sk[l0 + j * 64];
            val[j] = sv[l0 + j * 64];
        }
        __syncthreads();  // sk, sv are written again by the next pass
    }
#pragma unroll
    for (int j = 0; j < IPW; ++j) {
        const int i = l0 + j * 64;
        if (j < rounds && i < n) {
            keys[beg + i] = key[j];
            vals[beg + i] = val[j];
            if (ranges) {  // sk still holds the sorted keys
                const uint32_t c = key[j], p = i > 0 ? sk[i - 1] : 0u;
                if (i == 0 || p != c) {
                    if (i > 0 && p < nbins) ranges[p].y = (uint32_t)i;
                    if (c < nbins) ranges[c].x = (uint32_t)i;
                }
                if (i == n - 1 && c < nbins) ranges[c].y = (uint32_t)n;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// tile ranges, fills, sums
// ---------------------------------------------------------------------------

// [start, end) of every bin of sorted keys; keys at or past nbins (entries
// that belong nowhere, sorted last) are left out of every range.
template <typename KeyT>
__global__ void __launch_bounds__(256) tile_ranges_kernel(const KeyT* __restrict__ keys, int64_t Kcap,
                                                           const uint64_t* __restrict__ K_dev, int shift,
                                                           uint64_t nbins, uint2* __restrict__ ranges) {
    const int64_t K = live_count(Kcap, K_dev);
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    const uint64_t t = (uint64_t)(keys[k] >> shift);
    const bool tv = t < nbins;
    if (k == 0) {
        if (tv) ranges[t].x = 0;
    } else {
        const uint64_t p = (uint64_t)(keys[k - 1] >> shift);
        if (p != t) {
            if (p < nbins) ranges[p].y = (uint32_t)k;
            if (tv) ranges[t].x = (uint32_t)k;
        }
    }
    if (k == K - 1 && tv) ranges[t].y = (uint32_t)K;
}

// The same for 32-bit keys, four consecutive keys per thread (one 16-byte
// load of keys 4 j .. 4 j + 3 and the key before them), or 16-bit ones (8
// bytes).
template <typename KeyT>
__global__ void __launch_bounds__(256) tile_ranges4_kernel(const KeyT* __restrict__ keys, int64_t Kcap,
                                                            const uint64_t* __restrict__ K_dev, uint64_t nbins,
                                                            uint2* __restrict__ ranges) {
    const int64_t K = live_count(Kcap, K_dev);
    const int64_t k0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (k0 >= K) return;
    uint32_t v[4];
    if (k0 + 4 <= K) {
        if constexpr (sizeof(KeyT) == 2) {
            const uint2 q = *reinterpret_cast<const uint2*>(keys + k0);
            v[0] = q.x & 0xffffu; v[1] = q.x >> 16; v[2] = q.y & 0xffffu; v[3] = q.y >> 16;
        } else {
            const uint4 q = *reinterpret_cast<const uint4*>(keys + k0);
            v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = k0 + i < K ? keys[k0 + i] : 0u;
    }
    uint64_t p = k0 > 0 ? (uint64_t)keys[k0 - 1] : 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t k = k0 + i;
        if (k >= K) break;
        const uint64_t t = v[i];
        const bool tv = t < nbins;
        if (k == 0) {
            if (tv) ranges[t].x = 0;
        } else if (p != t) {
            if (p < nbins) ranges[p].y = (uint32_t)k;
            if (tv) ranges[t].x = (uint32_t)k;
        }
        if (k == K - 1 && tv) ranges[t].y = (uint32_t)K;
        p = t;
    }
}

__global__ void __launch_bounds__(256) fill_u32_kernel(uint32_t* __restrict__ p, int64_t n, uint32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Up to FILL_SPANS u32 spans in one launch
__global__ void __launch_bounds__(256) fill_set_kernel(FillSet fs) {
    fill_element(fs, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

__global__ void __launch_bounds__(256) fill_f32_kernel(float* __restrict__ p, int64_t n, float v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void __launch_bounds__(256) round_f64_kernel(const double* __restrict__ in, float* __restrict__ out,
                                                         int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (float)in[i];
}

__global__ void __launch_bounds__(NT) sum_i32x4_partial_kernel(const int4* __restrict__ in, int64_t n,
                                                                uint64_t* __restrict__ partial, int64_t nb) {
    __shared__ uint64_t sh[4][NT / 64];
    const int64_t base = (int64_t)blockIdx.x * TILE;
    uint64_t s[4] = {0, 0, 0, 0};
    for (int j = 0; j < IPT; ++j) {
        const int64_t i = base + j * NT + threadIdx.x;
        if (i < n) {
            const int4 v = in[i];
            s[0] += (uint64_t)(int64_t)v.x;
            s[1] += (uint64_t)(int64_t)v.y;
            s[2] += (uint64_t)(int64_t)v.z;
            s[3] += (uint64_t)(int64_t)v.w;
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint64_t x = wave_inclusive_scan(s[c]);
        if (lane_id() == 63) sh[c][threadIdx.x >> 6] = x;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        uint64_t t = 0;
        for (int i = 0; i < NT / 64; ++i) t += sh[threadIdx.x][i];
        partial[threadIdx.x * nb + blockIdx.x] = t;
    }
}

// seg_len > 0: the keys form segments of seg_len keys, each sorted on its own
// (no device-side count then); otherwise one segment.
// ranges, nbins: as launch_cell_sort; returns whether they were written.
// live (32-bit keys): a sort of the keys' indices (see SortSeg); *dropped tells
// whether live was written.
template <typename KeyT>
bool radix_sort_t(hipStream_t stream, KeyT* keys, uint32_t* vals, KeyT* keys_alt, uint32_t* vals_alt, int64_t K,
                  const uint64_t* K_dev, int begin_bit, int end_bit, void* scratch, bool* out_in_alt,
                  int64_t seg_len = 0, uint32_t* ranges = nullptr, int64_t nbins = 0, uint32_t* live = nullptr,
                  bool* dropped = nullptr) {
    *out_in_alt = false;
    if (dropped) *dropped = false;
    if (K <= (live ? 0 : 1) && !K_dev) return false;
    if (end_bit <= begin_bit) return false;
    if constexpr (sizeof(KeyT) == 4) {
        // short segments: one launch, in place (the lines between 8 and 16
        // keys per thread and at SHORT_MAX are those of its LDS)
        const int64_t sl = seg_len > 0 && seg_len < K && !K_dev ? seg_len : K;
        const unsigned ns = (unsigned)((K + sl - 1) / sl);
        if (sl <= SHORT_MAX) {
            uint2* r = ns == 1 ? reinterpret_cast<uint2*>(ranges) : nullptr;
#define MGS_SHORT(I)                                                                                               \
    hipLaunchKernelGGL(radix_short_kernel<I>, dim3(ns), dim3(SHORT_DT), 0, stream, keys, vals, K, K_dev, begin_bit, \
                       end_bit, sl, r, (uint32_t)nbins, live != nullptr)
            if (sl <= SHORT_DT * 8) MGS_SHORT(8);
            else MGS_SHORT(16);
#undef MGS_SHORT
            return r != nullptr;
        }
    }
    // about SORT_BLOCKS workgroups, each over a contiguous chunk of whole
    // tiles of one segment
    constexpr int64_t STILE = sort_tile<KeyT>();
    const bool segmented = seg_len > 0 && seg_len < K && !K_dev;
    const int64_t slen = segmented ? seg_len : (K > 0 ? K : 1);
    const int64_t nseg = segmented ? (K + seg_len - 1) / seg_len : 1;
    const int64_t per_seg = std::max<int64_t>(1, SORT_BLOCKS / nseg);
    const int64_t ntiles = (slen + STILE - 1) / STILE;
    const int64_t tiles_per_block = (ntiles + per_seg - 1) / per_seg;
    const int64_t chunk = tiles_per_block * STILE;
    const int64_t nbs = (ntiles + tiles_per_block - 1) / tiles_per_block;
    const int64_t nb = nseg * nbs;
    const int64_t seg_arg = segmented ? seg_len : INT64_MAX / 4;
    static_assert(SORT_BLOCKS % NT == 0, "row scan: whole runs per thread");
    const int64_t hn = nb * RADIX, rows = nseg * RADIX;
    uint32_t* hist = reinterpret_cast<uint32_t*>(scratch);
    uint32_t* row_pre = hist + hn;
    uint32_t* row_tot = row_pre + hn;
    KeyT* kin = keys;
    uint32_t* vin = vals;
    KeyT* kout = keys_alt;
    uint32_t* vout = vals_alt;
    const bool own_scan = nbs <= OWN_SCAN_BLOCKS;
    const bool drop = live && K >= DROP_MIN;
    if (dropped) *dropped = drop;
    uint32_t* later = drop ? live : nullptr;
    // the values' last buffer, where the first pass places the dead ones (an
    // even number of passes ends where it began: nothing reads vals then)
    uint32_t* dead_out = ((end_bit - begin_bit + 7) / 8) % 2 ? vals_alt : vals;
    for (int shift = begin_bit; shift < end_bit; shift += 8) {
        auto sweep = [&](auto first_c, auto own_c, auto copies_c) {
            constexpr int FIRST = decltype(first_c)::value, COPIES = decltype(copies_c)::value;
            constexpr bool OWN = decltype(own_c)::value;
            hipLaunchKernelGGL((radix_upsweep_kernel<KeyT, COPIES, OWN, FIRST == INDEX_DROP ? FIRST : LATER>),
                               dim3((unsigned)nb), dim3(NT), 0, stream, kin, K, K_dev, shift, hist, nb, chunk, seg_arg,
                               nbs, (const uint32_t*)later);
            if constexpr (!OWN)
                hipLaunchKernelGGL(radix_rowscan_kernel, dim3((unsigned)rows), dim3(NT), 0, stream,
                                   (const uint32_t*)hist, nbs, row_pre, row_tot);
            hipLaunchKernelGGL((radix_downsweep_kernel<KeyT, OWN, FIRST>), dim3((unsigned)nb), dim3(sort_dt<KeyT>()),
                               0, stream, kin, vin, kout, vout, K, K_dev, shift,
                               (const uint32_t*)(OWN ? hist : row_pre), (const uint32_t*)row_tot, nb, chunk, seg_arg,
                               nbs, later, dead_out);
        };
        auto by_scan = [&](auto first_c, auto copies_c) {
            if (own_scan) sweep(first_c, std::true_type{}, copies_c);
            else sweep(first_c, std::false_type{}, copies_c);
        };
        using One = std::integral_constant<int, 1>;
        using Four = std::integral_constant<int, 4>;
        if constexpr (sizeof(KeyT) == 4) {
            const bool first = live && shift == begin_bit;
            if (first && drop) by_scan(std::integral_constant<int, INDEX_DROP>{}, One{});
            else if (first) by_scan(std::integral_constant<int, INDEX>{}, One{});
            else if (live) by_scan(std::integral_constant<int, LATER>{}, One{});
            else by_scan(std::integral_constant<int, LATER>{}, Four{});
        } else {
            by_scan(std::integral_constant<int, LATER>{}, Four{});
        }
        KeyT* tk = kin; kin = kout; kout = tk;
        uint32_t* tv = vin; vin = vout; vout = tv;
        *out_in_alt = !*out_in_alt;
    }
    return false;
}

}  // namespace

size_t scan_scratch_bytes(int64_t n) { return (size_t)(nblocks(n) + 1) * sizeof(uint64_t) + 256; }

int64_t scan_noalloc_max_n() {
    // the scan needs (blocks + 1) u64 partial sums plus 256 bytes
    const int64_t blocks = (int64_t)((SCAN_NOALLOC_BYTES - 256) / sizeof(uint64_t)) - 1;
    return blocks * TILE;
}

hipError_t scan_noalloc_init(int device, void** out) {
    *out = nullptr;
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    if (!g_noalloc_ptr[device]) {
        // with `device` current: its own copy of the array
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_noalloc_ptr[device] = p;
    }
    *out = g_noalloc_ptr[device];
    return hipSuccess;
}

void launch_scan_u32(hipStream_t stream, const uint32_t* in, int64_t n, uint32_t* out, uint64_t* total_dev,
                     void* scratch) {
    const int64_t nb = nblocks(n);
    uint64_t* partial = reinterpret_cast<uint64_t*>(scratch);
    if (n == 0) {
        if (total_dev) hipLaunchKernelGGL(scan_partials_kernel, dim3(1), dim3(NT), 0, stream, partial, (int64_t)0,
                                          total_dev);
        return;
    }
    hipLaunchKernelGGL(scan_reduce_kernel, dim3((unsigned)nb), dim3(NT), 0, stream, in, n, partial);
    hipLaunchKernelGGL(scan_partials_kernel, dim3(1), dim3(NT), 0, stream, partial, nb, total_dev);
    hipLaunchKernelGGL(scan_down_kernel, dim3((unsigned)nb), dim3(NT), 0, stream, in, n,
                       (const uint64_t*)partial, out);
}

void launch_duplicate(hipStream_t stream, const float* rec, const float* radius, const float* depth,
                      const uint32_t* tiles, const uint32_t* offsets, int64_t n_records, int64_t n_per_view,
                      const ViewSet& views, const DevSettings& st, uint64_t* keys, uint32_t* vals, int64_t capacity,
                      uint32_t* flags) {
    if (n_records == 0) return;
    hipLaunchKernelGGL(duplicate_kernel, dim3((unsigned)((n_records + 255) / 256)), dim3(256), 0, stream,
                       reinterpret_cast<const float4*>(rec), radius, depth, tiles, offsets, n_records, n_per_view,
                       views, st, keys, vals, capacity, flags);
}

size_t sort_scratch_bytes(int64_t K) {
    // workgroups of a sort of K keys: at most one per tile of the smallest
    // tile size plus one per segment (at most MAX_SORT_SEGMENTS), and at
    // most SORT_BLOCKS (the launcher's bound)
    const int64_t nb = std::min<int64_t>(((K > 0 ? K : 1) + SORT_TILE_MIN - 1) / SORT_TILE_MIN + MAX_SORT_SEGMENTS,
                                         SORT_BLOCKS);
    const int64_t hist = nb * RADIX;
    return (size_t)(2 * hist + MAX_SORT_SEGMENTS * RADIX) * sizeof(uint32_t) + 1024;
}

void launch_radix_sort(hipStream_t stream, uint64_t* keys, uint32_t* vals, uint64_t* keys_alt, uint32_t* vals_alt,
                       int64_t K, const uint64_t* K_dev, int key_bits, void* scratch, bool* out_in_alt) {
    radix_sort_t<uint64_t>(stream, keys, vals, keys_alt, vals_alt, K, K_dev, 0, key_bits, scratch, out_in_alt);
}

bool cell_keys16(int64_t K, int64_t cells) { return cells < 0xffff && K > SHORT_MAX; }

bool launch_cell_sort(hipStream_t stream, void* keys, uint32_t* vals, void* keys_alt, uint32_t* vals_alt, bool keys16,
                      int64_t K, const uint64_t* K_dev, int bits, void* scratch, bool* out_in_alt, uint32_t* ranges,
                      int64_t nbins) {
    if (keys16)
        return radix_sort_t<uint16_t>(stream, (uint16_t*)keys, vals, (uint16_t*)keys_alt, vals_alt, K, K_dev, 0, bits,
                                      scratch, out_in_alt);
    return radix_sort_t<uint32_t>(stream, (uint32_t*)keys, vals, (uint32_t*)keys_alt, vals_alt, K, K_dev, 0, bits,
                                  scratch, out_in_alt, 0, ranges, nbins);
}

bool launch_depth_sort(hipStream_t stream, uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                       int64_t K, int64_t seg_len, void* scratch, bool* out_in_alt, uint32_t* live) {
    if (seg_len > 0 && (K + seg_len - 1) / seg_len > MAX_SORT_SEGMENTS) seg_len = 0;  // not reached: views <= 16
    bool dropped = false;
    radix_sort_t<uint32_t>(stream, keys, vals, keys_alt, vals_alt, K, nullptr, 0, 32, scratch, out_in_alt, seg_len,
                           nullptr, 0, live, &dropped);
    return dropped;
}

void launch_tile_ranges(hipStream_t stream, const uint64_t* keys, int64_t K, const uint64_t* K_dev,
                        int64_t total_tiles, uint32_t* ranges) {
    launch_fill_u32(stream, ranges, 2 * total_tiles, 0u);
    if (K == 0) return;
    hipLaunchKernelGGL(tile_ranges_kernel<uint64_t>, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, stream, keys, K,
                       K_dev, 32, (uint64_t)total_tiles, reinterpret_cast<uint2*>(ranges));
}

void launch_cell_ranges(hipStream_t stream, const void* keys, bool keys16, int64_t K, const uint64_t* K_dev,
                        int64_t cells, uint32_t* ranges) {
    if (K == 0) return;
    // keys come from the library's own buffers (16-byte aligned)
    const dim3 grid((unsigned)((K + 1023) / 1024));
    uint2* r = reinterpret_cast<uint2*>(ranges);
    if (keys16)
        hipLaunchKernelGGL(tile_ranges4_kernel<uint16_t>, grid, dim3(256), 0, stream, (const uint16_t*)keys, K, K_dev,
                           (uint64_t)cells, r);
    else
        hipLaunchKernelGGL(tile_ranges4_kernel<uint32_t>, grid, dim3(256), 0, stream, (const uint32_t*)keys, K, K_dev,
                           (uint64_t)cells, r);
}

void launch_fill_u32(hipStream_t stream, uint32_t* p, int64_t n, uint32_t value) {
    if (n <= 0) return;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p, n, value);
}

FillSet make_fill_set(const FillSpan* spans, int count) {
    FillSet fs{};
    for (int k = 0; k < count && fs.count < FILL_SPANS; ++k) {
        if (!spans[k].p || spans[k].n <= 0) continue;
        fs.total += spans[k].n;
        fs.p[fs.count] = spans[k].p;
        fs.end[fs.count] = fs.total;
        fs.v[fs.count] = spans[k].value;
        ++fs.count;
    }
    return fs;
}

void launch_fill_spans(hipStream_t stream, const FillSpan* spans, int count) {
    const FillSet fs = make_fill_set(spans, count);
    if (fs.total == 0) return;
    hipLaunchKernelGGL(fill_set_kernel, dim3((unsigned)((fs.total + 255) / 256)), dim3(256), 0, stream, fs);
}

void launch_round_f64(hipStream_t stream, const double* in, float* out, int64_t n) {
    if (n <= 0) return;
    hipLaunchKernelGGL(round_f64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, in, out, n);
}

void launch_fill_f32(hipStream_t stream, float* p, int64_t n, float value) {
    if (n <= 0) return;
    hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p, n, value);
}

void launch_sum_i32x4(hipStream_t stream, const int32_t* in, int64_t n, uint64_t* out_dev, void* scratch) {
    const int64_t nb = nblocks(n > 0 ? n : 1);
    uint64_t* partial = reinterpret_cast<uint64_t*>(scratch);
    hipLaunchKernelGGL(sum_i32x4_partial_kernel, dim3((unsigned)nb), dim3(NT), 0, stream,
                       reinterpret_cast<const int4*>(in), n, partial, nb);
    for (int c = 0; c < 4; ++c)
        hipLaunchKernelGGL(scan_partials_kernel, dim3(1), dim3(NT), 0, stream, partial + c * nb, nb, out_dev + c);
}

}  // namespace mgs
