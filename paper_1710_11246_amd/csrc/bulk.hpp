// Bulk form of the operations: a batch that holds several operations per bucket is split by
// bucket range first, so that every slab is read once per batch instead of once per operation.
// Included by slabhash.hip, inside its unnamed namespace.
//
//   split   each workgroup takes a tile of the batch and orders it by part (a part is `span`
//           consecutive buckets), in LDS; the tile's operations go to the caller's workspace in
//           that order, with each operation's place (16 bits) and the tile's part starts.
//   probe   one workgroup per part: the part's base slabs go to LDS, the part's operations are
//           gathered from every tile's run and answered there; results replace the operations.
//   merge   each tile's results go back to the batch's order, through LDS.
//
// Times of the kernels (us; 217,316 buckets at 2^22 operations, 3,477,982 at 2^26; searches: the
// mean of all present and all absent):
//
//                     plain   bulk   of it: split   probe / insert   later   merge
//   2^22 searches       149     67             16               42               9
//   2^26 searches      2890   1440            207             1070             167
//   2^22 inserts        239    110             21               73      11       5
//   2^26 inserts       4260   2060            298             1680      19      60
//
// The plain form reads 256 bytes at random per operation, and an insert swaps 8. Split and merge
// are bound by memory at 2^26 (split moves 11 bytes per search and 18 per insert: 3.7 and 4.1 TB/s;
// a searches' merge 12: 4.8), by the ends of their tiles' phases at 2^22. Probe and insert are
// bound by the chain of waits of a part (run starts, operations, slabs, and the swap and the stores
// of an insert), which other parts on the same compute unit cover: three of 8 wavefronts at 2^22
// operations, none at 2^26, where a part of 16 wavefronts and its slabs fill the LDS (parts that
// leave room for a second make the runs too short: 256 slabs instead of 340 took 2^26 searches
// 1.68 ms instead of 1.53). (Slabs left out of LDS, with only their tags there and a found pair
// read from L2: more parts per compute unit, but 2^22 searches 64 -> 73 us and 2^26 1533 -> 1762.)
//
// A run of a tile is a few operations (tile / parts), less than a cache line. Workgroups b,
// b + 8, b + 16, ... share an XCD, so they take consecutive parts: the lines their runs share
// then meet in that XCD's L2.

#include "bulk_plan.hpp"

// Inclusive sum over the wavefront's lanes: four shifts within rows of 16 lanes, then the sums of
// the rows before (lane 15 of rows 0 and 2 to rows 1 and 3, lane 31 to rows 2 and 3).
template <int Ctrl, int Rows>
__device__ __forceinline__ uint32_t add_dpp(uint32_t x)
{
    return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, Ctrl, Rows, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t x)
{
    x = add_dpp<0x111, 0xF>(x);
    x = add_dpp<0x112, 0xF>(x);
    x = add_dpp<0x114, 0xF>(x);
    x = add_dpp<0x118, 0xF>(x);
    x = add_dpp<0x142, 0xA>(x);
    return add_dpp<0x143, 0xC>(x);
}

// Exclusive sum over the workgroup's threads (NW wavefronts); *total receives the sum. `tmp`
// holds NW words of LDS; two barriers inside.
template <int NW>
__device__ __forceinline__ uint32_t block_scan(uint32_t x, uint32_t *tmp, uint32_t *total)
{
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
    const uint32_t incl = wave_scan(x);
    if (lane == 63)
        tmp[w] = incl;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const uint32_t v = tmp[i];
        before += (uint32_t)i < w ? v : 0u;
        sum += v;
    }
    __syncthreads();
    *total = sum;
    return before + incl - x;
}

// Popular keys repeat within a tile, and would all fall to one part's workgroup. Where a tile's
// run of one part is longer than distinct keys make it, the run's keys are entered in a small
// hash table, and a repeated key takes the place of its first operation: it is answered once per
// tile, and the merge hands the answer to every repetition.
//
// LDS: the tile's words (before they are staged, the repeated keys' table), the part counters
// (two 16-bit ones per word) and the scan's wavefront sums.
template <int R, bool Vals>
__global__ __launch_bounds__(kSplitThreads) void split_kernel(View T, Bulk A,
                                                              const uint32_t *__restrict__ keys,
                                                              const uint32_t *__restrict__ vals,
                                                              uint64_t n, uint32_t reserve_from)
{
    extern __shared__ uint32_t sm[];
    constexpr uint32_t kTile = kSplitThreads * R, kTable = kTile / 2;
    constexpr uint32_t kTableBits = __builtin_ctz(kTable);
    uint32_t *stage = sm, *cnt = sm + kTile, *tmp = cnt + A.row;
    uint32_t *tkey = stage, *trank = stage + kTable; // the table: keys and their ranks
    const uint32_t tid = threadIdx.x, tile = blockIdx.x;
    const uint64_t base = (uint64_t)tile * kTile;
    const uint32_t count = (n - base < kTile) ? (uint32_t)(n - base) : kTile;
    const uint32_t *in = keys + base;
    const bool wide = (reinterpret_cast<uintptr_t>(in) & 15u) == 0;
    auto index = [&](int j) { return (j / 4) * (4 * kSplitThreads) + tid * 4 + (j & 3); };
    uint32_t k[R], pr[R]; // keys; part << 16 | rank in the tile's run of the part
#pragma unroll
    for (int j = 0; j < R; j += 4) {
        const uint32_t i = index(j);
        if (wide && i + 4 <= count) {
            const uint4 v = *reinterpret_cast<const uint4 *>(in + i);
            k[j] = v.x, k[j + 1] = v.y, k[j + 2] = v.z, k[j + 3] = v.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                k[j + e] = i + e < count ? in[i + e] : 0u;
        }
    }
    for (uint32_t i = tid; i < A.row; i += kSplitThreads)
        cnt[i] = 0u;
    if (tid == 0)
        tmp[kSplitThreads / 64] = 0u;
    if (Vals && tile == 0 && tid == 0)
        *A.later_count = 0u;
    __syncthreads();
    auto rank_of = [&](uint32_t p) {
        const uint32_t sh = (p & 1u) * 16u;
        return (atomicAdd(&cnt[p >> 1], 1u << sh) >> sh) & 0xFFFFu;
    };
    bool bad = false;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (index(j) < count) {
            uint32_t rem;
            const uint32_t p = div_magic(bucket_of(T, k[j]), A.span, A.span_magic, &rem);
            pr[j] = (p << 16) | rank_of(p);
            bad = bad || k[j] >= reserve_from;
        }
    }
    const uint64_t bad_m = ballot(bad);
    if (bad_m)
        raise_error(T, SH_ERR_RESERVED_KEY, lane_id(), ffs0(bad_m));
    __syncthreads();
    const uint32_t per = (A.row + kSplitThreads - 1) / kSplitThreads;
    const uint32_t w0 = tid * per, w1 = w0 + per < A.row ? w0 + per : A.row;
    uint32_t sum = 0;
    bool hot = false;
    for (uint32_t w = w0; w < w1; ++w) {
        const uint32_t c = cnt[w];
        sum += (c & 0xFFFFu) + (c >> 16);
        hot = hot || (c & 0xFFFFu) > A.hot || (c >> 16) > A.hot;
    }
    if (hot)
        tmp[kSplitThreads / 64] = 1u;
    __syncthreads();
    const bool repeats = !Vals && tmp[kSplitThreads / 64] != 0;
    const uint16_t *start = reinterpret_cast<const uint16_t *>(cnt);
    uint32_t inhot = 0, first = 0; // bit j: key j is of a hot run; is its tile's first
    if (repeats) {
        for (uint32_t i = tid; i < kTable; i += kSplitThreads)
            tkey[i] = kEmpty;
        __syncthreads();
        // (eight keys of a thread at a time, their swaps in flight together)
        constexpr int kB = R < 8 ? R : 8;
#pragma unroll
        for (int j0 = 0; j0 < R; j0 += kB) {
            uint32_t h[kB], old[kB], left = 0;
#pragma unroll
            for (int j = 0; j < kB; ++j) {
                h[j] = (k[j0 + j] * 0x9E3779B1u) >> (32 - kTableBits);
                if (index(j0 + j) < count && start[pr[j0 + j] >> 16] > A.hot)
                    left |= 1u << j;
            }
            inhot |= left << j0;
            first |= left << j0;
            for (uint32_t d = 0; d < 8 && left; ++d) {
#pragma unroll
                for (int j = 0; j < kB; ++j)
                    if (((left >> j) & 1u) && k[j0 + j] != kEmpty) // (the empty entry's mark)
                        old[j] = atomicCAS(&tkey[h[j]], kEmpty, k[j0 + j]);
#pragma unroll
                for (int j = 0; j < kB; ++j)
                    if (((left >> j) & 1u) && k[j0 + j] != kEmpty) {
                        if (old[j] == kEmpty || old[j] == k[j0 + j]) {
                            left &= ~(1u << j);
                            if (old[j] != kEmpty)
                                first &= ~(1u << (j0 + j));
                            // the key's entry, in place of its rank
                            pr[j0 + j] = (pr[j0 + j] & 0xFFFF0000u) | h[j];
                        } else {
                            h[j] = (h[j] + 1) & (kTable - 1);
                        }
                    }
            }
            // a key that found no entry is counted as if it were the only one
#pragma unroll
            for (int j = 0; j < kB; ++j)
                if ((left >> j) & 1u)
                    pr[j0 + j] = (pr[j0 + j] & 0xFFFF0000u) | kTable;
        }
        __syncthreads();
        // the hot runs are counted again, without the repetitions
#pragma unroll
        for (int j = 0; j < R; ++j)
            if ((inhot >> j) & 1u)
                reinterpret_cast<uint16_t *>(cnt)[pr[j] >> 16] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < R; ++j)
            if ((first >> j) & 1u) {
                const uint32_t rank = rank_of(pr[j] >> 16), at = pr[j] & 0xFFFFu;
                if (at < kTable) {
                    trank[at] = rank;
                } else {
                    pr[j] = (pr[j] & 0xFFFF0000u) | rank;
                    inhot &= ~(1u << j);
                }
            }
        __syncthreads();
        sum = 0;
        for (uint32_t w = w0; w < w1; ++w)
            sum += (cnt[w] & 0xFFFFu) + (cnt[w] >> 16);
    }
    // counts become starts: each thread sums its words, in order
    uint32_t total;
    uint32_t at = block_scan<kSplitThreads / 64>(sum, tmp, &total);
    uint32_t *row = reinterpret_cast<uint32_t *>(A.starts) + (size_t)tile * A.row;
    for (uint32_t w = w0; w < w1; ++w) {
        const uint32_t c = cnt[w];
        const uint32_t s = at | ((at + (c & 0xFFFFu)) << 16);
        at += (c & 0xFFFFu) + (c >> 16);
        cnt[w] = s;
    }
    __syncthreads();
    for (uint32_t i = tid; i < A.row; i += kSplitThreads)
        row[i] = cnt[i];
#pragma unroll
    for (int j = 0; j < R; ++j)
        if (index(j) < count) {
            const uint32_t x = pr[j] & 0xFFFFu;
            pr[j] = start[pr[j] >> 16] + (((inhot >> j) & 1u) ? trank[x] : x);
        }
    if (repeats)
        __syncthreads(); // the table has been read
    // pr: places now
    uint16_t *place = A.place + base;
#pragma unroll
    for (int j = 0; j < R; j += 4) {
        const uint32_t i = index(j);
        uint32_t pos[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pos[e] = 0;
            if (i + e < count) {
                pos[e] = pr[j + e];
                if (!((inhot & ~first) >> (j + e) & 1u))
                    stage[pos[e]] = k[j + e];
            }
        }
        // the places of a tile start at a multiple of its size: always aligned
        if (i < count)
            *reinterpret_cast<uint2 *>(place + i) =
                make_uint2(pos[0] | (pos[1] << 16), pos[2] | (pos[3] << 16));
    }
    __syncthreads();
    uint32_t *out = A.key + base;
    for (uint32_t i = tid * 4; i < total; i += kSplitThreads * 4) {
        *reinterpret_cast<uint4 *>(out + i) = *reinterpret_cast<const uint4 *>(stage + i);
        if constexpr (!Vals)
            *reinterpret_cast<uint32_t *>(A.flag + base + i) = 0u;
    }
    if constexpr (Vals) {
        // the values the same way (no key of an insert is left out as a repetition)
        const uint32_t *vin = vals + base;
        const bool vwide = (reinterpret_cast<uintptr_t>(vin) & 15u) == 0;
#pragma unroll
        for (int j = 0; j < R; j += 4) {
            const uint32_t i = index(j);
            if (vwide && i + 4 <= count) {
                const uint4 v = *reinterpret_cast<const uint4 *>(vin + i);
                k[j] = v.x, k[j + 1] = v.y, k[j + 2] = v.z, k[j + 3] = v.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    k[j + e] = i + e < count ? vin[i + e] : 0u;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (index(j) < count)
                stage[pr[j]] = k[j];
        __syncthreads();
        out = A.val + base;
        for (uint32_t i = tid * 4; i < total; i += kSplitThreads * 4)
            *reinterpret_cast<uint4 *>(out + i) = *reinterpret_cast<const uint4 *>(stage + i);
    }
}

// A part's runs in LDS: first[t] operations of the part precede tile t's (first[tiles]: all of
// them), and operation q of the part, in tile t, is at shift[t] + q of the workspace's arrays.
struct Runs {
    uint32_t *first, *shift;
};

// Writes the runs of the wavefront's lanes (operations lo .. hi - 1 of the queue come from `tile`):
// each lane its own, the wavefront together the long ones.
__device__ __forceinline__ void write_owner(uint16_t *owner, uint32_t lo, uint32_t hi, uint32_t tile)
{
    const bool is_long = hi > lo && hi - lo > 64u;
    if (!is_long)
        for (uint32_t q = lo; q < hi; ++q)
            owner[q] = (uint16_t)tile;
    for (uint64_t m = ballot(is_long); m; m &= m - 1) {
        const uint32_t l = ffs0(m);
        const uint32_t end = rl(hi, l), t = rl(tile, l);
        for (uint32_t q = rl(lo, l) + lane_id(); q < end; q += 64)
            owner[q] = (uint16_t)t;
    }
}

// Reads the part's runs; returns the number of its operations. If one queue holds them all, their
// owners are written too.
template <int NW>
__device__ __forceinline__ uint32_t load_runs(const Bulk &A, uint32_t part, Runs R, uint32_t *tmp,
                                              uint16_t *owner)
{
    constexpr uint32_t kThreads = NW * 64;
    const uint32_t tid = threadIdx.x;
    const uint32_t per = (A.tiles + kThreads - 1) / kThreads;
    const uint32_t t0 = tid * per;
    uint32_t s[kMaxTiles / kThreads];
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < kMaxTiles / kThreads; ++j) {
        s[j] = 0;
        if (j < per && t0 + j < A.tiles) {
            const uint16_t *st = A.starts + (size_t)(t0 + j) * (2 * A.row) + part;
            s[j] = st[0] | ((uint32_t)st[1] << 16);
            sum += (s[j] >> 16) - (s[j] & 0xFFFFu);
        }
    }
    uint32_t total;
    uint32_t at = block_scan<NW>(sum, tmp, &total);
#pragma unroll
    for (uint32_t j = 0; j < kMaxTiles / kThreads; ++j) {
        if (j < per) {
            const uint32_t n = (s[j] >> 16) - (s[j] & 0xFFFFu);
            if (t0 + j < A.tiles) {
                R.first[t0 + j] = at;
                R.shift[t0 + j] = (t0 + j) * A.tile + (s[j] & 0xFFFFu) - at;
            }
            if (total <= A.queue)
                write_owner(owner, at, at + n, t0 + j);
            at += n;
        }
    }
    if (tid == 0)
        R.first[A.tiles] = total;
    return total;
}

// owner[q - q0] = the tile that operation q of the part comes from, for q0 <= q < q1: a part that
// is taken in pieces.
template <int NW>
__device__ __forceinline__ void own_runs(const Bulk &A, const Runs &R, uint32_t q0, uint32_t q1,
                                         uint16_t *owner)
{
    for (uint32_t t0 = threadIdx.x & ~63u; t0 < A.tiles; t0 += NW * 64) {
        const uint32_t t = t0 + lane_id();
        uint32_t lo = q0, hi = q0;
        if (t < A.tiles) {
            const uint32_t a = R.first[t], b = R.first[t + 1];
            lo = a < q0 ? q0 : a;
            hi = b < q1 ? b : q1;
        }
        write_owner(owner, lo - q0, hi < lo ? lo - q0 : hi - q0, t);
    }
}

// An 8-bit tag of a key; the tags of a slab's 32 words are kept so that word s has byte s / 8 of
// 32-bit group s % 8, and one comparison of a group yields the votes of words g, g + 8, ...
__device__ __forceinline__ uint32_t tag_of(uint32_t key) { return (key * 0x9E3779B1u) >> 24; }

// Bit s: word s of the row has the tag.
__device__ __forceinline__ uint32_t tag_votes(const uint32_t *row, uint32_t pattern)
{
    const uint4 a = *reinterpret_cast<const uint4 *>(row);
    const uint4 b = *reinterpret_cast<const uint4 *>(row + 4);
    const uint32_t g[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        // high bit of each zero byte (the borrow may also set bytes above one: a wrong vote
        // costs a comparison of the key)
        const uint32_t x = g[i] ^ pattern;
        m = (m >> 1) | ((x - 0x01010101u) & ~x & 0x80808080u);
    }
    return m;
}

// 32-bit words of tags per row: pairs have one tag per word, key-only slabs one for each of a
// word's two entries.
template <bool KO> constexpr uint32_t kTagWords = KO ? 16u : 8u;

// Searches of one part. LDS: the rows of the part's slabs, their tags, the runs, and a queue of
// the part's searches: their keys, which the results replace, and the tiles they come from. (A
// queue in LDS, not in registers: eight searches a thread in registers left three wavefronts per
// SIMD where this form runs six, and took 62 us where it takes 37: 2^22 searches, 2^22 keys.)
// Lists longer than one slab are taken level by level: while many searches still run, the next
// slab of every list with an open one replaces its row; a wavefront with few left walks their
// lists itself, one per half wavefront. A thread keeps the searches it has not answered as bits,
// search tid + i * threads of the queue in bit i.
template <bool KO, int NW>
__global__ __launch_bounds__(NW * 64) void probe_kernel(View T, Bulk A)
{
    extern __shared__ uint64_t sm8[];
    constexpr uint32_t kThreads = NW * 64;
    constexpr uint32_t kFew = 8; // searches that a wavefront walks itself
    uint64_t *rows = sm8;
    // 16-byte aligned: an even number of 8-byte words comes before it
    uint32_t *tags = reinterpret_cast<uint32_t *>(rows + ((A.span * kRowWords + 1) & ~1u));
    Runs R;
    R.first = tags + A.span * kTagWords<KO>;
    R.shift = R.first + A.tiles + 1;
    uint32_t *tmp = R.shift + A.tiles;
    uint32_t *sh = tmp + NW; // unanswered searches
    uint32_t *queue = sh + 1;
    uint16_t *owner = reinterpret_cast<uint16_t *>(queue + A.queue); // bit 15: found
    uint8_t *open_row = reinterpret_cast<uint8_t *>(owner + A.queue); // its list is read on
    const uint32_t tid = threadIdx.x, lane = lane_id(), wv = tid >> 6;
    const uint32_t half = lane >> 5, slot = lane & 31;
    const uint32_t limit = T.total_blocks * SH_BLOCK_SLABS; // no list has more pool slabs
    // consecutive parts to one XCD
    const uint32_t per_xcd = (A.parts + 7) / 8;
    const uint32_t part = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (part >= A.parts)
        return;
    const uint32_t b0 = part * A.span;
    const uint32_t nb = T.B - b0 < A.span ? T.B - b0 : A.span;

    auto put_row = [&](uint32_t r, uint64_t w) {
        rows[r * kRowWords + slot] = w;
        uint8_t *tg = reinterpret_cast<uint8_t *>(tags + r * kTagWords<KO>) + (slot & 7u) * 4 +
                      (slot >> 3);
        *tg = (uint8_t)tag_of((uint32_t)w);
        if constexpr (KO)
            tg[32] = (uint8_t)tag_of((uint32_t)(w >> 32));
    };
    // the part's base slabs, two per load: eight loads in flight per wavefront
    constexpr int kRowLoads = 8;
    uint64_t w[kRowLoads];
    auto fetch_rows = [&](uint32_t r0) {
#pragma unroll
        for (int u = 0; u < kRowLoads; ++u) {
            const uint32_t r = r0 + u * NW * 2 + half;
            w[u] = r < nb ? *gmem(T.base + (size_t)(b0 + r) * 32 + slot) : 0ull;
        }
    };
    auto put_rows = [&](uint32_t r0) {
#pragma unroll
        for (int u = 0; u < kRowLoads; ++u) {
            const uint32_t r = r0 + u * NW * 2 + half;
            if (r < nb)
                put_row(r, w[u]);
        }
    };
    fetch_rows(wv * 2); // in flight while the runs are read and summed
    for (uint32_t r = tid; r < A.span; r += kThreads)
        open_row[r] = 0;
    const uint32_t total = load_runs<NW>(A, part, R, tmp, owner);
    put_rows(wv * 2);
    bool fresh = true, have = true; // rows to be read; the first of them already there
    for (uint32_t q0 = 0; q0 < total; q0 += A.queue) {
        const uint32_t count = total - q0 < A.queue ? total - q0 : A.queue;
        if (total > A.queue) {
            __syncthreads(); // the runs are there, and the last piece is done
            own_runs<NW>(A, R, q0, q0 + count, owner);
        }
        if (fresh) {
            for (uint32_t r0 = wv * 2 + (have ? NW * 2 * kRowLoads : 0); r0 < nb;
                 r0 += NW * 2 * kRowLoads) {
                fetch_rows(r0);
                put_rows(r0);
            }
            have = fresh = false;
        }
        if (tid == 0)
            sh[0] = 0;
        __syncthreads();
        // each thread fetches the keys that it will look up: no barrier in between
        for (uint32_t i = tid; i < count; i += 4 * kThreads) {
            uint32_t k[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t q = i + u * kThreads;
                k[u] = q < count ? A.key[R.shift[owner[q]] + q0 + q] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u * kThreads < count)
                    queue[i + u * kThreads] = k[u];
        }

        uint64_t undone = 0;
        for (uint32_t level = 0;; ++level) {
            uint64_t bit = 1;
            for (uint32_t q = tid; q < count; q += kThreads, bit <<= 1) {
                if (level && !(undone & bit))
                    continue;
                const uint32_t key = queue[q];
                const uint32_t r = bucket_of(T, key) - b0;
                const uint64_t *row = rows + r * kRowWords;
                const uint32_t pattern = tag_of(key) * 0x01010101u;
                // reserved keys match nothing
                const bool valid = key < (KO ? kTombKey : kEmpty);
                uint32_t m = tag_votes(tags + r * kTagWords<KO>, pattern);
                if constexpr (KO)
                    m |= tag_votes(tags + r * kTagWords<KO> + 8, pattern);
                m &= valid ? (uint32_t)kSlotMask : 0u;
                bool hit = false;
                uint32_t val = kEmpty;
                while (m) {
                    const uint64_t x = row[__builtin_ctz(m)];
                    m &= m - 1u;
                    if ((uint32_t)x == key || (KO && (uint32_t)(x >> 32) == key)) {
                        hit = true;
                        val = KO ? key : (uint32_t)(x >> 32);
                        break; // the first of the list
                    }
                }
                const uint32_t next = (uint32_t)(row[31] >> 32);
                if (hit || next == kEmpty || !valid || level > limit) {
                    queue[q] = val;
                    if (hit)
                        owner[q] |= 0x8000u;
                    undone &= ~bit;
                } else {
                    undone |= bit;
                    open_row[r] = 1;
                }
            }
            uint32_t mine = (uint32_t)__popcll(undone);
            if (ballot(mine != 0)) {
                uint32_t open = rl(wave_scan(mine), 63);
                if (open <= kFew) {
                    for (uint32_t i = 0; open; ++i) {
                        const bool me = (undone >> i) & 1ull;
                        const uint32_t q = tid + i * kThreads;
                        const uint32_t key = me ? queue[q] : 0u;
                        const uint32_t next =
                            me ? (uint32_t)(rows[(bucket_of(T, key) - b0) * kRowWords + 31] >> 32)
                               : kEmpty;
                        for (uint64_t m = ballot(me); m;) {
                            const uint32_t ja = ffs0(m);
                            m &= m - 1;
                            const bool two = m != 0;
                            const uint32_t jb = two ? ffs0(m) : ja;
                            m = two ? m & (m - 1) : m;
                            open -= two ? 2u : 1u;
                            const uint32_t k = half ? rl(key, jb) : rl(key, ja);
                            uint32_t nx = half ? (two ? rl(next, jb) : kEmpty) : rl(next, ja);
                            uint32_t val = kEmpty, hit = 0, steps = 0;
                            bool go = nx != kEmpty && pool_in_range(T, nx);
                            while (ballot(go)) {
                                const uint64_t x = go ? *gmem(pool_slab(T, nx) + slot) : 0ull;
                                const bool is = go && slot < 31 &&
                                                ((uint32_t)x == k ||
                                                 (KO && (uint32_t)(x >> 32) == k));
                                const uint32_t mm = (uint32_t)(ballot(is) >> (lane & 32u));
                                const uint32_t src =
                                    (lane & 32u) | (mm ? (uint32_t)__builtin_ctz(mm) : 31u);
                                const uint32_t hv =
                                    (uint32_t)__shfl((int)(uint32_t)(x >> 32), (int)src, 64);
                                if (go && mm) {
                                    val = KO ? k : hv;
                                    hit = 1;
                                    go = false;
                                } else if (go) {
                                    nx = hv;
                                    go = nx != kEmpty && pool_in_range(T, nx) && ++steps <= limit;
                                }
                            }
                            const uint32_t va = rl(val, 0), vb = rl(val, 32);
                            const uint32_t ha = rl(hit, 0), hb = rl(hit, 32);
                            if (lane == ja || (two && lane == jb)) {
                                queue[q] = lane == ja ? va : vb;
                                if (lane == ja ? ha : hb)
                                    owner[q] |= 0x8000u;
                            }
                        }
                    }
                    undone = 0;
                } else if (lane == 63) {
                    atomicAdd(&sh[0], open);
                }
            }
            __syncthreads();
            if (sh[0] == 0)
                break;
            __syncthreads();
            if (tid == 0)
                sh[0] = 0;
            __syncthreads();
            // the next slab of every list with an open search replaces its row (a list without a
            // next slab has none)
            fresh = true;
            for (uint32_t r0 = wv * 2; r0 < nb; r0 += NW * 2 * kRowLoads) {
                uint32_t has = 0;
#pragma unroll
                for (int u = 0; u < kRowLoads; ++u) {
                    const uint32_t r = r0 + u * NW * 2 + half;
                    const uint32_t nx = r < nb && open_row[r]
                                            ? (uint32_t)(rows[r * kRowWords + 31] >> 32)
                                            : kEmpty;
                    has |= nx != kEmpty ? 1u << u : 0u;
                    w[u] = nx != kEmpty && pool_in_range(T, nx) ? *gmem(pool_slab(T, nx) + slot)
                                                                : ~0ull;
                }
#pragma unroll
                for (int u = 0; u < kRowLoads; ++u)
                    if ((has >> u) & 1u) {
                        put_row(r0 + u * NW * 2 + half, w[u]);
                        open_row[r0 + u * NW * 2 + half] = 0;
                    }
            }
            __syncthreads();
        }
        for (uint32_t q = tid; q < count; q += kThreads) {
            const uint32_t o = owner[q], at = R.shift[o & 0x7FFFu] + q0 + q;
            const uint32_t val = queue[q];
            A.key[at] = val;
            // Only what the value does not tell (split has written zeros, whole lines): a run's
            // flags are a few bytes of a line, and writing them all took 2^26 searches 96 us.
            if (val == kEmpty && (o >> 15))
                A.flag[at] = 1;
        }
    }
}

// Inserts of one part, on a unique-key pair table (REPLACE). They are gathered by bucket in LDS,
// and half a wavefront per slab commits them to the table: one that finds its key gives the slot
// its value (status 2), another takes the next empty slot (status 1).
//
//   new pairs    the first empty slot is swapped to kLockPair, the pairs of the slots after it
//                are stored in one piece, and the pair of the locked slot is stored last. Slots
//                fill in order: an insert of another kernel that has read the slab meets the lock
//                at the first empty slot and reads the slab again, so no key can enter twice.
//                (One new pair is swapped in as it is.)
//   new values   each replaced slot is swapped from what it holds now, key unchanged. Only pairs
//                whose bit of the bucket's 512 an insert has set (see below) are compared with the
//                inserts: comparing every pair took 2^22 inserts on 19 pairs a bucket, 6 more
//                each, 472 us where this takes 319 (plain 332).
//
// What a list of one slab has no room for goes to a new slab, whole before it is linked (left to
// the plain kernel, where a wavefront adds one slab a round, the 2500 such pairs of 2^22 took
// 17 us). What loses a swap to another kernel's update, and the inserts into longer lists, are
// listed for the plain kernel, which runs next. A half wavefront takes four slabs at a time, and
// their locks open together: after three memory round trips (its own swap, the stores, the opening)
// where no list grows, and after up to eleven more for each of the four that does (eight bitmap
// words tried, the new pairs, the link, and if it is lost the clearing). It waits for nothing else
// meanwhile. (Opening the locks of lists that do not grow first took the kernel 76.4 us instead of
// 75.1: 2^22 inserts in 217,000 buckets.)
//
// One swap a slab instead of one a pair, and stores of whole runs of slots: 2^22 random swaps
// take 158 us on this memory, swaps of 19 adjacent slots 49 us, stores of them 18 us.
//
// A bucket's inserts are lined up in LDS by counting, up to 32; the slab itself stays in
// registers, a slot per lane, and meets the lane that holds the insert of its place in line.
// Inserts of one key must not take two slots: each sets one of 512 bits of its bucket, and one
// that finds its bit set, or no place, looks through the line. Where the line holds its key, one
// of that key's inserts keeps its place for all of them: the one whose bit was clear, or else (two
// keys share the bit) the first of the line. It is made last, so its value stays and it finds the
// key there; a new key is new to one of the others. A popular key so costs one swap a piece and a
// look through LDS per insert, whatever the length of its run. (Comparing the groups of each key in
// the commit, and leaving what had no place in line to the plain kernel, took the kernel 31.7 us
// where this takes 21.1 with every key twice, 2^18 in 40,960 buckets; 92 us and 86 more in the
// plain kernel where this takes 71 and 9 with Zipf(0.8) keys, 2^18 in 21,845; and 71.8 us where
// this takes 73.8 with distinct keys, 2^22 in 217,000.)
template <int NW>
__global__ __launch_bounds__(NW * 64) void insert_kernel(View T, Bulk A)
{
    extern __shared__ uint64_t sm8[];
    constexpr uint32_t kThreads = NW * 64;
    constexpr uint32_t kLater = 3; // results beside the statuses 0, 1, 2
    constexpr uint32_t kNewOther = 4; // new to another insert of the key; this one replaced it
    constexpr uint32_t kNoLine = 0x8000u; // `line` of an insert without a place: | its result
    // `owner`: the tile, and whether the insert's key keeps another's place in line, and whether
    // this one is the insert that a new key is new to
    constexpr uint32_t kRepeat = 0x8000u, kNewTo = 0x4000u, kTileOf = 0x3FFFu;
    uint64_t *pairs = sm8; // the buckets' lines
    uint32_t *sig = reinterpret_cast<uint32_t *>(pairs + ((A.span * kRowWords + 1) & ~1u));
    uint8_t *res = reinterpret_cast<uint8_t *>(pairs); // a line's results, once its pairs are read
    uint32_t *cnt = sig + A.span * kSigWords;
    uint32_t *again = cnt + A.span;  // bit i: the line's insert i found its bit set
    uint32_t *shared = again + A.span; // bit i: it keeps its place for others of its key too
    Runs R;
    R.first = shared + A.span;
    R.shift = R.first + A.tiles + 1;
    uint32_t *tmp = R.shift + A.tiles;
    uint16_t *owner = reinterpret_cast<uint16_t *>(tmp + NW);
    uint16_t *line = owner + A.queue; // bucket * 32 + place in line
    const uint32_t tid = threadIdx.x, lane = lane_id(), wv = tid >> 6;
    const uint32_t half = lane >> 5, slot = lane & 31, hshift = lane & 32;
    const uint32_t below = (1u << slot) - 1u;
    const uint32_t per_xcd = (A.parts + 7) / 8;
    const uint32_t part = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if (part >= A.parts)
        return;
    const uint32_t b0 = part * A.span;
    const uint32_t nb = T.B - b0 < A.span ? T.B - b0 : A.span;

    // lists the inserts of the lanes that say so
    auto leave = [&](bool yes, uint32_t pos) {
        const uint64_t m = ballot(yes);
        if (!m)
            return;
        uint32_t at = 0;
        if (lane == ffs0(m))
            at = __hip_atomic_fetch_add(gmem(A.later_count), (uint32_t)__popcll(m),
                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        at = rl(at, ffs0(m)) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (yes)
            A.later[at] = pos;
    };
    auto half_of = [&](uint64_t m) { return (uint32_t)(m >> hshift); };
    // A new slab for the pairs of the half's lanes that say so, linked to the slab whose last word
    // is `last`; true for the lanes whose pair is in the table then. The slab is taken from the
    // table's own pool with one try per bitmap word, and a full pool, like a link lost to another
    // kernel's, leaves the pairs to the plain kernel. Where the caller holds the slab's lock the
    // link is not lost: no one else sees the slab full.
    auto add_slab = [&](uint64_t *last, bool over, uint64_t pair, uint32_t seed) {
        const uint32_t om = half_of(ballot(over));
        const uint32_t words = T.nblk * 64, place = (uint32_t)__popc(om & below);
        uint32_t idx = kEmpty, lk = 0;
        if (om && slot == 0 && words) {
            uint32_t at = __umulhi(seed, words);
            for (int tries = 0; tries < 8 && idx == kEmpty; ++tries) {
                const uint32_t bit = seed & 31u;
                if (!((or32(T.bitmap + at, 1u << bit) >> bit) & 1u))
                    idx = at * 32 + bit;
                seed = mix32(seed);
                at = at + 1 == words ? 0u : at + 1;
            }
        }
        idx = (uint32_t)__shfl((int)idx, (int)hshift, 64);
        const bool put = over && idx != kEmpty && place < 31;
        uint64_t *fresh = pool_slab(T, idx != kEmpty ? idx : 0u) + place;
        if (put)
            __hip_atomic_store(gmem(fresh), pair, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" ::: "memory");
        wait_vm_all(); // the pairs, and the stores before them, come before the link
        asm volatile("" ::: "memory");
        if (idx != kEmpty && slot == 0)
            lk = cas32(reinterpret_cast<uint32_t *>(last) + 1, kEmpty, idx);
        const bool linked = (uint32_t)__shfl((int)lk, (int)hshift, 64) == kEmpty;
        if (!linked) {
            // a free slab is all ones
            if (put)
                __hip_atomic_store(gmem(fresh), kEmptyPair, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("" ::: "memory");
            wait_vm_all();
            asm volatile("" ::: "memory");
            if (idx != kEmpty && slot == 0)
                slab_free(T, idx);
        }
        return put && linked;
    };
    constexpr int kRowLoads = 8;
    uint64_t w[kRowLoads];
    auto fetch_rows = [&](uint32_t r0) {
#pragma unroll
        for (int u = 0; u < kRowLoads; ++u) {
            const uint32_t r = r0 + u * NW * 2 + half;
            w[u] = r < nb ? load_slot<true>(T.base + (size_t)(b0 + r) * 32 + slot) : 0ull;
        }
    };
    fetch_rows(wv * 2); // in flight while the runs are read and summed
    const uint32_t total = load_runs<NW>(A, part, R, tmp, owner);
    bool have = true;
    for (uint32_t q0 = 0; q0 < total; q0 += A.queue) {
        const uint32_t count = total - q0 < A.queue ? total - q0 : A.queue;
        if (total > A.queue) {
            __syncthreads(); // the runs are there, and the last piece is done
            own_runs<NW>(A, R, q0, q0 + count, owner);
        }
        for (uint32_t i = tid; i < A.span * (kSigWords + 3); i += kThreads)
            sig[i] = 0u; // (and the counts)
        __syncthreads();
        uint32_t look = 0; // bit j: insert tid + j * kThreads looks through its line
        uint32_t j0 = 0;
        for (uint32_t i = tid; i < count; i += 4 * kThreads, j0 += 4) {
            uint32_t k[4], v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t q = i + u * kThreads;
                const uint32_t pos = q < count ? R.shift[owner[q]] + q0 + q : 0u;
                k[u] = q < count ? A.key[pos] : kEmpty;
                v[u] = q < count ? A.val[pos] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t q = i + u * kThreads;
                if (q >= count)
                    continue;
                uint32_t l = kNoLine;
                if (k[u] != kEmpty) {
                    const uint32_t r = bucket_of(T, k[u]) - b0;
                    const uint32_t at = atomicAdd(&cnt[r], 1u);
                    l = kNoLine | kLater;
                    bool looks = true;
                    if (at < 32u) {
                        pairs[r * kRowWords + at] = ((uint64_t)v[u] << 32) | k[u];
                        const uint32_t h = (k[u] * 0x9E3779B1u) >> 23;
                        const uint32_t old = atomicOr(&sig[r * kSigWords + (h >> 5)],
                                                      1u << (h & 31u));
                        looks = (old >> (h & 31u)) & 1u;
                        if (looks)
                            atomicOr(&again[r], 1u << at);
                        l = r * 32 + at;
                    }
                    look |= looks ? 1u << (j0 + u) : 0u;
                }
                line[q] = (uint16_t)l;
            }
        }
        __syncthreads();
        for (; look; look &= look - 1u) {
            const uint32_t q = tid + (uint32_t)__builtin_ctz(look) * kThreads;
            const uint32_t l = line[q];
            uint32_t r = l >> 5, key;
            if (l & kNoLine) {
                key = A.key[R.shift[owner[q]] + q0 + q];
                r = bucket_of(T, key) - b0;
            } else {
                key = (uint32_t)pairs[r * kRowWords + (l & 31u)];
            }
            const uint32_t c = cnt[r] < 32u ? cnt[r] : 32u;
            uint32_t is = 0; // the line's inserts of this key (a place given up in this loop
                             // meanwhile may be missing: it is not the one that is kept)
            for (uint32_t j = 0; j < c; j += 16)
#pragma unroll
                for (uint32_t i = 0; i < 16; ++i)
                    is |= (uint32_t)pairs[r * kRowWords + j + i] == key ? 1u << (j + i) : 0u;
            is &= c < 32u ? (1u << c) - 1u : ~0u;
            if (!is)
                continue; // (no place and no one to share one with)
            const uint32_t clear = is & ~again[r];
            const uint32_t kept = r * 32 + (uint32_t)__builtin_ctz(clear ? clear : is);
            if (kept == l)
                continue;
            const uint32_t bit = 1u << (kept & 31u);
            owner[q] |= (atomicOr(&shared[r], bit) & bit) ? kRepeat : kRepeat | kNewTo;
            line[q] = (uint16_t)kept;
            if (!(l & kNoLine))
                pairs[r * kRowWords + (l & 31u)] = kEmptyPair; // gives up its place
        }
        __syncthreads();
        for (uint32_t r0 = wv * 2; r0 < nb; r0 += NW * 2 * kRowLoads) {
            if (!have)
                fetch_rows(r0);
            have = false;
            constexpr int kC = 4; // slabs of a half wavefront whose swaps are in flight together
#pragma unroll
            for (int u0 = 0; u0 < kRowLoads; u0 += kC) {
                uint64_t pr[kC], old[kC], want[kC];
                uint32_t to[kC], out[kC]; // the slot; the result if all goes well
                uint32_t e[kC], fresh[kC];
                auto row_of = [&](int u) { return r0 + (u0 + u) * NW * 2 + half; };
                auto global = [&](int u, uint32_t s) {
                    return T.base + (size_t)(b0 + row_of(u)) * 32 + s;
                };
                auto new_to = [&](int u) { // the result of a lane's new key
                    return (shared[row_of(u)] >> slot) & 1u ? kNewOther : 1u;
                };
#pragma unroll
                for (int u = 0; u < kC; ++u) {
                    const uint64_t x = w[u0 + u];
                    const bool in = row_of(u) < nb;
                    const uint32_t c = in ? cnt[row_of(u)] : 0u;
                    pr[u] = slot < c ? pairs[row_of(u) * kRowWords + slot] : kEmptyPair;
                    const uint32_t key = (uint32_t)pr[u];
                    const bool has = key != kEmpty;
                    const uint32_t ev = half_of(ballot(x == kEmptyPair));
                    const uint32_t locked = half_of(ballot(x == kLockPair));
                    e[u] = locked ? 31u : (uint32_t)__builtin_ctz(ev | 0x80000000u);
                    to[u] = 32;
                    out[u] = has ? kLater : 0u;
                    want[u] = kEmptyPair;
                    // keys that are there: the live pairs whose bit an insert has set, one after
                    // another
                    const uint32_t h = ((uint32_t)x * 0x9E3779B1u) >> 23;
                    const uint32_t bits = in ? sig[row_of(u) * kSigWords + (h >> 5)] : 0u;
                    const uint64_t live = ballot(slot < 31 && (uint32_t)x != kEmpty &&
                                                 ((bits >> (h & 31u)) & 1u));
                    for (uint32_t m = (uint32_t)live | (uint32_t)(live >> 32); m; m &= m - 1) {
                        const uint32_t s = (uint32_t)__builtin_ctz(m);
                        const uint32_t ka = rl((uint32_t)x, s), kb = rl((uint32_t)x, s + 32);
                        const uint32_t va = rl((uint32_t)(x >> 32), s);
                        const uint32_t vb = rl((uint32_t)(x >> 32), s + 32);
                        if (has && key == (half ? kb : ka)) {
                            to[u] = s;
                            want[u] = ((uint64_t)(half ? vb : va) << 32) | key;
                        }
                    }
                    const uint32_t nm = half_of(ballot(has && to[u] == 32));
                    const uint32_t place = e[u] + (uint32_t)__popc(nm & below);
                    if (has && to[u] < 32) {
                        out[u] = 2;
                    } else if (has && place < 31) {
                        to[u] = place;
                        out[u] = new_to(u);
                    } else if (has && (ev >> 31) && !locked) {
                        to[u] = 33; // a list of one full slab
                    }
                    fresh[u] = nm ? (uint32_t)__popc(nm) : 0u;
                    if (fresh[u] > 31u - e[u])
                        fresh[u] = 31u - e[u];
                    const bool opens = has && want[u] == kEmptyPair && to[u] == e[u];
                    old[u] = want[u];
                    if (has && (opens ? to[u] < 31 : want[u] != kEmptyPair))
                        old[u] = cas64(global(u, to[u]), want[u],
                                       opens && fresh[u] > 1 ? kLockPair : pr[u]);
                }
#pragma unroll
                for (int u = 0; u < kC; ++u) {
                    const bool isnew = want[u] == kEmptyPair && to[u] < 31;
                    const bool no = half_of(ballot(isnew && old[u] != kEmptyPair)) != 0u;
                    if (old[u] != want[u] || (isnew && no))
                        out[u] = kLater;
                    else if (isnew && to[u] > e[u])
                        __hip_atomic_store(gmem(global(u, to[u])), pr[u], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    if (no)
                        fresh[u] = 0;
                    if (ballot(to[u] > 32)) {
                        const bool over = to[u] > 32 && !no;
                        if (add_slab(global(u, 31), over, pr[u], mix32(b0 + row_of(u))))
                            out[u] = new_to(u);
                    }
                }
                // the stores have reached memory before the locks open
                asm volatile("" ::: "memory");
                wait_vm_all();
                asm volatile("" ::: "memory");
#pragma unroll
                for (int u = 0; u < kC; ++u) {
                    if (want[u] == kEmptyPair && fresh[u] > 1 && to[u] == e[u])
                        __hip_atomic_store(gmem(global(u, to[u])), pr[u], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    if (row_of(u) < nb)
                        res[row_of(u) * (kRowWords * 8) + slot] = (uint8_t)out[u];
                }
            }
        }
        if (q0 + A.queue < total)
            wait_vm_all(); // the next piece reads the slabs again
        __syncthreads();
        for (uint32_t i = tid & ~63u; i < count; i += kThreads) {
            const uint32_t q = i + lane;
            uint32_t code = 0, pos = 0;
            if (q < count) {
                const uint32_t o = owner[q];
                pos = R.shift[o & kTileOf] + q0 + q;
                const uint32_t l = line[q];
                code = l & kNoLine ? l & 3u : res[(l >> 5) * (kRowWords * 8) + (l & 31u)];
                if (code == kNewOther)
                    code = o & kNewTo ? 1u : 2u;
                else if ((o & kRepeat) && code != kLater)
                    code = 2;
                if (code != kLater)
                    A.flag[pos] = (uint8_t)code;
            }
            leave(code == kLater, pos);
        }
    }
}

// The inserts that the parts' workgroups left, the plain way: their statuses go where theirs do.
template <int NQ>
__global__ __launch_bounds__(kBlock) void later_kernel(View T, Bulk A, uint32_t seq)
{
    __shared__ WaveLds lds[kWavesPerBlock];
    const uint32_t n = *A.later_count;
    const uint32_t wl_ = threadIdx.x >> 6, lane = lane_id();
    const uint32_t wave = blockIdx.x * kWavesPerBlock + wl_;
    const uint32_t nwaves = gridDim.x * kWavesPerBlock;
    // Inserts listed together share buckets. A lane takes `turns` neighbours one after another,
    // so that they do not race for the same slots; and as few inserts go to a wavefront at a time
    // as there are wavefronts for, since it grows one list a round.
    const uint32_t share = (n + nwaves - 1) / nwaves;
    const uint32_t C = share < 4 ? 4 : share < 2 * NQ ? share : 2 * NQ;
    const uint64_t lanes = (uint64_t)nwaves * C;
    const uint32_t turns = (uint32_t)((n + lanes - 1) / lanes);
    if ((uint64_t)wave * C * turns >= n)
        return;
    Alloc al;
    alloc_init(al, wave, seq);
    alloc_preload(T, al, lane);
    Counters cnt = {0, 0, 0, 0};
    for (uint32_t turn = 0; turn < turns; ++turn) {
        const uint64_t at = ((uint64_t)wave * C + lane) * turns + turn;
        const bool in = lane < C && at < n;
        const uint32_t count = (uint32_t)__popcll(ballot(in));
        const uint32_t pos = in ? A.later[at] : 0u;
        ChunkIn c;
        c.key = in ? A.key[pos] : kEmpty;
        c.val = in ? A.val[pos] : 0u;
        c.op = kInsert;
        run_chunk<kInsert, false, false, NQ, true>(T, al, cnt, lds[wl_], c, nullptr, A.flag, pos,
                                                   count, 0u);
    }
}

// Results back to the batch's order.
template <int R>
__global__ __launch_bounds__(kSplitThreads) void merge_kernel(Bulk A, uint64_t n,
                                                              uint32_t *__restrict__ vout,
                                                              uint8_t *__restrict__ sout)
{
    extern __shared__ uint32_t sm[];
    constexpr uint32_t kTile = kSplitThreads * R;
    uint32_t *val = sm;
    uint8_t *flag = reinterpret_cast<uint8_t *>(vout ? sm + kTile : sm);
    const uint32_t tid = threadIdx.x;
    const uint64_t base = (uint64_t)blockIdx.x * kTile;
    const uint32_t count = (n - base < kTile) ? (uint32_t)(n - base) : kTile;
    // the workspace's arrays hold whole tiles: the last tile's reads stay inside them
    for (uint32_t i = tid * 4; i < count; i += kSplitThreads * 4) {
        if (vout)
            *reinterpret_cast<uint4 *>(val + i) = *reinterpret_cast<const uint4 *>(A.key + base + i);
        if (sout)
            *reinterpret_cast<uint32_t *>(flag + i) =
                *reinterpret_cast<const uint32_t *>(A.flag + base + i);
    }
    __syncthreads();
    if (vout)
        vout += base;
    if (sout)
        sout += base;
    const bool wide = ((reinterpret_cast<uintptr_t>(vout) & 15u) |
                       (reinterpret_cast<uintptr_t>(sout) & 3u)) == 0;
    for (uint32_t i = tid * 4; i < count; i += kSplitThreads * 4) {
        const uint2 pl = *reinterpret_cast<const uint2 *>(A.place + base + i);
        const uint32_t p[4] = {pl.x & 0xFFFFu, pl.x >> 16, pl.y & 0xFFFFu, pl.y >> 16};
        if (wide && i + 4 <= count) {
            uint32_t found = 0; // searches that return a value: found whatever the flag
            if (vout) {
                const uint4 v = make_uint4(val[p[0]], val[p[1]], val[p[2]], val[p[3]]);
                *reinterpret_cast<uint4 *>(vout + i) = v;
                found = (v.x != kEmpty ? 1u : 0u) | (v.y != kEmpty ? 1u << 8 : 0u) |
                        (v.z != kEmpty ? 1u << 16 : 0u) | (v.w != kEmpty ? 1u << 24 : 0u);
            }
            if (sout)
                *reinterpret_cast<uint32_t *>(sout + i) =
                    found | flag[p[0]] | (flag[p[1]] << 8) | (flag[p[2]] << 16) |
                    (flag[p[3]] << 24);
        } else {
            for (uint32_t e = 0; e < 4 && i + e < count; ++e) {
                if (vout)
                    vout[i + e] = val[p[e]];
                if (sout)
                    sout[i + e] = flag[p[e]] | (vout && val[p[e]] != kEmpty ? 1 : 0);
            }
        }
    }
}
