// Host arithmetic of the bulk form: which calls have one, how a batch is cut into tiles and parts,
// and where its arrays lie in the workspace. Plain C++ (the test suite compiles it for the CPU);
// included by bulk.hpp, inside its unnamed namespace, after <math.h>, <stddef.h> and <stdint.h>.

constexpr uint32_t kSplitThreads = 1024;
constexpr uint32_t kMaxParts = 15872;     // a tile's part counters fit in LDS beside its keys
constexpr uint32_t kMaxTiles = 2048;      // run starts of one part, in LDS
constexpr uint32_t kMaxSpan = 1000;       // buckets of a part (insert_kernel's `line`)
constexpr uint32_t kRowWords = 33;        // a slab's row in LDS: 32 words and one of padding, so
                                          // that one slot of many rows spreads over the banks
constexpr uint32_t kSigWords = 16;        // an insert's bucket: 512 bits
// LDS per bucket of a part. Searches: the row, its tags and a byte; inserts: the line, the bits and
// three words.
constexpr uint32_t kPairRowBytes = kRowWords * 8 + 32 + 1, kKeyRowBytes = kRowWords * 8 + 64 + 1;
constexpr uint32_t kInsRowBytes = kRowWords * 8 + kSigWords * 4 + 12;
constexpr size_t kLdsBytes = 160 * 1024;

struct Bulk {
    uint32_t span, span_magic;   // buckets per part
    uint32_t parts, tiles, tile; // tile: operations per tile
    uint32_t row;                // 32-bit words of one tile's row of part starts
    uint32_t queue;              // operations a part's workgroup takes of its part at a time
    uint32_t hot;                // a longer run of one part in one tile repeats keys
    uint16_t *starts;            // tiles rows of parts + 1 starts
    uint32_t *key;               // operations in tile order; a search's results afterwards
    uint32_t *val;               // inserts: their values
    uint32_t *later;             // inserts left to the plain kernel: their positions
    uint32_t *later_count;
    uint16_t *place;             // place of each operation of the batch in its tile
    uint8_t *flag;               // per operation, in tile order
};

// A call, as far as its plan depends on it.
struct BulkCall {
    uint64_t n;
    uint32_t buckets, num_cu;
    bool insert;    // else a search
    bool keys_only;
    uint64_t since_reset; // inserts and operations of mixed batches, as far as the host knows
};

struct BulkPlan {
    uint32_t rows;  // operations per thread of a split workgroup (its tile / 1024)
    uint32_t waves; // wavefronts of a part's workgroup
    uint64_t chunk; // operations per pass over the kernels
    Bulk a;
    size_t starts, key, val, place, flag, later, total; // byte offsets
    size_t split_lds, part_lds, merge_lds;
};

// 32-bit words of one tile's part starts: two 16-bit ones each, and the end of the last.
constexpr uint32_t split_row_words(uint32_t parts) { return parts / 2 + 1; }

// The calls that have a bulk form (bulk_pays, below, has those for which it is the faster one):
constexpr uint64_t kBulkSearches = 1u << 21, kBulkInserts = 1u << 17; // the smallest batches
constexpr uint32_t kBulkCached = 1u << 15;  // base slabs that the L2s hold: 2^21 searches of them
constexpr uint64_t kBulkCachedSearches = 3u << 20; // take 42 us plain / 46, 2^22 85 / 65
constexpr uint32_t kBulkPerBucket = 6;      // operations per bucket, at least
constexpr uint32_t kBulkBuckets = 1u << 10; // a part has at least one, and parts fill the chip
constexpr uint32_t kBulkQueue = 1024;       // the shortest queue of a part taken in pieces
constexpr uint32_t kBulkFill = 26;          // since_reset + n per bucket, at most

// Whether the call has a bulk form, and how it runs. A part of about 2048 operations keeps a
// workgroup of 8 wavefronts busy while three of them share a compute unit's LDS (2^22 searches of
// 2^22 keys: 79, 62, 64 and 71 us with 1024, 2048, 2560 and 4096 parts); batches with more such
// parts than a tile can count take larger ones, 16 wavefronts each (2^26 searches: 1.54 ms
// against 1.92 ms with 8). Tiles grow with the batch: a tile per compute unit at least, and runs
// of several operations per part.
inline bool bulk_plan(const BulkCall &c, BulkPlan *P)
{
    const uint32_t B = c.buckets;
    const bool ins = c.insert;
    P->chunk = c.n < (1ull << 26) ? c.n : (1ull << 26);
    const uint64_t m = P->chunk;
    if (m < (ins ? kBulkInserts : B < kBulkCached ? kBulkCachedSearches : kBulkSearches) ||
        m / kBulkPerBucket < B || B < kBulkBuckets)
        return false;
    // inserts that the base slabs have no room for are made the plain way, after the others:
    // nothing is gained where they are many
    if (ins && c.since_reset + c.n > (uint64_t)B * kBulkFill)
        return false;
    P->rows = m <= (3u << 19) ? 4 : m <= (3u << 20) ? 8 : m <= (1u << 23) ? 16 : 32;
    Bulk &A = P->a;
    A = Bulk{};
    A.tile = P->rows * kSplitThreads;
    A.tiles = (uint32_t)((m + A.tile - 1) / A.tile);
    P->waves = 8;
    uint64_t parts = (m + 2047) / 2048;
    if (parts < B / 160)
        parts = B / 160; // few operations per bucket: the slabs bound the part
    if (parts > kMaxParts) {
        P->waves = 16;
        parts = (m + 6553) / 6554;
        if (parts < B / 400)
            parts = B / 400;
    }
    const uint64_t cus = c.num_cu, most = kMaxParts / cus * cus;
    parts = (parts + cus - 1) / cus * cus;
    if (parts > most)
        parts = most;
    const uint32_t row_bytes = ins ? kInsRowBytes : c.keys_only ? kKeyRowBytes : kPairRowBytes;
    const uint32_t queue_bytes = ins ? 4 : 6;
    const size_t runs = 8 + 8 * (size_t)A.tiles + 8 + 4 * P->waves;
    // More parts until one fits the LDS beside its queue; where that is not enough, a queue
    // shorter than a part, which is then taken in pieces. (Calls that went the plain way while a
    // part had to fit as it was: 2^26 searches at 16 per bucket 3.01 -> 1.49 ms, of keys alone at
    // 38 2.48 -> 1.40; 2^26 inserts at 16 per bucket 4.43 -> 2.14, 3 * 2^24 at 9.6 3.49 -> 2.09.)
    for (;; parts += cus) {
        A.span = (uint32_t)((B + parts - 1) / parts);
        A.parts = (B + A.span - 1) / A.span;
        // a part's share varies as a sum of independent operations does
        const double avg = (double)m / A.parts;
        A.queue = (uint32_t)(avg + 6 * sqrt(avg) + 64) & ~3u;
        if (A.queue > 32 * P->waves * 64)
            A.queue = 32 * P->waves * 64;
        P->part_lds = (size_t)A.span * row_bytes + runs + queue_bytes * (size_t)A.queue;
        if (P->part_lds <= kLdsBytes || parts + cus > most)
            break;
    }
    if (P->part_lds > kLdsBytes) {
        const size_t fixed = (size_t)A.span * row_bytes + runs;
        if (fixed + queue_bytes * (size_t)kBulkQueue > kLdsBytes)
            return false;
        A.queue = (uint32_t)((kLdsBytes - fixed) / queue_bytes) & ~3u;
        P->part_lds = fixed + queue_bytes * (size_t)A.queue;
    }
    if (A.tiles > kMaxTiles || A.span > kMaxSpan)
        return false;
    A.row = split_row_words(A.parts);
    // more of one part in a tile than distinct keys make by chance
    const double run = (double)A.tile / A.parts;
    A.hot = ins ? 0xFFFFu : (uint32_t)(run + 5 * sqrt(run)) + 4;
    P->split_lds = ((size_t)A.tile + A.row + kSplitThreads / 64 + 1) * 4;
    P->merge_lds = (size_t)A.tile * (ins ? 1 : 5);
    if (P->split_lds > kLdsBytes || P->merge_lds > kLdsBytes)
        return false;
    const size_t slots = (size_t)A.tiles * A.tile;
    size_t off = 256;
    auto take = [&off](size_t bytes) {
        const size_t at = off;
        off = (off + bytes + 255) & ~(size_t)255;
        return at;
    };
    P->starts = take((size_t)A.tiles * A.row * 4);
    P->key = take(slots * 4);
    P->place = take(slots * 2);
    P->flag = take(slots);
    P->val = ins ? take(slots * 4) : 0;
    P->later = ins ? take(slots * 4) : 0;
    P->total = off;
    return true;
}

// Whether the bulk form is the faster one for the call, whatever its keys: distinct, repeated or
// popular, present or absent. Each line lies where the slowest distribution measured is level with
// the plain form (us, plain / bulk; Zipf(0.8) and Zipf(1.1) ranks; "half": half of them absent):
//
//   searches   the plain form finds popular keys in the caches, and three launches instead of one
//              cost 10 us: 2.5 * 2^20 at 10 per bucket uniform 101 / 74 but Zipf(1.1) 74 / 80, half
//              76 / 86; at 40, 82 / 54, 63 / 62, 65 / 73. 3.5 * 2^20 at 10: 145 / 85, 100 / 90,
//              101 / 94. At 2^26 at 10: 3258 / 1885, 1521 / 1517. So 3.5 * 2^20, ten per bucket.
//              Longer lists than one slab are read level by level for all of a part: with 40 pairs
//              per bucket 2^22 at 10 197 / 148 but Zipf(0.8) 156 / 175, at 16 189 / 115, 152 / 145;
//              with 150, Zipf(1.1) at 16 190 / 222 (uniform 462 / 254), with 400 at 64 370 / 383.
//              So 16 per bucket, and 64, of tables that may hold that much.
//   inserts    into an empty table, every key once, and twice: 2^17 at 6.1 per bucket 26 / 26 and
//              22 / 27, at 10 35 / 24 and 26 / 25; 2^18 at 7 33 / 33 and 29 / 35, at 10 37 / 27 and
//              31 / 29; 3 * 2^17 at 6.1 39 / 33 and 36 / 34. Popular keys gain most. The host takes
//              16 us for such a call, 4 for a plain one: a pass of reset, inserts, search, delete
//              and search that is waited for takes at 2^17 and 10 per bucket 69 / 79, at 15 79 / 72;
//              3 * 2^16 at 10, with small searches, 65 / 71; 2^18 at 10 70 / 70. So 15, 10 and 6
//              per bucket from 2^17, 2^18 and 3 * 2^17 on.
//              Beside pairs that the table holds, fresh keys / keys that are all present: 2^18 at
//              12 on 12 held 47 / 30 and 23 / 37 (a plain insert finds such a key and swaps once);
//              2^20 92 / 55 and 68 / 69; 2^22 at 8 on 12 266 / 215 and 251 / 257, at 12 289 / 182
//              and 243 / 209. So 2^20 and 12 per bucket there.
//
// counted: no operations but those in since_reset have reached the table.
inline bool bulk_pays(const BulkCall &c, bool counted)
{
    const uint64_t m = c.n < (1ull << 26) ? c.n : (1ull << 26), B = c.buckets;
    const uint64_t slab = c.keys_only ? 62 : 31; // entries
    if (!c.insert) {
        const uint64_t held = c.since_reset;
        const uint64_t per = !counted || held > 2 * slab * B ? 64
                             : held > slab * B * 2 / 3       ? 16
                                                             : 10;
        return c.n >= (7u << 19) && m / per >= B;
    }
    if (c.since_reset == 0)
        return c.n >= (1u << 17) &&
               m / (c.n < (1u << 18) ? 15 : c.n < (3u << 17) ? 10 : 6) >= B;
    return c.n >= (1u << 20) && m / 12 >= B;
}
