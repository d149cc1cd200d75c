// Index arithmetic that memory safety rests on, free of HIP so that a host compiler can build it and
// the tests can go through it exhaustively.
#pragma once
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>

#ifdef __HIPCC__
#define QGX_PLAN __host__ __device__ __forceinline__
#else
#define QGX_PLAN inline
#endif

namespace qgx {

// The words of a worker's payload that hold bits start .. end of a chunk whose first word is `off`: `words`
// of them from payload word `at` on, the first one word w0 of the chunk; at, w0 and words are multiples of 4.
// `off`, `start` and `end` come from the stream's tables and may be anything; `cap` is the payload's size, a
// non-zero multiple of 4.  Not ok, with at = words = 0, when they are no place of 1 .. max_words words inside the
// payload.  Whoever reads max(words, 4) words from `at` thus stays inside it: an extent without words is refused like
// the others (a half chunk has at least a bit per coordinate), for at the payload's very end it would leave nothing
// to read.
struct HalfWords { uint64_t at; uint32_t w0, words; bool ok; };

QGX_PLAN HalfWords half_words(uint32_t off, uint32_t start, uint32_t end, uint32_t max_words, uint64_t cap)
{
    HalfWords h;
    h.w0 = (start >> 5) & ~3u;
    h.words = ((((end + 31u) >> 5) + 3u) & ~3u) - h.w0;       // (an end before the start: beyond max_words, or 0, or an empty run)
    h.at = (uint64_t)off + h.w0;
    h.ok = h.words - 1u < max_words && (off & 3u) == 0u && h.at + h.words <= cap;
    if (!h.ok) { h.at = 0; h.words = 0; }
    return h;
}

// ---- which worker's which unit of work a workgroup of the coding kernel takes ----------------------
// Workgroups are dealt to the eight XCDs by their number, each XCD starts its own in order, and no other XCD takes over
// what is queued behind a busy one.  Where workgroups share a bucket (`parts` of them) one that has started waits for its
// partners.  They take (bucket, part) from their worker's ticket counter, so of each worker only the newest bucket is
// incomplete and at most parts - 1 workgroups wait.  An XCD that is behind (the others have run out of work) can thus
// hold (parts - 1) x the workers that have workgroups on it, all waiting for partners in its own queue: a free place
// must always be left, so the workers on an XCD are kept below what `held`, the workgroups an XCD holds at once, allows.
constexpr uint32_t kXcds = 8;

// Blocks deal the workers round, in rows of `span` of which the first K are workers: block i is worker i % span's unit
// i / span.  With a span of K all workers can have workgroups on every XCD; with one that is a multiple of 2, 4 or 8 the
// workers k of one k mod 2 (4, 8) have the XCDs of that number mod 2 (4, 8) to themselves.

// The K workgroups of a unit on one XCD instead, one after the other: for operands that the workers share.  All workers
// have workgroups on every XCD.  Grid: K * units.
struct BlockWork { uint32_t k, unit; };

QGX_PLAN BlockWork block_by_unit(uint32_t i, uint32_t K, uint32_t units)
{
    const uint32_t even = units / kXcds * kXcds;              // units in whole rounds of the XCDs
    const uint32_t j = i / kXcds, rest = i - even * K;
    if (i < even * K) return BlockWork{j % K, j / K * kXcds + i % kXcds};
    return BlockWork{rest % K, even + rest / K};
}

// Where a worker's workgroups keep an order (compact placement, whole buckets) and K is a multiple of 8, the plain rows put each
// worker on one XCD, whose workgroups then all wait for the same straggler, go on together and are in step from there on. Rows
// turned against each other by 0, 2, 4 and 6 workers give a worker four XCDs.  What that gives grows with a worker's workgroups on an
// XCD, and with few of them plain rows are the better; the two meet at about 16 for each worker.  Plain / turned, us, buckets of
// 16384, 8 workers, 17 exponential levels: 2^21 coordinates (128 workgroups a worker) 31.1 / 29.2, 2^22 59.7 / 54.8, 2^24 219 / 167
// (without an order 138); 33 uniform ones: 2^20 17.2 / 18.9, 2^21 26.8 / 27.8, 2^22 52.7 / 52.5, 9.86 M 125 / 108, 2^24 198 / 164.  33 uniform
// levels, 16 workers: 128 workgroups 49.2 / 52.3, 256 91.5 / 92.1, 512 183 / 160; 24 workers: 192 92.2 / 97.2, 384 169 / 168, 576
// 269 / 241; 32 workers: 256 149 / 154, 512 285 / 283; 64 workers: 256 274 / 280.
QGX_PLAN uint32_t worker_spread(uint32_t k, uint32_t unit, uint32_t span) { return (k + 2u * (unit & 3u)) % span; }

inline bool spread_workers(uint32_t K, uint32_t units) { return K % kXcds == 0u && units >= 16u * K; }

// Workgroups of four waves that an XCD holds at once: a wave of each on every SIMD, and their LDS (in steps of 2 KiB).
inline uint32_t held_per_xcd(uint32_t waves_per_simd, size_t lds_bytes, uint32_t n_cu)
{
    const size_t fit = 160u * 1024u / ((lds_bytes + 2047u) / 2048u * 2048u);
    return (uint32_t)(fit < waves_per_simd ? fit : waves_per_simd) * (n_cu / kXcds);
}

// The shortest row that leaves an XCD a free place; a multiple of 8 if none does.
inline uint32_t worker_span(uint32_t K, uint32_t parts, uint32_t held)
{
    uint32_t groups = 1;
    while (groups < kXcds && (parts - 1u) * ((K + groups - 1u) / groups) >= held) groups *= 2;
    return (K + groups - 1u) / groups * groups;
}

// Whole buckets to a workgroup of the coding kernel, where buckets have few chunks (a wave each): four waves then share the
// tables in LDS, and a compute unit's places hold as many waves whatever the bucket.  A small launch is over sooner with more and
// smaller workgroups, unless they have to keep an order, which has the fewer members.  Measured, one bucket to a workgroup /
// four waves, us, 8 workers in buckets of one chunk and of two.  In slots: 256 chunks 9.0 / 9.9 and 9.0 / 9.7, 2048 14.2 / 14.6
// and 14.1 / 14.4, 4096 23.8 / 24.4 and 23.7 / 24.2, 8192 41.6 / 42.0 and 41.0 / 41.4, 16384 76.0 / 75.5 and 75.7 / 75.1, 19257
// 84.5 / 83.1 and 83.0 / 83.0.  In order: 128 10.8 / 11.5 and 10.6 / 11.3, 256 11.4 / 11.7 and 11.0 / 11.5, 512 13.9 / 12.4 and
// 11.6 / 12.2, 1024 15.9 / 13.0 and 14.6 / 12.9, 4096 37.3 / 29.7 and 32.1 / 29.4, 16384 123 / 95.9 and 105 / 95.0.  (The lines
// were drawn at five waves per SIMD; with look-ups ahead, small launches in slots gain nothing from sharing up to twice the line.)
inline uint32_t buckets_per_group(uint32_t waves_per_bucket, uint64_t chunks_of_all, bool ordered)
{
    if (waves_per_bucket > 2u || chunks_of_all < (ordered ? 256u : 4096u)) return 1u;
    return 4u / waves_per_bucket;
}

// Waves of a workgroup of `group` buckets that have one: fewer in a worker's last workgroup.
QGX_PLAN uint32_t waves_with_a_bucket(uint32_t unit, uint32_t group, uint32_t waves_per_bucket, uint32_t NB)
{
    const uint32_t left = NB - unit * group;
    return (left < group ? left : group) * waves_per_bucket;
}

// The coding kernel's form with look-ups ahead at four waves per SIMD, or five waves: a wave per chunk, up to two rounds of four.
// Beyond that, chunks in order lose more with it than those in slots gain.  Five waves / look-ups ahead, us, 8 workers in buckets of
// 16384, 17 levels, in slots: 512 chunks 10.6 / 9.6, 2048 14.7 / 14.0, 4096 24.5 / 23.7, 6144 32.1 / 31.6, 8192 41.2 / 41.0, 9216 45.0 /
// 44.0, 10240 49.0 / 48.5, 12288 57.4 / 56.5, 16384 74.1 / 74.5, 24576 104 / 104; in order: 512 13.0 / 11.9, 2048 19.5 / 18.4, 4096
// 29.3 / 28.6, 6144 46.1 / 46.5, 8192 56.8 / 54.4, 9216 59.2 / 64.6, 10240 62.0 / 69.5, 12288 77.0 / 76.1, 16384 92.5 / 96.5.  In slots,
// 4096 and 8192 chunks, with 33 levels 23.8 / 22.7 and 39.5 / 38.5, 65 23.2 / 22.2 and 39.4 / 38.1, 127 24.8 / 23.2 and 42.9 /
// 40.5; L-infinity norm 24.9 / 24.2 and 41.8 / 41.0, q = 3 59.5 / 58.6 and 116 / 114.
inline bool use_staged(uint64_t chunks_of_all, uint32_t n_simd) { return chunks_of_all <= 8u * (uint64_t)n_simd; }

// The coding kernel's form with four waves to a chunk, `per_bucket` chunks to a workgroup where buckets do not share chunks: as long as the
// waves find places, in slots and with unshared chunks with at most eight of them to a workgroup, so that no compute unit has more while others are
// empty (shared chunks in order come four to a ticket, and thus sixteen waves to a workgroup).  A wave per chunk / four,
// us, kernel alone, 8 workers and 17 levels if not said otherwise.  In slots, shared chunks (buckets of 1024): 512 chunks 13.3 / 8.1,
// 1024 14.4 / 11.1, 2048 19.8 / 18.7, 4096 31.6 / 29.6, 8192 49.2 / 51.7; of 256: 4096 39.2 / 36.9, 8192 63.6 / 66.3.  One or
// two chunks to a bucket: buckets of 8192, 512 10.0 / 8.2, 1024 13.5 / 11.9, 1280 15.0 / 14.8, 2048 17.4 / 19.2; of 6000, 816 11.6 / 9.6,
// 1408 12.8 / 13.5.  Four: 256 10.0 / 10.6, 1024 11.8 / 12.7.  One chunk of 1024 coordinates 5.7 / 5.1.  In order, shared
// chunks, four to a workgroup: 256 15.4 / 12.2, 1024 18.5 / 14.6, 1280 20.8 / 25.0, 2048 22.8 / 27.6; one or two to a bucket: 16 11.0 / 9.0,
// 128 11.1 / 9.4, from 256 on a workgroup has four: 13.0 / 13.6.
inline bool use_columns(uint64_t chunks_of_all, uint32_t per_bucket, bool shared, bool ordered, uint32_t n_simd)
{
    if (shared) return chunks_of_all <= (ordered ? 1u : 4u) * (uint64_t)n_simd;
    return per_bucket <= 2u && (ordered ? chunks_of_all < 256u : chunks_of_all <= n_simd);
}

// What that form gives depends on the work in a chunk besides.  Its lanes have 16 rows in 4, 2 or 1 of their own (`rows`: those of the
// longest bucket's last chunk, of 256 coordinates each), and lanes past the chunk's end work for nothing: quarters of n_simd up to which it
// is no slower, L2 and L-infinity norms on the left, q norms (powers in binary64, row by row from memory) on the right.  A wave per chunk /
// four, us or as 1 / the ratio, 8 workers in slots, 17 exponential levels: 1 row, 248 chunks 5.4 / 5.3, 512 5.7 / 6.3, 1024 6.1 / 7.9, q = 3 6.3 / 6.7 and
// 7.1 / 9.8; 2 rows, 512 1 / 0.98, 1024 1 / 1.13, q = 3, 256 1 / 1.0, 384 1 / 1.10; 5 rows, 640 1 / 1.10; 9 rows, 192 1 / 1.02, 384 1 / 1.25; 10
// rows, 256 1 / 1.0, 384 1 / 1.05, 640 1 / 1.22; 12 rows, 512 1 / 0.93, 1024 1 / 1.13, q = 3 1 / 0.83; 14 rows, 1024 1 / 1.0; 16 and 9,
// 512 1 / 0.92, 640 1 / 1.08.  (15 uniform levels, nearly all zeros after L2, 1 / 1.08 where others have 1 / 0.95.)  In order
// (below 256 chunks): 1 row 1 / 0.98, q = 3 1 / 1.07, 9 rows 1 / 1.07, the others gain.
// Four waves load a large table sooner (127 levels, 1 row, 248 chunks 7.1 / 5.4, 512 7.3 / 6.4, 1024 1 / 1.02, 2 rows, 1024 1 / 0.93, 10 rows, 512
// 1 / 0.87, 640 1 / 1.03; 34 to 65 levels, 1 row, 256 1 / 0.87, 384 1 / 0.98, 3 rows, 1024 1 / 0.9), and where the levels are too close for the cells
// (`crowded`, known of tables that were set), a row takes several times as long: 1 / 0.8 to 1 / 0.6 from 3 rows on, but 1 / 1.13 with one row.
// Fitted tables of 18 to 33 levels can be such: 1 row 1 / 1.11, 9 rows 1 / 0.63.
// Shared chunks in slots, with buckets of 8 rows, which go through all the lanes' turns: 1536 chunks 1 / 0.87, 2048 1 / 1.06, 4096 1 / 1.09, q = 3 1 / 0.69, 1 / 1.11
// and 1 / 1.31; 127 levels (LDS for fewer workgroups) 1280 1 / 0.97, 1536 1 / 1.04, 4096 1 / 1.18, in shorter buckets 1536 1 / 0.9, 3072 1 / 1.11; crowded 4096 1 / 0.8,
// q = 3 1 / 1.13 (2560 1 / 0.89).
inline bool columns_pay(uint64_t chunks_of_all, uint32_t per_bucket, uint32_t rows, bool shared, bool ordered, bool powers, bool crowded, uint32_t n_sym, uint32_t n_simd)
{
    const bool large = n_sym > 65u;
    uint32_t quarters = 16u;
    if (shared) {                                      // (rows: of a bucket)
        if (ordered) return true;
        if (crowded) quarters = rows == 8u && powers ? 12u : 16u;
        else if (large) quarters = rows == 8u ? 5u : powers ? 16u : 6u;
        else if (rows == 8u) quarters = 6u;
    } else if (per_bucket == 2u) {
        quarters = !powers && !crowded && (rows == 9u || rows == 10u) ? 2u : 4u;
    } else if (!(crowded && rows > 2u)) {
        constexpr uint8_t kQuarters[17][2] = {{0, 0}, {0, 0}, {2, 1}, {3, 2}, {4, 4}, {2, 2}, {3, 4}, {4, 4}, {4, 4}, {0, 2}, {1, 4}, {2, 4}, {2, 4}, {3, 4}, {4, 4}, {4, 4}, {4, 4}};
        quarters = kQuarters[rows < 16u ? rows : 16u][powers ? 1 : 0];
        if (!crowded) {
            quarters += large ? (rows > 8u ? 1u : 2u) : n_sym > 33u && rows <= 8u ? 1u : 0u;
            if (quarters == 0u && (rows == 9u ? n_sym > 17u : n_sym <= 17u && !powers)) quarters = 1u;
        }
        if (quarters > 4u) quarters = 4u;
    }
    return 4u * chunks_of_all <= (uint64_t)quarters * n_simd;
}

// Two levels strictly inside one cell of the look-up (qgx_tables.hip): rows then go through the levels one by one.
inline bool levels_crowded(const float* levels, uint32_t n_sym, int cell_mant, int octaves)
{
    auto cell_of = [&](float x, bool* edge) {
        uint32_t u;
        std::memcpy(&u, &x, sizeof(u));
        const int64_t c = (int64_t)(u >> (23 - cell_mant)) - ((int64_t)(127 - octaves) << cell_mant);
        *edge = c > 0 && (u & ((1u << (23 - cell_mant)) - 1u)) == 0u;
        return c > 0 ? c : 0;
    };
    for (uint32_t j = 1; j + 2u < n_sym; ++j) {
        bool at_edge, unused;
        const int64_t a = cell_of(levels[j], &at_edge), b = cell_of(levels[j + 1u], &unused);
        if (a == b && !at_edge) return true;
    }
    return false;
}

// ---- waves to a task of the fused decoders (1, 2 or 4, and see eight_waves): each takes a run of the K workers, and they join their sums --
// x = f * tasks against the wave slots (8 per SIMD with one stream, 4 with two).  A launch is bound by latency,
// ceil(K / f) workers one after the other (a worker's chain of look-ups takes 2.2 us with one stream, 3.3 with two, however
// few waves there are), or by throughput, x K / f of the time that full slots take for a worker (7.7 and 7.1 us, the unit
// below); where a last round fills a part of the slots, that part counts max(0.36, 0.15 + 0.85 x).  Joining costs more the
// more waves do it.  Measured with 1 / 2 / 4 waves, us: first half-step, 512 tasks of 8 workers 23.3 / 15.1 / 12.6, 1024 of 5
// 17.8 / 14.8 / 16.3, 2048 of 8 30.2 / 26.2 / 30.7, of 12 39.7 / 33.1 / 37.6, 4096 of 8 40.8 / 45.7 / 53.2; second, 512 of 8
// 37.3 / 26.0 / 22.0, 2048 of 8 51.6 / 51.0 / 57.3, 4096 of 8 81.8 / 87.9 / 97.1, 4816 of 8 113 / 105 / 112.
inline uint32_t waves_per_task(uint32_t n_tasks, uint32_t workers, uint32_t n_simd, uint32_t streams)
{
    const bool two = streams == 2u;
    const double K = workers, tasks = n_tasks / (n_simd * (two ? 4.0 : 8.0));
    auto cost = [&](uint32_t f) {
        const double x = f * tasks, whole = std::floor(x), part = x - whole;
        const double rounds = whole > 0.0 && part > 0.0 ? whole + std::fmax(0.36, 0.15 + 0.85 * part) : x;
        const double latency = (two ? 0.47 : 0.28) * std::ceil(K / f), throughput = rounds * K / f;
        const double join = f == 1u ? 0.0 : f == 2u ? (two ? 0.28 : 0.10) + 0.28 * x : two ? 0.28 + 0.42 * x : 0.22 + 0.58 * x;
        return std::sqrt(std::hypot(latency * latency, throughput * throughput)) + join;      // (the larger of the two, rounded off)
    };
    uint32_t best = 1;
    for (uint32_t f = 2; f <= 4u && f <= workers; f *= 2)
        if (cost(f) < cost(best)) best = f;
    return best;
}

// Eight waves to a task instead, for eight workers and more: where even so a SIMD has no more than two or three of them, the workers
// that a wave goes through one after the other are all that counts.  At four waves per SIMD also with one stream (at eight the join spilled 140
// bytes a lane and took what it gave).  Four waves / eight, us: first half-step, 4 tasks of 8 workers 9.7 / 7.7, 128 11.8 / 8.6, 256 11.6 /
// 9.0, 512 12.9 / 12.4, 768 14.1 / 19.0, of 12 256 12.5 / 11.2, 512 14.3 / 15.0, of 32 256 23.2 / 17.0, 512 26.5 / 22.2; second, 4 of 8
// 12.4 / 10.6, 32 12.8 / 11.2, 256 12.2 / 11.6, 512 15.4 / 17.6, of 16 256 19.1 / 15.4, 512 24.1 / 25.8, of 32 32.0 / 23.6 and 40.2 / 42.6.
// Between 256 and 384 tasks of one stream: means of 8 workers, 320 10.4 / 11.0 and 384 10.2 / 11.1, of 12 12.6 / 13.0 and 12.5 / 13.2, of 16 14.8 / 14.1 and
// 14.8 / 14.3, of 32 24.3 / 20.6 and 24.5 / 21.2; first half-steps (which have the means' rule) of 8 11.2 / 11.3 and 11.2 / 11.4, of 12 13.4 / 13.4 and
// 13.8 / 13.4; second ones without a previous stream (`second`) of 8 17.0 / 16.6 and 17.4 / 17.2, of 12 20.2 / 18.7 and 19.9 / 19.0.
inline bool eight_waves(uint32_t n_tasks, uint32_t workers, uint32_t n_simd, uint32_t streams, bool second = true)
{
    const bool longer = streams == 1u && (second || workers >= 16u);
    return workers >= 8u && n_tasks <= (longer ? n_simd / 8u * 3u : n_simd / 4u);
}

}  // namespace qgx
