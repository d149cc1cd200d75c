// Index arithmetic that memory safety rests on, free of HIP so that a host compiler can build it and
// the tests can go through it exhaustively.
#pragma once
#include <cmath>
#include <cstddef>
#include <cstdint>

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
// turned against each other by 0, 2, 4 and 6 workers give a worker four XCDs.  8 workers in buckets of 16384, us, plain / turned:
// 2^20 coordinates 20.1 / 20.7, 2^21 34.5 / 31.1, 2^22 64.9 / 56.7, 9.86 M 141 / 108, 2^24 224 / 166 (without an order 145);
// 16 workers, 2^22 103 / 95, 2^23 201 / 162.  With more workers to an XCD each has fewer workgroups there and the wait is a
// part of it: 24 workers of 2^21 70 / 80, 32 of 2^20 50 / 60, of 2^22 157 / 161.
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
// tables in LDS, and a compute unit holds twenty waves whatever the bucket.  A small launch is over sooner with more and
// smaller workgroups, unless they have to keep an order, which has the fewer members.  Measured, one bucket to a workgroup /
// four waves, us, in slots: 256 chunks 9.9 / 10.6, 2048 15.8 / 16.3, 3665 24.2 / 24.5, 5005 (half of them short) 26.3 / 25.1,
// 8192 47.1 / 45.6; in order: 256 chunks 13.7 / 13.8 and (a chunk to a bucket) 15.3 / 13.9, 2048 20.8 / 21.1 and 30.2 / 20.5,
// 8192 81.6 / 68.3 and 88.4 / 69.1.
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
// Measured, us, five waves / look-ups ahead: 256 chunks 10.6 / 9.6, 2048 15.9 / 15.2, 4096 27.7 / 27.0, 8192 46.7 / 45.4 (in order
// 13.7 / 12.7, 19.9 / 19.7, 31.7 / 30.9, 59.8 / 58.0); 19328 84.0 / 85.5, 32768 137 / 137.
inline bool use_staged(uint64_t chunks_of_all, uint32_t n_simd) { return chunks_of_all <= 8u * (uint64_t)n_simd; }

// ---- waves to a task of the fused decoders (1, 2 or 4): each takes a run of the K workers, and they join their sums --
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

}  // namespace qgx
