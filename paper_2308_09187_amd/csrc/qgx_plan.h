// Index arithmetic that memory safety rests on, free of HIP so that a host compiler can build it and
// the tests can go through it exhaustively.
#pragma once
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

}  // namespace qgx
