// DEQ o CODE and everything fused onto it: plain decode, the mean over K workers, and the two
// extra-gradient half-steps with the step-size accumulator.
// (Section 3.2 / Appendix J for the decoding; Algorithm 1 and eq. (Q-GenX) for the updates;
// Theorem 3 for gamma_t.)
//
// A wave's task is half a chunk position: 2048 coordinates, of which every lane parses one run of 32
// (a sub-chunk), starting at the bit offset the sub-chunk table gives.  The wave copies its half of a
// worker's chunk from the payload into LDS with coalesced 16-byte loads, then every lane parses its
// run: a 64-bit window from three LDS words per four symbols, one table look-up by the next 13 (or 11)
// stream bits for each symbol's length and level, the sign bit, one multiply by the bucket norm.  A symbol's
// length decides where the next one starts, so a parse is one long dependent chain of LDS look-ups.
// The K decoded values of a coordinate are summed in registers in worker order, so decoded vectors
// never go to HBM in the fused modes.
//
// Two shapes, eight chains per SIMD either way (LDS holds no more):
//   one stream (mean, first half-step): one chain per lane, 64 registers, eight waves per SIMD, whose
//     loads, parses and updates cover each other;
//   two streams (second half-step): two chains per lane, a worker's two streams, 128 registers, four waves
//     per SIMD; the next worker's half chunks travel ahead in registers.  Plain decoding has this shape too,
//     with two workers' chunks.
// Why half a position: a wave per whole position held 64 sums per lane, which left four (one stream) or two
// (two streams) waves per SIMD, and a launch of a round or two of equal waves in step.  Measured, whole position
// -> half: second half-step of 16 x 2^26 coordinates 1.246 -> 1.02 ms, of 8 x 9.86 M 0.150 -> 0.115 ms; first
// half-step 0.593 -> 0.497 and 0.085 -> 0.057 ms, of 8 x 2^24 73 us as before in a loop of coding and half-step, but
// 69 -> 74 us inside a whole iteration: it reads 10 MB more (a chunk's extents and the line that its halves share are asked for
// by two waves).
// Positions of fewer than 4096 coordinates are the same tasks with some lanes' symbols masked out; a half
// without coordinates is no task at all.  (A workgroup per such position, its workers spread over the waves, took
// 0.168 ms for the second half-step of 5 x 3 M coordinates in buckets of 6000, this takes 0.035.)
#include "qgx_device.h"
#include "qgx_plan.h"

namespace qgx {

constexpr int kHalfCoords = kChunk / 2;               // coordinates of a task, a run of kSub per lane
constexpr int kPre = 3;                               // uint4 per lane that travel ahead: 768 words, 12 bits per coordinate
static_assert(kHalfCoords * kMaxSymBits / 32 + 8 <= (kPre + 1) * kWave * 4, "one more covers any half chunk");
template <DecMode MODE, bool PREV> constexpr bool two_chains() { return PREV || MODE == DecMode::Decode; }
// Most waves per workgroup; they share the decode table.  Two tables leave LDS for one workgroup of eight waves with two chains
// to a compute unit, and for one of sixteen: second half-step of 8 x 2^24 coordinates, two tables, 191 -> 164 us (180 with a wave per whole position).
template <DecMode MODE, bool PREV, bool TWO> constexpr int most_waves() { return two_chains<MODE, PREV>() && !TWO ? 8 : 16; }
static_assert(kSub * kWave == kHalfCoords && kSubs == 2 * kWave, "a sub-chunk per lane, two tasks per chunk");

// Staged words in LDS.  Lane j parses the j-th run of the half, whose bits start roughly bits-per-coordinate
// words after lane j-1's: often a stride that would put all lanes on a few banks.  So two pad words
// are inserted after every 32 words (word i lives at i + 2 (i / 32)), and the pad slots repeat the two
// words that follow them, so that a lane always finds the three words of its 64-bit window next to
// each other.
__device__ __forceinline__ uint32_t staged(uint32_t i) { return i + ((i >> 5) << 1); }

// One worker's stream as this wave reads it (wave-uniform): its chunk's entry in the offset table, its row of
// sub-chunk ends, its norms and its payload; stepped from worker to worker.
struct StreamAt {
    const uint32_t* off;
    const uint16_t* ends;
    const float* norms;
    const uint32_t* payload;
};

__device__ __forceinline__ StreamAt stream_at(const uint32_t* chunk_off, const uint16_t* sub_end, const float* norms,
                                              const uint32_t* payload, uint64_t cap, uint32_t k, uint32_t c, const Layout& lay)
{
    return StreamAt{chunk_off + (size_t)k * (lay.NC + 1) + c, sub_end + ((size_t)k * lay.NC + c) * kSubs,
                    norms + (size_t)k * lay.NB, payload + (size_t)k * cap};
}

__device__ __forceinline__ void step_workers(StreamAt& s, uint64_t cap, uint32_t n, const Layout& lay)
{
    s.off += (size_t)n * (lay.NC + 1);
    s.ends += (size_t)n * lay.NC * kSubs;
    s.norms += (size_t)n * lay.NB;
    s.payload += (size_t)n * cap;
}

// Where half a chunk lies (wave-uniform): the chunk's first word in the worker's payload, and the bits of
// the chunk at which the half starts and ends.
struct Extent { uint32_t off, start, end; };

__device__ __forceinline__ Extent load_extent(const StreamAt& s, uint32_t half)
{
    Extent x;                                             // (rows of 256 bytes: pairs of entries are words)
    x.off = scalar_load(s.off);
    x.start = half ? scalar_load(s.ends + kWave - 2) >> 16 : 0u;
    x.end = scalar_load(s.ends + kWave * (half + 1u) - 2u) >> 16;
    return x;
}

// What a lane needs of it: where its run ends (the lane before it: where it starts), and its bucket's norm.
struct RunMeta { uint32_t hi; float n; };

// The words that hold the half's bits.  A half's extent comes from the sub-chunk table, so
// compact and slotted placements read alike; words counts from w0, both multiples of 4.
struct HalfRef {
    const uint4* src;
    uint32_t w0, words, start;
};

__device__ __forceinline__ HalfRef half_ref(const uint32_t* payload, uint64_t cap, const Extent& x, uint32_t max_words, Scalars* sc)
{
    const HalfWords h = half_words(x.off, x.start, x.end, max_words, cap);
    if (!h.ok && lane_id() == 0) raise_error(sc, QGX_EBIT_STREAM);     // (nothing is staged: what was staged before is parsed)
    return HalfRef{reinterpret_cast<const uint4*>(payload + h.at), h.w0, h.words, x.start};
}

// Lanes past the half's words read its last piece once more (no branch per load); nobody stages it.  With no words
// (half_words refused the extent) that is the first piece of the worker's payload, which holds at least one.
__device__ __forceinline__ void prefetch_half(const HalfRef& hr, uint4 (&pre)[kPre], uint32_t lane)
{
    const uint32_t last = max(hr.words >> 2, 1u) - 1u;
#pragma unroll
    for (int q = 0; q < kPre; ++q) pre[q] = nt_load4u(hr.src + min(lane + (uint32_t)q * kWave, last));
}

// The half chunk goes to LDS back to front: its bit t (counted from word w0) goes to bit
// 32 (kTail + stage_words) - 1 - t of the buffer (word w to place kTail + stage_words - 1 - w, its bits
// turned round), so that a plain funnel shift of buffer words gives a window with the FIRST stream bit on
// top, which is how the decode tables are indexed, and no window has to be turned round when it is read:
// a word is turned once here instead of twice per three symbols there.  kTail zero words lie below the
// end (the windows of the last symbols reach there), and the buffer's slack above the first word
// stays zero as well (a cursor may point one bit before it).
// `words`: the half's own size; pieces of 256 words that lie beyond it are left as they are (a valid
// stream's symbols never depend on what follows its last bit).
constexpr int kTail = 4;
__device__ __forceinline__ void commit_half(uint32_t* stage, const uint4 (&pre)[kPre], const HalfRef& hr, uint32_t stage_words,
                                            uint32_t lane)
{
    static_assert(kTail % 4 == 0, "16-byte pieces stay aligned");
    constexpr uint32_t kStep = kWave * 4u + kWave * 4u / 16u;                 // a piece of 256 words and its pads
    const uint32_t j0 = (uint32_t)kTail + stage_words - 4u - 4u * lane;       // place of the lane's LAST word of piece 0
    uint32_t* at0 = stage + (int)staged(j0);                                  // (piece q: whole steps of 32 words below)
    const bool pads = (j0 & 31u) == 0u;
#pragma unroll
    for (int q = 0; q <= kPre; ++q) {
        const uint32_t left = hr.words - (uint32_t)q * (kWave * 4u);          // words from this piece on
        if ((int)left <= 0) break;                                            // (wave-uniform)
        uint4 x;
        if (q < kPre) x = pre[q < kPre ? q : 0];
        // the end of a half chunk of the longest codes: asked for only here (its registers are better spent)
        else x = nt_load4u(hr.src + min(lane + (uint32_t)q * kWave, (hr.words >> 2) - 1u));
        if (4u * lane < left) {
            uint2* at = reinterpret_cast<uint2*>(at0 - q * (int)kStep);
            const uint2 low = make_uint2(__brev(x.w), __brev(x.z));
            at[0] = low;
            at[1] = make_uint2(__brev(x.y), __brev(x.x));
            if (pads) at[-1] = low;                                           // (j0 - 256 q >= kTail: never the buffer's first word)
        }
    }
}

// LDS tables of the decoder in one array: level values first, then the decode table, so that the
// level of a reject entry still lands inside the array.
constexpr int kTabLevelsAt = 16, kTabDlutAt = kTabLevelsAt + kSymMax * 4;
constexpr int kTabBytes = kTabDlutAt + kDlut * 2;
static_assert(kTabLevelsAt + 4 * (kDlutReject >> 6) + 4 <= kTabBytes, "the level of a reject entry");

// Symbols are parsed in groups of four from one 64-bit window (three LDS words): a symbol takes at most 14 bits with
// its sign, so two leave the first word's last bits to shift from, and the fourth starts before bit 42 and has its 14 bits
// in the window.  (Groups of three need a shift less and three windows more a run: first half-step of 8 x 2^24
// coordinates 74.8 us, now 69.8; of 8 x 9.86 M 56.7, now 53.5; second 99.6, now 92.8.)
constexpr int kGroup = 4;
static_assert(kSub % kGroup == 0 && 2 * kMaxSymBits < 32 && 3 * kMaxSymBits + kMaxSymBits <= 63 && kGroup * kMaxSymBits < 64, "a group in a window");
struct Window { uint32_t w0, w1, w2; };

__device__ __forceinline__ Window read_window(const uint32_t* stage, uint32_t p)
{
    // (the two shift-and-adds spelled out: the compiler would shift and mask each part, an instruction more)
    uint32_t at = lds_address(stage);
    asm("v_lshl_add_u32 %0, %1, 1, %2" : "=v"(p) : "v"(p >> 10), "v"(p >> 5));
    asm("v_lshl_add_u32 %0, %1, 2, %2" : "=v"(at) : "v"(p), "s"(at));
    return Window{lds_load_u32(at), lds_load_u32(at + 4u), lds_load_u32(at + 8u)};
}

// The dependent chain: window i needs the lengths of the symbols before it.  The cursor r is a bit position
// in the buffer and moves DOWN, the three words from it give the 64 bits with the first stream bit on top by
// two funnel shifts and nothing else.
// The windows are taken one bit early: r + 63 is the buffer bit of the stream bit BEFORE the next symbol,
// so bit 31 of a symbol's window is the last bit of the symbol before it, which is that symbol's sign
// if it has one.  The sign of a symbol is thus read off the window of the next one with a single
// AND-OR, no shift by its length: W[i + 1] for symbol i, the next group's W[0] for a group's last
// symbol, and for the last group of a run (LAST) the window after its last symbol, W[4].
// The table index sits one bit lower (bits 30..20 resp. 30..18).
// `seen` gathers the sums of the groups' halves: a reject entry leaves a one in bit 15 or 16, valid entries never do, so no
// per-symbol flag is kept.
// WIDE: the 8-byte table, which has the level beside the count.
template <bool WIDE, bool LAST>
__device__ __forceinline__ void parse_group(const Window& w, const unsigned char* tab, uint32_t& r,
                                            uint32_t (&W)[kGroup + 1], uint32_t (&e)[kGroup], float (&lv)[kGroup], uint32_t& seen)
{
    auto look_up = [&](int i) __attribute__((always_inline)) {
        if constexpr (WIDE) {
            const uint2 t = *reinterpret_cast<const uint2*>(tab + kTabDlutAt + ((W[i] >> 17) & 0x3FF8u));
            e[i] = t.x;
            lv[i] = __uint_as_float(t.y);
        } else {
            e[i] = *reinterpret_cast<const uint16_t*>(tab + kTabDlutAt + ((W[i] >> 17) & 0x3FFEu));
        }
    };
    const uint32_t nxt = __builtin_amdgcn_alignbit(w.w1, w.w0, r);
    W[0] = __builtin_amdgcn_alignbit(w.w2, w.w1, r);                          // shifts use r mod 32
    look_up(0);
    W[1] = __builtin_amdgcn_alignbit(W[0], nxt, e[0]);                        // (W[0]:nxt) << used, upper word
    look_up(1);
    const uint32_t half0 = e[0] + e[1];
    W[2] = __builtin_amdgcn_alignbit(W[0], nxt, half0);
    const uint32_t after = __builtin_amdgcn_alignbit(nxt, 0u, half0);         // what follows W[2]
    look_up(2);
    W[3] = __builtin_amdgcn_alignbit(W[2], after, e[2]);
    look_up(3);
    const uint32_t half1 = e[2] + e[3];
    if constexpr (LAST) W[4] = __builtin_amdgcn_alignbit(W[2], after, half1);        // at least two bits used: never a shift by 0
    seen |= half0 | half1;
    r += (half0 + half1) | 0xFFFFFFC0u;                                       // down by the bits used
}

// norm with the sign of the symbol whose last bit is bit 31 of `w_next` (norms are not negative)
__device__ __forceinline__ float signed_norm(uint32_t w_next, float n)
{
    return __uint_as_float((w_next & 0x80000000u) | __float_as_uint(n));
}

// +-(norm * level), one binary32 product, sign from the window of the next symbol
// EXACT_ZERO: +0 for the zero symbol, whose sign bit is not in the stream (the level 0 is the only one
// that is zero)
template <bool EXACT_ZERO>
__device__ __forceinline__ float symbol_value(uint32_t w_next, float lv, float n)
{
    const float val = __uint_as_float((w_next & 0x80000000u) | __float_as_uint(n * lv));
    if (EXACT_ZERO) return lv == 0.0f ? 0.0f : val;
    return val;
}

// (64 less a symbol's bits has ones in bits 4 and 5: an entry over 16 is 4 idx + 3)
static_assert(64 - kMaxSymBits >= 48, "bits 4 and 5");
__device__ __forceinline__ float level_of(const unsigned char* tab, uint32_t e)
{
    return *reinterpret_cast<const float*>(tab + (kTabLevelsAt - 3) + (e >> 4));
}

// Level values and decode table of one Tables object into the decoder's LDS array (WIDE: the table of
// 8-byte entries, which has the same size and holds the level values itself).
template <bool WIDE>
__device__ __forceinline__ void load_tables(unsigned char* s_tab, const Tables* __restrict__ tab, int tid, int nthreads)
{
    static_assert(kWide * sizeof(uint2) == kDlut * sizeof(uint16_t), "the two decode tables share one LDS area");
    static_assert(offsetof(Tables, dlut) % 16 == 0 && offsetof(Tables, dlutw) % 16 == 0 && sizeof(Tables) % 16 == 0, "16-byte copies");
    static_assert(kTabDlutAt % 16 == 0, "16-byte copies");
    if constexpr (!WIDE) {
        for (int i = tid; i < kSymMax; i += nthreads) reinterpret_cast<float*>(s_tab + kTabLevelsAt)[i] = tab->lval[i];
    }
    const uint4* src = WIDE ? reinterpret_cast<const uint4*>(tab->dlutw) : reinterpret_cast<const uint4*>(tab->dlut);
    for (int i = tid; i < kDlut / 8; i += nthreads) reinterpret_cast<uint4*>(s_tab + kTabDlutAt)[i] = src[i];
}

// First coordinate, length and bucket of chunk position c.
__device__ __forceinline__ void chunk_geometry(const Layout& lay, uint32_t c, uint32_t& clo, uint32_t& clen, uint32_t& bkt)
{
    if (lay.uniform_bucket) {                             // one segment: chunk geometry is arithmetic
        bkt = c / lay.waves_per_bucket;
        const uint32_t lo = bkt * lay.uniform_bucket, hi = min(lo + lay.uniform_bucket, lay.d);
        clo = lo + (c - bkt * lay.waves_per_bucket) * (uint32_t)kChunk;
        clen = min((uint32_t)kChunk, hi - clo);
    } else {
        clo = lay.chunk_start[c];
        clen = lay.chunk_start[c + 1] - clo;
        bkt = lay.chunk_bucket[c];
    }
}

// S, gamma_{t+1}, t at the end of the second half-step, from S; what the update multiplies by comes back.
__device__ __forceinline__ float step_size(double S, uint32_t K) { return (float)((double)K / sqrt(1.0 + S)); }      // Theorem 3: gamma_t = K (1 + sum ...)^(-1/2)

__device__ __forceinline__ void finish_scalars(Scalars* sc, double S, uint32_t K)
{
    sc->S = S;
    sc->gamma = (double)K / sqrt(1.0 + S);
    sc->gamma_f = step_size(S, K);
    sc->t += 1ull;
}

// X_{t+1} = X_1 + gamma Y by threads `at` of `step`: four coordinates at a time (X, Y and the anchor are 16-byte aligned), the last
// d mod 4 by the first threads.
__device__ __forceinline__ void x_from_y(float gam, uint32_t d, const float* Y, const float* anchor, float* X, uint32_t at, uint32_t step)
{
    const uint32_t quads = d / 4u;
    for (uint32_t q = at; q < quads; q += step) {
        const float4 y = reinterpret_cast<const float4*>(Y)[q];
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (anchor) x = reinterpret_cast<const float4*>(anchor)[q];
        x.x += gam * y.x; x.y += gam * y.y; x.z += gam * y.z; x.w += gam * y.w;
        reinterpret_cast<float4*>(X)[q] = x;
    }
    if (at < (d & 3u)) X[4u * quads + at] = (anchor ? anchor[4u * quads + at] : 0.0f) + gam * Y[4u * quads + at];
}

template <bool B> struct BoolTag { static constexpr bool value = B; };

// Four consecutive floats; a decoded vector of an odd length puts them at any multiple of 4 bytes.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// PREV (Half1): the previous half-step's streams are there; without them the vectors count as zero.
// TWO: those were coded with another level table and code (a.tab_p) than the current ones.
// WIDE: the first kWideBits bits of a code word always tell which one it is, so the 8-byte decode table
// is there (of both codes, with TWO).
// KSPLIT = 2, 4 or 8: that many neighbouring waves share a task, each takes a run of the workers (as
// equal as K allows, the longer runs first), and they add their sums through LDS before the update
// (for layouts with too few tasks to fill the GPU's wave slots).
// What bounds it: the parse, whose chains wait for their look-ups (with two streams vector ALUs busy for 73 % of the time, LDS
// for 55 %), and at the largest sizes of one stream the memory path.
template <DecMode MODE, bool PREV, bool TWO, bool WIDE, int KSPLIT>
__global__ __launch_bounds__((most_waves<MODE, PREV, TWO>()) * kWave) __attribute__((amdgpu_waves_per_eu((two_chains<MODE, PREV>() || KSPLIT == 8) ? 4 : 8)))
void k_decode(Layout lay, const Tables* __restrict__ tab, Scalars* sc, DecodeArgs a)
{
    static_assert(!PREV || MODE == DecMode::Half1, "only the second half-step reads two streams");
    static_assert(!TWO || PREV, "a second table only comes with a second stream");
    static_assert(KSPLIT == 1 || KSPLIT == 2 || KSPLIT == 4 || KSPLIT == 8, "the waves of a workgroup in groups of 1, 2, 4 or 8");
    static_assert(KSPLIT == 1 || MODE != DecMode::Decode, "plain decoding has nothing to add up");
    extern __shared__ __align__(16) uint32_t s_dyn[];    // [waves][2][stage_stride]
    __shared__ double s_sd[KSPLIT > 1 || MODE == DecMode::Half1 ? most_waves<MODE, PREV, TWO>() : 1];
    constexpr bool kTwo = two_chains<MODE, PREV>();       // chains per lane
    constexpr uint32_t kBufs = kTwo ? 2u : 1u;
    __shared__ __align__(16) unsigned char s_tab[kTabBytes];
    __shared__ __align__(16) unsigned char s_tab2[TWO ? kTabBytes : 16];
    const unsigned char* s_tab_b = TWO ? s_tab2 : s_tab;

    const int tid = (int)threadIdx.x, w = __builtin_amdgcn_readfirstlane(wave_id());
    int lane = lane_id();
    const uint32_t nwaves = blockDim.x >> 6;
    const int part = w & (KSPLIT - 1);                   // this wave's place in its group
    const uint32_t stage_words = a.stage_words;          // words half a chunk of this code can touch
    const uint32_t stage_stride = a.stage_stride;        // padded size of one staging buffer, words
    uint32_t* stage = s_dyn + (size_t)w * kBufs * stage_stride;
    uint32_t* stage_b = stage + stage_stride;

    if constexpr (WIDE) {
        bool ok = tab->wide_ok != 0u;
        if constexpr (TWO) ok = ok && a.tab_p->wide_ok != 0u;
        if (!ok) {                                        // the host chose this variant for another code
            if (tid == 0) raise_error(sc, QGX_EBIT_STATE);
            return;
        }
    }

    // ---- the task ---------------------------------------------------------------------------------
    // The chains of a lane: worker k; and its previous stream (PREV), or worker k + 1 (Decode).
    constexpr uint32_t kStep = MODE == DecMode::Decode ? 2u : 1u;
    const uint32_t g = blockIdx.x * nwaves + (uint32_t)w;                        // global wave number
    uint32_t task, k_first, k_count;
    bool mine;                                           // wave-uniform: there is such a task
    if (MODE == DecMode::Decode) {                       // a task of two workers
        const uint32_t pair = g / lay.n_tasks;
        task = g - pair * lay.n_tasks;
        mine = 2u * pair < lay.K;
        k_first = mine ? 2u * pair : 0u;
        k_count = min(2u, lay.K - k_first);
    } else {
        const uint32_t each = lay.K / KSPLIT, more = lay.K % KSPLIT;   // `more` runs of each + 1, then runs of each
        task = g / KSPLIT;
        mine = task < lay.n_tasks;
        k_first = (uint32_t)part * each + min((uint32_t)part, more);
        k_count = each + ((uint32_t)part < more ? 1u : 0u);            // (the host: KSPLIT <= K)
    }
    if (!mine) task = 0u;                                // (KSPLIT > 1: does its work for nobody; workgroup barriers below)
    const uint32_t ch = lay.task ? scalar_load(lay.task + task) : task;
    const uint32_t c = ch >> 1, half = ch & 1u;
    uint32_t clo, clen, bkt;
    chunk_geometry(lay, c, clo, clen, bkt);
    const uint32_t cend = clo + clen;
    const uint32_t base = clo + (uint32_t)kHalfCoords * half;                    // first coordinate of the task
    const bool full = base + (uint32_t)kHalfCoords <= cend;                      // (wave-uniform)
    // The loop with a look-ahead and, with two streams, squared differences in binary32 groups; the first half of a
    // short position has all its coordinates, but the sum of a short position is formed in binary64 throughout.
    const bool straight = PREV ? clen == (uint32_t)kChunk : full;

    StreamAt sa = stream_at(a.chunk_off, a.sub_end, a.norms, a.payload, a.cap_words, k_first, c, lay), sb = sa;
    if constexpr (PREV) sb = stream_at(a.chunk_off_p, a.sub_end_p, a.norms_p, a.payload_p, a.cap_words_p, k_first, c, lay);
    else if (kTwo && k_count > 1u) step_workers(sb, a.cap_words, 1u, lay);              // (an odd worker out: itself again, for nothing)
    const uint64_t cap_b = PREV ? a.cap_words_p : a.cap_words;
    auto meta_of = [&](const StreamAt& s, uint32_t ln) {
        // the lane's 32 coordinates lie in one bucket: the chunk's own, or with shared chunks one further on
        // (a lane past the end of a short chunk has nothing to decode: its index is kept inside the table)
        const uint32_t run = (uint32_t)kWave * half + ln;
        const uint32_t bucket = min(bkt + ((run * (uint32_t)kSub) >> lay.bucket_shift), lay.NB - 1u);
        return RunMeta{s.ends[run], s.norms[bucket]};
    };
    // Ahead of the parse travel, in registers, the next half chunks with their runs' ends and norms, and (scalar)
    // the extents of the ones after them, which have to be known before their words can be asked for.
    RunMeta ma{}, mb{};
    HalfRef ra{}, rb{};
    Extent xa{}, xb{};
    uint4 pre_a[kPre], pre_b[kPre];
    auto fetch = [&](uint32_t i, uint32_t ln) {
        ra = half_ref(sa.payload, a.cap_words, xa, stage_words, sc);
        prefetch_half(ra, pre_a, ln);
        ma = meta_of(sa, ln);
        if constexpr (kTwo) {
            rb = half_ref(sb.payload, cap_b, xb, stage_words, sc);
            prefetch_half(rb, pre_b, ln);
            mb = meta_of(sb, ln);
        }
        if (i + kStep < k_count) {
            step_workers(sa, a.cap_words, kStep, lay);
            xa = load_extent(sa, half);
            if constexpr (kTwo) {
                if (PREV || i + kStep + 1u < k_count) step_workers(sb, cap_b, kStep, lay);
                xb = load_extent(sb, half);
            }
        }
    };
    uint32_t fresh = (uint32_t)lane;
    xa = load_extent(sa, half);
    if constexpr (kTwo) xb = load_extent(sb, half);
    if (kTwo && straight) fetch(0u, fresh);
    load_tables<WIDE>(s_tab, tab, tid, (int)blockDim.x);
    if constexpr (TWO) load_tables<WIDE>(s_tab2, a.tab_p, tid, (int)blockDim.x);
    // words past a half chunk's end are read by the window of its last symbols: keep them defined
    for (uint32_t q = (uint32_t)lane; q < kBufs * stage_stride; q += kWave) stage[q] = 0;
    __syncthreads();
    if constexpr (KSPLIT == 1) {
        if (!mine && (MODE != DecMode::Half1 || a.end == kEndSums)) return;
    }                                                    // (else: the waves meet at workgroup barriers below)

    // From bit t of the staged words to the buffer bit r with the bit before t on top of the 64 bits
    // from r: r = r_base - t (they lie back to front).
    const uint32_t r_base = 32u * ((uint32_t)kTail + stage_words) - 63u;
    // A cursor from a corrupt table is pulled back so that a chain of 32 symbols from it stays inside
    // the buffer.  No valid cursor is beyond that: the last run of a half starts after 2016 symbols of
    // at most sym_bits each and up to 127 bits of the run before, and the buffer holds 2048 and 256 bits.
    const uint32_t p_limit = stage_words * 32u - (uint32_t)kSub * a.sym_bits;
    auto symbols_of = [&](uint32_t ln) {                  // symbols of lane ln's run
        const uint32_t at0 = base + (uint32_t)kSub * ln;
        return full ? kSub : (int)min((uint32_t)kSub, cend > at0 ? cend - at0 : 0u);
    };

    float acc[kSub], acc_b[MODE == DecMode::Decode ? kSub : 1];
#pragma unroll
    for (int s = 0; s < kSub; ++s) acc[s] = 0.0f;
    double sdiff = 0.0;
    uint32_t seen = 0;
    uint32_t bad = 0;                                    // not 0: malformed

    // RAG: a short half, or with two streams a half of a short position.  The symbols past a lane's count are parsed
    // like the others (from a cursor below p_limit 32 of them stay inside the buffer, and any window finds a table
    // entry) and count for nothing.  It has a loop of its own, without a look-ahead, so that what it holds on top costs
    // the full halves no registers.
    auto all_workers = [&](auto rag_tag) __attribute__((always_inline)) {
    constexpr bool RAG = decltype(rag_tag)::value;
    uint32_t i = 0;
    do {
        // (the lane number anew, so that the addresses made from it are worked out here and not held in two dozen
        // registers around the loop)
        asm volatile("" : "+v"(fresh));
        if (RAG || !kTwo) fetch(i, fresh);
        wave_lds_fence();                                     // the windows of the workers before have been read
        commit_half(stage, pre_a, ra, stage_words, fresh);
        if constexpr (kTwo) commit_half(stage_b, pre_b, rb, stage_words, fresh);
        wave_lds_fence();                                     // a lane parses words that other lanes stored
        const bool have_b = PREV || (kTwo && i + 1u < k_count);         // wave-uniform
        const float n = ma.n, nB = have_b ? mb.n : 0.0f;
        // first and last bit of the lane's runs, from the staged words' start (they wrap past p_limit if before it)
        const uint32_t t_end = ma.hi - 32u * ra.w0, tb_end = mb.hi - 32u * rb.w0;
        uint32_t t = wave_shift_in(ma.hi, ra.start) - 32u * ra.w0, tb = wave_shift_in(mb.hi, rb.start) - 32u * rb.w0;
        {
            const bool any = !RAG || symbols_of(fresh) > 0;
            bad |= (t > p_limit) & any;
            bad |= (tb > p_limit) & any & have_b;
        }
        t = min(t, p_limit);
        tb = min(tb, p_limit);
        if (!RAG && kTwo && i + kStep < k_count) fetch(i + kStep, fresh);
        // Squared differences: six at a time in binary32 (at most six roundings on a sum of
        // non-negative terms), the groups in binary64.  The differences are scaled by a power of two
        // taken from the larger of the lane's two norms, so that no square leaves the range of
        // binary32 whatever the scale of the vectors; the sum is scaled back in binary64.
        const uint32_t ex = min((__float_as_uint(fmaxf(n, nB)) >> 23) & 0xFFu, 253u);        // (254 - ex = 0 would be no power of two)
        const float down = __uint_as_float((254u - ex) << 23);                       // 2^(127 - ex)
        const double up2 = __longlong_as_double((long long)(2 * (int)ex - 254 + 1023) << 52);   // 2^(2 ex - 254)
        float sd32 = 0.0f;
        double sw = 0.0;

        auto parse = [&](auto pair_tag) __attribute__((always_inline)) {
            constexpr bool PAIR = decltype(pair_tag)::value;                    // both chains
            uint32_t q = r_base - t, qb = r_base - tb;
            uint32_t W[kGroup + 1], e[kGroup], W_b[kGroup + 1], e_b[kGroup];
            float held = 0.0f, held_b = 0.0f;
            uint32_t used = 0, used_b = 0, ignored = 0;
            const int cnt = RAG ? symbols_of(fresh) : kSub;
            Window wn = read_window(stage, q), wn_b{};
            if constexpr (PAIR) wn_b = read_window(stage_b, qb);
            auto emit = [&](int at, uint32_t w_next, float lv, uint32_t w_next_b, float lv_b) __attribute__((always_inline)) {
                if constexpr (MODE == DecMode::Decode) {
                    acc[at] = symbol_value<true>(w_next, lv, n);
                    if constexpr (PAIR) acc_b[at] = symbol_value<true>(w_next_b, lv_b, nB);
                } else if constexpr (PREV) {
                    const float val = symbol_value<false>(w_next, lv, n);
                    acc[at] += val;
                    const float val_p = symbol_value<false>(w_next_b, lv_b, nB);   // (a stray sign on a zero does not show in a difference)
                    if constexpr (RAG) {                                  // (short positions are few: every term in binary64)
                        const double df = (double)val_p - (double)val;
                        sdiff = fma(df, df, sdiff);
                    } else {
                        const float df = (val_p - val) * down;
                        sd32 = fmaf(df, df, sd32);
                        if (at % 6 == 4 || at == kSub - 1) { sw += (double)sd32; sd32 = 0.0f; }
                    }
                } else if constexpr (MODE == DecMode::Half1) {           // no previous streams: the vectors of t count as zero
                    const float val = symbol_value<false>(w_next, lv, n);
                    acc[at] += val;
                    sdiff = fma((double)val, (double)val, sdiff);
                    if constexpr (PAIR) {
                        const float val_b = symbol_value<false>(w_next_b, lv_b, nB);
                        acc[at] += val_b;
                        sdiff = fma((double)val_b, (double)val_b, sdiff);
                    }
                } else {
                    acc[at] = fmaf(signed_norm(w_next, n), lv, acc[at]);    // (a stray sign on a zero adds nothing)
                    if constexpr (PAIR) acc[at] = fmaf(signed_norm(w_next_b, nB), lv_b, acc[at]);
                }
            };
#pragma unroll
            for (int s = 0; s < kSub; s += kGroup) {
                // a group's last symbol is finished when the next group's first window (its sign on top) is there
                float lv[kGroup] = {0.f, 0.f, 0.f, 0.f}, lv_b[kGroup] = {0.f, 0.f, 0.f, 0.f};
                const bool last = s + kGroup == kSub;
                if (!last) {
                    parse_group<WIDE, false>(wn, s_tab, q, W, e, lv, RAG ? ignored : seen);
                    wn = read_window(stage, q);
                    if constexpr (PAIR) {
                        parse_group<WIDE, false>(wn_b, s_tab_b, qb, W_b, e_b, lv_b, RAG ? ignored : seen);
                        wn_b = read_window(stage_b, qb);
                    }
                } else {
                    parse_group<WIDE, true>(wn, s_tab, q, W, e, lv, RAG ? ignored : seen);
                    if constexpr (PAIR) parse_group<WIDE, true>(wn_b, s_tab_b, qb, W_b, e_b, lv_b, RAG ? ignored : seen);
                }
#pragma unroll
                for (int j = 0; j < kGroup; ++j) {
                    if constexpr (!WIDE) {
                        lv[j] = level_of(s_tab, e[j]);
                        if constexpr (PAIR) lv_b[j] = level_of(s_tab_b, e_b[j]);
                    }
                    if constexpr (RAG) {                                  // (a symbol past the count: one bit, no value)
                        const bool in = s + j < cnt;
                        e[j] = in ? e[j] : 63u;
                        lv[j] = in ? lv[j] : 0.0f;
                        if constexpr (PAIR) {
                            e_b[j] = in ? e_b[j] : 63u;
                            lv_b[j] = in ? lv_b[j] : 0.0f;
                        }
                    }
                }
                if constexpr (RAG) {
                    used -= (e[0] + e[1] + e[2] + e[3]) | 0xFFFFFFC0u;
                    seen |= (e[0] + e[1]) | (e[2] + e[3]);
                    if constexpr (PAIR) {
                        used_b -= (e_b[0] + e_b[1] + e_b[2] + e_b[3]) | 0xFFFFFFC0u;
                        seen |= (e_b[0] + e_b[1]) | (e_b[2] + e_b[3]);
                    }
                }
                if (s > 0) emit(s - 1, W[0], held, W_b[0], held_b);
#pragma unroll
                for (int j = 0; j < (last ? kGroup : kGroup - 1); ++j) emit(s + j, W[j + 1], lv[j], W_b[j + 1], lv_b[j]);
                held = lv[kGroup - 1]; held_b = lv_b[kGroup - 1];
                // A group's values are done before the next group's look-ups.  The compiler would move them behind
                // the whole chain of look-ups (into the block after the parse, and the scheduler again inside it)
                // and keep every entry and window until then, hundreds of registers.
#pragma unroll
                for (int at = s > 0 ? s - 1 : 0; at < s + (last ? kGroup : kGroup - 1); ++at) {
                    asm volatile("" : "+v"(acc[at]));
                    if constexpr (MODE == DecMode::Decode && PAIR) asm volatile("" : "+v"(acc_b[at]));
                }
                asm volatile("" : "+v"(seen), "+v"(bad));
                if constexpr (PREV && !RAG) asm volatile("" : "+v"(sd32), "+v"(sw));
                else if constexpr (MODE == DecMode::Half1) asm volatile("" : "+v"(sdiff));
                if constexpr (RAG) asm volatile("" : "+v"(used));
                if constexpr (RAG && PAIR) asm volatile("" : "+v"(used_b));
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (RAG) {
                const uint32_t rest = (uint32_t)(kSub - cnt);
                bad |= ((cnt > 0) & (t + used != t_end + rest)) | ((cnt > 0) & have_b & (tb + used_b != tb_end + rest));
            } else {
                bad |= (r_base - q) ^ t_end;
                if constexpr (PAIR) bad |= (r_base - qb) ^ tb_end;
            }
        };
        if constexpr (!kTwo) parse(BoolTag<false>{});
        else if (RAG || have_b) parse(BoolTag<true>{});       // (Decode of a short half, an odd worker out: a second chain for nothing)
        else parse(BoolTag<false>{});
        if constexpr (PREV && !RAG) sdiff = fma(sw, up2, sdiff);
        i += kStep;
    } while (i < k_count);
    };
    // (A wave without a task of its own, KSPLIT == 1, only meets the scalar end's barrier.  When it parsed task 0 for nobody, the second
    // half-step of 4 x 8392704 coordinates, 4098 tasks, took 66.8 us, now 64.6.)
    if (KSPLIT > 1 || mine) {
        if (straight) all_workers(BoolTag<false>{});
        else all_workers(BoolTag<true>{});
    }
    bad |= seen >> 15;                                   // (a reject entry among those parsed)
    if (__any(bad != 0u) && lane == 0) raise_error(sc, QGX_EBIT_STREAM);

    // ---- aggregate and update ---------------------------------------------------------------------
    // Lane L holds coordinates 32 L .. 32 L + 31 of the task.  Through LDS the wave turns them, kTurn lanes
    // at a time, so that eight lanes own a row of 32 consecutive floats and global accesses touch whole
    // 128-byte lines.
    // At 64 registers the loop has none to hold the lane's number in.  (Spilled, it and what is made from it cost the first
    // half-step of 8 x 2^24 coordinates 1.5 us, 8 bytes a lane written and read; the second half-step without a
    // previous stream then spills its sum's registers instead and is no faster.)
    if constexpr (!kTwo && MODE != DecMode::Half1) lane = late_lane_id();
    constexpr int kPitch = kSub + 4;                            // rows of 36 floats
    constexpr int kTurn = kTwo ? 32 : 16;                       // 1152 floats in two staging buffers, or 576 in one
    constexpr int kPasses = kWave / kTurn, kReads = kTurn / 8;
    float* tr = reinterpret_cast<float*>(stage);
    auto put_rows = [&](const float (&v)[kSub], int q, float scale) __attribute__((always_inline)) {
        if (mine && lane / kTurn == q) {
#pragma unroll
            for (int j = 0; j < kSub / 4; ++j)
                *reinterpret_cast<float4*>(tr + (lane % kTurn) * kPitch + 4 * j) =
                    make_float4(v[4 * j] * scale, v[4 * j + 1] * scale, v[4 * j + 2] * scale, v[4 * j + 3] * scale);
        }
    };
    const int row0 = lane >> 3, col = lane & 7;
    auto place = [&](int q, int i) -> uint32_t {                // this lane's i-th float4 of pass q
        return base + (uint32_t)(kSub * (kTurn * q + row0 + 8 * i) + 4 * col);
    };
    if constexpr (MODE == DecMode::Decode) {
        auto write_out = [&](const float (&v)[kSub], uint32_t k) __attribute__((always_inline)) {
            float* __restrict__ out = a.out + (size_t)k * lay.d;
#pragma unroll
            for (int q = 0; q < kPasses; ++q) {
                wave_lds_fence();
                put_rows(v, q, 1.0f);
                wave_lds_fence();
                if (full) {
#pragma unroll
                    for (int i = 0; i < kReads; ++i) {
                        const float4 m = *reinterpret_cast<const float4*>(tr + (row0 + 8 * i) * kPitch + 4 * col);
                        const f32x4_any o = {m.x, m.y, m.z, m.w};
                        *reinterpret_cast<f32x4_any*>(out + place(q, i)) = o;
                    }
                } else {
#pragma unroll 1
                    for (uint32_t f = (uint32_t)lane; f < (uint32_t)(kTurn * kSub); f += kWave) {
                        const uint32_t at = base + (uint32_t)(kTurn * kSub * q) + f;
                        if (at < cend) out[at] = tr[(f >> 5) * kPitch + (f & 31u)];
                    }
                }
            }
        };
        write_out(acc, k_first);
        if (k_count > 1u) write_out(acc_b, k_first + 1u);
        return;
    } else {
    const float invK = 1.0f / (float)lay.K;
    const float gam = sc->gamma_f;
    // (asked for early, and by a launch of one workgroup alone: the others' last barrier would wait for it, and only the last to arrive needs it)
    const double S_before = MODE == DecMode::Half1 && a.end == kEndAll ? sc->S : 0.0;
    if constexpr (MODE == DecMode::Half0) {               // one more term of the ergodic average
        if (a.x_sum && blockIdx.x == 0 && w == 0 && lane == 0) sc->avg_count += 1ull;
    }
    if constexpr (MODE == DecMode::Half1) {
        sdiff = wave_sum(sdiff);
        if (lane == 0) s_sd[w] = mine ? sdiff : 0.0;      // joined below, after a barrier
        if (KSPLIT == 1 && lane == 0 && a.end == kEndSums) a.s_partial[task] = sdiff;
    }
    // KSPLIT: all waves of the group put their sums there, and after a barrier each of them adds them
    // up (in the order of the workers' runs) for its share of the rows and does the update for those.
    const float* tr0 = KSPLIT > 1 ? reinterpret_cast<const float*>(s_dyn + (size_t)(w - part) * kBufs * stage_stride) : tr;
    const size_t tr_step = kBufs * (size_t)stage_stride;     // from one wave's buffer to the next, in words
    const float scale = KSPLIT > 1 ? 1.0f : invK;         // KSPLIT: the division comes after the group's sum
    // A piece of Y is asked for as soon as the piece before it in the same registers has been used, a pass
    // ahead of its own use: a load issued where it is used would be waited for in full.
    constexpr bool kYAhead = kTwo;                        // (with eight waves per SIMD the others cover it)
    float4 y_ahead[kReads];
    auto load_y = [&](int q, int i) {
        y_ahead[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (KSPLIT > 1 && ((q * kReads + i) & (KSPLIT - 1)) != part) return;
        if (mine && full) y_ahead[i] = *reinterpret_cast<const float4*>(a.Y + place(q, i));
    };
    if constexpr (kYAhead) {
#pragma unroll
        for (int i = 0; i < kReads; ++i) load_y(0, i);
    }
#pragma unroll
    for (int q = 0; q < kPasses; ++q) {
        wave_lds_fence();                                     // (the windows, the rows of the pass before: read)
        put_rows(acc, q, scale);
        wave_lds_fence();                                     // the rows are read by other lanes than wrote them
        if constexpr (KSPLIT > 1) {
            __syncthreads();
        }
        if (mine && full) {
#pragma unroll
            for (int i = 0; i < kReads; ++i) {
                if (kYAhead && q + 1 < kPasses && KSPLIT > 1 && ((q * kReads + i) & (KSPLIT - 1)) != part) { load_y(q + 1, i); continue; }
                if (KSPLIT > 1 && ((q * kReads + i) & (KSPLIT - 1)) != part) continue;   // a share of the rows for each wave of the group
                const int at_lds = (row0 + 8 * i) * kPitch + 4 * col;
                float4 m = *reinterpret_cast<const float4*>(tr0 + at_lds);
                if constexpr (KSPLIT > 1) {
#pragma unroll
                    for (int j = 1; j < KSPLIT; ++j) {
                        const float4 h4 = *reinterpret_cast<const float4*>(tr0 + j * tr_step + at_lds);
                        m.x += h4.x; m.y += h4.y; m.z += h4.z; m.w += h4.w;
                    }
                    m.x *= invK; m.y *= invK; m.z *= invK; m.w *= invK;
                }
                const uint32_t at = place(q, i);
                if (MODE == DecMode::Average) {
                    *reinterpret_cast<float4*>(a.out + at) = m;
                } else if (MODE == DecMode::Half0) {
                    const float4 y = kYAhead ? y_ahead[i] : *reinterpret_cast<const float4*>(a.Y + at);
                    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (a.anchor) x = *reinterpret_cast<const float4*>(a.anchor + at);
                    x.x = (x.x + gam * y.x) - gam * m.x;
                    x.y = (x.y + gam * y.y) - gam * m.y;
                    x.z = (x.z + gam * y.z) - gam * m.z;
                    x.w = (x.w + gam * y.w) - gam * m.w;
                    *reinterpret_cast<float4*>(a.out + at) = x;
                    if (kYAhead && q + 1 < kPasses) load_y(q + 1, i);
                    if (a.x_sum) {                               // ergodic average: sum of the half-step iterates
                        double2* xs = reinterpret_cast<double2*>(a.x_sum + at);
                        double2 s0 = xs[0], s1 = xs[1];
                        s0.x += (double)x.x; s0.y += (double)x.y; s1.x += (double)x.z; s1.y += (double)x.w;
                        xs[0] = s0; xs[1] = s1;
                    }
                } else {
                    float4 y = kYAhead ? y_ahead[i] : *reinterpret_cast<const float4*>(a.Y + at);
                    y.x -= m.x; y.y -= m.y; y.z -= m.z; y.w -= m.w;
                    *reinterpret_cast<float4*>(a.Y + at) = y;
                    if (kYAhead && q + 1 < kPasses) load_y(q + 1, i);
                }
            }
        } else if (mine) {
            // a short half: coordinate by coordinate, each wave of a group its share of the rows
#pragma unroll 1
            for (uint32_t f = (uint32_t)(kTurn * kSub / KSPLIT * part + lane); f < (uint32_t)(kTurn * kSub / KSPLIT * (part + 1)); f += kWave) {
                const uint32_t at = base + (uint32_t)(kTurn * kSub * q) + f;
                if (at >= cend) break;
                const uint32_t at_lds = (f >> 5) * (uint32_t)kPitch + (f & 31u);
                float m = tr0[at_lds];
                if constexpr (KSPLIT > 1) {
                    for (int j = 1; j < KSPLIT; ++j) m += tr0[j * tr_step + at_lds];
                    m *= invK;
                }
                if (MODE == DecMode::Average) {
                    a.out[at] = m;
                } else if (MODE == DecMode::Half0) {
                    const float x = ((a.anchor ? a.anchor[at] : 0.0f) + gam * a.Y[at]) - gam * m;
                    a.out[at] = x;
                    if (a.x_sum) a.x_sum[at] += (double)x;
                } else {
                    a.Y[at] -= m;
                }
            }
        }
        if constexpr (KSPLIT > 1) {
            if (q + 1 < kPasses) __syncthreads();             // the partners have read these rows
        }
    }
    // As much of the scalar end as the launch has been given (Half1End).  Where that is only sums (KSPLIT 1: left above; else the waves have put
    // theirs down since the first of the barriers), the waves go one by one: with a barrier here a worker of 19.7 M coordinates took 51.4 us, now
    // 48.5, and two of 1 M 11.0, now 10.5.
    if constexpr (MODE == DecMode::Half1) {
        if (a.end == kEndSums) {
            if (KSPLIT > 1 && mine && part == 0 && lane == 0) {
                double sd = s_sd[w];
                for (int j = 1; j < KSPLIT; ++j) sd += s_sd[w + j];
                a.s_partial[task] = sd;
            }
            return;
        }
        if (KSPLIT > 1 && a.end == kEndGroupSums) {
            if (tid == 0) {
                double sd = 0.0;
                for (uint32_t i = 0; i < nwaves; ++i) sd += s_sd[i];
                a.s_partial[blockIdx.x] = sd;
            }
            return;
        }
        __syncthreads();
        double own = 0.0;
        for (uint32_t i = 0; i < nwaves; ++i) own += s_sd[i];
        if (a.end == kEndAll) {                               // one workgroup: Y is its own work
            const double S = own + S_before;
            if (tid == 0) finish_scalars(sc, S, lay.K);
            x_from_y(step_size(S, lay.K), lay.d, a.Y, a.anchor, a.x_out, (uint32_t)tid, blockDim.x);
        } else if (w == 0) {
            // each leaves its sum and counts itself (release), and the last one to arrive (acquire) adds up the sums
            uint32_t before = 0;
            if (lane == 0) {
                __hip_atomic_store(&a.s_partial[blockIdx.x], own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                before = __hip_atomic_fetch_add(&sc->arrived, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            }
            if ((uint32_t)__builtin_amdgcn_readfirstlane((int)before) + 1u == gridDim.x) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                const double sum = wave_sum((uint32_t)lane < gridDim.x ? __hip_atomic_load(&a.s_partial[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0);
                if (lane == 0) {
                    finish_scalars(sc, sum + sc->S, lay.K);
                    __hip_atomic_store(&sc->arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
    }
    }
}

constexpr uint32_t kFinishThreads = 1024;      // of k_finish_half1

template <DecMode MODE, bool PREV, bool TWO, bool WIDE, int KSPLIT>
static hipError_t launch_as(const Layout& lay, const Tables* tab, Scalars* sc, const DecodeArgs& a, hipStream_t st, Half1End* left)
{
    const uint64_t nwaves = MODE == DecMode::Decode ? (uint64_t)lay.n_tasks * ((lay.K + 1u) / 2u) : (uint64_t)lay.n_tasks * (uint32_t)KSPLIT;
    // Workgroups of four waves spread over the compute units and are replaced as soon as four waves are done, but
    // each has tables of its own: the smallest with which the launch's waves all fit the LDS at once, and
    // where they do not fit anyway the largest, of which LDS holds the most waves (decode of 2^22 coordinates of
    // eight workers, 4096 waves: 26.5 us in workgroups of four, 28 to 30 in workgroups of sixteen).
    const size_t wave_lds = (size_t)(two_chains<MODE, PREV>() ? 2 : 1) * a.stage_stride * sizeof(uint32_t);
    const size_t tables_lds = (size_t)(TWO ? 2 : 1) * kTabBytes + 256;
    auto held = [&](uint32_t n) {                            // waves on a compute unit in workgroups of n
        return min((uint64_t)(160u * 1024u / (n * wave_lds + tables_lds)) * n, (uint64_t)(two_chains<MODE, PREV>() ? 16 : 32));
    };
    uint32_t per = (uint32_t)most_waves<MODE, PREV, TWO>();
    if (TWO && held(8) >= held(16)) per = 8;                 // (short codes: two of eight beside each other, 160 us to 164)
    for (uint32_t small = KSPLIT > 4 ? (uint32_t)KSPLIT : 4u; small < per; small *= 2)
        if (nwaves <= held(small) * a.n_cu) { per = small; break; }
    // The scalar end in the same launch, as long as a wave has a lane for each workgroup.  Second half-step of 8 workers, us, in a
    // launch of its own / in this one: 2 workgroups 15.8 / 14.5, 16 16.2 / 15.2, 64 16.4 / 15.6; with lanes that add up several sums
    // 65 18.2 / 17.6, 128 16.9 / 17.9, 256 17.6 / 22.2.  (A release and an acquire around the count cost nothing beside relaxed accesses.)
    // One workgroup, whose coordinates are all its own, writes X_{t+1} as well: an iteration of one bucket 30.9 us, now 28.0.
    const uint64_t grid = (nwaves + per - 1u) / per;
    DecodeArgs b = a;
    // A sum per workgroup (where its waves meet anyway) as soon as the next launch's threads would have more than one each to read: iterations of
    // 8 x 2^22 coordinates 146.0 us, with a sum per task 147.2.
    b.end = grid == 1u && a.x_out ? kEndAll : grid <= kWave ? kEndScalars : KSPLIT > 1 && lay.n_tasks > kFinishThreads ? kEndGroupSums : kEndSums;
    if (left) *left = Half1End{b.end == kEndSums ? lay.n_tasks : (uint32_t)grid, b.end};
    const size_t lds = (size_t)per * wave_lds;
    static LdsLimit limit;
    hipError_t e = limit.ensure(reinterpret_cast<const void*>(&k_decode<MODE, PREV, TWO, WIDE, KSPLIT>), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_decode<MODE, PREV, TWO, WIDE, KSPLIT>), dim3((uint32_t)grid), dim3(per * kWave), lds, st,
                       lay, tab, sc, b);
    return hipGetLastError();
}

template <DecMode MODE, bool PREV, bool TWO = false>
static hipError_t launch_mode(const Layout& lay, const Tables* tab, Scalars* sc, const DecodeArgs& a, hipStream_t st, Half1End* left)
{
    if constexpr (MODE != DecMode::Decode) {
        if (a.ksplit == 2u) {
            if (a.wide) return launch_as<MODE, PREV, TWO, true, 2>(lay, tab, sc, a, st, left);
            return launch_as<MODE, PREV, TWO, false, 2>(lay, tab, sc, a, st, left);
        }
        if (a.ksplit == 4u) {
            if (a.wide) return launch_as<MODE, PREV, TWO, true, 4>(lay, tab, sc, a, st, left);
            return launch_as<MODE, PREV, TWO, false, 4>(lay, tab, sc, a, st, left);
        }
        if (a.ksplit == 8u) {
            if (a.wide) return launch_as<MODE, PREV, TWO, true, 8>(lay, tab, sc, a, st, left);
            return launch_as<MODE, PREV, TWO, false, 8>(lay, tab, sc, a, st, left);
        }
    }
    if (a.wide) return launch_as<MODE, PREV, TWO, true, 1>(lay, tab, sc, a, st, left);
    return launch_as<MODE, PREV, TWO, false, 1>(lay, tab, sc, a, st, left);
}

hipError_t launch_decode(DecMode mode, const Layout& lay, const Tables* tab, Scalars* sc, const DecodeArgs& a,
                         hipStream_t st, Half1End* left)
{
    switch (mode) {
        case DecMode::Decode: return launch_mode<DecMode::Decode, false>(lay, tab, sc, a, st, left);
        case DecMode::Average: return launch_mode<DecMode::Average, false>(lay, tab, sc, a, st, left);
        case DecMode::Half0: return launch_mode<DecMode::Half0, false>(lay, tab, sc, a, st, left);
        default:
            if (a.payload_p == nullptr) return launch_mode<DecMode::Half1, false>(lay, tab, sc, a, st, left);
            return a.tab_p ? launch_mode<DecMode::Half1, true, true>(lay, tab, sc, a, st, left)
                           : launch_mode<DecMode::Half1, true>(lay, tab, sc, a, st, left);
    }
}

// ---- the scalar end of the second half-step: S, gamma_{t+1}, t; and X_{t+1} on request -----------
__global__ __launch_bounds__(kFinishThreads) void k_finish_half1(uint32_t n_sums, uint32_t K, Scalars* sc, const double* __restrict__ sums)
{
    __shared__ double s_red[kFinishThreads / kWave];
    double acc = 0.0;
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < n_sums; i += kFinishThreads) acc += sums[i];     // fixed order: reproducible
    acc = wave_sum(acc);
    if (lane_id() == 0) s_red[wave_id()] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double S = 0.0;
        for (uint32_t w = 0; w < kFinishThreads / kWave; ++w) S += s_red[w];
        finish_scalars(sc, S + sc->S, K);
    }
}

__global__ __launch_bounds__(256) void k_x_from_y(uint32_t d, const Scalars* sc, const float* __restrict__ Y,
                                                  const float* __restrict__ anchor, float* __restrict__ X)
{
    x_from_y(sc->gamma_f, d, Y, anchor, X, blockIdx.x * 256u + threadIdx.x, gridDim.x * 256u);
}

// Two launches, the second only, or none, by what the half-step has left.  (In one launch, each workgroup of the second adding up the
// sums, one of the half-step's workgroups each, by itself: no faster, iterations of 5 x 3 M 115.6 us, 115.7 with two, of 8 x 9.86 M 328.7 and 328.4.)
hipError_t launch_finish_half1(const Layout& lay, Scalars* sc, const double* s_partial, const float* Y,
                               const float* anchor, float* X_out, const Half1End& left, hipStream_t st)
{
    hipError_t e = hipSuccess;
    if (left.end == kEndSums || left.end == kEndGroupSums) {
        hipLaunchKernelGGL(k_finish_half1, dim3(1), dim3(kFinishThreads), 0, st, left.sums, lay.K, sc, s_partial);
        e = hipGetLastError();
    }
    if (e != hipSuccess || X_out == nullptr || left.end == kEndAll) return e;
    const uint32_t grid = min(lay.d / 1024u + 1u, 16384u);
    hipLaunchKernelGGL(k_x_from_y, dim3(grid), dim3(256), 0, st, lay.d, sc, Y, anchor, X_out);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_state_init(uint32_t d, uint32_t K, Scalars* sc, float* Y, float* anchor,
                                                    const float* X1)
{
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < d; i += gridDim.x * 256u) {
        Y[i] = 0.0f;
        anchor[i] = X1 ? X1[i] : 0.0f;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc->S = 0.0; sc->gamma = (double)K; sc->gamma_f = (float)K; sc->t = 1ull;
    }
}

hipError_t launch_state_init(const Layout& lay, Scalars* sc, float* Y, float* anchor, const float* X1, hipStream_t st)
{
    const uint32_t grid = min((lay.d + 255u) / 256u, 4096u);
    hipLaunchKernelGGL(k_state_init, dim3(grid), dim3(256), 0, st, lay.d, lay.K, sc, Y, anchor, X1);
    return hipGetLastError();
}

// Ergodic average of the half-step iterates: out = x_sum / count, the count kept on the device (so
// that the half-steps of a replayed graph are counted too); clearing the sum.
__global__ __launch_bounds__(256) void k_average(uint32_t d, const double* __restrict__ x_sum, const Scalars* sc,
                                                 float* __restrict__ out)
{
    const double count = (double)sc->avg_count;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < d; i += gridDim.x * 256u) out[i] = (float)(x_sum[i] / count);
}

hipError_t launch_average(uint32_t d, const double* x_sum, const Scalars* sc, float* out, hipStream_t st)
{
    const uint32_t grid = min((d + 255u) / 256u, 4096u);
    hipLaunchKernelGGL(k_average, dim3(grid), dim3(256), 0, st, d, x_sum, sc, out);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_average_reset(uint32_t d, double* __restrict__ x_sum, Scalars* sc)
{
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < d; i += gridDim.x * 256u) x_sum[i] = 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->avg_count = 0ull;
}

hipError_t launch_average_reset(uint32_t d, double* x_sum, Scalars* sc, hipStream_t st)
{
    const uint32_t grid = min((d + 255u) / 256u, 4096u);
    hipLaunchKernelGGL(k_average_reset, dim3(grid), dim3(256), 0, st, d, x_sum, sc);
    return hipGetLastError();
}

__global__ void k_state_set(Scalars* sc, double S, unsigned long long t, uint32_t K)
{
    const double gamma = (double)K / sqrt(1.0 + S);
    sc->S = S; sc->gamma = gamma; sc->gamma_f = (float)gamma; sc->t = t;
}

hipError_t launch_state_set(Scalars* sc, double S, unsigned long long t, uint32_t K, hipStream_t st)
{
    hipLaunchKernelGGL(k_state_set, dim3(1), dim3(1), 0, st, sc, S, t, K);
    return hipGetLastError();
}

// Bits of the last coded streams, without padding: the last sub-chunk entry of every chunk.
__global__ __launch_bounds__(256) void k_sum_bits(uint64_t n_chunks, const uint16_t* sub_end, Scalars* sc)
{
    __shared__ unsigned long long s_red[256];
    unsigned long long acc = 0;
    for (uint64_t i = threadIdx.x; i < n_chunks; i += 256) acc += sub_end[i * kSubs + (kSubs - 1)];
    s_red[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) s_red[threadIdx.x] += s_red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) sc->total_bits = s_red[0];
}

hipError_t launch_sum_bits(const Layout& lay, const uint16_t* sub_end, Scalars* sc, hipStream_t st)
{
    hipLaunchKernelGGL(k_sum_bits, dim3(1), dim3(256), 0, st, (uint64_t)lay.K * lay.NC, sub_end, sc);
    return hipGetLastError();
}

// ---- slotted -> compact ---------------------------------------------------------------------------
// One workgroup per worker scans the chunk sizes (from the bit lengths) into exclusive offsets; then
// one wave per chunk copies its words.
__device__ __forceinline__ uint32_t chunk_words_of(const uint16_t* __restrict__ sub_end, size_t chunk)
{
    const uint32_t bits = sub_end[chunk * kSubs + (kSubs - 1)];
    return (((bits + 31u) >> 5) + 3u) & ~3u;
}

__global__ __launch_bounds__(1024) void k_compact_offsets(uint32_t NC, const uint16_t* __restrict__ sub_end,
                                                          uint32_t* __restrict__ out_off, uint64_t out_cap, Scalars* sc)
{
    __shared__ uint32_t s_wave[16];
    const uint32_t k = blockIdx.x, tid = threadIdx.x;
    const int lane = lane_id(), w = wave_id();
    // a thread's chunks are consecutive, so its own running sum is all it carries between the two passes
    const uint32_t per = (NC + 1023u) / 1024u;
    const uint32_t c0 = min(tid * per, NC), c1 = min(c0 + per, NC);
    uint32_t sum = 0;
    for (uint32_t c = c0; c < c1; ++c) sum += chunk_words_of(sub_end, (size_t)k * NC + c);
    const uint32_t incl = wave_incl_scan(sum);
    if (lane == kWave - 1) s_wave[w] = incl;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (int i = 0; i < 16; ++i) {
        if (i == w) before = total;
        total += s_wave[i];
    }
    if (tid == 0) {
        out_off[(size_t)k * (NC + 1) + NC] = total;
        if ((uint64_t)total > out_cap) raise_error(sc, QGX_EBIT_CAPACITY);
    }
    uint32_t run = before + incl - sum;
    for (uint32_t c = c0; c < c1; ++c) {
        out_off[(size_t)k * (NC + 1) + c] = run;
        run += chunk_words_of(sub_end, (size_t)k * NC + c);
    }
}

constexpr int kChunkPieces = kChunkWordsMax / (kWave * 4);   // 7 x uint4 per lane cover a worst-case chunk

__global__ __launch_bounds__(256) void k_compact_copy(uint32_t NC, uint32_t K, const uint16_t* __restrict__ sub_end,
                                                      const uint32_t* __restrict__ in_off, const uint32_t* __restrict__ in_payload,
                                                      uint64_t in_cap, const uint32_t* __restrict__ out_off,
                                                      uint32_t* __restrict__ out_payload, uint64_t out_cap, Scalars* sc)
{
    const uint32_t g = blockIdx.x * (blockDim.x >> 6) + (uint32_t)wave_id();
    if (g >= K * NC) return;
    const uint32_t k = g / NC, c = g - k * NC, lane = (uint32_t)lane_id();
    const uint32_t words = chunk_words_of(sub_end, (size_t)k * NC + c);
    const uint32_t src = in_off[(size_t)k * (NC + 1) + c], dst = out_off[(size_t)k * (NC + 1) + c];
    if ((src & 3u) || (uint64_t)src + words > in_cap || (uint64_t)dst + words > out_cap) {
        if (lane == 0) raise_error(sc, (uint64_t)dst + words > out_cap ? QGX_EBIT_CAPACITY : QGX_EBIT_STREAM);
        return;
    }
    const uint4* s = reinterpret_cast<const uint4*>(in_payload + (size_t)k * in_cap + src);
    uint4* d = reinterpret_cast<uint4*>(out_payload + (size_t)k * out_cap + dst);
    // a chunk of the largest size is kChunkPieces pieces per lane: all of a lane's loads are on their way before
    // its first store (a chunk of some other origin may be longer: the loop goes on)
    for (uint32_t q0 = 0; q0 < (words >> 2); q0 += (uint32_t)(kChunkPieces * kWave)) {
        uint4 held[kChunkPieces];
#pragma unroll
        for (int j = 0; j < kChunkPieces; ++j) {
            const uint32_t q = q0 + lane + (uint32_t)j * kWave;
            held[j] = q < (words >> 2) ? nt_load4u(s + q) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < kChunkPieces; ++j) {
            const uint32_t q = q0 + lane + (uint32_t)j * kWave;
            if (q < (words >> 2)) d[q] = held[j];
        }
    }
}

hipError_t launch_compact(const Layout& lay, const uint16_t* sub_end, const uint32_t* in_off, const uint32_t* in_payload,
                          uint64_t in_cap, uint32_t* out_off, uint32_t* out_payload, uint64_t out_cap, Scalars* sc,
                          hipStream_t st)
{
    hipLaunchKernelGGL(k_compact_offsets, dim3(lay.K), dim3(1024), 0, st, lay.NC, sub_end, out_off, out_cap, sc);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const uint32_t grid = (lay.K * lay.NC + 3u) / 4u;
    hipLaunchKernelGGL(k_compact_copy, dim3(grid), dim3(256), 0, st, lay.NC, lay.K, sub_end, in_off, in_payload, in_cap,
                       out_off, out_payload, out_cap, sc);
    return hipGetLastError();
}

}  // namespace qgx
