// CODE o Q in one pass: per-bucket norm, normalise, level lookup, stochastic rounding, code lookup,
// bit packing through LDS, ordered placement of the chunks in the payload.
// (Definition 1; Section 3.2; Appendix J "Encoding".)
//
// Work decomposition for 64-wide wavefronts: one workgroup per (worker, bucket), per few short ones (buckets_per_group), or
// several per bucket when it is longer than four chunks (see exchange_parts); one wave per chunk of
// 4096 coordinates.  A wave holds its chunk in registers as 16 rows of 256 coordinates, lane L owning
// the four consecutive coordinates 4L..4L+3 of every row, so that (a) every global load is a fully
// coalesced 16-byte-per-lane access, (b) the bucket is read from HBM once and stays in registers
// between the norm reduction and the rounding pass, (c) one Philox4x32 block (four words) serves
// exactly the four coordinates of a lane and row.
//
// The vector ALUs' issue bounds it (112 instructions per row of four coordinates a lane, a third of them the generator), the
// memory system is next (5.4 TB/s of the 6.2 that the best streaming kernel reaches), so the per-coordinate path is kept to a
// straight line: u -> cell (1/16, 1/32 or 1/64 of an octave, by the table's size) -> (boundary level, lower candidate level)
// -> one 16-byte LDS row holding the level, the scaled gap and the two candidate code words with the sign
// already appended -> compare against the Philox draw -> select.  A chunk's short last row, buckets
// whose norm is zero or has no finite reciprocal and level tables too fine for the cell table take a general path, row by row from memory.
// Measured, us (120 instructions a row, tables waited for before a chunk is asked for, a workgroup per bucket -> now):
// 8 x 2^24 coordinates 147 -> 138, 8 x 9.86 M in buckets of 8192 96 -> 83, of 1024 101 -> 86, 5 x 3000001 in buckets of 6000
// 35 -> 28, 2^20 coordinates 11.7 -> 9.9.
//
// The stream keeps coordinate order: the lanes' code lengths are prefix-summed across the wave (DPP, two rows in
// one scan) and every lane ORs its (at most 56) bits into the wave's LDS staging buffer.  No branch lies between
// the rows of a full chunk.  (A scan per row and a branch around the store of the sub-chunk ends: 160
// instructions a row, 8 x 2^24 coordinates 173 us; without 163.)
// Placement of the chunks in the payload.  Slotted: chunk c goes to c * slot_words; no workgroup waits
// for another.  Compact: chunks in chunk order without gaps, so a workgroup needs the total length of
// all earlier buckets of its worker: a decoupled look-back over per-bucket (flag, length) words gives
// it without a second pass over V.  There a workgroup's worker is fixed by its block index and its
// buckets come from that worker's atomic ticket, so every bucket a waiting workgroup depends on is
// held by a running workgroup that needs nothing from later tickets; the wait is bounded all the same.
#include "qgx_device.h"
#include "qgx_plan.h"

namespace qgx {

constexpr unsigned kSpinLimit = 1u << 22;
constexpr float kNoReciprocal = 0x1p-128f;        // 1 / n overflows binary32 for n up to this

// Exclusive prefix of `agg` over buckets 0..b-1 of one worker (decoupled look-back, one wave).
// state[] entries: high word = epoch << 2 | status (1 = aggregate, 2 = inclusive prefix), low word = value.
__device__ uint32_t lookback_exclusive(unsigned long long* state, uint32_t b, uint32_t agg, uint32_t epoch,
                                       Scalars* sc)
{
    const int lane = lane_id();
    const unsigned long long tag_agg = (unsigned long long)((epoch << 2) | 1u) << 32;
    const unsigned long long tag_pre = (unsigned long long)((epoch << 2) | 2u) << 32;
    if (b == 0) {
        if (lane == 0) __hip_atomic_store(&state[0], tag_pre | agg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return 0;
    }
    if (lane == 0) __hip_atomic_store(&state[b], tag_agg | agg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t excl = 0;
    int pos = (int)b - 1;
    unsigned spins = 0;
    for (;;) {
        const int i = pos - lane;
        unsigned long long s = 0;
        bool ready = i < 0;
        unsigned long long done, pre;
        for (;;) {
            if (!ready) {                         // (what has been seen is not asked for again)
                s = __hip_atomic_load(&state[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint32_t flag = (uint32_t)(s >> 32);
                ready = ((flag >> 2) == epoch) && ((flag & 3u) != 0u);
            }
            done = __ballot(ready);
            pre = __ballot(ready && i >= 0 && ((uint32_t)(s >> 32) & 3u) == 2u);
            // the nearest full prefix and everything since, or the whole window
            if (pre != 0ull ? (~done & (pre & (0ull - pre)) - 1ull) == 0ull : done == ~0ull) break;
            if (++spins > kSpinLimit) {           // never expected: every predecessor is already running
                if (lane == 0) raise_error(sc, QGX_EBIT_STATE);
                if (!ready) s = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
        const uint32_t val = i >= 0 ? (uint32_t)s : 0u;
        if (pre != 0ull) {
            const int first = __ffsll((long long)pre) - 1;    // nearest predecessor with a full prefix
            excl += wave_sum_u32(lane <= first ? val : 0u);
            break;
        }
        excl += wave_sum_u32(val);
        if (pos < kWave) break;
        pos -= kWave;
    }
    if (lane == 0)
        __hip_atomic_store(&state[b], tag_pre | (unsigned long long)(excl + agg), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    return excl;
}

// Buckets longer than four chunks are shared by several workgroups of four waves (parts), which a
// compute unit holds five of (four in the forms with look-ups ahead) at different points of their life, where one workgroup of sixteen waves
// would have the unit to itself and leave the memory system idle while it computes and the ALUs idle
// while it loads.  What the parts must agree on is the bucket's norm: every part publishes its
// partial sum (or maximum) and reads the others'.  A published value is two words, each tagged with
// the launch's epoch, so a reader knows a word is this launch's without any ordering between
// stores.  The wait cannot deadlock: parts take their (bucket, part) from the worker's ticket
// counter, so at most the bucket of the newest tickets is incomplete, and every other waiting
// workgroup has all its partners running; for the partners of the newest there is always a place on the
// XCD whose queue they are in (worker_span).  The wait is bounded all the same.
// Called by one whole wave; returns the parts' values combined in part order in every lane.
__device__ double exchange_parts(unsigned long long* words /* [parts][2 phases][2] of this bucket */, uint32_t parts,
                                 uint32_t part, uint32_t phase, double mine, bool take_max, uint32_t epoch, Scalars* sc)
{
    const int lane = lane_id();
    const unsigned long long tag = (unsigned long long)epoch << 32;
    const unsigned long long bits = (unsigned long long)__double_as_longlong(mine);
    if (lane < 2)
        __hip_atomic_store(&words[(part * 2u + phase) * 2u + (uint32_t)lane],
                           tag | (lane ? (bits >> 32) : (bits & 0xFFFFFFFFull)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool reader = (uint32_t)lane < 2u * parts;
    const uint32_t at = (((uint32_t)lane >> 1) * 2u + phase) * 2u + ((uint32_t)lane & 1u);
    unsigned long long s = 0;
    unsigned spins = 0;
    for (;;) {
        bool ready = true;
        if (reader) {
            s = __hip_atomic_load(&words[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ready = (uint32_t)(s >> 32) == epoch;
        }
        if (__all(ready)) break;
        if (++spins > kSpinLimit) {               // never expected: see above
            if (lane == 0) raise_error(sc, QGX_EBIT_STATE);
            if (!ready) s = 0;
            break;
        }
        __builtin_amdgcn_s_sleep(8);
    }
    double tot = 0.0;
    for (uint32_t p = 0; p < parts; ++p) {
        const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)s, (int)(2u * p), kWave);
        const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)s, (int)(2u * p + 1u), kWave);
        const double x = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
        if (take_max) tot = (x > tot || x != x) ? x : tot;
        else tot += x;
    }
    return tot;
}

// The encoder's tables start at LDS address 0 (checked at entry), so that where they lie is known at compile time: the
// cells, then the level rows (Tables::enc).  CM: the table's cell size, mantissa bits per octave.
template <int CM> constexpr uint32_t kCellShift = 23u - CM;                              // bits of u >> that: cell number + kCellKey0
template <int CM> constexpr uint32_t kCellKey0 = (uint32_t)(127 - kCellOct) << CM;       // (everything below goes to the first cell, too)
template <int CM> constexpr uint32_t kLevAt = lev_piece0(CM) * 16u;                      // LDS address of the level rows

// tau(u) by the general route: start at the cell's lower level and walk up.
template <int CM>
__device__ __forceinline__ uint32_t level_general(float u, uint32_t n_sym)
{
    const float um = fminf(fmaxf(u, __uint_as_float(kCellKey0<CM> << kCellShift<CM>)), 1.0f);
    uint32_t j = lds_load_u2(((__float_as_uint(um) >> kCellShift<CM>) - kCellKey0<CM>) * 8u).y;
    while (j + 2 < n_sym && __uint_as_float(lds_load_u32(kLevAt<CM> + 32u * (j + 1u))) <= u) ++j;
    return j;
}

// One coordinate's way to the code entry E(idx, sign) of q_l(u) with its sign, in three parts, so that other work can stand
// between a look-up and its use: the cell of u, the level row, the decision.  Straight-line cell route: valid when u <= 1 up
// to rounding (so the clamp of u to 1 can be left out: at u >= 1 the coordinate rounds up whatever the draw) and no cell
// holds two levels.
// first_cell: kCellKey0 << kCellShift.
template <int CM>
__device__ __forceinline__ uint2 cell_of(float u, uint32_t first_cell)
{
    // cell number times eight; a saturating subtraction sends everything below the first cell there
    static_assert(((uint32_t)((kCellOct << CM) + 1) * 8u) <= 0x10000u, "cell numbers times eight fit 16 bits");
    return lds_load_u2((__builtin_elementwise_sub_sat(__float_as_uint(u), first_cell) >> (kCellShift<CM> - 3u)) & 0xFFF8u);
}

__device__ __forceinline__ uint32_t level_in_cell(float u, uint2 c) { return c.y + (u >= __uint_as_float(c.x) ? 1u : 0u); }

template <int CM>
__device__ __forceinline__ uint4 level_row(uint32_t j, float x)
{
    return lds_load_u4(__builtin_amdgcn_alignbit(j, __float_as_uint(x), 31) * 16u + kLevAt<CM>);       // row 2 j + sign
}

// Up with probability xi = (u - l_j) / (l_{j+1} - l_j):  r * gap < u - l_j, r = top 24 bits * 2^-24.
__device__ __forceinline__ bool rounds_up(float u, uint4 t, uint32_t rnd)
{
    return (float)(rnd >> 8) * __uint_as_float(t.y) < u - __uint_as_float(t.x);      // (t.y = gap * 2^-24: exact scaling)
}

// Where a chunk's sub-chunk ends go, eight lanes of a row one 16-byte piece: the row of the table as a buffer
// of 256 bytes.  A run's last lane writes; the others' offset lies outside the buffer, and such stores are dropped:
// no branch, so that the rows of a chunk are one straight line for the scheduler.
struct SubEnds {
    __amdgpu_buffer_rsrc_t row;
    uint32_t at;                 // 2 * (the lane's run in a row), or outside
    __device__ __forceinline__ SubEnds(uint16_t* table_row, int lane)
        : row(__builtin_amdgcn_make_buffer_rsrc(table_row, 0, kSubs * (int)sizeof(uint16_t), 0x00027000)),
          at((lane & 7) == 7 ? 2u * (uint32_t)(lane >> 3) : 0x40000000u) {}
    __device__ __forceinline__ void put(int r, uint32_t end) const
    {
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)end, row, (int)(at + 16u * (uint32_t)r), 0, 0);
    }
};

// A lane's four entries of a row joined: their bits one after the other (<= 56), and the sum of the entries, whose byte 1 is
// their number.  (An entry: the code word at the top, its length from bit 8 on, 32 less the length in the low five bits.)
struct RowCode { uint32_t sum, lo, hi; };

// {hi, lo} >> (s mod 32), the low word
__device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t s) { return __builtin_amdgcn_alignbit(hi, lo, s); }

// Every shift count is the low five bits of an entry or of a sum of entries, which the hardware takes as they are: a word
// comes down from the top by its own entry, and the funnel shift by the entry before it puts the word behind that one, whose
// low bits it drops.  Entries of 0 (no symbol) come last and add nothing.
__device__ __forceinline__ RowCode join_row(const uint32_t (&e)[4])
{
    const uint32_t c01 = funnel(e[1] >> (e[1] & 31u), e[0], e[0]);         // <= 28 bits
    const uint32_t c23 = funnel(e[3] >> (e[3] & 31u), e[2], e[2]);
    const uint32_t s01 = e[0] + e[1];                                      // low five bits: 32 less the bits of c01
    return RowCode{s01 + e[2] + e[3], funnel(c23, c01 << (s01 & 31u), s01), c23 >> (s01 & 31u)};
}

// The bits go to bit P + 1 of LDS (P counts from LDS address 0): with the place less one at hand no shift count is 32.
__device__ __forceinline__ void place_row(uint32_t P, const RowCode& c)
{
    const uint32_t up = ~P;                                                // 32 less the place's bit in its word, mod 32
    auto* at = reinterpret_cast<__attribute__((address_space(3))) uint32_t*>((uintptr_t)((P >> 3) & ~3u));
    __hip_atomic_fetch_or(at, funnel(c.lo, 0u, up), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_or(at + 1, funnel(c.hi, c.lo, up), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_or(at + 2, c.hi >> (up & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Appends row r (four entries per lane) to the wave's staging buffer, whose first bit is bit stage0 + 1 of LDS; returns the
// row's bit count.
// BRANCH: the sub-chunk ends' store behind a branch after all, for the rolled loop, whose rows no scheduler mixes: dropped
// stores are not free (symbols of 8 x 2^22 coordinates in words of three bits coded in 28 us instead of 31).
template <bool BRANCH>
__device__ __forceinline__ uint32_t pack_row(uint32_t stage0, const SubEnds& ends, int r, uint32_t row_base, const uint32_t (&e)[4])
{
    const RowCode c = join_row(e);
    const uint32_t len = (c.sum >> 8) & 0xFFu, incl = wave_incl_scan(len);
    place_row(stage0 + row_base + incl - len, c);
    if (!BRANCH || ends.at < (uint32_t)kSubs) ends.put(r, row_base + incl);
    return (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
}

// The same for rows r and r + 1: a row's bit count (at most 64 * 56) fits 16 bits, so one scan across the wave
// does both.
__device__ __forceinline__ uint32_t pack_two_rows(uint32_t stage0, const SubEnds& ends, int r, uint32_t row_base,
                                                  const uint32_t (&ea)[4], const uint32_t (&eb)[4])
{
    const RowCode a = join_row(ea), b = join_row(eb);
    const uint32_t both = __builtin_amdgcn_perm(b.sum, a.sum, 0x0C050C01u);       // the two lengths: byte 1 of each sum
    const uint32_t incl = wave_incl_scan(both), excl = incl - both;
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    const uint32_t second = row_base + (total & 0xFFFFu);
    place_row(stage0 + row_base + (excl & 0xFFFFu), a);
    ends.put(r, row_base + (incl & 0xFFFFu));
    place_row(stage0 + second + (excl >> 16), b);
    ends.put(r + 1, second + (incl >> 16));
    return (total & 0xFFFFu) + (total >> 16);
}

struct ChunkGeom {            // one wave's share of a bucket
    uint32_t c;               // chunk number
    uint32_t clo, clen, cend; // first coordinate, length, one past the last
    int nrows;                // rows of 256 coordinates that hold data
    bool full;                // all 4096 coordinates present
    uint32_t bparts;          // workgroups that share the bucket (groups of four chunks that hold data)
};

// Chunk w of bucket b; no chunk (clen = 0) past the bucket's last one, or with !there.
__device__ __forceinline__ ChunkGeom chunk_geom(const Layout& lay, uint32_t b, uint32_t w, bool there)
{
    uint32_t lo, hi, c0;
    if (lay.uniform_bucket) {                      // one segment: no table look-ups on the critical path
        lo = b * lay.uniform_bucket;
        hi = min(lo + lay.uniform_bucket, lay.d);
        c0 = b * lay.waves_per_bucket;
    } else {
        lo = scalar_load(lay.bucket_start + b); hi = scalar_load(lay.bucket_start + b + 1); c0 = scalar_load(lay.bucket_chunk0 + b);
    }
    ChunkGeom g;
    g.c = c0 + w;
    g.clo = lo + w * kChunk;
    g.clen = there && g.clo < hi ? min((uint32_t)kChunk, hi - g.clo) : 0u;
    g.cend = g.clo + g.clen;
    g.nrows = (int)((g.clen + 255u) >> 8);
    g.full = g.clen == (uint32_t)kChunk;
    g.bparts = ((hi - lo + (uint32_t)kChunk - 1u) / (uint32_t)kChunk + 3u) >> 2;
    return g;
}

// Shared chunks (buckets of 256..2048 coordinates): a wave's chunk holds up to 16 buckets, each a run
// of whole rows, so the wave works out their norms by itself, one wave reduction at the last row of
// every bucket, and leaves 1 / norm (0 for a bucket that is all zero or rejected) in LDS for the
// rounding pass.  Returns whether the straight-line rounding path applies to the whole chunk: every
// bucket live, no coordinate above its norm, and no norm so small that its reciprocal overflows.
template <EncMode MODE>
__device__ __forceinline__ bool shared_chunk_norms(const float4 (&v)[kRows], const float* __restrict__ Vk,
                                                   const ChunkGeom& g, const Layout& lay, const EncodeArgs& a,
                                                   Scalars* sc, uint32_t k, uint32_t bucket0, float* rinv_out, int lane)
{
    const uint32_t bshift = lay.bucket_shift, rshift = bshift - 8u;
    const uint32_t rows_mask = (1u << rshift) - 1u;
    const bool l2 = a.norm_kind == QGX_NORM_L2;
    bool plain = true;
    float p0 = 0.0f, p1 = 0.0f, p2 = 0.0f, p3 = 0.0f;
    float mx = 0.0f;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        if (l2) {
            p0 = fmaf(v[r].x, v[r].x, p0);
            p1 = fmaf(v[r].y, v[r].y, p1);
            p2 = fmaf(v[r].z, v[r].z, p2);
            p3 = fmaf(v[r].w, v[r].w, p3);
        } else {
            mx = largest_of(v[r], mx);
        }
        if ((((uint32_t)r + 1u) & rows_mask) != 0u) continue;             // wave-uniform: the bucket goes on
        const uint32_t gb = (uint32_t)r >> rshift;
        const uint32_t lo = g.clo + (gb << bshift);
        if (lo < g.cend) {
            const uint32_t hi = min(lo + (1u << bshift), g.cend);
            double tot;
            if (l2) {
                tot = wave_sum(((double)p0 + (double)p1) + ((double)p2 + (double)p3));
                if (!(tot >= 0x1p-60 && tot <= 0x1p100)) {                // as in the kernel: redo in binary64
                    double acc = 0.0;
#pragma unroll 1
                    for (uint32_t i = lo + (uint32_t)lane; i < hi; i += kWave) acc = fma((double)Vk[i], (double)Vk[i], acc);
                    tot = wave_sum(acc);
                }
            } else {
                tot = (double)__uint_as_float(wave_max_u32(__float_as_uint(mx)));
            }
            float n = l2 ? (float)sqrt(tot) : (float)tot;
            if (!l2 && a.norm_kind != QGX_NORM_LINF && tot > 0.0 && tot <= 3.402823466e+38) {
                const double inv_m = 1.0 / tot;
                double acc = 0.0;
#pragma unroll 1
                for (uint32_t i = lo + (uint32_t)lane; i < hi; i += kWave)
                    acc += pow_int(fabs((double)Vk[i]) * inv_m, (uint32_t)a.norm_kind);
                n = (float)(tot * root_int(wave_sum(acc), (uint32_t)a.norm_kind));
            }
            bool u_le_1 = true;
            if (a.norms_in) {
                const float forced = a.norms_in[(size_t)k * lay.NB + bucket0 + gb];
                u_le_1 = forced >= n;
                n = (n == n && fabsf(n) <= 3.402823466e+38f) ? forced : n;
            }
            const bool bucket_bad = !(fabsf(n) <= 3.402823466e+38f);
            if (bucket_bad) n = 0.0f;
            const bool live = n > 0.0f;
            if (lane == 0) {
                if (bucket_bad) raise_error(sc, QGX_EBIT_NONFINITE);
                if (a.norms_out) a.norms_out[(size_t)k * lay.NB + bucket0 + gb] = n;
                rinv_out[gb] = live ? 1.0f / n : 0.0f;                    // one IEEE division per bucket
            }
            plain = plain && n > kNoReciprocal && u_le_1;
        }
        p0 = p1 = p2 = p3 = 0.0f;
        mx = 0.0f;
    }
    return plain;
}

// One workgroup per (worker, bucket), group of short buckets or part of a long one.  Workgroups are short-lived on purpose: with five of
// them (four with look-ups ahead) per compute unit at different points of their life, the load, ticket and look-back latencies of one
// overlap the arithmetic of the others (a persistent, lock-stepped variant measured slower).
// GROUPED: the layout has shared chunks; a workgroup is four waves with a chunk each, and every wave
// finds the norms of its chunk's buckets by itself.
// CM: cell_mant of the level table, so that the rounding pass has the cell size as a constant.
// STAGED: a row's four look-ups are asked for together, cells before the generator and level rows after it, at four waves
// per SIMD, whose registers hold it (at five 17 were spilled: 8 x 2^24 coordinates 148 us instead of 137).  The game's form, whose
// second generator and transcendentals need the registers anyway, always: 16 x 2^26 coordinates 2.02 -> 1.93 ms.  Where V is
// read, launches of few waves, which wait for their look-ups with little else to do (use_staged).
template <EncMode MODE> constexpr bool kWaits = MODE != EncMode::EncodeOnly;     // for partners: it needs the bucket's norm
template <bool STAGED> constexpr int kSimdWaves = STAGED ? 4 : 5;
template <EncMode MODE, bool GROUPED, int CM, bool STAGED>
// (On a page: up to 78 KB of code, more than the instruction cache holds, so that where it lies counts.  The kernels ahead of it in the object
// moved it by 3.5 KB: an iteration of 8 x 9.86 M in buckets of 1024 336.6 us on a page, 338.6 off it; other layouts 0.2 % either way.)
__global__ __launch_bounds__(GROUPED ? 256 : 1024) __attribute__((amdgpu_waves_per_eu(kSimdWaves<STAGED>), aligned(4096)))
void k_encode(Layout lay, const Tables* __restrict__ tab, Scalars* sc, EncodeArgs a)
{
    extern __shared__ __align__(16) unsigned char s_all[];
    const int tid = (int)threadIdx.x, lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(wave_id());    // (scalar, and all of the chunk's geometry with it)
    const int nwaves = (int)(blockDim.x >> 6);
    // The worker and, without tickets, the unit of work are fixed by the block.
    uint32_t k = blockIdx.x % a.span, own_unit = blockIdx.x / a.span;
    if (a.spread) k = worker_spread(k, own_unit, a.span);
    if (MODE == EncMode::Generate && a.by_unit) {
        const BlockWork own = block_by_unit(blockIdx.x, lay.K, a.units);
        k = own.k; own_unit = own.unit;
    }

    // LDS plan: [tables][reduction scratch][one staging buffer per wave]
    uint4* s_enc = reinterpret_cast<uint4*>(s_all);
    double* s_red = reinterpret_cast<double*>(s_enc + a.pieces);
    double* s_tot = s_red + 2 * nwaves;                                       // second set: the general-q sum
    uint32_t* s_words = reinterpret_cast<uint32_t*>(s_tot + 2);               // bucket totals of a split bucket
    uint32_t* s_misc = s_words + (nwaves + 3) / 4 * 4;
    float* s_rinv = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(s_misc) + 32);      // GROUPED: [waves][16]
    uint32_t* stage = reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(s_misc) + 32 +
                                                  (GROUPED ? (size_t)nwaves * 64 : 0) + (size_t)w * a.stage_bytes);
    // The lookups address the tables by number: the kernel has no static LDS, so the dynamic array (and
    // with it the tables) starts at address 0.
    if (lds_address(s_all) != 0u) {
        if (tid == 0) raise_error(sc, QGX_EBIT_STATE);
        return;
    }

    // The tables are asked for first, the chunk's rows before the tables are waited for: a workgroup's two trips to memory
    // lie side by side.
    const uint32_t nthreads = blockDim.x;
    for (uint32_t i = (uint32_t)tid + 2u * nthreads; i < a.pieces; i += nthreads) s_enc[i] = tab->enc[i];
    const uint32_t piece0 = min((uint32_t)tid, a.pieces - 1u), piece1 = min((uint32_t)tid + nthreads, a.pieces - 1u);
    const nt_u32x4 ahead0 = reinterpret_cast<const nt_u32x4*>(tab->enc)[piece0];
    const nt_u32x4 ahead1 = reinterpret_cast<const nt_u32x4*>(tab->enc)[piece1];

    // Compact placement: buckets by ticket.
    // Slotted placement and plain quantisation have no order to keep: the bucket is the block's own.
    // Split buckets: (bucket, part) by ticket as well, whatever the placement (see exchange_parts).
    const bool ordered = MODE != EncMode::QuantOnly && a.slot_words == 0u;
    const bool ticketed = ordered || a.parts > 1u;
    // A worker's counter only ever grows, and every launch of a context that takes tickets takes the
    // same number from it, so a ticket tells both the unit inside this launch and the number of the
    // launch, which tags what the workgroups publish to each other (30 bits, never 0: untouched
    // words hold 0).  Nothing about it comes from the host: a captured graph can be replayed.
    if (ticketed) {
        if (tid == 0 && (!kWaits<MODE> || k < lay.K)) {
            const unsigned long long per_launch = a.units;
            const unsigned long long raw = atomicAdd(a.tickets + k * kTicketStride, 1ull);
            const unsigned long long launch = raw / per_launch;
            s_misc[2] = (uint32_t)(raw - launch * per_launch);
            s_misc[3] = (uint32_t)(launch % 0x3FFFFFFFull) + 1u;
        }
        __syncthreads();
    }

    if (kWaits<MODE> && k >= lay.K) return;             // a row's end (asked before the ticket it costs compact placement 1 %)
    const size_t kbase = (size_t)k * lay.d;
    const bool vec_ok = MODE == EncMode::Generate || (kbase & 3u) == 0;    // 16-byte aligned rows for this worker
    // the number of this quantisation call: given, or taken from the iteration counter (replayed graphs)
    const uint32_t call_id = a.call_mode ? 2u * (scalar_load(&sc->t) - 1u) + (a.call_mode - 1u) : a.call_id;
    const float* __restrict__ Vk = (MODE == EncMode::Fused || MODE == EncMode::QuantOnly) ? a.V + kbase : nullptr;
    // one coordinate of the worker's vector again, for the rolled paths: from memory, or (Generate) formed again
    auto value_at = [&](uint32_t i) -> float {
        if constexpr (MODE == EncMode::Generate) {
            const float4 row = game_dual_row(a.game, i & ~3u, k, call_id);
            const uint32_t q = i & 3u;
            return q == 0u ? row.x : q == 1u ? row.y : q == 2u ? row.z : row.w;
        } else {
            return Vk[i];
        }
    };
    const uint32_t unit = ticketed ? (uint32_t)__builtin_amdgcn_readfirstlane((int)s_misc[2]) : own_unit;
    const uint32_t epoch = ticketed ? (uint32_t)__builtin_amdgcn_readfirstlane((int)s_misc[3]) : 0u;
    // Short buckets: a workgroup takes `group` of them (buckets_per_group).
    const uint32_t per_bucket = a.group > 1u ? lay.waves_per_bucket : (uint32_t)nwaves;            // waves to a bucket
    const uint32_t mine = a.group > 1u ? (uint32_t)w / per_bucket : 0u, w0 = mine * per_bucket;    // the wave's bucket, and its first wave
    uint32_t b = a.parts > 1u ? unit / a.parts : unit * a.group + mine;  // the bucket; with shared chunks the first of the wave's chunk
    const uint32_t part = GROUPED || a.parts == 1u ? 0u : unit - b * a.parts;
    const bool there = GROUPED || b < lay.NB;           // (a worker's last workgroup: no bucket for some waves)
    ChunkGeom g;
    if constexpr (GROUPED) {
        if (unit * 4u >= lay.NC) return;               // cannot happen: one workgroup per four chunks and worker
        g.c = unit * 4u + (uint32_t)w;
        const bool have = g.c < lay.NC;
        g.clo = have ? scalar_load(lay.chunk_start + g.c) : 0u;
        g.clen = have ? scalar_load(lay.chunk_start + g.c + 1) - g.clo : 0u;
        g.cend = g.clo + g.clen;
        g.nrows = (int)((g.clen + 255u) >> 8);
        g.full = g.clen == (uint32_t)kChunk;
        g.bparts = 1u;
        b = have ? scalar_load(lay.chunk_bucket + g.c) : 0u;
    } else {
        if (b - mine >= lay.NB) return;                // cannot happen: one workgroup per unit and worker
        if (!there) b = lay.NB - 1u;
        g = chunk_geom(lay, b, part * 4u + (uint32_t)w - w0, there);
    }
    if (part >= g.bparts) {
        // a short bucket has nothing for this part; no partner waits for it, but in compact placement
        // the units after it look back over its (empty) aggregate
        if (ordered && tid == 0)
            __hip_atomic_store(a.scan_state + (size_t)k * lay.NB * a.parts + unit,
                               (unsigned long long)((epoch << 2) | 1u) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    const bool split = a.parts > 1u && g.bparts > 1u;
    unsigned long long* xch = a.xch + ((size_t)k * lay.NB + b) * a.parts * 4u;
    // The sub-chunk ends go straight to the table in global memory: staging them in LDS would cost the fifth
    // workgroup of a compute unit.
    uint16_t* __restrict__ sub_g =
        MODE != EncMode::QuantOnly ? a.sub_end + ((size_t)k * lay.NC + g.c) * kSubs : nullptr;
    const SubEnds ends(reinterpret_cast<uint16_t*>(uniform_address(sub_g)), lane);
    float4 v[kRows];
    if constexpr (MODE == EncMode::Fused || MODE == EncMode::QuantOnly) load_rows(v, chunk_rows(Vk + g.clo, g.clen), lane);
    // (by all threads: a branch would leave it open what is still under way)
    reinterpret_cast<nt_u32x4*>(s_enc)[piece0] = ahead0;
    reinterpret_cast<nt_u32x4*>(s_enc)[piece1] = ahead1;
    if (MODE != EncMode::QuantOnly) {
        for (uint32_t q = (uint32_t)lane; q < a.stage_bytes / 16; q += kWave)
            reinterpret_cast<uint4*>(stage)[q] = make_uint4(0, 0, 0, 0);
    }
    // (the table builder and the host take the cell size from the table's length by the same rule)
    const uint32_t n_sym = tab->n_sym;
    const uint32_t cell_exact = (tab->cell_exact != 0u && (uint32_t)cell_mant(n_sym) == a.cell_mant) ? 1u : 0u;
    __syncthreads();
    if constexpr (MODE == EncMode::Fused || MODE == EncMode::QuantOnly) load_rest(v, Vk + g.clo, g.clen, lane);
    if constexpr (MODE == EncMode::Generate) {
        // the dual vector is formed here instead of read: operator and noise for four coordinates per lane and row
        // (every bucket and vector length is a multiple of four in this mode).  The operands are buffers, zeros past the chunk's
        // end, so that no branch divides the rows and a row's operands are asked for while the row before it is worked out
        // (16 x 2^26 coordinates 1.96 ms with a branch and a wait in every row, 1.66 without).
        const GameRows rows = game_rows(a.game, g.clo, g.clen);
        GameOperands next = load_game_operands(rows, 0, lane);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const uint32_t i0 = g.clo + (uint32_t)r * 256u + (uint32_t)lane * 4u;
            const GameOperands now = next;
            if (r + 1 < kRows) next = load_game_operands(rows, r + 1, lane);
            v[r] = game_noisy_row(a.game, game_operator_row(a.game, now), i0, k, call_id);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!g.full) {                                 // no noise past the chunk's end (selected in every row: two of its 210 instructions)
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const uint32_t i0 = g.clo + (uint32_t)r * 256u + (uint32_t)lane * 4u;
                if (i0 >= g.cend) v[r] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        if (a.game.V_out) {
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const uint32_t i0 = g.clo + (uint32_t)r * 256u + (uint32_t)lane * 4u;
                if (i0 < g.cend) *reinterpret_cast<float4*>(a.game.V_out + kbase + i0) = v[r];
            }
        }
    }
    {

        // ---- norm of the bucket from the rows in registers ---------------------------------------
        float n = 0.0f;
        bool u_le_1 = true;
        bool plain = true;                             // GROUPED: every bucket of the chunk live, no u above 1
        if constexpr (GROUPED) {
            if (MODE != EncMode::EncodeOnly && g.clen != 0u)
                plain = shared_chunk_norms<MODE>(v, Vk, g, lay, a, sc, k, b, s_rinv + w * 16, lane);
            wave_lds_fence();                              // lane 0 left the buckets' 1 / norm for all lanes
        } else if (MODE != EncMode::EncodeOnly) {
            // A non-finite coordinate shows in the reduced value itself (a sum of squares with a NaN
            // or an infinity in it, a maximum taken on magnitude bits).
            double red;
            if (a.norm_kind == QGX_NORM_L2) {
                // four binary32 runs of 16 fused multiply-adds per lane (error of a run at most
                // 15 roundings, 1e-6 relative, half of that on the norm), everything after in
                // binary64; sums outside the range where binary32 squares are safe are redone below
                float p0 = 0.0f, p1 = 0.0f, p2 = 0.0f, p3 = 0.0f;
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    p0 = fmaf(v[r].x, v[r].x, p0);
                    p1 = fmaf(v[r].y, v[r].y, p1);
                    p2 = fmaf(v[r].z, v[r].z, p2);
                    p3 = fmaf(v[r].w, v[r].w, p3);
                }
                red = wave_sum(((double)p0 + (double)p1) + ((double)p2 + (double)p3));
            } else {
                float mx = 0.0f;
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    mx = largest_of(v[r], mx);
                }
                red = (double)__uint_as_float(wave_max_u32(__float_as_uint(mx)));      // inf or NaN bits survive the conversion
            }
            if (lane == 0) s_red[w] = red;
            __syncthreads();
            auto bucket_total = [&](const double* part_of) {      // the values of the bucket's waves, in order
                double t = 0.0;
                for (uint32_t i = 0; i < per_bucket; ++i) {
                    if (a.norm_kind == QGX_NORM_L2) t += part_of[i];
                    else t = (part_of[i] > t || part_of[i] != part_of[i]) ? part_of[i] : t;
                }
                return t;
            };
            double tot = bucket_total(s_red + w0);
            if (split) {
                if (w == 0) {
                    const double t = exchange_parts(xch, g.bparts, part, 0u, tot, a.norm_kind != QGX_NORM_L2, epoch, sc);
                    if (lane == 0) s_tot[0] = t;
                }
                __syncthreads();
                tot = s_tot[0];
            }
            // squares that overflow or go subnormal in binary32 (or a non-finite input): the sum again in binary64, from
            // memory (the rolled loop keeps the register copy intact), by the waves of the buckets that need it; the others of
            // the workgroup wait.  (A wave without a bucket has a sum of zero and needs nothing; when it had all of its
            // workgroup, a worker's last, sum again, coding 5 x 4.2 M coordinates in 513 buckets of 8192 took 37.8 us in slots and 66.2
            // in order, now 29.1 and 44.7; one vector of 2^20 in 350 buckets of 3000, in order, 17.2, now 14.0.)
            auto beyond = [&](double t) { return a.norm_kind == QGX_NORM_L2 && !(t >= 0x1p-60 && t <= 0x1p100); };
            const bool again = there && beyond(tot);
            bool any_again = again;
            if (a.group > 1u) {
                const uint32_t waves = waves_with_a_bucket(unit, a.group, per_bucket, lay.NB);
                for (uint32_t f = 0; f < waves; f += per_bucket) any_again = any_again || beyond(bucket_total(s_red + f));
            }
            if (any_again) {
                double acc = 0.0;
                if (again) {
#pragma unroll 1
                    for (uint32_t i = g.clo + (uint32_t)lane; i < g.cend; i += kWave) { const double x = (double)value_at(i); acc = fma(x, x, acc); }
                }
                acc = wave_sum(acc);
                if (lane == 0) s_red[nwaves + w] = acc;
                __syncthreads();
                double sum = 0.0;
                for (uint32_t i = 0; i < per_bucket; ++i) sum += s_red[nwaves + w0 + i];
                if (split) {
                    if (w == 0) {
                        const double t = exchange_parts(xch, g.bparts, part, 1u, sum, false, epoch, sc);
                        if (lane == 0) s_tot[1] = t;
                    }
                    __syncthreads();
                    sum = s_tot[1];
                }
                if (again) tot = sum;
            }
            n = (a.norm_kind == QGX_NORM_L2) ? (float)sqrt(tot) : (float)tot;
            if (a.norm_kind != QGX_NORM_L2 && a.norm_kind != QGX_NORM_LINF) {
                // any other q of Definition 1: (sum |v_i|^q)^(1/q), relative to the largest magnitude
                // found above so that no power leaves the range of binary64
                const bool sound = tot > 0.0 && tot <= 3.402823466e+38;       // (the parts of a split bucket agree on it)
                const double inv_m = 1.0 / tot;
                const uint32_t q = (uint32_t)a.norm_kind;
                double acc = 0.0;
                // (a rolled loop over memory: indexing the register copy by a run-time row would
                // push it out of registers for the common norms as well)
                if (sound) {
#pragma unroll 1
                    for (uint32_t i = g.clo + (uint32_t)lane; i < g.cend; i += kWave)
                        acc += pow_int(fabs((double)value_at(i)) * inv_m, q);
                }
                acc = wave_sum(acc);
                if (lane == 0) s_red[nwaves + w] = acc;
                __syncthreads();
                double sum = 0.0;
                for (uint32_t i = 0; i < per_bucket; ++i) sum += s_red[nwaves + w0 + i];
                if (split && sound) {
                    if (w == 0) {
                        const double t = exchange_parts(xch, g.bparts, part, 1u, sum, false, epoch, sc);
                        if (lane == 0) s_tot[1] = t;
                    }
                    __syncthreads();
                    sum = s_tot[1];
                }
                if (sound) n = (float)(tot * root_int(sum, q));
            }
            if (a.norms_in) {
                const float forced = a.norms_in[(size_t)k * lay.NB + b];
                u_le_1 = forced >= n;                                        // else |v| / norm may exceed 1
                n = (n == n && fabsf(n) <= 3.402823466e+38f) ? forced : n;   // a poisoned bucket stays rejected
            }
            const bool bucket_bad = !(fabsf(n) <= 3.402823466e+38f);
            if (bucket_bad) n = 0.0f;
            if (there && (uint32_t)w == w0 && lane == 0) {
                if (bucket_bad) raise_error(sc, QGX_EBIT_NONFINITE);
                if (a.norms_out && part == 0u) a.norms_out[(size_t)k * lay.NB + b] = n;
            }
        }
        const float rinv = GROUPED ? 0.0f : 1.0f / n;  // one IEEE division per bucket
        const bool live = GROUPED ? plain : n > 0.0f;
        // The straight path's look-ups lie inside the tables for u <= 1 up to a rounding only: a norm of 2^-128 or less, whose
        // reciprocal overflows and makes u infinite or NaN, takes the general path, which clamps u (as a chunk's last
        // row does, if short).
        const bool fast = live && (GROUPED || n > kNoReciprocal) && (vec_ok || MODE != EncMode::QuantOnly) && u_le_1 && (cell_exact != 0u) && MODE != EncMode::EncodeOnly;
        const uint32_t rshift = GROUPED ? lay.bucket_shift - 8u : 0u;         // rows per bucket, as a shift

        // ---- per row: quantise, code, pack -------------------------------------------------------
        uint32_t first_cell = kCellKey0<CM> << kCellShift<CM>;
        asm("" : "+v"(first_cell));
        const uint32_t stage0 = 8u * (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_address(stage)) - 1u;     // (see place_row)
        uint32_t row_base = 0;                         // bits of this chunk written so far (wave-uniform)
        int rows_done = 0;
        const uint32_t block0 = (g.clo >> 2) + (uint32_t)lane;                // Philox block of row 0 (chunks start at multiples of 4)
        const PhiloxKeys keys = philox_keys(a.seed_lo, a.seed_hi);
        auto quantize_row = [&](int r, uint32_t (&e)[4]) __attribute__((always_inline)) {
            const float xs[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
            const float rinv_r = GROUPED ? s_rinv[w * 16 + (int)((uint32_t)r >> rshift)] : rinv;
            uint32_t rnd[4], pk = 0;
            auto decide = [&](int q, float u, uint32_t j, uint4 t) __attribute__((always_inline)) {
                const bool up = rounds_up(u, t, rnd[q]);
                e[q] = up ? t.w : t.z;
                if (MODE == EncMode::QuantOnly) pk |= (j + (up ? 1u : 0u) + ((__float_as_uint(xs[q]) >> 31) << 7)) << (8 * q);
            };
            if constexpr (STAGED) {
                float u[4];
                uint2 c[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) { u[q] = fabsf(xs[q]) * rinv_r; c[q] = cell_of<CM>(u[q], first_cell); }      // |v| / ||v||
                __builtin_amdgcn_sched_barrier(0);
                philox4x32_10(block0 + 64u * (uint32_t)r, 0u, k, call_id, keys, rnd);
                __builtin_amdgcn_sched_barrier(0);
                uint32_t j[4];
                uint4 t[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) { j[q] = level_in_cell(u[q], c[q]); t[q] = level_row<CM>(j[q], xs[q]); }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < 4; ++q) decide(q, u[q], j[q], t[q]);
            } else {
                philox4x32_10(block0 + 64u * (uint32_t)r, 0u, k, call_id, keys, rnd);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float u = fabsf(xs[q]) * rinv_r;                                                           // |v| / ||v||
                    const uint32_t j = level_in_cell(u, cell_of<CM>(u, first_cell));
                    decide(q, u, j, level_row<CM>(j, xs[q]));
                }
            }
            if (MODE == EncMode::QuantOnly) *reinterpret_cast<uint32_t*>(a.sym_out + kbase + 4u * (size_t)(block0 + 64u * (uint32_t)r)) = pk;
        };
        if (fast && g.full) {
#pragma unroll
            for (int r = 0; r < kRows; r += 2) {
                uint32_t ea[4], eb[4];
                quantize_row(r, ea);
                quantize_row(r + 1, eb);
                if (MODE != EncMode::QuantOnly) row_base += pack_two_rows(stage0, ends, r, row_base, ea, eb);
                __builtin_amdgcn_sched_barrier(0);     // (two rows at a time: more of them in flight spill)
            }
            rows_done = kRows;
        } else if (fast) {
            const int whole = (int)(g.clen >> 8);
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                if (r < whole) {                       // (wave-uniform)
                    uint32_t e[4];
                    quantize_row(r, e);
                    if (MODE != EncMode::QuantOnly) row_base += pack_row<false>(stage0, ends, r, row_base, e);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            rows_done = whole;
        }
        {
#pragma unroll 1
            for (int r = rows_done; r < g.nrows; ++r) {
                const uint32_t i0 = g.clo + (uint32_t)r * 256u + (uint32_t)lane * 4u;
                uint32_t e[4], idx[4], neg[4];
                if (MODE == EncMode::EncodeOnly) {
                    const uint8_t* __restrict__ Sk = a.sym_in + kbase;
                    bool unknown = false;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t by = (i0 + (uint32_t)q < g.cend) ? (uint32_t)Sk[i0 + q] : 0u;
                        idx[q] = by & 0x7Fu;
                        neg[q] = by >> 7;
                        if (idx[q] >= n_sym) { idx[q] = 0; unknown = true; }
                    }
                    if (__any(unknown) && lane == 0) raise_error(sc, QGX_EBIT_STREAM);
                } else {
                    uint32_t rnd[4];
                    philox4x32_10(i0 >> 2, 0u, k, call_id, philox_keys(a.seed_lo, a.seed_hi), rnd);
                    // the register copy is indexed by compile-time row numbers only: this path reads the row again
                    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
                    if constexpr (MODE == EncMode::Generate) {
                        if (i0 < g.cend) x = game_dual_row(a.game, i0, k, call_id);
                    } else {
                        if (i0 < g.cend) x.x = Vk[i0];
                        if (i0 + 1 < g.cend) x.y = Vk[i0 + 1];
                        if (i0 + 2 < g.cend) x.z = Vk[i0 + 2];
                        if (i0 + 3 < g.cend) x.w = Vk[i0 + 3];
                    }
                    const float xs[4] = {x.x, x.y, x.z, x.w};
                    const float rinv_r = GROUPED ? s_rinv[w * 16 + (int)((uint32_t)r >> rshift)] : rinv;
                    const bool live_r = GROUPED ? rinv_r != 0.0f : live;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        idx[q] = 0;
                        neg[q] = __float_as_uint(xs[q]) >> 31;
                        if (live_r) {
                            const float u = fminf(fabsf(xs[q]) * rinv_r, 1.0f);
                            const uint32_t j = level_general<CM>(u, n_sym);
                            idx[q] = j + (rounds_up(u, level_row<CM>(j, xs[q]), rnd[q]) ? 1u : 0u);
                        }
                    }
                }
                if (MODE == EncMode::QuantOnly) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (i0 + (uint32_t)q < g.cend) a.sym_out[kbase + i0 + q] = (uint8_t)(idx[q] | (neg[q] << 7));
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        // E(idx, sign) from the table row of idx (its third word), nothing for a padded slot
                        uint32_t code = lds_load_u32(kLevAt<CM> + 8u + (2u * idx[q] + neg[q]) * 16u);
                        asm("" : "+v"(code));                  // (read by all lanes: four branches a row cost more)
                        e[q] = (i0 + (uint32_t)q < g.cend) ? code : 0u;
                    }
                    row_base += pack_row<true>(stage0, ends, r, row_base, e);
                }
            }
        }

        // ---- sizes, ordered offsets, flush ---------------------------------------------------------
        const uint32_t total_bits = row_base;
        uint32_t words = (total_bits + 31u) >> 5;
        words = (words + (kAlignWords - 1)) & ~(uint32_t)(kAlignWords - 1);
        if (MODE != EncMode::QuantOnly) {
            if (g.clen != 0) {
                for (int j = lane; j < kSubs; j += kWave)
                    if (j >= 8 * g.nrows) sub_g[j] = (uint16_t)total_bits;
            }
            if (lane == 0 && ordered) s_words[w] = words;
        }
        if (MODE != EncMode::QuantOnly) {
            uint32_t off;
            if (ordered) {
                __syncthreads();
                uint32_t bucket_words = 0, wave_excl = 0;
                for (int i = 0; i < nwaves; ++i) {
                    if (i == w) wave_excl = bucket_words;
                    bucket_words += s_words[i];
                }
                if (w == 0) {
                    const uint32_t excl = lookback_exclusive(a.scan_state + (size_t)k * lay.NB * a.parts, unit, bucket_words, epoch, sc);
                    if (lane == 0) s_misc[1] = excl;
                }
                __syncthreads();
                off = s_misc[1] + wave_excl;
            } else {
                off = g.c * a.slot_words;
            }
            if (g.clen != 0) {
                if (lane == 0) {
                    a.chunk_off[(size_t)k * (lay.NC + 1) + g.c] = off;
                    if (g.c + 1 == lay.NC) a.chunk_off[(size_t)k * (lay.NC + 1) + lay.NC] = off + (ordered ? words : a.slot_words);
                }
                if ((uint64_t)off + words > a.cap_words) {
                    if (lane == 0) raise_error(sc, QGX_EBIT_CAPACITY);
                } else {
                    uint4* __restrict__ dst = reinterpret_cast<uint4*>(a.payload + (size_t)k * a.cap_words + off);
                    uint4* src = reinterpret_cast<uint4*>(stage);
                    wave_lds_fence();                          // a lane stores words that all lanes' codes went into
                    for (uint32_t q = (uint32_t)lane; q < (words >> 2); q += kWave) dst[q] = src[q];
                }
            }
        }
    }
}

// The coding kernel where V is read and chunks are few: four waves to a chunk.  Such a launch takes as long as one wave lives, of
// which a third is the straight line of its rows (a wave alone on its SIMD issues every 6.4 clocks, 5 us for sixteen rows), while most
// of the GPU's places for waves are empty.
// A wave has 16 of the 64 columns of four coordinates, lane 16 i + j rows 4 i .. 4 i + 3 of its column j (a short chunk: as
// many rows as it takes, 4 i -> slots * i): a column's sums of squares thus go from row to row inside a wave, by lane
// swaps, and are the sums of k_encode bit for bit.  The codes' lengths are summed across 16 lanes, and a row's four pieces
// find their places through the chunk's 64 counts in LDS.
// What bounds it is still latency: launch, tables and rows 2.3 us, the norm with its two barriers 1.2, a row at a time 0.4, flush 0.5.
// Kernel alone, a wave per chunk -> four, us: 256 chunks in slots, buckets of 1024 13.1 -> 7.0, of 6000 9.8 -> 7.4, of 8192 (L-infinity
// norm) 9.6 -> 7.7; one bucket of 1024 6.3 -> 5.0; in order, 16 chunks in buckets of 1024 14.2 -> 10.7, of 8192 11.0 -> 9.0; where not: use_columns.
// (A quarter of the rows to a wave, the sums handed on through LDS with a barrier each: 6.1, 9.5, 7.2 and 6.8.)
// Units, tickets and look-back are those of k_encode; a workgroup is a whole bucket (a.parts is 1), or with shared chunks a chunk, or
// four where they keep an order.
constexpr int kSlots = kRows / 4;       // rows of a lane
struct ColumnLds {                      // LDS after the tables, in bytes, for a workgroup of `chunks` chunks
    uint32_t sums, misc, rinv, fine, counts, totals, stage, buckets;
    __host__ __device__ ColumnLds(uint32_t pieces, uint32_t chunks, bool grouped)
    {
        buckets = grouped ? 16u : 1u;                               // of a chunk
        sums = pieces * 16u;                                        // [chunks][buckets][64] double: a bucket's columns
        misc = sums + chunks * buckets * (uint32_t)kWave * 8u;      // 4 words
        rinv = misc + 16u;                                          // [chunks][16] float: 1 / norm of the buckets that share a chunk
        fine = rinv + (grouped ? chunks * 64u : 0u);                // [chunks][16] words: the straight route applies to them
        counts = fine + (grouped ? chunks * 64u : 0u);              // [chunks][64]: bits of row r's columns 16 q and on, at 4 r + q
        totals = counts + chunks * 256u;                            // [4] words of the unit's chunks
        stage = totals + 16u;
    }
};

// From the lanes of a row of 16 to the lanes of the next row: FROM 0 -> 1 and 2 -> 3 (even), 1 -> 2 (odd).
template <bool ODD>
__device__ __forceinline__ float next_sixteen(float x)
{
    const LanePair p = lane_pair<16>(__float_as_uint(x));
    if constexpr (!ODD) return __uint_as_float(p.a);
    return __uint_as_float(lane_pair<32>(p.b).a);
}

template <bool GROUPED, int CM>
__global__ __launch_bounds__(1024) void k_encode_columns(Layout lay, const Tables* __restrict__ tab, Scalars* sc, EncodeArgs a)
{
    extern __shared__ __align__(16) unsigned char s_all[];
    const int tid = (int)threadIdx.x, lane = lane_id();
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane(wave_id()), cw = w >> 2, part = w & 3u;
    const uint32_t nthreads = blockDim.x, nchunks = nthreads >> 8;
    uint32_t k = blockIdx.x % lay.K;
    const uint32_t own_unit = blockIdx.x / lay.K;
    if (a.spread) k = worker_spread(k, own_unit, lay.K);
    const ColumnLds at(a.pieces, nchunks, GROUPED);
    uint4* s_enc = reinterpret_cast<uint4*>(s_all);
    double* s_sums = reinterpret_cast<double*>(s_all + at.sums);
    uint32_t* s_misc = reinterpret_cast<uint32_t*>(s_all + at.misc);
    float* s_rinv = reinterpret_cast<float*>(s_all + at.rinv) + cw * 16u;
    uint32_t* s_fine = reinterpret_cast<uint32_t*>(s_all + at.fine) + cw * 16u;
    uint32_t* s_counts = reinterpret_cast<uint32_t*>(s_all + at.counts) + cw * 64u;
    uint32_t* s_totals = reinterpret_cast<uint32_t*>(s_all + at.totals);
    uint32_t* stage = reinterpret_cast<uint32_t*>(s_all + at.stage + (size_t)cw * a.stage_bytes);
    if (lds_address(s_all) != 0u) {                    // the look-ups address the tables by number (see k_encode)
        if (tid == 0) raise_error(sc, QGX_EBIT_STATE);
        return;
    }
    for (uint32_t i = (uint32_t)tid + 2u * nthreads; i < a.pieces; i += nthreads) s_enc[i] = tab->enc[i];
    const uint32_t piece0 = min((uint32_t)tid, a.pieces - 1u), piece1 = min((uint32_t)tid + nthreads, a.pieces - 1u);
    const nt_u32x4 ahead0 = reinterpret_cast<const nt_u32x4*>(tab->enc)[piece0];
    const nt_u32x4 ahead1 = reinterpret_cast<const nt_u32x4*>(tab->enc)[piece1];

    const bool ordered = a.slot_words == 0u;
    if (ordered) {                                     // (the unit and the launch's number from the ticket: see k_encode)
        if (tid == 0) {
            const unsigned long long per_launch = a.units;
            const unsigned long long raw = atomicAdd(a.tickets + k * kTicketStride, 1ull);
            const unsigned long long launch = raw / per_launch;
            s_misc[2] = (uint32_t)(raw - launch * per_launch);
            s_misc[3] = (uint32_t)(launch % 0x3FFFFFFFull) + 1u;
        }
        __syncthreads();
    }
    const uint32_t unit = ordered ? (uint32_t)__builtin_amdgcn_readfirstlane((int)s_misc[2]) : own_unit;
    const uint32_t epoch = ordered ? (uint32_t)__builtin_amdgcn_readfirstlane((int)s_misc[3]) : 0u;
    if (unit >= a.units) return;                       // cannot happen
    const uint32_t call_id = a.call_mode ? 2u * (scalar_load(&sc->t) - 1u) + (a.call_mode - 1u) : a.call_id;
    const float* __restrict__ Vk = a.V + (size_t)k * lay.d;

    // the wave's chunk and bucket (with shared chunks: the chunk's first)
    ChunkGeom g;
    uint32_t b;
    if constexpr (GROUPED) {
        g.c = unit * nchunks + cw;
        const bool there = g.c < lay.NC;
        g.clo = there ? scalar_load(lay.chunk_start + g.c) : 0u;
        g.clen = there ? scalar_load(lay.chunk_start + g.c + 1) - g.clo : 0u;
        g.cend = g.clo + g.clen;
        g.nrows = (int)((g.clen + 255u) >> 8);
        g.full = g.clen == (uint32_t)kChunk;
        b = there ? scalar_load(lay.chunk_bucket + g.c) : 0u;
    } else {
        b = unit;
        g = chunk_geom(lay, b, cw, true);
    }
    // rows to a lane: 4, 2 or 1
    const int slots = g.nrows > 8 ? 4 : g.nrows > 4 ? 2 : 1;
    const uint32_t column = 16u * part + ((uint32_t)lane & 15u);
    const uint32_t row0 = ((uint32_t)lane >> 4) * (uint32_t)slots;
    const uint32_t at0 = g.clo + row0 * 256u + column * 4u;            // the lane's first coordinate; slot s: 256 s further on

    float4 v[kSlots];
    {
        const __amdgpu_buffer_rsrc_t rows = chunk_rows(Vk + g.clo, g.clen);
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            v[s] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (s < slots) v[s] = load_row(rows, s, (int)(row0 * 64u + column));
        }
    }
    reinterpret_cast<nt_u32x4*>(s_enc)[piece0] = ahead0;
    reinterpret_cast<nt_u32x4*>(s_enc)[piece1] = ahead1;
    for (uint32_t i = part * kWave + (uint32_t)lane; i < a.stage_bytes / 16; i += 4u * kWave)
        reinterpret_cast<uint4*>(stage)[i] = make_uint4(0, 0, 0, 0);
    if (part == 0u) s_counts[lane] = 0u;
    const uint32_t n_sym = tab->n_sym;
    const bool cell_exact = tab->cell_exact != 0u && (uint32_t)cell_mant(n_sym) == a.cell_mant;
    __syncthreads();
    if ((g.clen & 3u) != 0u) {                         // the last one to three coordinates of an odd vector (load_rest)
        const uint32_t rest = g.clo + (g.clen & ~3u);
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        x.x = Vk[rest];
        if ((g.clen & 3u) > 1u) x.y = Vk[rest + 1u];
        if ((g.clen & 3u) > 2u) x.z = Vk[rest + 2u];
#pragma unroll
        for (int s = 0; s < kSlots; ++s)
            if (s < slots && at0 + 256u * (uint32_t)s == rest) v[s] = x;
    }

    // ---- norms -----------------------------------------------------------------------------------
    const bool l2 = a.norm_kind == QGX_NORM_L2;
    const uint32_t rshift = GROUPED ? lay.bucket_shift - 8u : 4u;      // rows to a bucket of the chunk, as a shift
    // A column's four runs of squares (largest magnitude) of a bucket's rows, in row order, to bucket t's columns in LDS.
    auto leave = [&](uint32_t t, const float4& p, float mx) {
        s_sums[(cw * at.buckets + t) * (uint32_t)kWave + column] =
            l2 ? ((double)p.x + (double)p.y) + ((double)p.z + (double)p.w) : (double)mx;       // inf or NaN survive the conversion
    };
    auto add_slot = [&](float4& p, float& mx, int s) {
        if (l2) {
            p.x = fmaf(v[s].x, v[s].x, p.x);
            p.y = fmaf(v[s].y, v[s].y, p.y);
            p.z = fmaf(v[s].z, v[s].z, p.z);
            p.w = fmaf(v[s].w, v[s].w, p.w);
        } else {
            mx = largest_of(v[s], mx);
        }
    };
    if ((1 << rshift) <= slots) {                      // (shared chunks) a lane's rows are whole buckets
        float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
        float mx = 0.0f;
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            if (s >= slots) break;
            add_slot(p, mx, s);
            if ((((uint32_t)s + 1u) & ((1u << rshift) - 1u)) != 0u) continue;
            leave((row0 + (uint32_t)s) >> rshift, p, mx);
            p = make_float4(0.f, 0.f, 0.f, 0.f);
            mx = 0.0f;
        }
    } else {
        // from one row of 16 lanes to the next, but where a bucket begins
        const uint32_t in_bucket = row0 & ((1u << rshift) - 1u);
        float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
        float mx = 0.0f;
#pragma unroll
        for (int turn = 0; turn < 4; ++turn) {
            if (turn > 0) {
                auto pass = [&](float x) { return turn == 2 ? next_sixteen<true>(x) : next_sixteen<false>(x); };
                p = make_float4(pass(p.x), pass(p.y), pass(p.z), pass(p.w));
                mx = pass(mx);
                if (in_bucket == 0u) { p = make_float4(0.f, 0.f, 0.f, 0.f); mx = 0.0f; }
            }
#pragma unroll
            for (int s = 0; s < kSlots; ++s)
                if (s < slots) add_slot(p, mx, s);
            // (the lanes whose turn it is, where the bucket or the chunk ends)
            if ((lane >> 4) == turn && (turn == 3 || in_bucket + (uint32_t)slots == (1u << rshift))) leave(row0 >> rshift, p, mx);
        }
    }
    __syncthreads();
    auto column_total = [&](uint32_t chunk, uint32_t t) -> double {    // (a whole wave)
        const double x = s_sums[(chunk * at.buckets + t) * (uint32_t)kWave + (uint32_t)lane];
        return l2 ? wave_sum(x) : (double)__uint_as_float(wave_max_u32(__float_as_uint((float)x)));
    };
    auto beyond = [&](double t) { return l2 && !(t >= 0x1p-60 && t <= 0x1p100); };
    auto finite = [](float x) { return fabsf(x) <= 3.402823466e+38f; };
    float n = 0.0f;
    bool fast = cell_exact;                            // the straight route applies: see k_encode
    if constexpr (GROUPED) {
        // a wave to a bucket of its chunk
        for (uint32_t t = part; t < 16u >> rshift; t += 4u) {
            const uint32_t lo = g.clo + (t << lay.bucket_shift);
            if (lo >= g.cend) break;
            const uint32_t hi = min(lo + (1u << lay.bucket_shift), g.cend);
            double tot = column_total(cw, t);
            if (beyond(tot)) {
                double acc = 0.0;
#pragma unroll 1
                for (uint32_t i = lo + (uint32_t)lane; i < hi; i += kWave) acc = fma((double)Vk[i], (double)Vk[i], acc);
                tot = wave_sum(acc);
            }
            float nt = l2 ? (float)sqrt(tot) : (float)tot;
            if (!l2 && a.norm_kind != QGX_NORM_LINF && tot > 0.0 && tot <= 3.402823466e+38) {
                const double inv_m = 1.0 / tot;
                double acc = 0.0;
#pragma unroll 1
                for (uint32_t i = lo + (uint32_t)lane; i < hi; i += kWave)
                    acc += pow_int(fabs((double)Vk[i]) * inv_m, (uint32_t)a.norm_kind);
                nt = (float)(tot * root_int(wave_sum(acc), (uint32_t)a.norm_kind));
            }
            bool u_le_1 = true;
            if (a.norms_in) {
                const float forced = a.norms_in[(size_t)k * lay.NB + b + t];
                u_le_1 = forced >= nt;
                nt = finite(nt) ? forced : nt;
            }
            const bool bad = !finite(nt);
            if (bad) nt = 0.0f;
            if (lane == 0) {
                if (bad) raise_error(sc, QGX_EBIT_NONFINITE);
                if (a.norms_out) a.norms_out[(size_t)k * lay.NB + b + t] = nt;
                s_rinv[t] = nt > 0.0f ? 1.0f / nt : 0.0f;
                s_fine[t] = nt > kNoReciprocal && u_le_1 ? 1u : 0u;
            }
        }
        __syncthreads();
    } else {
        // The bucket's sum of term(v) over its coordinates, from memory, by all waves of the workgroup, in the order of k_encode (an order of
        // its own would turn a norm between two binary32 numbers the other way): a lane of a chunk adds the coordinates 64 apart.  Each
        // wave works out a quarter of them, and the quarters are added one after the other.
        auto sum_again = [&](auto term) {
            constexpr int kTerms = kChunk / 4 / kWave;
            double x[kTerms], acc = 0.0;
#pragma unroll
            for (int j = 0; j < kTerms; ++j) {
                const uint32_t i = g.clo + part * (kChunk / 4u) + (uint32_t)(j * kWave + lane);
                x[j] = i < g.cend ? term(Vk[i]) : 0.0;
            }
            double* sums = s_sums + cw * (uint32_t)kWave + (uint32_t)lane;
            __syncthreads();                           // (the columns' sums have been read)
            // (a short chunk of a workgroup's own: only the quarters that it reaches into)
            const uint32_t turns = nchunks > 1u ? 4u : (g.clen + kChunk / 4u - 1u) / (kChunk / 4u);
            for (uint32_t turn = 0; turn < turns; ++turn) {
                if (part == turn) {
                    if (turn > 0u) acc = *sums;
#pragma unroll
                    for (int j = 0; j < kTerms; ++j) acc += x[j];
                    *sums = acc;
                }
                __syncthreads();
            }
            double t = 0.0;
            for (uint32_t c = 0; c < nchunks; ++c) t += wave_sum(s_sums[c * (uint32_t)kWave + (uint32_t)lane]);
            return t;
        };
        double tot = 0.0;
        for (uint32_t c = 0; c < nchunks; ++c) {       // the bucket's chunks, in order
            const double x = column_total(c, 0u);
            if (l2) tot += x;
            else tot = (x > tot || x != x) ? x : tot;
        }
        // as in k_encode: the sum again in binary64 (where a square is exact)
        if (beyond(tot)) tot = sum_again([](float v) { return (double)v * (double)v; });
        n = l2 ? (float)sqrt(tot) : (float)tot;
        if (!l2 && a.norm_kind != QGX_NORM_LINF && tot > 0.0 && tot <= 3.402823466e+38) {
            const double inv_m = 1.0 / tot;
            const double sum = sum_again([&](float v) { return pow_int(fabs((double)v) * inv_m, (uint32_t)a.norm_kind); });
            n = (float)(tot * root_int(sum, (uint32_t)a.norm_kind));
        }
        bool u_le_1 = true;
        if (a.norms_in) {
            const float forced = a.norms_in[(size_t)k * lay.NB + b];
            u_le_1 = forced >= n;
            n = finite(n) ? forced : n;
        }
        const bool bad = !finite(n);
        if (bad) n = 0.0f;
        if (tid == 0) {
            if (bad) raise_error(sc, QGX_EBIT_NONFINITE);
            if (a.norms_out) a.norms_out[(size_t)k * lay.NB + b] = n;
        }
        fast = fast && n > kNoReciprocal && u_le_1;
    }
    const float rinv = GROUPED ? 0.0f : 1.0f / n;
    const bool live = n > 0.0f;

    // ---- the rows: quantise, code ------------------------------------------------------------------
    uint32_t first_cell = kCellKey0<CM> << kCellShift<CM>;
    asm("" : "+v"(first_cell));
    const PhiloxKeys keys = philox_keys(a.seed_lo, a.seed_hi);
    float rinv_s[kSlots];
#pragma unroll
    for (int s = 0; s < kSlots; ++s) {
        rinv_s[s] = rinv;
        if constexpr (GROUPED) {
            if (s < slots) {
                const uint32_t t = (row0 + (uint32_t)s) >> rshift;
                const bool inside = g.clo + (t << lay.bucket_shift) < g.cend;
                rinv_s[s] = inside ? s_rinv[t] : 0.0f;
                fast = fast && !__any(inside && s_fine[t] == 0u);
            }
        }
    }
    RowCode code[kSlots];
    uint32_t length[kSlots], end[kSlots];
    auto put_entries = [&](int s, uint32_t (&e)[4]) __attribute__((always_inline)) {
        if (!g.full) {                                 // nothing past the chunk's end (wave-uniform)
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i] = at0 + 256u * (uint32_t)s + (uint32_t)i < g.cend ? e[i] : 0u;
        }
        code[s] = join_row(e);
    };
    auto fast_row = [&](int s) __attribute__((always_inline)) {
        const float xs[4] = {v[s].x, v[s].y, v[s].z, v[s].w};
        float u[4];
        uint2 c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { u[i] = fabsf(xs[i]) * rinv_s[s]; c[i] = cell_of<CM>(u[i], first_cell); }
        uint32_t rnd[4], e[4];
        philox4x32_10((at0 >> 2) + 64u * (uint32_t)s, 0u, k, call_id, keys, rnd);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 t = level_row<CM>(level_in_cell(u[i], c[i]), xs[i]);
            e[i] = rounds_up(u[i], t, rnd[i]) ? t.w : t.z;
        }
        put_entries(s, e);
    };
    if (fast && slots == kSlots) {
#pragma unroll
        for (int s = 0; s < kSlots; ++s) fast_row(s);
    } else {
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            code[s] = RowCode{0u, 0u, 0u};
            if (s >= slots) continue;
            if (fast) {
                fast_row(s);
            } else {                                   // a norm of zero or without a reciprocal, u above 1, crowded cells
                const float xs[4] = {v[s].x, v[s].y, v[s].z, v[s].w};
                const bool live_s = GROUPED ? rinv_s[s] != 0.0f : live;
                uint32_t rnd[4], e[4];
                philox4x32_10((at0 >> 2) + 64u * (uint32_t)s, 0u, k, call_id, keys, rnd);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t idx = 0;
                    const uint32_t neg = __float_as_uint(xs[i]) >> 31;
                    if (live_s) {
                        const float u = fminf(fabsf(xs[i]) * rinv_s[s], 1.0f);
                        const uint32_t j = level_general<CM>(u, n_sym);
                        idx = j + (rounds_up(u, level_row<CM>(j, xs[i]), rnd[i]) ? 1u : 0u);
                    }
                    uint32_t entry = lds_load_u32(kLevAt<CM> + 8u + (2u * idx + neg) * 16u);
                    asm("" : "+v"(entry));
                    e[i] = entry;
                }
                put_entries(s, e);
            }
        }
    }
    // each lane's place among its row's 16 columns, two slots to a scan; the rows' pieces through LDS
#pragma unroll
    for (int s = 0; s < kSlots; s += 2) {
        const uint32_t both = __builtin_amdgcn_perm(code[s + 1].sum, code[s].sum, 0x0C050C01u);
        uint32_t incl = both;
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x112, 0xf, 0xf, false);
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x114, 0xf, 0xf, false);
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x118, 0xf, 0xf, false);
        length[s] = both & 0xFFFFu;
        length[s + 1] = both >> 16;
        end[s] = incl & 0xFFFFu;
        end[s + 1] = incl >> 16;
        if ((lane & 15) == 15) {
            if (s < slots) s_counts[4u * (row0 + (uint32_t)s) + part] = end[s];
            if (s + 1 < slots) s_counts[4u * (row0 + (uint32_t)s + 1u) + part] = end[s + 1];
        }
    }
    __syncthreads();
    const uint32_t count = s_counts[lane], upto = wave_incl_scan(count);
    const uint32_t total_bits = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
    const uint32_t words = (((total_bits + 31u) >> 5) + (kAlignWords - 1)) & ~(uint32_t)(kAlignWords - 1);
    if (ordered && part == 0u && lane == 0) s_totals[cw] = words;
    if (g.clen != 0u) {
        uint16_t* __restrict__ sub_g = a.sub_end + ((size_t)k * lay.NC + g.c) * kSubs;
        const __amdgpu_buffer_rsrc_t ends = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(uniform_address(sub_g)), 0, kSubs * (int)sizeof(uint16_t), 0x00027000);
        const uint32_t stage0 = 8u * (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_address(stage)) - 1u;      // (see place_row)
#pragma unroll
        for (int s = 0; s < kSlots; ++s) {
            if (s >= slots) break;
            const uint32_t row = row0 + (uint32_t)s;
            const uint32_t base = (uint32_t)__shfl((int)(upto - count), (int)(4u * row + part), kWave);
            place_row(stage0 + base + end[s] - length[s], code[s]);
            // a run's last lane stores where it ends, the others outside the buffer; a row without symbols: where the chunk ends
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(base + end[s]), ends, (lane & 7) == 7 ? (int)(16u * row + 2u * (column >> 3)) : 0x40000000, 0, 0);
        }
        // the rows that no slot stands for
        for (uint32_t i = 32u * (uint32_t)slots + part * kWave + (uint32_t)lane; i < (uint32_t)kSubs; i += 4u * kWave) sub_g[i] = (uint16_t)total_bits;
    }
    uint32_t words_before = 0;
    if (ordered) {
        __syncthreads();
        uint32_t unit_words = 0;
        for (uint32_t c = 0; c < nchunks; ++c) {
            if (c == cw) words_before = unit_words;
            unit_words += s_totals[c];
        }
        if (w == 0u) {
            const uint32_t excl = lookback_exclusive(a.scan_state + (size_t)k * lay.NB * a.parts, unit, unit_words, epoch, sc);
            if (lane == 0) s_misc[1] = excl;
        }
    }
    __syncthreads();                                   // the chunk's codes are all there
    if (g.clen == 0u) return;
    const uint32_t off = ordered ? s_misc[1] + words_before : g.c * a.slot_words;
    if (part == 0u && lane == 0) {
        a.chunk_off[(size_t)k * (lay.NC + 1) + g.c] = off;
        if (g.c + 1 == lay.NC) a.chunk_off[(size_t)k * (lay.NC + 1) + lay.NC] = off + (ordered ? words : a.slot_words);
    }
    if ((uint64_t)off + words > a.cap_words) {
        if (part == 0u && lane == 0) raise_error(sc, QGX_EBIT_CAPACITY);
    } else {
        uint4* __restrict__ dst = reinterpret_cast<uint4*>(a.payload + (size_t)k * a.cap_words + off);
        const uint4* src = reinterpret_cast<const uint4*>(stage);
        for (uint32_t i = part * kWave + (uint32_t)lane; i < (words >> 2); i += 4u * kWave) dst[i] = src[i];
    }
}

static size_t encode_lds_bytes(int waves, const EncodeArgs& a, bool with_stage, bool grouped)
{
    size_t n = (size_t)a.pieces * sizeof(uint4) + (grouped ? (size_t)waves * 64 : 0) +
               (2 * (size_t)waves + 2) * sizeof(double) + (size_t)(waves + 3) / 4 * 4 * sizeof(uint32_t) + 32;
    if (with_stage) n += (size_t)waves * a.stage_bytes;
    return n;
}

template <EncMode MODE, bool GROUPED, int CM, bool STAGED = false>
static hipError_t launch_mode(const Layout& lay, const Tables* tab, Scalars* sc, const EncodeArgs& a, hipStream_t st)
{
    EncodeArgs b = a;
    const bool ordered = MODE != EncMode::QuantOnly && a.slot_words == 0u;
    b.group = GROUPED || a.parts > 1u ? 1u : buckets_per_group(lay.waves_per_bucket, (uint64_t)lay.K * lay.NC, ordered);
    const int waves = (GROUPED || a.parts > 1u) ? 4 : (int)(b.group * lay.waves_per_bucket);
    const size_t lds = encode_lds_bytes(waves, a, MODE != EncMode::QuantOnly, GROUPED);
    static LdsLimit limit;
    hipError_t e = limit.ensure(reinterpret_cast<const void*>(&k_encode<MODE, GROUPED, CM, STAGED>), 160 * 1024);
    if (e != hipSuccess) return e;
    // one workgroup per bucket or group of buckets, per part of a bucket, or (shared chunks) per four chunks; in compact
    // placement and with split buckets each takes one ticket of its worker
    b.units = GROUPED ? (lay.NC + 3u) / 4u : a.parts > 1u ? lay.NB * a.parts : (lay.NB + b.group - 1u) / b.group;
    // Where the workgroups of a bucket wait for each other, no XCD may have more workers than leave it a place to
    // start one in (see worker_span).  The game's form puts the K workgroups of a unit on one XCD, which all K workers
    // then share, as long as that holds for K (42 workers with four workgroups to a compute unit, 31 with three).
    const uint32_t held = held_per_xcd(kSimdWaves<STAGED>, lds, a.n_cu);
    b.span = kWaits<MODE> && a.parts > 1u ? worker_span(lay.K, a.parts, held) : lay.K;
    b.spread = ordered && a.parts == 1u && spread_workers(lay.K, b.units) ? 1u : 0u;
    b.by_unit = MODE == EncMode::Generate && (a.parts == 1u || (a.parts - 1u) * lay.K < held) ? 1u : 0u;
    const uint32_t grid = b.span * b.units;
    hipLaunchKernelGGL((k_encode<MODE, GROUPED, CM, STAGED>), dim3(grid), dim3(waves * kWave), lds, st, lay, tab, sc, b);
    return hipGetLastError();
}

template <bool GROUPED, int CM>
static hipError_t launch_columns(const Layout& lay, const Tables* tab, Scalars* sc, const EncodeArgs& a, hipStream_t st)
{
    EncodeArgs b = a;
    const bool ordered = a.slot_words == 0u;
    // (where units are ticketed these are those of k_encode: a context's launches share the counters)
    const uint32_t chunks = GROUPED ? (ordered ? 4u : 1u) : lay.waves_per_bucket;
    b.units = GROUPED ? (lay.NC + chunks - 1u) / chunks : lay.NB;
    b.spread = ordered && spread_workers(lay.K, b.units) ? 1u : 0u;
    const size_t lds = ColumnLds(a.pieces, chunks, GROUPED).stage + (size_t)chunks * a.stage_bytes;
    static LdsLimit limit;
    const hipError_t e = limit.ensure(reinterpret_cast<const void*>(&k_encode_columns<GROUPED, CM>), 160 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_encode_columns<GROUPED, CM>), dim3(lay.K * b.units), dim3(chunks * 4u * kWave), lds, st, lay, tab, sc, b);
    return hipGetLastError();
}

template <EncMode MODE, int CM>
static hipError_t launch_size(const Layout& lay, const Tables* tab, Scalars* sc, const EncodeArgs& a, hipStream_t st)
{
    if constexpr (MODE == EncMode::Fused) {
        if (a.columns)
            return lay.shared_chunks ? launch_columns<true, CM>(lay, tab, sc, a, st) : launch_columns<false, CM>(lay, tab, sc, a, st);
    }
    if (lay.shared_chunks) return launch_mode<MODE, true, CM>(lay, tab, sc, a, st);
    if constexpr (MODE == EncMode::Fused) {
        if (use_staged((uint64_t)lay.K * lay.NC, 4u * a.n_cu)) return launch_mode<MODE, false, CM, true>(lay, tab, sc, a, st);
    }
    return launch_mode<MODE, false, CM>(lay, tab, sc, a, st);
}

template <EncMode MODE>
static hipError_t launch_kind(const Layout& lay, const Tables* tab, Scalars* sc, const EncodeArgs& a, hipStream_t st)
{
    switch (a.cell_mant) {
        case 4: return launch_size<MODE, 4>(lay, tab, sc, a, st);
        case 5: return launch_size<MODE, 5>(lay, tab, sc, a, st);
        default: return launch_size<MODE, 6>(lay, tab, sc, a, st);
    }
}

hipError_t launch_encode(EncMode mode, const Layout& lay, const Tables* tab, Scalars* sc, const EncodeArgs& a,
                         hipStream_t st)
{
    switch (mode) {
        case EncMode::Fused: return launch_kind<EncMode::Fused>(lay, tab, sc, a, st);
        case EncMode::Generate:
            if (lay.shared_chunks) return hipErrorInvalidValue;          // (the host side has refused this layout)
            switch (a.cell_mant) {
                case 4: return launch_mode<EncMode::Generate, false, 4, true>(lay, tab, sc, a, st);
                case 5: return launch_mode<EncMode::Generate, false, 5, true>(lay, tab, sc, a, st);
                default: return launch_mode<EncMode::Generate, false, 6, true>(lay, tab, sc, a, st);
            }
        case EncMode::QuantOnly: return launch_kind<EncMode::QuantOnly>(lay, tab, sc, a, st);
        default: return launch_kind<EncMode::EncodeOnly>(lay, tab, sc, a, st);
    }
}

}  // namespace qgx
