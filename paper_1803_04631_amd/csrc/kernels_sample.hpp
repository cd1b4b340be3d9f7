// Sampling kernel: one pass of the sparsity-aware sampler (paper Section 6.1, Eq. 6-8,
// Algorithm 2) over word-sorted tokens.
//
// Mapping to gfx950 (the paper's own mapping, one 32-wide warp per sampler with 32-way
// index trees, was made for NVIDIA warps; measured here, a whole 64-lane wave per token is
// bound by VALU issue, not by HBM):
//   - a workgroup of four (twelve or sixteen for large K) waves, or a single wave where the tile is small and the
//     column of topics short, works on one tile = up to 1024 (4096 for large K) consecutive tokens of ONE
//     word and stages that word's p*(k) (Eq. 8, rounded to fp32) once in LDS, widened to fp64 where
//     K <= 2048 and rows are not the shortest, with fp64 prefix sums over groups of 4 (or 16) topics
//     (Section 6.1.2: samplers of a block share the word's data);
//     for large K, as many workgroups as the chip holds take tile after tile from a counter, the many words of
//     few tokens last, and turn p* of one such word into p* of the next; where K is too large for p* to fit the
//     LDS, the topics that have no room are staged in a strip of device memory that the workgroup owns;
//   - each wave takes 64 tokens at a time (fewer when a large-K tile is too small to give every
//     wave that many).  What is per token and needs no cooperation is
//     done one token per LANE: the Philox uniform, the token's own-count correction of
//     p*(o), and the search in the dense bucket p2 (binary search over the group prefixes,
//     then the group's topics);
//   - the walk over the token's sparse theta row (S and the p1 prefix sums, Eq. 6-7) is done
//     by a GROUP of 4, 8, 16, 32 or 64 lanes per token, chosen per pass from the row lengths
//     so that a lane owns at most three 16-byte units of entries (16, 8, 4, 2 or 1 tokens per
//     pass: the fixed cost of a pass is shared by as many tokens as their rows allow).  Groups
//     narrower than a DPP row of 16 lanes are interleaved inside the row (4 or 2 tokens side by
//     side), so that plain row shifts scan every group at once.  Every lane owns a contiguous
//     run of entries, accumulates them in fp64 and keeps the sum at the end of each unit; a DPP
//     scan over the group gives the prefix over lanes.  The lane whose range holds the draw
//     names the unit that holds it and what is left of the draw there; "the smallest k whose
//     prefix exceeds it" (Section 6.1.1) among that unit's few entries is found afterwards, one
//     token per lane again, for all tokens of the batch at once.  Rows too long for three
//     units per lane of a whole wave are walked twice by the wave.  Token parameters and
//     results travel between the per-lane and per-group phases through small per-wave LDS
//     records;
//   - tokens of one document and word stand next to each other; where most tokens of a batch have such
//     company, a row is walked once for all of them, its prefix sums go to LDS, and every token
//     corrects them for its own topic and looks its draw up there, one token per lane;
//   - a theta row is a run of entries (topic, count) in ascending topic order, 2 bytes each
//     where K <= 2048 (3, 5 or 6 bits of count; 4 bytes for documents long beside the topics, and
//     for the shortest), else 4 bytes (16 bits of topic, 14 of count); a count too large for its field is written
//     as several entries of the same topic, one after the other, which changes no sum.  Only
//     the first entry of the token's own topic gives up the token itself;
//   - the row walk is a chain of dependent loads (record, then a random row in HBM), so the
//     loads of the next pass are issued before the current pass is worked on.
#pragma once
#include <type_traits>
#include "chunk_layout.hpp"
#include "device_util.hpp"
#include "row_sums.hpp"

namespace mlda {

// phi (Section 6.1.3: short integers for the dense model).  A word with fewer than 2^16 tokens
// can never overflow a 16-bit count: its row lives in `narrow`.  The few heavier words have an
// int32 row in `wide` (wide_row[v] = its index there, -1 for the others) and their rows in
// `narrow` stay zero, so that sums over all cells of both matrices count every token once.
constexpr int kNarrowWordLimit = 1 << 16;   // tokens of a word from which its row is wide
struct PhiView {
    uint16_t* narrow;           // [V][K]
    int32_t* wide;              // [n_wide][K]
    const int32_t* wide_row;    // [V]
};

struct SampleArgs {
    const Tile* tiles;
    const uint32_t* tok_slot;   // [T] slot of the theta row of each word-major token's document
    const int32_t* tok_id;      // [T] its index in the caller's document-major order
    const uint16_t* z_cur;      // [T] word-major, frozen for the pass
    uint16_t* z_next;           // [T] word-major, written
    // theta rows: a slot (offset in 16-byte units) starts with a header of kRowHeader bytes
    // whose first word is the row's number of entries and whose last bytes are a padding
    // entry, then holds the entries in one of the layouts below (PackedRows, TinyRows, CountedRows),
    // filled up to a whole 16-byte unit with padding entries (count 0, topic K)
    const unsigned char* slots;
    PhiView phi;
    const int32_t* n_k;         // [K]
    int32_t K, Kpad;            // Kpad = K+1 rounded up to a multiple of the dense group: p*(K..Kpad-1) = 0
    double alpha, beta, beta_V;
    uint64_t seed;
    uint32_t iter;
    // The tiles from n_single on each hold a whole word of few tokens (see Form)
    int32_t n_tiles, n_single;
    // Form::queued and split: workgroup b takes tile b, then those that next_tile (zero before and after the launch)
    // hands out from the grid's size on.
    uint32_t* next_tile;
    // Form::split: workgroup b keeps p* of the topics near_topics (a multiple of 16) and on in its strip of
    // far_strip_cells(Kpad, near_topics) from far_pstar on, from the kFarFirst-th of them
    float* far_pstar;
    int32_t near_topics;
    int32_t min_batch;          // K <= 2048: tokens a wave takes at a time at least
    // Tokens that share the walks over their rows: how many passes, and (fp64 weights) units of them, a wave keeps
    // the sums of at a time; none: every token walks by itself.  (fp32 weights: a sum per lane and pass)
    int32_t kept_passes, kept_sums;
    uint32_t sum_slack;         // shared walks, fp64 weights: see kNearlyAll (bits of a double's exponent, in its upper dword)
    unsigned long long* started;    // see stamp_start
};

constexpr int kRowHeader = 16;  // bytes before a theta row's entries
// Topics per fp64 prefix group of the dense bucket: 4 where LDS has room (workgroups of up to four
// waves, K <= 2048), 16 for the large-K workgroups, 32 where p* does not fit beside the groups' sums.
__host__ __device__ constexpr int dense_group(int waves, bool far = false) { return waves <= 4 ? 4 : far ? 32 : 16; }
constexpr int kKeptUnits = 3;   // 16-byte units of entries a lane keeps in registers at most
constexpr int kMostKeptUnits = kWave * kKeptUnits;  // of a row that is walked once
constexpr int kMinBatch = 8;    // tokens a wave takes at a time at least

// Once a token's pass has read its record, the record takes the result back to the per-lane
// phase: `nnz` says what kind (below), `off` and `u` hold it.
struct __align__(16) TokenRec { // per-lane phase -> per-group phase, 32 bytes
    uint32_t off;               // slot offset of the token's theta row, 16-byte units
    int32_t nnz;                // 16-byte units of entries of the row
    int32_t o;                  // current topic
    float w_o;                  // p*(o) with the token itself removed
    double u;
    double Qp;                  // alpha * sum_k p*'(k)
};
constexpr int kDrawInUnit = -1; // off = the 16-byte unit of the slot buffer that holds the draw,
                                // u = what is left of the draw at the unit's start
constexpr int kDrawDense = -2;  // the draw falls into the dense bucket p2; u = its position there
constexpr int kDrawTopic = -3;  // off = the new topic itself

// p* of the tile's word is staged as fp64 or fp32 (Layout::kDoubleWeights), as fp32 always in the
// workgroups of twelve and sixteen waves, where fp64 would cost a CU its second workgroup or LDS its topics.
//
// Large K: a wave keeps the sums of at least so many passes, which takes no more than its records do.
constexpr int kLeastKeptPasses = 2;
// (a sum per lane and pass; the rows' lengths take two bytes each, 64 bytes more than the shorter ones below)
__host__ __device__ constexpr int lane_sums_for(int kept_passes) { return kept_passes * kWave + 8; }
// What a wave keeps in LDS: the records of its tokens, or (shared walks) the sums of up to kept_sums units
// and the first topics of the lanes of kept_passes passes, then 64 rows' slots and lengths.
__host__ __device__ constexpr int sample_wave_bytes(int kept_passes, int kept_sums) {
    const int shared = kept_sums * 8 + kept_passes * kWave * 2 + kWave * 5, records = kWave * (int)sizeof(TokenRec);
    return shared > records ? shared : records;
}
// LDS bytes of sample_kernel<kWaves> for a given Kpad and bytes of a staged weight: p*, the prefix sums, the word's least
// weight (in 16 bytes), the waves' own.
__host__ __device__ constexpr size_t sample_lds_bytes(int Kpad, int waves, int weight_bytes, int kept_passes = 0, int kept_sums = 0) {
    return (size_t)Kpad * weight_bytes + (size_t)((Kpad / dense_group(waves) + 1) & ~1) * 8 + 16 +
           (size_t)waves * sample_wave_bytes(kept_passes, kept_sums);
}
// What small tiles that follow one another keep in LDS besides: the groups' own sums (the prefix sums are made
// from them again after every change) and one bit per group for "changed".
__host__ __device__ constexpr size_t sample_run_lds_bytes(int Kpad, int waves, bool far = false) {
    const size_t ng = (size_t)(Kpad / dense_group(waves, far));
    return ((ng + 1) & ~(size_t)1) * 8 + ((ng + 31) / 32 * 4 + 15 & ~(size_t)15);
}
// Cells of a workgroup's strip of device memory: those of the topics from `near` on, and four of 0 before them.
constexpr int kFarFirst = 16;
__host__ __device__ constexpr size_t far_strip_cells(int Kpad, int near) { return (size_t)(Kpad - near + kFarFirst); }
// The same when p* of the topics from `near` on stays in device memory (four cells of 0 stand for those).
__host__ __device__ constexpr size_t sample_far_lds_bytes(int Kpad, int waves, int near) {
    return (size_t)(near + 4) * 4 + (size_t)((Kpad / dense_group(waves, true) + 1) & ~1) * 8 + 16 +
           (size_t)waves * sample_wave_bytes(kLeastKeptPasses, lane_sums_for(kLeastKeptPasses)) + sample_run_lds_bytes(Kpad, waves, true);
}
constexpr int kRunTileTokens = 1024;    // a tile of a run holds a whole word of at most this many tokens

// A count becomes a factor without a conversion: its bits, taken as the upper dword of a double
// whose lower dword is zero, are the denormal number count * kCountUnit.  The weights staged in
// LDS carry kWeightScale, so a product (exact, as before) is count * p* * kSumScale: powers of two
// that change no rounding anywhere.  p* <= 1, hence a weight stays finite; an fp32 p* other than 0
// is at least 2^-149, hence no product comes near the denormal numbers again.
constexpr double kWeightScale = 0x1p1000;
constexpr double kCountUnit = 0x1p-1042;
constexpr double kSumScale = kWeightScale * kCountUnit;
constexpr int kSumScaleLog2 = 1000 - 1042;
// Shared walks, fp64 weights: sums of up to 2^sum_slack times what is exact round in a last bit or three where sub-lanes are
// added up, as they do in a walk of the token's own, and are let where the row's sum with all of the own topic in it is at
// most so many times the token's total.  Where the row's units end, error against __float128 in 2^-53 of the total, of such
// tokens in books late in training (7 % of the tokens there, at beta = 0.01): root mean square 0.3949, at most 2.55, both as in a
// walk of their own.  At beta = 1e-3 0.4846 against 0.4844; at 1e-5, where none are let, up to 2 % more or less.
constexpr double kNearlyAll = 1.02;
// Q' times kSumScale is a normal number from here on.  A smaller one (alpha below 1e-290 or so) decides
// draws of tokens that are alone in their document only; their place in p2 is worked out without the scale.
constexpr double kSmallestScaled = 0x1p-900;

// A staged weight of either form without its scale.
__device__ __forceinline__ double plain_weight(float w) { return (double)w; }
__device__ __forceinline__ double plain_weight(double w) { return w * (1.0 / kWeightScale); }

// Dense bucket (p2 = alpha p*', Eq. 6): smallest k with alpha * prefix'(k) > y, where
// prefix' is the prefix sum of p* with the entry of the token's own topic o replaced by
// w_o (delta = w_o - p*(o)).  One lane per token.
// four(k): the weights of the topics k .. k + 3 without their scale, k a multiple of 4.
template <int kGroup, class Four>
__device__ __forceinline__ int dense_bucket_search(const Four& four, const double* cp, int K,
                                                   int ng, double alpha, double y, int o,
                                                   float w_o, double delta) {
    // Bisection with steps of falling powers of two: `lo` counts the groups known to lie
    // before the draw.  Every lane makes the same number of steps, so the scalar unit runs the
    // loop, and a step is one LDS read, the correction and one comparison.
    const int o_group = o / kGroup;        // groups from here on hold the own topic's correction
    int lo = 0;
    for (int step = 1 << (31 - __builtin_clz(ng)); step > 0; step >>= 1) {
        const int upto = lo + step;        // would groups 0 .. upto - 1 all lie before the draw?
        if (upto <= ng) {
            const double pre = cp[upto - 1] + (upto > o_group ? delta : 0.0);
            if (!(alpha * pre > y)) lo = upto;
        }
    }
    if (lo >= ng) return K - 1;
    const int k0 = lo * kGroup;
    const double before = (lo > 0 ? cp[lo - 1] : 0.0) + (k0 > o ? delta : 0.0);
    // the group's topics, four in a read (p* beyond K is 0 and adds nothing)
    double acc = before;
    int found = k0 + kGroup - 1;
#pragma unroll 1
    for (int j = k0; j < k0 + kGroup; j += 4) {
        const double4 w = four(j);
        const double a0 = acc + (j == o ? (double)w_o : w.x);
        const double a1 = a0 + (j + 1 == o ? (double)w_o : w.y);
        const double a2 = a1 + (j + 2 == o ? (double)w_o : w.z);
        acc = a2 + (j + 3 == o ? (double)w_o : w.w);
        const int k = alpha * a0 > y ? j : alpha * a1 > y ? j + 1 : alpha * a2 > y ? j + 2 : j + 3;
        if (kGroup == 4 || alpha * acc > y) { found = k; break; }
    }
    return min(found, K - 1);
}

// DPP move of a double with full row and bank masks; lanes without a source read 0.
template <int kCtrl>
__device__ __forceinline__ double dpp_move_all0(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Lane layout of a pass with kLanes lanes per token.  Groups of 16, 32 or 64 lanes are runs
// of consecutive lanes.  Groups of 8 or 4 lanes are interleaved inside each row of 16 lanes:
// with g = 16 / kLanes tokens per row, lane l of the row works for token l % g as its
// sub-lane l / g.
//
// Inclusive prefix sum over the sub-lanes of every group.  Every lane must be active.
// Shifts inside each row of 16 lanes (starting at the interleave distance); for wider groups
// lane 15 of the even rows is added to the odd rows, and for the whole wave lane 31 to rows
// 2 and 3.
template <int kLanes>
__device__ __forceinline__ double group_inclusive_sum(double v) {
    if (kLanes >= 16) v += dpp_move_all0<0x111>(v);   // row_shr:1
    if (kLanes >= 8) v += dpp_move_all0<0x112>(v);    // row_shr:2
    v += dpp_move_all0<0x114>(v);                      // row_shr:4
    v += dpp_move_all0<0x118>(v);                      // row_shr:8
    if (kLanes >= 32) v += dpp_move0<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    if (kLanes >= 64) v += dpp_move0<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

// Value of the sub-lane before this one inside the group, 0 for the group's first sub-lane.
template <int kLanes>
__device__ __forceinline__ double group_previous(double incl, int sl) {
    if (kLanes == 16) return dpp_move_all0<0x111>(incl);          // row_shr:1
    if (kLanes == 8) return dpp_move_all0<0x112>(incl);           // row_shr:2
    if (kLanes == 4) return dpp_move_all0<0x114>(incl);           // row_shr:4
    const double up = dpp_move_all0<0x138>(incl);                  // wave_shr:1
    return sl == 0 ? 0.0 : up;
}

// Lane that holds the group's last sub-lane.
template <int kLanes>
__device__ __forceinline__ int group_last_lane(int lane) {
    return kLanes >= 16 ? (lane | (kLanes - 1)) : (lane | (16 - 16 / kLanes));
}

// Value of the sub-lane before this one inside the group (garbage for the group's first).
template <int kLanes>
__device__ __forceinline__ int group_previous_int(int v) {
    if (kLanes == 16) return __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    if (kLanes == 8) return __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);    // row_shr:2
    if (kLanes == 4) return __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);    // row_shr:4
    return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true);                      // wave_shr:1
}

// ---------------------------------------------------------------- theta row layouts
// A row's entries follow its 16-byte header in ascending topic order and are read in units of
// 16 bytes.  A count beyond an entry's field is spread over several entries of the same topic.
// key = the byte offset of p*(topic).

// 4 bytes per entry: count << 18 | topic << 2.  Any K; p* in fp32.
struct PackedRows {
    typedef uint32_t Entry;
    static constexpr int kEntryBytes = 4, kUnitEntries = 4;
    static constexpr int kMaxCount = (1 << 14) - 1;
    static constexpr int kWavesPerSimd = 6;
    static constexpr bool kOneEntryPerTopic = false, kDoubleWeights = false, kShares = true;
    static __host__ __device__ __forceinline__ Entry make(int count, int topic) {
        return ((uint32_t)count << 18) | ((uint32_t)topic << 2);
    }
    static __host__ __device__ __forceinline__ int entry_topic(Entry e) { return (int)((e >> 2) & 0xffffu); }
    static __host__ __device__ __forceinline__ int entry_count(Entry e) { return (int)(e >> 18); }
    static __device__ __forceinline__ uint32_t word(const uint4& u, int j) {
        return j == 0 ? u.x : j == 1 ? u.y : j == 2 ? u.z : u.w;
    }
    static __device__ __forceinline__ int key_of_topic(int k) { return k << 2; }
    static __device__ __forceinline__ int key(const uint4& u, int j) { return (int)(word(u, j) & 0x3fffcu); }
    static __device__ __forceinline__ int count(const uint4& u, int j) { return (int)(word(u, j) >> 18); }
};

// The same when no document has more tokens than an entry counts (the host checks): every topic
// then has one entry, the row walk needs no look at the entry before, and with so few entries
// per unit the search for the draw's entry is cheapest inside the pass itself.
struct PackedRowsShort : PackedRows {
    static constexpr bool kOneEntryPerTopic = true;
};
// The same for documents so short that tokens hardly share a walk over their row.
struct PackedRowsAlone : PackedRowsShort {
    static constexpr bool kShares = false;
};

// The two layouts of K <= 2048, whose p* is staged in fp64.  An entry holds its topic above its
// count: entries of a row rise as numbers, and "(o, kMaxCount) - entry", as an unsigned number, is at
// most kMaxCount for the entries of topic o only.
//
// 2 bytes per entry: topic << kCountBits | count.  With three bits of count a topic's place in the
// entry is the byte offset of its p*; with more of them (five for K < 2048, six for K < 1024: all that
// the topics leave) a pair of entries is shifted there by one instruction more, which short documents
// need not pay: row_kind_for.
template <int kCountBits>
struct TinyRows {
    typedef uint16_t Entry;
    static constexpr int kEntryBytes = 2, kUnitEntries = 8;
    static constexpr int kMaxCount = (1 << kCountBits) - 1;
    static constexpr int kMaxK = (1 << (16 - kCountBits)) - 1;      // topics 0 .. K, K being the padding entries'
    static constexpr int kWavesPerSimd = 5;
    static constexpr bool kOneEntryPerTopic = false, kDoubleWeights = true, kShares = true;
    typedef uint16_t Pair __attribute__((ext_vector_type(2)));
    static __host__ __device__ __forceinline__ Entry make(int count, int topic) {
        return (Entry)(((uint32_t)topic << kCountBits) | (uint32_t)count);
    }
    static __host__ __device__ __forceinline__ int entry_topic(Entry e) { return (int)(e >> kCountBits); }
    static __host__ __device__ __forceinline__ int entry_count(Entry e) { return (int)(e & (uint32_t)kMaxCount); }
    static __device__ __forceinline__ uint32_t word(const uint4& u, int i) {
        return i == 0 ? u.x : i == 1 ? u.y : i == 2 ? u.z : u.w;
    }
    static __device__ __forceinline__ int key_of_topic(int k) { return k << 3; }
    static __device__ __forceinline__ int key(const uint4& u, int j) {
        const Pair both = __builtin_bit_cast(Pair, word(u, j >> 1));
        const uint32_t d = __builtin_bit_cast(uint32_t, kCountBits > 3 ? both >> (uint16_t)(kCountBits - 3) : both);
        if ((j & 1) == 0) return (int)(d & 0xfff8u);
        uint32_t k;                 // the upper half, masked: one instruction
        asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD"
            : "=v"(k) : "v"(d), "s"(0xfff8u));
        return (int)k;
    }
    static __device__ __forceinline__ int count(const uint4& u, int j) {
        const uint32_t d = word(u, j >> 1);
        return (j & 1) ? (int)__builtin_amdgcn_ubfe(d, 16, kCountBits) : (int)(d & (uint32_t)kMaxCount);
    }
    // The entries of topic o lose their tokens, which are added to n: of the distances to (o,
    // kMaxCount), as unsigned numbers, those of kMaxCount and less are the entries of o, and what they
    // lack to kMaxCount the count.
    static __device__ __forceinline__ void take_out(uint4& u, int o, uint32_t& n) {
        const Pair most = Pair((uint16_t)make(kMaxCount, o)), one = Pair(1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t& d = i == 0 ? u.x : i == 1 ? u.y : i == 2 ? u.z : u.w;
            const Pair own = __builtin_elementwise_sub_sat(Pair(kMaxCount), most - __builtin_bit_cast(Pair, d));
            n = __builtin_amdgcn_udot2(own, one, n, false);
            d -= __builtin_bit_cast(uint32_t, own);         // (no half below zero: own is its count, or 0)
        }
    }
    // n += the tokens of topic o (as take_out, the entries stay)
    static __device__ __forceinline__ void count_own(const uint4& u, int o, uint32_t& n) {
        const Pair most = Pair((uint16_t)make(kMaxCount, o)), one = Pair(1);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            n = __builtin_amdgcn_udot2(__builtin_elementwise_sub_sat(Pair(kMaxCount), most - __builtin_bit_cast(Pair, word(u, i))), one, n, false);
    }
    // acc += count * weight over the eight entries, in their order
    static __device__ __forceinline__ void add_products(const uint4& u, const double* w, double& acc) {
        add_four(u.x, u.y, w, acc);
        add_four(u.z, u.w, w + 4, acc);
    }
    static __device__ __forceinline__ void add_four(uint32_t d0, uint32_t d1, const double* w, double& acc) {
        asm("v_mov_b32 v72, 0\n\tv_mov_b32 v74, 0\n\t"
            "v_and_b32 v73, %7, %1\n\tv_bfe_u32 v75, %1, 16, %8\n\t"
            "v_fma_f64 %0, v[72:73], %3, %0\n\tv_and_b32 v73, %7, %2\n\t"
            "v_fma_f64 %0, v[74:75], %4, %0\n\tv_bfe_u32 v75, %2, 16, %8\n\t"
            "v_fma_f64 %0, v[72:73], %5, %0\n\t"
            "v_fma_f64 %0, v[74:75], %6, %0"
            : "+&v"(acc)
            : "v"(d0), "v"(d1), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "n"(kMaxCount), "n"(kCountBits)
            : "v72", "v73", "v74", "v75");
    }
};

// 4 bytes per entry: topic << 16 | count (13 bits), for long documents over few topics.
struct CountedRows {
    typedef uint32_t Entry;
    static constexpr int kEntryBytes = 4, kUnitEntries = 4;
    static constexpr int kMaxCount = (1 << 13) - 1;
    static constexpr int kWavesPerSimd = 5;
    static constexpr bool kOneEntryPerTopic = false, kDoubleWeights = true, kShares = true;
    static __host__ __device__ __forceinline__ Entry make(int count, int topic) {
        return ((uint32_t)topic << 16) | (uint32_t)count;
    }
    static __host__ __device__ __forceinline__ int entry_topic(Entry e) { return (int)(e >> 16); }
    static __host__ __device__ __forceinline__ int entry_count(Entry e) { return (int)(e & 0x1fffu); }
    static __device__ __forceinline__ uint32_t word(const uint4& u, int j) {
        return j == 0 ? u.x : j == 1 ? u.y : j == 2 ? u.z : u.w;
    }
    static __device__ __forceinline__ int key_of_topic(int k) { return k << 3; }
    static __device__ __forceinline__ int key(const uint4& u, int j) { return (int)(word(u, j) >> 13); }
    static __device__ __forceinline__ int count(const uint4& u, int j) { return (int)(word(u, j) & 0x1fffu); }
    static __device__ __forceinline__ void take_out(uint4& u, int o, uint32_t& n) {     // as above
        const uint32_t most = make(kMaxCount, o);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t& d = i == 0 ? u.x : i == 1 ? u.y : i == 2 ? u.z : u.w;
            const uint32_t own = __builtin_elementwise_sub_sat((uint32_t)kMaxCount, most - d);
            n += own;
            d -= own;
        }
    }
    static __device__ __forceinline__ void count_own(const uint4& u, int o, uint32_t& n) {
        const uint32_t most = make(kMaxCount, o);
#pragma unroll
        for (int i = 0; i < 4; ++i) n += __builtin_elementwise_sub_sat((uint32_t)kMaxCount, most - word(u, i));
    }
    static __device__ __forceinline__ void add_products(const uint4& u, const double* w, double& acc) {
        asm("v_mov_b32 v72, 0\n\tv_mov_b32 v74, 0\n\t"
            "v_and_b32 v73, 0x1fff, %1\n\tv_and_b32 v75, 0x1fff, %2\n\t"
            "v_fma_f64 %0, v[72:73], %5, %0\n\tv_and_b32 v73, 0x1fff, %3\n\t"
            "v_fma_f64 %0, v[74:75], %6, %0\n\tv_and_b32 v75, 0x1fff, %4\n\t"
            "v_fma_f64 %0, v[72:73], %7, %0\n\t"
            "v_fma_f64 %0, v[74:75], %8, %0"
            : "+&v"(acc)
            : "v"(u.x), "v"(u.y), "v"(u.z), "v"(u.w), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3])
            : "v72", "v73", "v74", "v75");
    }
};

// Unit `unit` of the row in slot `off`.  Every lane loads: a lane without entries reads the
// padding entries that the library keeps in the first 64 bytes of the slot buffer (no slot
// starts there).
__device__ __forceinline__ uint4 load_unit(const unsigned char* slots, uint32_t off, int unit, bool on) {
    static_assert(kRowHeader == 16, "a row's entries start one 16-byte unit into its slot");
    uint32_t at = on ? off + 1u + (uint32_t)unit : 0u;
    // the choice is made on the 32-bit unit number, before it becomes a 64-bit address
    asm volatile("" : "+v"(at));
    return *reinterpret_cast<const uint4*>(slots + (size_t)at * 16u);
}

// The same for a slot buffer smaller than 4 GiB.  `row_bytes` is the byte offset of the lane's
// first unit, `c` (a constant) the unit's number among the lane's units; a lane without that
// unit reads padding unit c (the buffer starts with kKeptUnits + 1 of them).
__device__ __forceinline__ uint4 load_unit_near(const unsigned char* slots, uint32_t row_bytes, int c, bool on) {
    uint32_t at = on ? row_bytes : 0u;
    asm volatile("" : "+v"(at));
    return *reinterpret_cast<const uint4*>(slots + (size_t)at + (size_t)(c * 16));
}

// A load and a store at a 32-bit byte offset from a base that is the same for the whole wave:
// the base stays in scalar registers and the offset is all a lane computes.
template <class T>
__device__ __forceinline__ T load_at(const void* base, uint32_t byte_offset) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(base) + byte_offset);
}
template <class T>
__device__ __forceinline__ void store_at(void* base, uint32_t byte_offset, T v) {
    *reinterpret_cast<T*>(reinterpret_cast<unsigned char*>(base) + byte_offset) = v;
}

// Key of the entry that lies just before a unit in memory (a row's header ends in a padding
// entry, so this is always an entry).
template <class Layout>
__device__ __forceinline__ int key_before_unit(const unsigned char* unit_ptr) {
    typedef typename Layout::Entry Entry;
    return Layout::key_of_topic(Layout::entry_topic(*reinterpret_cast<const Entry*>(unit_ptr - sizeof(Entry))));
}

// p*(k) is staged at the very start of the workgroup's LDS, so a topic's key (4 k, 8 k for fp64)
// is the LDS address of its weight.
__device__ __forceinline__ float lds_float_at(uint32_t byte_address) {
    typedef __attribute__((address_space(3))) const float* lds_float_ptr;
    return *(lds_float_ptr)(uintptr_t)byte_address;
}
__device__ __forceinline__ double lds_double_at(uint32_t byte_address) {
    typedef __attribute__((address_space(3))) const double* lds_double_ptr;
    return *(lds_double_ptr)(uintptr_t)byte_address;
}

// Where the walk over a row finds p*(k) by the entry's key 4 k: in LDS ...
struct LdsWeights {
    __device__ __forceinline__ float operator()(uint32_t key) const { return lds_float_at(key); }
};
// ... or, when K is too large for that, there up to near_key (where a 0 lies) and from there on in the workgroup's
// own strip of device memory (written by the workgroup itself before a barrier, and read through the CU's own cache;
// in front of its first cell lies a 0).  Every lane reads both places: those whose topic is near all read the
// strip's one 0, so that a gather from it costs what its far topics do.
struct SplitWeights {
    const unsigned char* strip;
    uint32_t near_key;
    __device__ __forceinline__ float operator()(uint32_t key) const {
        return lds_float_at(min(key, near_key)) + *reinterpret_cast<const float*>(strip + max(key, near_key - 4u));
    }
};

// p1 = theta' p*' over the entries of one unit (Eq. 6), accumulated onto `acc` in entry order
// (each product is exact in fp64).  The token's own topic o weighs w_o in all its entries and
// its first entry counts one less: the token itself.  `prev_own`: the lanes whose entry before
// this unit belongs to their o; on return: those whose last entry of the unit does.  ("Own and
// first" is worked out on these lane masks, by the scalar unit.)
// This form leaves the sum at the unit's end only.  (Every entry added with its whole count, and w_o given back at the
// end, takes an instruction less per entry; but w_o may be 1 / beta times all the rest, of which nothing is then left.)
template <class Layout, class Weights>
__device__ __forceinline__ void unit_sum(const Weights& weight_at, const uint4& raw, int o_key, float w_o,
                                         uint64_t& prev_own, double& acc) {
    constexpr int n = Layout::kUnitEntries;
#pragma unroll
    for (int h = 0; h < n; h += 4) {       // four gathers of p* on their way at a time
        int key[4];
        float w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            key[j] = Layout::key(raw, h + j);
            w[j] = weight_at((uint32_t)key[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool own = key[j] == o_key;
            const uint64_t own_lanes = __ballot(own);
            const bool first = __builtin_amdgcn_inverse_ballot_w64(own_lanes & ~prev_own);
            prev_own = own_lanes;
            acc = fma((double)(Layout::count(raw, h + j) - (first ? 1 : 0)), (double)(own ? w_o : w[j]), acc);
        }
    }
}

// The same with the running sum after every entry and the entries' keys kept.
template <class Layout, class Weights>
__device__ __forceinline__ void unit_prefix_sums(const Weights& weight_at, const uint4& raw, int o_key, float w_o,
                                                 uint64_t& prev_own, double& acc, double* sums, int* keys) {
    constexpr int n = Layout::kUnitEntries;
#pragma unroll
    for (int j = 0; j < n; ++j) {
        const int key = Layout::key(raw, j);
        const bool own = key == o_key;
        const uint64_t own_lanes = __ballot(own);
        const bool first = __builtin_amdgcn_inverse_ballot_w64(own_lanes & ~prev_own);
        prev_own = own_lanes;
        acc = fma((double)(Layout::count(raw, j) - (first ? 1 : 0)),
                  (double)(own ? w_o : weight_at((uint32_t)key)), acc);
        sums[j] = acc;
        keys[j] = key;
    }
}

// What the lanes of a group need of their token for the walk, read back from its record.
struct RowCtx {
    uint32_t off;           // slot of the row
    int o_key;              // 4 * current topic (a topic's key is its byte offset in p*)
    float w_o;
};

__device__ __forceinline__ RowCtx row_ctx(const TokenRec* rec) {
    const int4 head = *reinterpret_cast<const int4*>(rec);
    RowCtx r;
    r.off = (uint32_t)head.x; r.o_key = head.z << 2; r.w_o = __int_as_float(head.w);
    return r;
}

// Row total S (Eq. 7), the draw x = u (S + Q'), and whether this lane's entries hold it.
struct RowDraw {
    double S, x, y;         // y = x - (sum of the group's sub-lanes before this one)
    bool sparse, hit;
};

// (kScaled: the sums carry kSumScale, and so do the draw and what follows from it)
template <int kLanes, bool kScaled = false>
__device__ __forceinline__ RowDraw row_draw(double lane_sum, const TokenRec* rec, int sl, int lane) {
    RowDraw d;
    const double incl = group_inclusive_sum<kLanes>(lane_sum);
    const double excl = group_previous<kLanes>(incl, sl);
    // (the lane that holds the group's total is worked out here, every time: hoisted out of
    // the loop over passes, one such constant per shape would each hold a register for good)
    asm volatile("" : "+v"(lane));
    d.S = __shfl(incl, group_last_lane<kLanes>(lane), kWave);
    const double2 uq = *reinterpret_cast<const double2*>(&rec->u);     // the uniform, and Q'
    d.x = uq.x * (kScaled ? fma(uq.y, kSumScale, d.S) : d.S + uq.y);
    d.sparse = d.x < d.S;
    d.hit = d.sparse && (incl > d.x) && !(excl > d.x);
    d.y = d.x - excl;
    return d;
}

// A token whose draw falls into the dense bucket p2: recorded once, by its first sub-lane.
__device__ __forceinline__ void record_dense(TokenRec* rec, int sl, const RowDraw& d) {
    if (!d.sparse && sl == 0) {
        rec->nnz = kDrawDense;
        rec->u = d.x - d.S;
    }
}

// Rows whose sub-lanes own at most kUnits units, already loaded (sub-lane sl owns the units from
// sl * kUnits on).  Every lane keeps its sum at the end of each unit; the lane that holds
// the draw records which unit holds it and the rest of the draw there.
// Rows with one entry per topic, already loaded: every lane keeps the running sum after each of
// its entries, and the lane that holds the draw finds its entry at once.
template <class Layout, int kLanes, int kUnits, class Weights>
__device__ __forceinline__ void row_pass_searched(const Weights& weight_at, TokenRec* rec, int sl,
                                                  const uint4* raw, int lane) {
    constexpr int UE = Layout::kUnitEntries, n = kUnits * UE;
    const RowCtx r = row_ctx(rec);
    double sums[n];
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < kUnits; ++c) {
        int key[UE];
        float w[UE];
#pragma unroll
        for (int j = 0; j < UE; ++j) {
            key[j] = Layout::key(raw[c], j);
            w[j] = weight_at((uint32_t)key[j]);
        }
#pragma unroll
        for (int j = 0; j < UE; ++j) {
            const bool own = key[j] == r.o_key;
            acc = fma((double)(Layout::count(raw[c], j) - (own ? 1 : 0)), (double)(own ? r.w_o : w[j]), acc);
            sums[c * UE + j] = acc;
        }
    }
    const RowDraw d = row_draw<kLanes>(acc, rec, sl, lane);
    // smallest entry whose sum exceeds y (the sums never decrease)
    uint32_t entry = Layout::word(raw[kUnits - 1], UE - 1);
#pragma unroll
    for (int i = n - 2; i >= 0; --i)
        if (sums[i] > d.y) entry = Layout::word(raw[i / UE], i % UE);
    if (__builtin_expect(__ballot(d.hit && !(acc > d.y)) != 0, 0)) {   // rounding left no sum above the draw:
        asm volatile("");                            // (a branch of its own: it is almost never taken)
        if (d.hit && !(acc > d.y)) {                 // take the lane's last entry with weight
            double before = 0.0;
#pragma unroll
            for (int i = 0; i < n; ++i) {
                if (sums[i] > before) entry = Layout::word(raw[i / UE], i % UE);
                before = sums[i];
            }
        }
    }
    if (d.hit) {
        rec->off = (uint32_t)Layout::entry_topic(entry);
        rec->nnz = kDrawTopic;
    }
    record_dense(rec, sl, d);
}

template <class Layout, int kLanes, int kUnits, class Weights>
__device__ __forceinline__ void row_pass_kept(const Weights& weight_at, TokenRec* rec, int sl,
                                              const uint4* raw, int lane) {
    const int first_unit = sl * kUnits;
    if constexpr (Layout::kOneEntryPerTopic) {
        row_pass_searched<Layout, kLanes, kUnits>(weight_at, rec, sl, raw, lane);
        return;
    }
    const RowCtx r = row_ctx(rec);
    // does the entry before this lane's first one belong to the token's own topic?  (the
    // previous sub-lane's last entry; a sub-lane past the row's end holds padding entries)
    const int before = group_previous_int<kLanes>(Layout::key(raw[kUnits - 1], Layout::kUnitEntries - 1));
    uint64_t prev_own = __ballot(sl > 0 && before == r.o_key);
    double at_end[kUnits];
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < kUnits; ++c) {
        unit_sum<Layout>(weight_at, raw[c], r.o_key, r.w_o, prev_own, acc);
        at_end[c] = acc;
    }
    const RowDraw d = row_draw<kLanes>(acc, rec, sl, lane);
    // first unit whose end exceeds y (the sums never decrease), and the sum before it
    int unit = kUnits - 1;
#pragma unroll
    for (int c = kUnits - 2; c >= 0; --c)
        if (at_end[c] > d.y) unit = c;
    if (__builtin_expect(__ballot(d.hit && !(acc > d.y)) != 0, 0)) {   // rounding left no sum above the draw:
        asm volatile("");                            // (a branch of its own: it is almost never taken)
        if (d.hit && !(acc > d.y)) {                 // take the lane's last unit with weight
            double before_unit = 0.0;
#pragma unroll
            for (int c = 0; c < kUnits; ++c) {
                if (at_end[c] > before_unit) unit = c;
                before_unit = at_end[c];
            }
        }
    }
    double base = 0.0;
#pragma unroll
    for (int c = 1; c < kUnits; ++c)
        if (unit >= c) base = at_end[c - 1];
    if (d.hit) {
        rec->off = r.off + 1u + (uint32_t)(first_unit + unit);
        rec->nnz = kDrawInUnit;
        rec->u = d.y - base;
    }
    record_dense(rec, sl, d);
}

// ---- the walk with fp64 weights (kDoubleWeights).  VALU issue bounds the walk (85 % of the SIMDs'
// cycles on 7.4e8 tokens at K = 1,000), so what counts is instructions per entry.  With fp32
// weights an entry takes seven: key, count, two conversions to fp64, a comparison with the own
// topic and a select, fma.  Here it takes three (key, count, fma), and two (4-byte entries: four) for
// the token's own topic: its entries are taken out of the row first, so that p*(o) is in no sum.  (It
// may be any number of times larger than all the rest: 1 / beta times for a word seen once.)  Its
// tokens, without the one that is sampled, weigh w_o where the unit ends.
// An 8-byte gather from random places of LDS costs what a 4-byte one does (7.4 cycles per wave and CU).
// Measured, sampling launch: fp32 weights 32.1 ms for 7.4e8 tokens at K = 1,000 and 6.65 ms for 9.9e7
// late in training, this walk 30.5 and 6.36 ms.  The own topic added with p*(o) and corrected where its
// unit ends: 30.3 and 6.61 ms (split rows went a longer way), and a fifth of the draws wrong at
// beta = 1e-30.  Finding its unit before the passes, one token per lane: 37.9 ms (two or three more
// scattered loads per token); four and six waves per SIMD: 32.6 and 30.5 ms.

// acc += count * weight over the entries of one unit.
template <class Layout>
__device__ __forceinline__ void unit_sum_plain(const uint4& raw, double& acc) {
    double w[Layout::kUnitEntries];
#pragma unroll
    for (int j = 0; j < Layout::kUnitEntries; ++j) w[j] = lds_double_at((uint32_t)Layout::key(raw, j));
    Layout::add_products(raw, w, acc);
}

// The sum at the end of a unit whose sum without the own topic is `others`, `n` the own topic's
// tokens up to there: one less where the lane has the topic's first entry (`itself` = 1), whose
// count holds the token itself.
__device__ __forceinline__ double with_own_topic(double others, uint32_t n, uint32_t itself, double w_o) {
    return fma(__hiloint2double((int)__builtin_elementwise_sub_sat(n, itself), 0), w_o, others);
}

template <class Layout, int kLanes, int kUnits>
__device__ __forceinline__ void row_pass_double(TokenRec* rec, int sl, const uint4* raw, int lane) {
    const int4 head = *reinterpret_cast<const int4*>(rec);     // off, units, o, w_o
    const uint32_t off = (uint32_t)head.x;
    const int own_key = Layout::key_of_topic(head.z), first_unit = sl * kUnits;
    const double w_o = kWeightScale * (double)__int_as_float(head.w);       // as the staged weights
    // the topic's first entry is this lane's unless the previous sub-lane's last one is of the topic
    const int before = group_previous_int<kLanes>(Layout::key(raw[kUnits - 1], Layout::kUnitEntries - 1));
    const uint32_t itself = sl > 0 && before == own_key ? 0u : 1u;
    double at_end[kUnits];
    double acc = 0.0;
    uint32_t n_own = 0;
#pragma unroll
    for (int c = 0; c < kUnits; ++c) {
        uint4 unit = raw[c];
        Layout::take_out(unit, head.z, n_own);
        unit_sum_plain<Layout>(unit, acc);
        at_end[c] = with_own_topic(acc, n_own, itself, w_o);
    }
    acc = at_end[kUnits - 1];
    const RowDraw d = row_draw<kLanes, true>(acc, rec, sl, lane);
    // first unit whose end exceeds y (the sums never decrease), and the sum before it
    int unit = kUnits - 1;
#pragma unroll
    for (int c = kUnits - 2; c >= 0; --c)
        if (at_end[c] > d.y) unit = c;
    if (__builtin_expect(__ballot(d.hit && !(acc > d.y)) != 0, 0)) {   // rounding left no sum above the draw:
        asm volatile("");                            // (a branch of its own: it is almost never taken)
        if (d.hit && !(acc > d.y)) {                 // take the lane's last unit with weight
            double before_unit = 0.0;
#pragma unroll
            for (int c = 0; c < kUnits; ++c) {
                if (at_end[c] > before_unit) unit = c;
                before_unit = at_end[c];
            }
        }
    }
    double base = 0.0;
#pragma unroll
    for (int c = 1; c < kUnits; ++c)
        if (unit >= c) base = at_end[c - 1];
    if (d.hit) {
        rec->off = off + 1u + (uint32_t)(first_unit + unit);
        rec->nnz = kDrawInUnit;
        rec->u = d.y - base;
    }
    record_dense(rec, sl, d);
}

// The walk over a row for all the tokens that share it: what the row's sub-lanes have summed up at the end
// of each of their units, every entry with p*, goes to LDS (`sums`, the row's units one after the other; the last one of
// a sub-lane with the sub-lanes before it), with the topic of each sub-lane's first entry.  Three instructions per
// entry and no draw.
template <class Layout, int kLanes, int kUnits>
__device__ __forceinline__ void row_pass_shared(double* sums, uint16_t* first_topic, int rel, int sl, const uint4* raw) {
    double at_end[kUnits];
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < kUnits; ++c) {
        unit_sum_plain<Layout>(raw[c], acc);
        at_end[c] = acc;
    }
    const double incl = group_inclusive_sum<kLanes>(acc);
    const int lane_at = rel * kLanes + sl;
#pragma unroll
    for (int c = 0; c + 1 < kUnits; ++c) sums[lane_at * kUnits + c] = at_end[c];
    sums[lane_at * kUnits + kUnits - 1] = incl;
    first_topic[lane_at] = (uint16_t)Layout::entry_topic((typename Layout::Entry)raw[0].x);
}

// The same for rows too long for the kept shapes, one per wave (sub-lane = lane): one walk for
// the sums, a second one over the hit lane's units.  Lane l owns the units [n l, n (l + 1)).
template <class Layout>
__device__ __forceinline__ void row_pass_double_long(const unsigned char* slots, TokenRec* rec, int lane) {
    const int4 head = *reinterpret_cast<const int4*>(rec);
    const uint32_t off = (uint32_t)head.x;
    const int n_units = head.y, n = (n_units + kWave - 1) / kWave, u0 = lane * n;
    const int own_key = Layout::key_of_topic(head.z);
    const double w_o = kWeightScale * (double)__int_as_float(head.w);
    // the entry before the lane's first one (lanes past the row's end have no entries at all)
    const uint32_t itself = u0 < n_units &&
        key_before_unit<Layout>(slots + ((size_t)off + 1u + (size_t)u0) * 16u) == own_key ? 0u : 1u;
    uint32_t own = 0;
    double others = 0.0;
    auto next_end = [&](uint4 unit) {       // the sum at the end of this unit
        Layout::take_out(unit, head.z, own);
        unit_sum_plain<Layout>(unit, others);
        return with_own_topic(others, own, itself, w_o);
    };
    double acc = 0.0;
    for (int c = 0; c < n; ++c) acc = next_end(load_unit(slots, off, u0 + c, u0 + c < n_units));
    const RowDraw d = row_draw<kWave, true>(acc, rec, lane, lane);
    if (__ballot(d.hit) != 0) {
        bool found = false;
        int unit = 0, last_unit = 0;
        double base = 0.0, last_base = 0.0, before = 0.0;
        own = 0;
        others = 0.0;
        for (int c = 0; c < n; ++c) {
            const double end = next_end(load_unit(slots, off, u0 + c, d.hit && u0 + c < n_units));
            if (!found && end > d.y) { unit = c; base = before; found = true; }
            if (end > before) { last_unit = c; last_base = before; }
            before = end;
        }
        if (d.hit) {
            rec->off = off + 1u + (uint32_t)(u0 + (found ? unit : last_unit));
            rec->nnz = kDrawInUnit;
            rec->u = d.y - (found ? base : last_base);
        }
    }
    record_dense(rec, lane, d);
}

// The entry of one unit that holds the draw y (measured from the unit's start), as
// topic_in_unit below: the first whose running sum exceeds y, else (rounding) the last one with
// weight.  One token per lane.  Bound by instruction issue: the sums are kept and searched from the end (a compare and a select
// an entry; it was two of each), the last entry with weight is looked for only in a batch that has a token without a sum above
// its draw.  Sampling launch at K = 1,000 of 7.4e8 tokens 29.72 -> 29.54 ms, of 9.9e7 late in training 5.16 -> 5.11 ms, at 128
// of 1e6 55.3 -> 54.5 us.
template <class Layout, bool kNear>
__device__ __forceinline__ int topic_in_unit_double(const unsigned char* slots, uint32_t unit, int o, float w_o_f,
                                                    double y) {
    constexpr int n = Layout::kUnitEntries;
    const unsigned char* p = kNear ? slots + (size_t)(uint32_t)(unit << 4) : slots + (size_t)unit * 16u;
    const uint4 raw = *reinterpret_cast<const uint4*>(p);
    const int own_key = Layout::key_of_topic(o);
    const double w_o = kWeightScale * (double)w_o_f;    // as the staged weights
    bool prev_own = key_before_unit<Layout>(p) == own_key;
    double sums[n];
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < n; ++j) {
        const int key = Layout::key(raw, j);
        const bool own = key == own_key, first = own && !prev_own;
        prev_own = own;
        acc = fma(__hiloint2double(Layout::count(raw, j) - (first ? 1 : 0), 0),
                  own ? w_o : lds_double_at((uint32_t)key), acc);
        sums[j] = acc;
    }
    int found = Layout::key(raw, n - 1);        // keys; the sums never fall
#pragma unroll
    for (int j = n - 2; j >= 0; --j)
        if (sums[j] > y) found = Layout::key(raw, j);
    if (__builtin_expect(__ballot(!(acc > y)) != 0, 0)) {
        asm volatile("");       // a branch, not selects
        if (!(acc > y)) {
            double before = 0.0;
            found = Layout::key(raw, 0);
#pragma unroll
            for (int j = 0; j < n; ++j) {
                if (sums[j] > before) found = Layout::key(raw, j);
                before = sums[j];
            }
        }
    }
    return found >> 3;
}

// The entry of one unit that holds the draw y (measured from the unit's start): the first
// whose running sum exceeds y, else (rounding) the last one with weight.  One token per lane.
template <class Layout, bool kNear, class Weights>
__device__ __forceinline__ int topic_in_unit(const Weights& weight_at, const unsigned char* slots, uint32_t unit,
                                             int o_key, float w_o, double y) {
    constexpr int n = Layout::kUnitEntries;
    const unsigned char* p = kNear ? slots + (size_t)(uint32_t)(unit << 4) : slots + (size_t)unit * 16u;
    const uint4 raw = *reinterpret_cast<const uint4*>(p);
    uint64_t prev_own = __ballot(key_before_unit<Layout>(p) == o_key);
    double acc = 0.0;
    int found = -1, last = Layout::key(raw, 0);     // keys: the first above y, the last with weight
#pragma unroll
    for (int j = 0; j < n; ++j) {
        const int key = Layout::key(raw, j);
        const uint64_t own_lanes = __ballot(key == o_key);
        const bool own = __builtin_amdgcn_inverse_ballot_w64(own_lanes);
        const bool first = __builtin_amdgcn_inverse_ballot_w64(own_lanes & ~prev_own);
        prev_own = own_lanes;
        const double before = acc;
        acc = fma((double)(Layout::count(raw, j) - (first ? 1 : 0)),
                  (double)(own ? w_o : weight_at((uint32_t)key)), acc);
        if (acc > before) last = key;
        if (found < 0 && acc > y) found = key;
    }
    return (found >= 0 ? found : last) >> 2;
}

// The walk over a row for all the tokens that share it, fp32 weights: the sums at the ends of the sub-lanes,
// every entry with p*, go to LDS with the topic of each sub-lane's first entry.
template <class Layout, class Weights>
__device__ __forceinline__ void unit_sum_shared(const Weights& weight_at, const uint4& raw, double& acc) {
    float w[Layout::kUnitEntries];
#pragma unroll
    for (int j = 0; j < Layout::kUnitEntries; ++j) w[j] = weight_at((uint32_t)Layout::key(raw, j));
#pragma unroll
    for (int j = 0; j < Layout::kUnitEntries; ++j) acc = fma((double)Layout::count(raw, j), (double)w[j], acc);
}
template <class Layout, int kLanes, int kUnits, class Weights>
__device__ __forceinline__ void row_pass_lanes(const Weights& weight_at, double* sums, uint16_t* first_topic, int rel, int sl,
                                               const uint4* raw) {
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < kUnits; ++c) unit_sum_shared<Layout>(weight_at, raw[c], acc);
    const double incl = group_inclusive_sum<kLanes>(acc);
    sums[rel * kLanes + sl] = incl;
    first_topic[rel * kLanes + sl] = (uint16_t)Layout::entry_topic((typename Layout::Entry)raw[0].x);
}

// The entry that holds the draw y (measured from the first unit's start) among the `n_units` units from `unit`
// on, which have all entries of o or none: as topic_in_unit.  One token per lane.
template <class Layout, class Weights>
__device__ __forceinline__ int topic_in_units(const Weights& weight_at, const unsigned char* slots, uint32_t unit, int n_units,
                                              int o, float w_o, double y) {
    const int o_key = Layout::key_of_topic(o);
    bool own_before = false;
    double acc = 0.0;
    int found = -1, last = -1;
    for (int c = 0; c < n_units && found < 0; ++c) {
        const uint4 raw = *reinterpret_cast<const uint4*>(slots + ((size_t)unit + (size_t)c) * 16u);
#pragma unroll
        for (int j = 0; j < Layout::kUnitEntries; ++j) {
            const int key = Layout::key(raw, j);
            const bool own = key == o_key, first = own && !own_before;
            own_before = own_before || own;
            const double before = acc;
            acc = fma((double)(Layout::count(raw, j) - (first ? 1 : 0)), (double)(own ? w_o : weight_at((uint32_t)key)), acc);
            if (acc > before || last < 0) last = key;
            if (found < 0 && acc > y) found = key;
        }
    }
    return (found >= 0 ? found : last) >> 2;
}

// Rows too long for the kept shapes, one per wave (sub-lane = lane): one walk for the sums, a
// second one over the hit lane's entries.  Lane l owns the units [n l, n (l + 1)).
template <class Layout, class Weights>
__device__ __forceinline__ void row_pass_long(const Weights& weight_at, const unsigned char* slots, TokenRec* rec,
                                              int lane) {
    constexpr int UE = Layout::kUnitEntries;
    const RowCtx r = row_ctx(rec);
    const int n_units = rec->nnz, n = (n_units + kWave - 1) / kWave;
    const int u0 = lane * n;
    // the entry before the lane's first one (lanes past the row's end have no entries at all)
    const bool own_before = u0 < n_units &&
        key_before_unit<Layout>(slots + ((size_t)r.off + 1u + (size_t)u0) * 16u) == r.o_key;
    uint64_t prev_own = __ballot(own_before);
    double acc = 0.0;
    for (int c = 0; c < n; ++c)
        unit_sum<Layout>(weight_at, load_unit(slots, r.off, u0 + c, u0 + c < n_units), r.o_key, r.w_o, prev_own,
                         acc);
    const RowDraw d = row_draw<kWave>(acc, rec, lane, lane);
    if (__ballot(d.hit) != 0) {
        bool found = false;
        int k_sel = 0, last_k = 0;
        prev_own = __ballot(own_before);
        acc = 0.0;
        for (int c = 0; c < n; ++c) {
            double sums[UE];
            int keys[UE];
            const double before_unit = acc;
            unit_prefix_sums<Layout>(weight_at, load_unit(slots, r.off, u0 + c, d.hit && u0 + c < n_units),
                                     r.o_key, r.w_o, prev_own, acc, sums, keys);
#pragma unroll
            for (int j = 0; j < UE; ++j) {
                const double before = (j == 0) ? before_unit : sums[j - 1];
                if (!found && sums[j] > d.y) { k_sel = keys[j] >> 2; found = true; }
                if (sums[j] > before) last_k = keys[j] >> 2;
            }
        }
        if (d.hit) {
            rec->off = (uint32_t)(found ? k_sel : last_k);
            rec->nnz = kDrawTopic;
        }
    }
    record_dense(rec, lane, d);
}

template <int kValue> using Int = std::integral_constant<int, kValue>;

// How a launch's workgroups meet its tiles.  once: a workgroup per tile.  queued: as many workgroups as the chip holds, each
// of which takes tiles until there are none left; the small ones (from n_single on) come last, and p* of a small one is made
// from that of the small one before.  split: the same where K is too large for p* to fit a workgroup's LDS: p* of the topics
// that do not fit then lives in the workgroup's own strip of device memory.
enum class Form { once, queued, split };

// kNear: every byte of the slot buffer has a 32-bit offset; a pass then finds its units with
// 32-bit arithmetic (one offset per lane, the unit's place in the load's own offset field).
template <int kWaves, class Layout, Form kForm = Form::once, bool kNear = false>
// Six waves per SIMD (80 VGPRs), five (96) with fp64 weights: the walk hides HBM latency by occupancy as
// well as by the early loads.
// (A workgroup of sixteen waves has a CU for itself.)
__attribute__((amdgpu_waves_per_eu(kWaves == 16 ? 4 : Layout::kWavesPerSimd)))
__global__ __launch_bounds__(kWaves * kWave) void sample_kernel(const SampleArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr bool kFar = kForm == Form::split, kQueue = kForm != Form::once;
    constexpr int kGroup = dense_group(kWaves, kFar);
    stamp_start(a.started);
    const int K = a.K, Kpad = a.Kpad, ng = Kpad / kGroup;
    constexpr bool kDouble = Layout::kDoubleWeights;
    static_assert(!(kDouble && (kFar || kWaves > 4)), "fp64 weights: workgroups of up to four waves, in LDS");
    typedef typename std::conditional<kDouble, double, float>::type Weight;
    // (what a staged weight, and a sum over a row, carry as a factor)
    constexpr double kStagedScale = kDouble ? kWeightScale : 1.0, kRowScale = kDouble ? kSumScale : 1.0;
    const size_t pstar_lds = kFar ? (size_t)(a.near_topics + 4) * 4 : (size_t)Kpad * sizeof(Weight);
    Weight* pstar = reinterpret_cast<Weight*>(lds);
    // (by topic: strip[near_topics] is the first of its own)
    [[maybe_unused]] float* strip = kFar ? a.far_pstar + (size_t)blockIdx.x * far_strip_cells(Kpad, a.near_topics) + kFarFirst - a.near_topics : nullptr;
    double* cp = reinterpret_cast<double*>(lds + pstar_lds);
    const int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);      // wave-uniform, in an SGPR
    constexpr bool kShares = Layout::kShares;
    unsigned char* wave_base = lds + pstar_lds + (size_t)((ng + 1) & ~1) * 8 + (kShares || kQueue ? 16 : 0);
    const int wave_bytes = kShares ? sample_wave_bytes(a.kept_passes, a.kept_sums) : kWave * (int)sizeof(TokenRec);
    TokenRec* my_rec = reinterpret_cast<TokenRec*>(wave_base + wave * wave_bytes);
    typedef typename std::conditional<kFar, SplitWeights, LdsWeights>::type Weights;
    [[maybe_unused]] Weights weight_at;
    if constexpr (kFar) {
        weight_at.strip = reinterpret_cast<const unsigned char*>(strip);
        weight_at.near_key = (uint32_t)a.near_topics << 2;
        if (tid < 4) {                  // (no topic is staged in these places)
            pstar[a.near_topics + tid] = 0.f;
            strip[a.near_topics - 4 + tid] = 0.f;
        }
    }
    // p*(k) of the tile's word: put, read, and read four at a time without its scale (k a multiple of 4)
    auto put_cell = [&](int k, Weight w) {
        if (kFar && k >= a.near_topics) strip[k] = (float)w;
        else pstar[k] = w;
    };
    auto cell = [&](int k) -> Weight {
        if constexpr (kFar) return weight_at((uint32_t)k << 2);
        else return pstar[k];
    };
    auto four_cells = [&](int k) {
        if constexpr (kDouble) {
            return make_double4(plain_weight(pstar[k]), plain_weight(pstar[k + 1]), plain_weight(pstar[k + 2]), plain_weight(pstar[k + 3]));
        } else {
            float4 w = *reinterpret_cast<const float4*>(pstar + (kFar ? min(k, a.near_topics) : k));
            if constexpr (kFar) {
                const float4 f = *reinterpret_cast<const float4*>(strip + max(k, a.near_topics - 4));
                w.x += f.x; w.y += f.y; w.z += f.z; w.w += f.w;
            }
            return make_double4((double)w.x, (double)w.y, (double)w.z, (double)w.w);
        }
    };
    auto group_total = [&](int g) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < kGroup; j += 4) {
            const double4 w = four_cells(g * kGroup + j);
            s += w.x; s += w.y; s += w.z; s += w.w;
        }
        return s;
    };

    double* group_sum = reinterpret_cast<double*>(wave_base + (size_t)kWaves * wave_bytes);
    uint32_t* changed = reinterpret_cast<uint32_t*>(group_sum + ((ng + 1) & ~1));
    if (kQueue) {
        for (int w = tid; w < (ng + 31) / 32; w += kWaves * kWave) changed[w] = 0u;
    }
    // Shared walks: no weight of the tile's word is less than the fp32 number with these bits (see row_sums.hpp; bits of
    // numbers that are not negative are in the numbers' order).  Every wave notes its own least in the LDS of its records;
    // the second one collects them while the first adds up the groups' sums.
    [[maybe_unused]] uint32_t* least = reinterpret_cast<uint32_t*>(wave_base) - 4;
    auto note_least = [&](uint32_t v) {
        if constexpr (kShares) {
            v = wave_min_at_last(v);
            if (lane == kWave - 1) *(kWaves == 1 ? least : reinterpret_cast<uint32_t*>(my_rec)) = v;
        }
    };
    auto collect_least = [&](bool beside) {         // (beside: of the words before in the run, too)
        if constexpr (kShares && kWaves > 1) {
            uint32_t v = 0xffffffffu;
            if (lane < kWaves) v = *reinterpret_cast<const uint32_t*>(wave_base + lane * wave_bytes);
            v = wave_min_at_last(v);
            if (lane == kWave - 1) *least = beside ? min(v, *least) : v;
        }
    };
    [[maybe_unused]] int last_ti = -1;          // kQueue: the tile before
    for (int ti = (int)blockIdx.x;;) {
    const bool small = kQueue && ti >= a.n_single, follows = small && last_ti >= a.n_single;
    // The inclusive prefix over the groups' sums, 64 at a time (chunks of a wave's lanes, then the chunks before).  Where there are
    // more than four chunks the waves scan them side by side, with the same additions in the same order: a tile of few
    // tokens waits for little else.  One wave / all, sampling launch: 5e5 tokens, 20,000 words, K = 20,000 584 / 503 us, 3e6,
    // K = 12,000 1,232 / 1,131; with two or three chunks (K < 4,096) the second barrier costs what it saves.
    auto add_up_groups = [&](const double* sums, bool beside) {
        const int n_chunks = (ng + kWave - 1) / kWave;
        if (!kQueue || n_chunks <= 4) {
            if (wave == 0) {
                double carry = 0.0;
                for (int base = 0; base < ng; base += kWave) {
                    const int g = base + lane;
                    double x = (g < ng) ? sums[g] : 0.0;
                    x = wave_inclusive_sum(x) + carry;
                    if (g < ng) cp[g] = x;
                    carry = read_lane(x, kWave - 1);
                }
            } else if (wave == 1) {
                collect_least(beside);
            }
            __syncthreads();
            return;
        }
        // (in the records of a wave that are not in use yet, behind its least weight)
        double* totals = reinterpret_cast<double*>(wave_base + 3 * wave_bytes + 64);
        for (int c = wave; c < n_chunks; c += kWaves) {
            const int g = c * kWave + lane;
            const double x = wave_inclusive_sum((g < ng) ? sums[g] : 0.0);
            if (g < ng) cp[g] = x;
            if (lane == kWave - 1) totals[c] = x;
        }
        if (wave == 1) collect_least(beside);
        __syncthreads();
        for (int c = wave; c < n_chunks; c += kWaves) {
            double carry = 0.0;
            for (int i = 0; i < c; ++i) carry = totals[i] + carry;
            const int g = c * kWave + lane;
            if (g < ng) cp[g] = cp[g] + carry;
        }
        __syncthreads();
    };
    Tile tl = a.tiles[ti];                 // the same for every lane: keep it in SGPRs
    tl.word = __builtin_amdgcn_readfirstlane(tl.word);
    tl.begin = __builtin_amdgcn_readfirstlane(tl.begin);
    tl.count = __builtin_amdgcn_readfirstlane(tl.count);
    // the word's row of phi: 16-bit or 32-bit cells, the same for the whole workgroup
    const int wide_row = __builtin_amdgcn_readfirstlane(tl.whole);    // (kept in the tile: one load less in the chain)
    const bool wide = wide_row >= 0;
    const unsigned char* phi_cells = wide ? reinterpret_cast<const unsigned char*>(a.phi.wide)
                                          : reinterpret_cast<const unsigned char*>(a.phi.narrow);
    const size_t phi_cell0 = (size_t)(wide ? wide_row : tl.word) * (size_t)K;
    const uint32_t phi_shift = wide ? 2u : 1u, phi_mask = wide ? 0xffffffffu : 0xffffu;

    if (kQueue && follows) {
        const Tile prev = a.tiles[last_ti];
        const int prev_begin = __builtin_amdgcn_readfirstlane(prev.begin);
        const int prev_count = __builtin_amdgcn_readfirstlane(prev.count);
        // ---- p* of the previous word becomes p* of this one.  Both words have all their
        // tokens in their tile, so a cell of phi is non-zero exactly for the topics of the
        // tile's tokens: only those cells differ from beta / (n_k + beta V).  Every changed cell
        // gets the value a fresh staging would give it, and the sums of the groups that hold
        // one are added up again in the same order, so the result is the fresh staging's, bit
        // for bit.  (The least weight so far stays a bound: a cell that changes counts with every value it is given.)
        uint32_t my_least = 0xffffffffu;
        for (int idx = tid; idx < prev_count; idx += kWaves * kWave) {
            const int k = (int)a.z_cur[prev_begin + idx];
            const float w = (float)((0.0 + a.beta) / ((double)a.n_k[k] + a.beta_V));
            put_cell(k, w);
            my_least = min(my_least, __float_as_uint(w));
            atomicOr(&changed[(k / kGroup) >> 5], 1u << ((k / kGroup) & 31));
        }
        __syncthreads();
        const uint16_t* phi_v = reinterpret_cast<const uint16_t*>(phi_cells) + phi_cell0;   // (never a wide row)
        for (int idx = tid; idx < tl.count; idx += kWaves * kWave) {
            const int k = (int)a.z_cur[tl.begin + idx];
            const float w = (float)(((double)phi_v[k] + a.beta) / ((double)a.n_k[k] + a.beta_V));
            put_cell(k, w);
            my_least = min(my_least, __float_as_uint(w));
            atomicOr(&changed[(k / kGroup) >> 5], 1u << ((k / kGroup) & 31));
        }
        note_least(my_least);
        __syncthreads();
        for (int g = tid; g < ng; g += kWaves * kWave)
            if ((changed[g >> 5] >> (g & 31)) & 1u) group_sum[g] = group_total(g);
        __syncthreads();
        if (wave == 3)
            for (int w = lane; w < (ng + 31) / 32; w += kWave) changed[w] = 0u;
        add_up_groups(group_sum, true);
    } else {
    // ---- stage p*(k) = (phi_kv + beta)/(n_k + beta V) as fp32 (Eq. 8)
    uint32_t my_least = 0xffffffffu;
    if (wide) {
        const int32_t* phi_v = reinterpret_cast<const int32_t*>(phi_cells) + phi_cell0;
        for (int k = tid; k < Kpad; k += kWaves * kWave) {
            float w = 0.f;
            if (k < K) {
                w = (float)(((double)phi_v[k] + a.beta) / ((double)a.n_k[k] + a.beta_V));
                my_least = min(my_least, __float_as_uint(w));
            }
            put_cell(k, (Weight)(kStagedScale * (double)w));
        }
    } else {
        const uint16_t* phi_v = reinterpret_cast<const uint16_t*>(phi_cells) + phi_cell0;
        for (int k = tid; k < Kpad; k += kWaves * kWave) {
            float w = 0.f;
            if (k < K) {
                w = (float)(((double)phi_v[k] + a.beta) / ((double)a.n_k[k] + a.beta_V));
                my_least = min(my_least, __float_as_uint(w));
            }
            put_cell(k, (Weight)(kStagedScale * (double)w));
        }
    }
    note_least(my_least);
    __syncthreads();
    for (int g = tid; g < ng; g += kWaves * kWave) {
        const double s = group_total(g);
        cp[g] = s;
        if (small) group_sum[g] = s;
    }
    __syncthreads();
    add_up_groups(cp, false);
    }

    // a pass shape's lane geometry: token of the lane relative to the pass's first, the lane's
    // place inside its group, its first unit of entries
    int geo_shape = -1, geo_rel = 0, geo_sl = 0, geo_q0 = 0;
    // A wave takes up to 64 tokens at a time.  A tile too small to give every wave such a batch
    // is dealt out in smaller batches, so that all waves work on it side by side: the passes
    // of one batch follow each other, each waiting for its rows.
    // (Full batches are less work in all, which is what counts where the chip is full; at K > 2048,
    // and where there are few tiles, it is the time of one tile.)
    const int batch = min(kWave, max(kWaves <= 4 ? a.min_batch : kMinBatch,
                                     ((tl.count + kWaves - 1) / kWaves + 3) & ~3));
    const int n_batches = (tl.count + batch - 1) / batch;
    [[maybe_unused]] int kept_own = 0;     // tokens of the wave's last shared batch that walked by themselves: with many, the rest do not share in vain
    for (int b = wave; b < n_batches; b += kWaves) {
        // ---- one token per lane: token, uniform, own-count correction
        const int idx = b * batch + lane;
        const bool valid = lane < batch && idx < tl.count;
        TokenRec mine;
        mine.off = 0; mine.nnz = 0; mine.o = 0; mine.w_o = 0.f; mine.u = 0.0; mine.Qp = 0.0;
        double delta = 0.0;
        // What the per-token phases read of the kernel's arguments is fetched from the argument
        // block again in every batch (scalar loads) instead of being kept in scalar registers
        // through the passes: there are not enough of those, and what does not fit is parked in
        // lanes of a vector register, every read of which takes a vector issue slot.
        // (SampleArgs is the kernel's only parameter, so the argument block starts with it.)
        typedef __attribute__((address_space(4))) const SampleArgs* ArgsPtr;
        ArgsPtr ka = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(ka));
        if (valid) {
            // (the tile's part of every per-token array starts at a scalar base)
            mine.off = load_at<uint32_t>(ka->tok_slot + tl.begin, (uint32_t)idx << 2);
            mine.o = (int)load_at<uint16_t>(ka->z_cur + tl.begin, (uint32_t)idx << 1);
            const uint64_t id = (uint64_t)load_at<uint32_t>(ka->tok_id + tl.begin, (uint32_t)idx << 2);
            // the row's length sits in front of its entries: this read also brings the row's
            // first line on its way
            const uint32_t entries = kNear ? load_at<uint32_t>(a.slots, mine.off << 4)
                                           : *reinterpret_cast<const uint32_t*>(a.slots + (size_t)mine.off * 16u);
            mine.nnz = (int)((entries + (uint32_t)(Layout::kUnitEntries - 1)) / (uint32_t)Layout::kUnitEntries);
            // (the seed too: the ten rounds' keys are then made where they are used, by the scalar
            // unit, and not once per kernel)
            mine.u = token_uniform(ka->seed, ka->iter, id);
            // the token itself is taken out of phi and n_k at its own topic
            // (its cell of phi, of either width, is cut out of the aligned dword that holds it)
            const size_t row_byte = phi_cell0 << phi_shift;        // the word's row: scalar
            const uint32_t own_byte = ((uint32_t)row_byte & 3u) + ((uint32_t)mine.o << phi_shift);
            const uint32_t own_dword = load_at<uint32_t>(phi_cells + (row_byte & ~(size_t)3), own_byte & ~3u);
            const int32_t phi_own = (int32_t)((own_dword >> ((own_byte & 2u) << 3)) & phi_mask);
            mine.w_o = (float)(((double)(phi_own - 1) + ka->beta) /
                               ((double)(ka->n_k[mine.o] - 1) + ka->beta_V));
            delta = (double)mine.w_o - plain_weight(cell(mine.o));
            // cp[ng - 1] = sum_k p*(k), read from LDS where it is needed; Q = alpha sum (Eq. 7)
            mine.Qp = ka->alpha * (cp[ng - 1] + delta);
        }
        // Which rows of the batch (tokens, or rows that tokens share) are beyond each of the pass shapes'
        // lengths: the shape of every pass follows from these masks.
        //   0 (4,1)   1 (4,2)   2 (4,3)   3 (8,2)   4 (8,3)   5 (16,2)   6 (16,3)
        //   7 (32,2)   8 (32,3)   9 (64,2)   10 (64,3)   11 = one longer row
        // (lanes per row, units per lane: a row may have up to lanes * units * (entries per unit) entries)
        static_assert(kKeptUnits == 3, "the pass shapes assume three kept units per lane");
        uint64_t over_4_1, over_4_2, over_4_3, over_8_2, over_8_3, over_16_2, over_16_3, over_32_2, over_32_3, over_64_2, over_64_3;
        auto learn_shapes = [&](int units) {
            over_4_1 = __ballot(units > 4); over_4_2 = __ballot(units > 8);
            over_4_3 = __ballot(units > 12); over_8_2 = __ballot(units > 16);
            over_8_3 = __ballot(units > 24); over_16_2 = __ballot(units > 32);
            over_16_3 = __ballot(units > 48); over_32_2 = __ballot(units > 64);
            over_32_3 = __ballot(units > 96); over_64_2 = __ballot(units > 128);
            over_64_3 = __ballot(units > 192);
        };
        auto any = [](uint64_t mask, int t0, uint32_t window) {      // 1 if a row of the window is set
            const uint32_t w = (uint32_t)(mask >> t0) & window;
            return min(1, (int)__builtin_popcount(w));      // stays scalar arithmetic
        };
        auto shape_at = [&](int t0) {
            if (!any(over_4_3, t0, 0xffffu)) return any(over_4_1, t0, 0xffffu) + any(over_4_2, t0, 0xffffu);
            if (!any(over_8_3, t0, 0xffu)) return 3 + any(over_8_2, t0, 0xffu);
            if (!any(over_16_3, t0, 0xfu)) return 5 + any(over_16_2, t0, 0xfu);
            if (!any(over_32_3, t0, 0x3u)) return 7 + any(over_32_2, t0, 0x3u);
            if (!any(over_64_3, t0, 0x1u)) return 9 + any(over_64_2, t0, 0x1u);
            return 11;
        };
        constexpr int kNoPass = 12;
        auto lanes_log2 = [](int shape) { return (int)((0x666554433222ull >> (4 * shape)) & 0xfull); };
        auto units_of = [](int shape) { return (int)((0x032323232321ull >> (4 * shape)) & 0xfull); };
        auto place_lanes = [&](int shape) {     // the lanes' places change only with the shape
            if (shape == geo_shape) return;
            const int lg = lanes_log2(shape);
            const int g = lg < 4 ? 4 - lg : 0, hs = lg < 4 ? 4 : lg;    // interleave, run length
            geo_shape = shape;
            geo_rel = ((lane >> hs) << g) | (lane & ((1 << g) - 1));
            geo_sl = (lane & ((1 << hs) - 1)) >> g;
            geo_q0 = geo_sl * units_of(shape);        // the lane's first unit
        };

        // ---- one token per lane at last: the entry inside the unit that holds the draw, or the
        // dense bucket; store
        auto finish = [&](int found, int kind, int o, float w_o, double u, double Qp) {
            int z_new = found;
            if (kind == kDrawInUnit) {
                if constexpr (kDouble)
                    z_new = topic_in_unit_double<Layout, kNear>(a.slots, (uint32_t)found, o, w_o, u);
                else
                    z_new = topic_in_unit<Layout, kNear>(weight_at, a.slots, (uint32_t)found, o << 2, w_o, u);
            }
            if (kind == kDrawDense) {
                double y = u * (1.0 / kRowScale);
                if (kDouble && __builtin_expect(Qp < kSmallestScaled, 0))
                    y = Qp * token_uniform(ka->seed, ka->iter,
                                           (uint64_t)load_at<uint32_t>(ka->tok_id + tl.begin, (uint32_t)(b * batch + lane) << 2));
                z_new = dense_bucket_search<kGroup>(four_cells, cp, K, ng, ka->alpha, y, o,
                                                    w_o, (double)w_o - plain_weight(cell(o)));
            }
            store_at<uint16_t>(ka->z_next + tl.begin, (uint32_t)(b * batch + lane) << 1, (uint16_t)z_new);
        };

        // ---- Tokens of one document and word stand next to each other and walk the same row with the same
        // p*: where rows are shared, a row is walked once for all its tokens of the batch.  The sums at the
        // ends of its units go to LDS, and each token, one per lane, then finds its topic among the row's
        // sub-lanes, counts it, corrects the sums from there on and looks its draw up among them.
        // Sums that hold no rounding are what a walk of the token's own would have found, to the last bit, and so is the
        // draw.  Tokens whose row's sum is too large for that (weights of the row far apart; at beta = 0.01 next to none), and those
        // with their topic spread over several units, take that walk below.
        bool in_rest = valid, shared = false;
        // (lane 0 is given slot 0, which no document has)
        const bool head = valid && mine.off != (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine.off, 0x138, 0xf, 0xf, true);
        const uint64_t heads = kShares ? __ballot(head) : 0;
        const int n_rows = __popcll(heads);
        // Sums whose upper dword is less are exact (with w_o in the place of p*(o), too)
        auto exact_below = [&]() {
            // (the address is made here, every time: hoisted, it would hold a register for good)
            int at = (int)(reinterpret_cast<unsigned char*>(least) - lds);
            asm volatile("" : "+v"(at));
            const uint32_t smallest = min(*reinterpret_cast<const uint32_t*>(lds + at), __float_as_uint(mine.w_o));
            return exact_sums_below(smallest, kDouble ? kSumScaleLog2 : 0);
        };
        // Sharing costs a search per token among its row's sums and a wait for units of the row, once for every
        // time that the kept sums fill up; it saves the walks that are not made, and a quarter of each that
        // is.  So: at most two rows for three tokens, and two passes saved.  Sampling
        // launch, ms, no sharing / rows up to 16 of 16, 16 of 20, 16 of 24 (and two passes saved):
        //   9.9e7 tokens, K = 1,000, late       6.26   6.04   5.16   5.16      1.8e8, K = 1,000   7.47   8.20   7.15   7.14
        //   6.3e6, K = 1,537                    0.62   0.78   0.55   0.55      1e6, K = 128      0.058  0.071  0.056  0.056
        //   8.6e6, documents of 30,000, K = 299 1.42   0.53   0.47   0.47      1e5, K = 32       12.3us 16.0   12.4   12.4
        //   1.2e7, documents of 4,000, K = 2,000 5.76  5.36   3.93   3.87
        // Rows of up to 8 units (late in training, or few topics) take so short a pass that the search is the larger part: only
        // where one pass stands for four.  2e7 tokens late in training, us, two passes saved / with this:
        //   K = 80, documents of 92, 769 words   860  757 (684 without sharing, in tiles of 1,024)       20,000 words  629  604
        //   K = 200, documents of 92, 800 words  626  603     K = 80, documents of 300  546  548     K = 24, of 2,000  432  433
        auto share_walks = [&]() {
            const int n = min(batch, tl.count - b * batch);
            if (kDouble && a.kept_passes == 0) return false;
            if (4 * kept_own > kWave || 3 * n_rows > 2 * n || (kDouble && __ballot(mine.nnz > kMostKeptUnits) != 0)) return false;
            const int rows_per_pass = __ballot(mine.nnz > 12) == 0 ? 16 : __ballot(mine.nnz > 24) == 0 ? 8 : __ballot(mine.nnz > 48) == 0 ? 4 : 1;
            const int least_saved = kDouble && __ballot(mine.nnz > 8) == 0 ? 13 : 8;
            return 4 * n - 3 * n_rows >= least_saved * rows_per_pass;
        };
        if constexpr (kDouble) if (share_walks()) {
            in_rest = false;
            shared = true;
            double* sums = reinterpret_cast<double*>(my_rec);
            uint16_t* first_topic = reinterpret_cast<uint16_t*>(sums + a.kept_sums);
            uint32_t* row_slot = reinterpret_cast<uint32_t*>(first_topic + a.kept_passes * kWave);
            unsigned char* row_units = reinterpret_cast<unsigned char*>(row_slot + kWave);
            const int row = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(heads >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)heads, 0u)) +
                            (head ? 0 : -1);
            if (head) {
                row_slot[row] = mine.off;
                row_units[row] = (unsigned char)mine.nnz;
            }
            int at = lane;              // (addresses made here, every time: hoisted, they would hold registers for good)
            asm volatile("" : "+v"(at));
            if (at >= n_rows) {
                row_slot[at] = 0;
                row_units[at] = 0;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            learn_shapes((int)row_units[at]);
            auto request = [&](int t0, int shape, uint4* raw, bool live) {
                place_lanes(shape);
                const int r = min(t0 + geo_rel, kWave - 1);
                const uint32_t off = row_slot[r];
                const int n_mine = live ? min((int)row_units[r] - geo_q0, units_of(shape)) : 0;
                if constexpr (kNear) {
                    const uint32_t row_bytes = (off + 1u + (uint32_t)geo_q0) << 4;
#pragma unroll
                    for (int c = 0; c < kKeptUnits; ++c) raw[c] = load_unit_near(a.slots, row_bytes, c, c < n_mine);
                } else {
#pragma unroll
                    for (int c = 0; c < kKeptUnits; ++c) raw[c] = load_unit(a.slots, off, geo_q0 + c, c < n_mine);
                }
            };
            uint4 raw_next[kKeptUnits];
            int t_next = 0, shape_next = shape_at(0);
            request(0, shape_next, raw_next, true);
            do {                // as many passes as there is room for, then the tokens of their rows
                const int row0 = t_next;
                int n_passes = 0, n_sums = 0, most_lanes = 4;
                do {
                    const int shape = shape_next, rel = geo_rel, sl = geo_sl, t0 = t_next;
                    uint4 raw[kKeptUnits];
#pragma unroll
                    for (int c = 0; c < kKeptUnits; ++c) raw[c] = raw_next[c];
                    const int lanes = 1 << lanes_log2(shape), nu = units_of(shape);
                    t_next += kWave / lanes;
                    most_lanes = max(most_lanes, lanes);
                    const int t_req = min(t_next, kWave - 1);
                    shape_next = shape_at(t_req);
                    request(t_req, shape_next, raw_next, t_next < n_rows);
                    double* s = sums + n_sums;
                    uint16_t* ft = first_topic + n_passes * kWave;
                    switch (shape) {
                    case 0: row_pass_shared<Layout, 4, 1>(s, ft, rel, sl, raw); break;
                    case 1: row_pass_shared<Layout, 4, 2>(s, ft, rel, sl, raw); break;
                    case 2: row_pass_shared<Layout, 4, 3>(s, ft, rel, sl, raw); break;
                    case 3: row_pass_shared<Layout, 8, 2>(s, ft, rel, sl, raw); break;
                    case 4: row_pass_shared<Layout, 8, 3>(s, ft, rel, sl, raw); break;
                    case 5: row_pass_shared<Layout, 16, 2>(s, ft, rel, sl, raw); break;
                    case 6: row_pass_shared<Layout, 16, 3>(s, ft, rel, sl, raw); break;
                    case 7: row_pass_shared<Layout, 32, 2>(s, ft, rel, sl, raw); break;
                    case 8: row_pass_shared<Layout, 32, 3>(s, ft, rel, sl, raw); break;
                    case 9: row_pass_shared<Layout, 64, 2>(s, ft, rel, sl, raw); break;
                    case 10: row_pass_shared<Layout, 64, 3>(s, ft, rel, sl, raw); break;
                    }
                    // where the row's sums are | its first sub-lane's place | units per lane | log2 of its lanes
                    if (sl == 0 && t0 + rel < n_rows)
                        row_slot[t0 + rel] = (uint32_t)(n_sums + rel * lanes * nu) | (uint32_t)(n_passes * kWave + rel * lanes) << 12 |
                                             (uint32_t)nu << 24 | (uint32_t)lanes_log2(shape) << 28;
                    ++n_passes;
                    n_sums += kWave * nu;
                } while (t_next < n_rows && n_passes < a.kept_passes && n_sums + kWave * units_of(shape_next) <= a.kept_sums);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                if (valid && row >= row0 && row < t_next) {
                    const uint32_t info = row_slot[row];
                    const int lane0 = (int)((info >> 12) & 0xfffu), nu = (int)((info >> 24) & 3u), lanes = 1 << (info >> 28);
                    const double* row_sums = sums + (info & 0xfffu);
                    const int n_units = mine.nnz, o = mine.o;
                    // the last sub-lane whose first topic is not above o
                    int holder = 0;
                    for (int step = most_lanes >> 1; step > 0; step >>= 1) {
                        const int at = min(holder + step, lanes - 1);
                        if (holder + step < lanes && (int)first_topic[lane0 + at] <= o) holder = at;
                    }
                    // its units: where o is, and o's tokens
                    const int q0 = holder * nu;
                    uint32_t n_to[kKeptUnits], n_o = 0;
                    uint4 held[kKeptUnits];
#pragma unroll
                    for (int c = 0; c < kKeptUnits; ++c) held[c] = load_unit(a.slots, mine.off, q0 + c, c < nu && q0 + c < n_units);
#pragma unroll
                    for (int c = 0; c < kKeptUnits; ++c) {
                        Layout::count_own(held[c], o, n_o);
                        n_to[c] = n_o;
                    }
                    const int c_o = n_to[0] > 0 ? 0 : n_to[1] > 0 ? 1 : 2;
                    if ((n_to[0] > 0 ? n_to[0] : n_to[1] > 0 ? n_to[1] : n_to[2]) != n_o) in_rest = true;
                    if (holder > 0 && (int)first_topic[lane0 + holder] == o &&
                        key_before_unit<Layout>(a.slots + ((size_t)mine.off + 1u + (size_t)q0) * 16u) == Layout::key_of_topic(o))
                        in_rest = true;
                    const double w_o = kWeightScale * (double)mine.w_o;
                    const double shift = fma(__hiloint2double((int)n_o - 1, 0), w_o,
                                             -(__hiloint2double((int)n_o, 0) * (double)pstar[o]));
                    const double S_all = row_sums[lanes * nu - 1];
                    const double S = S_all + shift, total = fma(mine.Qp, kSumScale, S);
                    const uint32_t below = exact_below(), sum_hi = (uint32_t)__double2hiint(S_all);
                    const bool exact = sum_hi < below;
                    if (!exact && !(sum_hi < below + a.sum_slack && S_all <= kNearlyAll * total)) in_rest = true;
                    if (!(mine.Qp >= kSmallestScaled)) in_rest = true;
                    const double x = mine.u * total;
                    int sub = 0;            // sub-lanes known to lie before the draw
                    double before = 0.0;
                    for (int step = most_lanes; step > 0; step >>= 1) {
                        const int upto = sub + step;
                        if (upto <= lanes) {
                            const double e = row_sums[upto * nu - 1] + (upto > holder ? shift : 0.0);
                            if (!(e > x)) { sub = upto; before = e; }
                        }
                    }
                    sub = min(sub, lanes - 1);      // (the last sum is S: above x, if the draw is in the row)
                    const double y = x - before;
                    int c_x = 0;
                    double base = 0.0;
                    const int c_shift = sub == holder ? c_o : kKeptUnits;       // its units from here on have the correction in their sums
                    const double* unit_sums = row_sums + sub * nu;
#pragma unroll
                    for (int c = 0; c + 1 < kKeptUnits; ++c) {
                        if (c_x == c && c + 1 < nu) {
                            const double e = unit_sums[c] + (c >= c_shift ? shift : 0.0);
                            if (!(e > y)) { c_x = c + 1; base = e; }
                        }
                    }
                    // (sums that round may leave the draw a last unit without weight)
                    if (!exact && c_x + 1 == nu && !(row_sums[sub * nu + nu - 1] + (sub >= holder ? shift : 0.0) - before > base))
                        in_rest = true;
                    if (!in_rest) {
                        const bool sparse = x < S;
                        mine.nnz = sparse ? kDrawInUnit : kDrawDense;
                        mine.off += 1u + (uint32_t)min(sub * nu + c_x, n_units - 1);
                        mine.u = sparse ? y - base : x - S;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            } while (t_next < n_rows);
            if (valid && !in_rest) finish((int)mine.off, mine.nnz, mine.o, mine.w_o, mine.u, mine.Qp);
        }
        if constexpr (kShares && !kDouble) if (share_walks()) {
            // The same with a sum per sub-lane: a unit has four entries here, and a token looks through the units of
            // its sub-lane itself.  Rows of any length: beyond the kept shapes a lane of the whole wave owns as many
            // units as it takes, read in threes.  Sampling launch, random topics, before / after:
            //   1.5e5 tokens in documents of 3,000, K = 4,983   4.28 / 0.97 ms     5e6 of 286, K = 2,218    0.84 / 0.49 ms
            //   9.9e7 of 330, K = 10,000                        39.3 / 32.6        2e6 of 250, K = 40,000   4.38 / 3.75
            in_rest = false;
            shared = true;
            double* sums = reinterpret_cast<double*>(my_rec);
            uint16_t* first_topic = reinterpret_cast<uint16_t*>(sums + a.kept_passes * kWave);
            uint32_t* row_slot = reinterpret_cast<uint32_t*>(first_topic + a.kept_passes * kWave);
            uint16_t* row_units = reinterpret_cast<uint16_t*>(row_slot + kWave);
            const int row = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(heads >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)heads, 0u)) +
                            (head ? 0 : -1);
            if (head) {
                row_slot[row] = mine.off;
                row_units[row] = (uint16_t)mine.nnz;
            }
            int at = lane;              // (addresses made here, every time: hoisted, they would hold registers for good)
            asm volatile("" : "+v"(at));
            if (at >= n_rows) {
                row_slot[at] = 0;
                row_units[at] = 0;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            learn_shapes((int)row_units[at]);
            int t_next = 0, scan_units = 0;
            do {                // as many passes as there is room for, then the tokens of their rows
                const int row0 = t_next;
                int n_passes = 0, most_lanes = 4, most_units = 1;
                do {
                    const int shape = shape_at(t_next), t0 = t_next;
                    place_lanes(shape);
                    const int lanes = 1 << lanes_log2(shape);
                    const int r = min(t0 + geo_rel, kWave - 1);
                    const uint32_t off = row_slot[r];
                    const int n_units = (int)row_units[r];
                    const int nu = shape < 11 ? units_of(shape) : __builtin_amdgcn_readfirstlane((n_units + kWave - 1) / kWave);
                    const int q0 = geo_sl * nu;
                    t_next += kWave / lanes;
                    most_lanes = max(most_lanes, lanes);
                    most_units = max(most_units, nu);
                    double* s = sums + n_passes * kWave;
                    uint16_t* ft = first_topic + n_passes * kWave;
                    uint4 raw[kKeptUnits];
#pragma unroll
                    for (int c = 0; c < kKeptUnits; ++c) raw[c] = load_unit(a.slots, off, q0 + c, c < nu && q0 + c < n_units);
                    switch (shape) {
                    case 0: row_pass_lanes<Layout, 4, 1>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 1: row_pass_lanes<Layout, 4, 2>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 2: row_pass_lanes<Layout, 4, 3>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 3: row_pass_lanes<Layout, 8, 2>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 4: row_pass_lanes<Layout, 8, 3>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 5: row_pass_lanes<Layout, 16, 2>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 6: row_pass_lanes<Layout, 16, 3>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 7: row_pass_lanes<Layout, 32, 2>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 8: row_pass_lanes<Layout, 32, 3>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 9: row_pass_lanes<Layout, 64, 2>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    case 10: row_pass_lanes<Layout, 64, 3>(weight_at, s, ft, geo_rel, geo_sl, raw); break;
                    default: {
                        ft[lane] = (uint16_t)Layout::entry_topic((typename Layout::Entry)raw[0].x);
                        double acc = 0.0;
                        for (int c0 = 0; c0 < nu; c0 += kKeptUnits) {
                            uint4 ahead[kKeptUnits];
#pragma unroll
                            for (int c = 0; c < kKeptUnits; ++c) {
                                const int q = c0 + kKeptUnits + c;
                                ahead[c] = load_unit(a.slots, off, q0 + q, q < nu && q0 + q < n_units);
                            }
#pragma unroll
                            for (int c = 0; c < kKeptUnits; ++c) {
                                unit_sum_shared<Layout>(weight_at, raw[c], acc);
                                raw[c] = ahead[c];
                            }
                        }
                        s[lane] = group_inclusive_sum<kWave>(acc);
                        break;
                    }
                    }
                    // where the row's sums are | units per lane | log2 of its lanes
                    if (geo_sl == 0 && t0 + geo_rel < n_rows)
                        row_slot[t0 + geo_rel] = (uint32_t)(n_passes * kWave + geo_rel * lanes) | (uint32_t)nu << 12 |
                                                 (uint32_t)lanes_log2(shape) << 28;
                    ++n_passes;
                } while (t_next < n_rows && n_passes < a.kept_passes);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                if (valid && row >= row0 && row < t_next) {
                    const uint32_t info = row_slot[row];
                    const int lane0 = (int)(info & 0xfffu), nu = (int)((info >> 12) & 0xffffu), lanes = 1 << (info >> 28);
                    const int n_units = mine.nnz, o = mine.o, n_lanes = (n_units + nu - 1) / nu;
                    int holder = 0;             // the last sub-lane whose first topic is not above o
                    for (int step = most_lanes >> 1; step > 0; step >>= 1) {
                        const int at = min(holder + step, lanes - 1);
                        if (holder + step < lanes && (int)first_topic[lane0 + at] <= o) holder = at;
                    }
                    const int q0 = holder * nu, o_key = Layout::key_of_topic(o);
                    int n_o = 0;
                    for (int c = 0; c < most_units; ++c) {
                        const uint4 unit = load_unit(a.slots, mine.off, q0 + c, c < nu && q0 + c < n_units);
#pragma unroll
                        for (int j = 0; j < Layout::kUnitEntries; ++j)
                            n_o += Layout::key(unit, j) == o_key ? Layout::count(unit, j) : 0;
                    }
                    if (!Layout::kOneEntryPerTopic && holder > 0 && (int)first_topic[lane0 + holder] == o &&
                        key_before_unit<Layout>(a.slots + ((size_t)mine.off + 1u + (size_t)q0) * 16u) == o_key)
                        in_rest = true;         // the sub-lane before has some of o's entries, too
                    const double shift = fma((double)(n_o - 1), (double)mine.w_o, -((double)n_o * (double)cell(o)));
                    const double S_all = sums[lane0 + n_lanes - 1];
                    const double S = S_all + shift, total = mine.Qp + S;
                    if (!((uint32_t)__double2hiint(S_all) < exact_below())) in_rest = true;
                    const double x = mine.u * total;
                    int sub = 0;                // sub-lanes known to lie before the draw
                    double before = 0.0;
                    for (int step = most_lanes; step > 0; step >>= 1) {
                        const int upto = sub + step;
                        if (upto <= n_lanes) {
                            const double e = sums[lane0 + upto - 1] + (upto > holder ? shift : 0.0);
                            if (!(e > x)) { sub = upto; before = e; }
                        }
                    }
                    if (!in_rest) {
                        const bool sparse = x < S;
                        sub = min(sub, n_lanes - 1);        // (the last sum is S: above x)
                        scan_units = sparse ? min(nu, n_units - sub * nu) : 0;
                        mine.off += 1u + (uint32_t)(sub * nu);
                        mine.u = x - (sparse ? before : S);
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            } while (t_next < n_rows);
            if (valid && !in_rest) {
                if (scan_units > 0) finish(topic_in_units<Layout>(weight_at, a.slots, mine.off, scan_units, mine.o, mine.w_o, mine.u),
                                           kDrawTopic, mine.o, mine.w_o, 0.0, 0.0);
                else finish(0, kDrawDense, mine.o, mine.w_o, mine.u, mine.Qp);
            }
        }
        // (the tokens that have no result yet, side by side)
        int n_here = min(batch, tl.count - b * batch), my_place = lane;
        if (kShares && shared) {
            const uint64_t rest = __ballot(in_rest);
            kept_own = n_here = __popcll(rest);
            if (n_here == 0) continue;
            my_place = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(rest >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)rest, 0u));
            if (!in_rest) {             // (behind the records in use)
                mine.off = 0; mine.nnz = 0;
                my_place = n_here + lane - my_place;
            }
        }
        my_rec[my_place] = mine;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // ---- one token per group of 4 .. 64 lanes.  A pass takes the next 16, 8, 4, 2 or 1
        // tokens, as many as lets every lane own at most kKeptUnits units; the rows of the
        // following pass are requested from memory before this one is worked on.
        int units = mine.nnz;
        if (kShares && shared) units = my_rec[lane].nnz;
        learn_shapes(units);
        // where a pass's rows are, and the loads of the units its lanes keep.  `rec` is the
        // record of the lane's token, `sl` the lane's place inside its group.  A pass that
        // would run past the batch's 64 records works on the last one several times over.
        auto request = [&](int t0, int shape, TokenRec*& rec, int& sl, uint4* raw, bool live) {
            const int nu = units_of(shape);
            place_lanes(shape);
            sl = geo_sl;
            rec = my_rec + min(t0 + geo_rel, kWave - 1);
            const uint2 where = *reinterpret_cast<const uint2*>(rec);
            // units the lane loads: those of the shape that the row still has from its first on
            const int n_mine = live ? min((int)where.y - geo_q0, nu) : 0;
            if constexpr (kNear) {
                const uint32_t row_bytes = (where.x + 1u + (uint32_t)geo_q0) << 4;
#pragma unroll
                for (int c = 0; c < kKeptUnits; ++c)
                    raw[c] = load_unit_near(a.slots, row_bytes, c, c < n_mine);
            } else {
#pragma unroll
                for (int c = 0; c < kKeptUnits; ++c)
                    raw[c] = load_unit(a.slots, where.x, geo_q0 + c, c < n_mine);
            }
        };
        int t_next = 0, shape_next = shape_at(0), sl_next;
        TokenRec* rec_next;
        // one pass: `mine_raw` holds its rows, already requested; the following pass's rows
        // go to `next_raw`.  The two buffers swap roles from pass to pass.
        auto pass = [&](uint4* mine_raw, uint4* next_raw) {
            const int shape = shape_next, sl = sl_next;
            TokenRec* rec = rec_next;
            const int n_tokens = kWave >> lanes_log2(shape);
            t_next += n_tokens;
            // The request is made whether or not a pass follows (after the batch's last pass
            // every lane loads padding units): the number of loads in flight behind this
            // pass's own is then the same on every path, and the pass waits for its own rows
            // only, not for the first of the following pass's as well.
            const int t_req = min(t_next, kWave - 1);
            shape_next = !kDouble || t_next < n_here ? shape_at(t_req) : kNoPass;
            request(t_req, shape_next, rec_next, sl_next, next_raw, t_next < n_here);
            // (one walk per layout family; all have the same shapes)
            auto row_pass = [&](auto lanes, auto units) {
                if constexpr (kDouble) row_pass_double<Layout, lanes.value, units.value>(rec, sl, mine_raw, lane);
                else row_pass_kept<Layout, lanes.value, units.value>(weight_at, rec, sl, mine_raw, lane);
            };
            switch (shape) {
            case 0: row_pass(Int<4>(), Int<1>()); break;
            case 1: row_pass(Int<4>(), Int<2>()); break;
            case 2: row_pass(Int<4>(), Int<3>()); break;
            case 3: row_pass(Int<8>(), Int<2>()); break;
            case 4: row_pass(Int<8>(), Int<3>()); break;
            case 5: row_pass(Int<16>(), Int<2>()); break;
            case 6: row_pass(Int<16>(), Int<3>()); break;
            case 7: row_pass(Int<32>(), Int<2>()); break;
            case 8: row_pass(Int<32>(), Int<3>()); break;
            case 9: row_pass(Int<64>(), Int<2>()); break;
            case 10: row_pass(Int<64>(), Int<3>()); break;
            case 11:
                if constexpr (kDouble) row_pass_double_long<Layout>(a.slots, rec, lane);
                if constexpr (kDouble) break;
                [[fallthrough]];
            default:                // (kDouble: kNoPass)
                if constexpr (!kDouble) row_pass_long<Layout>(weight_at, a.slots, rec, lane);
                break;
            }
        };
        uint4 raw_a[kKeptUnits], raw_b[kKeptUnits];
        request(0, shape_next, rec_next, sl_next, raw_a, true);
        if constexpr (kDouble) {
            // Always in twos, with a pass of nothing after an odd number: a way back to the loop's head
            // from between the two would make the compiler wait, in front of the first one's request,
            // for the rows it is about to work on.  (The twelve-wave kernels are 1 % slower with it:
            // they spill more registers.)
            do {
                pass(raw_a, raw_b);
                pass(raw_b, raw_a);
            } while (t_next < n_here);
        } else {
            while (t_next < n_here) {
                pass(raw_a, raw_b);
                if (t_next < n_here) pass(raw_b, raw_a);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // (the token's topic and corrected weight are read back from its record rather than
        // kept in registers across the passes)
        if (kShares ? in_rest : lane < batch && b * batch + lane < tl.count) {
            const TokenRec* rec = &my_rec[my_place];
            const int4 head_of = *reinterpret_cast<const int4*>(rec);     // off, kind, o, w_o
            finish(head_of.x, head_of.y, head_of.z, __int_as_float(head_of.w), rec->u, rec->Qp);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if constexpr (!kQueue) break;
    last_ti = ti;
    // The next tile is asked for by the wave that has the fewest batches, when it is done with them.  (Asked for beside the groups'
    // sums its time would not show, but a workgroup would hold it while it works on a long tile, and do long ones one after the
    // other for which others are free.)  Sampling launch, us, a workgroup for every tile / asked for beside the sums / when done:
    //   6.6e6 tokens in 300 documents, 139 words, K = 5,741       2,490 / 3,777 / 2,190     5,000 words   1,326 / 1,351 / 1,000
    //   1.9e6 in 87, K = 3,000     669 / 810 / 670                9.9e7 in 3e5, 102,000 words, K = 10,000 10,362 / 8,977 / 8,900
    //   3.8e6 in 15,000, 60,000 words, K = 9,000 1,108 / 849 / 828     2e6 in 8,009, K = 40,000 - / 455 / 449
    if (wave == kWaves - 1 && lane == 0) {
        const uint32_t taken = atomicAdd(a.next_tile, 1u);
        least[1] = taken + gridDim.x;
        // (every workgroup asks until there is no tile left: n_tiles times in all)
        if (taken + 1u == (uint32_t)a.n_tiles) atomicExch(a.next_tile, 0u);
    }
    __syncthreads();                // (and every wave is done with this word's p*)
    ti = __builtin_amdgcn_readfirstlane((int)least[1]);
    if (ti >= a.n_tiles) break;
    }
}

// Initial topics: z = floor(u(seed, 0, token) K), in word-major order.
__global__ void init_topics_kernel(const int32_t* tok_id, uint16_t* z, int64_t T, int32_t K,
                                   uint64_t seed) {
    const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (pos >= T) return;
    const double u = token_uniform(seed, 0u, (uint64_t)(uint32_t)tok_id[pos]);
    int k = (int)(u * (double)K);
    if (k > K - 1) k = K - 1;
    z[pos] = (uint16_t)k;
}

__global__ void philox_uniform_kernel(uint64_t seed, uint32_t iter, uint64_t token0, int64_t n,
                                      double* out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = token_uniform(seed, iter, token0 + (uint64_t)i);
}

}  // namespace mlda
