// libmlda.so: C ABI, context and host-side preprocessing (see include/mlda.h).
//
// Paper sections behind the host steps: Section 6.1.2 (tokens are sorted word-first and
// the tokens of heavy words are split over several workgroups), Section 6.2 (a
// document->token map lets the theta update find a document's tokens in the word-sorted
// arrays; the paper builds it on the CPU, here it is derived on the device), Section 4 and Algorithm 1 (the corpus is partitioned by document
// into chunks; WorkSchedule1: one chunk, transferred once, iterated on the device;
// WorkSchedule2: several chunks per GPU, transferred every iteration while phi stays).
//
// A context is the model (phi, n_k, tables) plus the chunk that is attached at the moment:
// with one chunk it is attached once and for all, with several each is attached in turn.
#include "../../include/mlda.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "chunk_layout.hpp"
#include "kernels_rebuild.hpp"
#include "kernels_sample.hpp"
#include "switches.hpp"

namespace {

thread_local std::string g_last_error;

int fail(int code, const std::string& msg) {
    g_last_error = msg;
    return code;
}

#define HIP_TRY(expr)                                                                  \
    do {                                                                               \
        hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess)                                                          \
            return fail(MLDA_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

#define RC_TRY(expr)                   \
    do {                               \
        const int rc_ = (expr);        \
        if (rc_ != MLDA_OK) return rc_; \
    } while (0)

using mlda::kAlign;
using mlda::align_up;
using mlda::ChunkLayout;
using mlda::chunk_first;
using mlda::chunk_layout;
constexpr size_t kSlotAlign = 64;     // theta row slot alignment (bytes)
constexpr size_t kLdsPerWorkgroup = 160 * 1024;
// waves per sampling workgroup: more of them share one staged p* column when K is large
// (twelve: two such workgroups fill a CU's six waves per SIMD, and their LDS fits twice; sixteen
// where it does not, from K = 11,440 on: 4e6 tokens at K = 13,000 608 us against 697, 2e6 at 29,000 910 against 1,085)
size_t queued_lds_bytes(int32_t K, int waves) {
    const int32_t g = mlda::dense_group(waves), Kpad = (K + g) / g * g;
    return mlda::sample_lds_bytes(Kpad, waves, 4) + mlda::sample_run_lds_bytes(Kpad, waves);
}
int sample_waves_for(int32_t K) { return K <= 2048 ? 4 : 2 * queued_lds_bytes(K, 12) <= kLdsPerWorkgroup ? 12 : 16; }

// How a chunk's theta rows are laid out: 4-byte entries of any K for the workgroups of twelve waves,
// and for those of four (K <= 2048) where rows are shortest; else for these 2-byte entries with 3, 5 or
// 6 bits of count, or 4-byte entries with long counts.
enum class RowKind { packed, tiny3, tiny5, tiny6, counted };

// f(layout) for the layout of that kind.
template <class F>
auto with_layout(RowKind rows, F&& f) {
    switch (rows) {
    case RowKind::tiny3: return f(mlda::TinyRows<3>());
    case RowKind::tiny5: return f(mlda::TinyRows<5>());
    case RowKind::tiny6: return f(mlda::TinyRows<6>());
    case RowKind::counted: return f(mlda::CountedRows());
    default: return f(mlda::PackedRows());
    }
}

// What the sampler's LDS holds besides p* itself belongs to K as well: Kpad = K + 1 rounded up to
// a multiple of the dense bucket's group (one zero entry of p* past the last topic: padding
// entries of theta rows point at it).
//
// p* of one word beside the prefix sums and the waves' records: where that exceeds the LDS a
// workgroup can have on this chip (K beyond about 26,100), p* of the topics that do not fit lives in device memory
// instead, one strip per workgroup of a launch of at most kFarStrips workgroups.
constexpr int kFarStrips = 256;
bool far_weights_for(int32_t K) { return sample_waves_for(K) == 16 && queued_lds_bytes(K, 16) > kLdsPerWorkgroup; }
int32_t kpad_for(int32_t K) {
    const int32_t g = mlda::dense_group(sample_waves_for(K), far_weights_for(K));
    return (K + g) / g * g;
}
// The topics whose p* stays in LDS then: as many as have room.
int32_t near_topics_for(int32_t K) {
    const size_t rest = mlda::sample_far_lds_bytes(kpad_for(K), sample_waves_for(K), 0);
    return (int32_t)std::min<size_t>((kLdsPerWorkgroup - rest) / 4, (size_t)kpad_for(K)) & ~15;
}
// What the others take of the workspace.  (Beyond kFarColumnsFrom topics, where a whole column beside twelve waves' records
// exceeds the LDS, callers are told of kFarColumns whole ones on top: the bound that mlda.h has named from the start.  The
// strips need no more than 42 MB of it, at K = 65,535.)
constexpr int32_t kFarColumnsFrom = 30943;
constexpr int kFarColumns = 512;
size_t far_bytes_for(int32_t K) {
    if (!far_weights_for(K)) return 0;
    return mlda::far_strip_cells(kpad_for(K), near_topics_for(K)) * kFarStrips * 4 +
           (K > kFarColumnsFrom ? (size_t)kpad_for(K) * kFarColumns * 4 : 0);
}

// short_docs: no document has more tokens than a 4-byte entry counts; near: the theta slots of
// the chunk end below 4 GiB, so that 32-bit byte offsets reach them
template <bool kNear>
const void* sample_kernel_of(int32_t K, RowKind rows, bool short_docs, bool alone) {
    if (far_weights_for(K)) return (const void*)mlda::sample_kernel<16, mlda::PackedRows, mlda::Form::split, kNear>;
    if (rows == RowKind::packed && sample_waves_for(K) == 4) return (const void*)mlda::sample_kernel<4, mlda::PackedRowsAlone, mlda::Form::once, kNear>;
    if (rows == RowKind::packed) {
        auto of_waves = [&](auto waves) {
            if (short_docs && alone) return (const void*)mlda::sample_kernel<waves.value, mlda::PackedRowsAlone, mlda::Form::queued, kNear>;
            if (short_docs) return (const void*)mlda::sample_kernel<waves.value, mlda::PackedRowsShort, mlda::Form::queued, kNear>;
            return (const void*)mlda::sample_kernel<waves.value, mlda::PackedRows, mlda::Form::queued, kNear>;
        };
        return sample_waves_for(K) == 12 ? of_waves(mlda::Int<12>()) : of_waves(mlda::Int<16>());
    }
    return with_layout(rows, [](auto layout) {
        typedef decltype(layout) Layout;
        return (const void*)mlda::sample_kernel<4, Layout, mlda::Form::once, kNear>;
    });
}
const void* sample_kernel_for(int32_t K, RowKind rows, bool short_docs, bool alone, bool near) {
    return near ? sample_kernel_of<true>(K, rows, short_docs, alone) : sample_kernel_of<false>(K, rows, short_docs, alone);
}
// (a wave per tile, K <= 2048)
template <bool kNear>
const void* sample_solo_kernel_of(RowKind rows) {
    if (rows == RowKind::packed) return (const void*)mlda::sample_kernel<1, mlda::PackedRowsAlone, mlda::Form::once, kNear>;
    return with_layout(rows, [](auto layout) {
        typedef decltype(layout) Layout;
        typedef typename std::conditional<Layout::kDoubleWeights, Layout, mlda::PackedRowsAlone>::type Rows;
        return (const void*)mlda::sample_kernel<1, Rows, mlda::Form::once, kNear>;
    });
}
bool slots_near(size_t slots_bytes) { return slots_bytes <= 0xffffffffull; }
// Few long documents are counted by kLongDocWaves waves each.  Measured, theta rebuild of D equal
// documents at K = 500 with one wave each / sixteen, us (24 and 3,000 topics alike):
//   tokens   D = 256     512       768        1,024      2,048
//    4,200    34/ 20    38/ 34    42/ 48     47/ 61     71/115
//   10,000    54/ 26    58/ 46    62/ 67     75/ 86    155/181
//   30,000   137/ 49   158/ 92   214/159    298/211
// Up to one document per CU from a few thousand tokens on, then the longer the more documents
// there are; and, up to eight per CU, where the longest alone would take a wave longer (4.7 ns a token)
// than all of them take sixteen waves each (about 8 us per document and CU and 1.2 ns per token and CU): 1,024
// documents of 10,000 tokens, the longest of 87,000, 478/166 us; 2,040 with 84,000 787/398.
bool long_docs_for(int64_t D, int64_t T, int64_t longest, int n_cus) {
    if (D <= 0 || D > (int64_t)n_cus * 8 || T / D < 4096) return false;
    return (D <= (int64_t)n_cus * 4 && T / D >= D * 4096 / n_cus) ||
           longest >= D * 1700 / n_cus + T / (4 * n_cus);
}
// (with a dense row)
const void* theta_kernel_for(RowKind rows, bool wide_counters, bool long_docs) {
    return with_layout(rows, [&](auto layout) {
        typedef decltype(layout) Layout;
        if (long_docs)
            return wide_counters ? (const void*)mlda::theta_rows_kernel<Layout, true, mlda::kLongDocWaves>
                                 : (const void*)mlda::theta_rows_kernel<Layout, false, mlda::kLongDocWaves>;
        return wide_counters ? (const void*)mlda::theta_rows_kernel<Layout, true, 1>
                             : (const void*)mlda::theta_rows_kernel<Layout, false, 1>;
    });
}
// (by ranks; `docs` documents per wave, two for K <= kPairMaxK)
const void* theta_ranked_kernel_for(RowKind rows, int docs) {
    return with_layout(rows, [&](auto layout) {
        typedef decltype(layout) Layout;
        return docs == 2 ? (const void*)mlda::theta_ranked_kernel<Layout, 2> : (const void*)mlda::theta_ranked_kernel<Layout, 1>;
    });
}
// What a wave of the sampler with fp64 weights keeps of shared walks: as much as leaves a CU its twenty waves
// (five per SIMD; LDS is dealt out in 128 pieces of 1,280 bytes), where that is at least one pass.  Units,
// sampling launch, ms:            192    384    576    768
//   K = 299, documents of 30,000 0.632  0.549  0.520  0.519
//   K = 1,000, 3.3e7 tokens       2.63   2.46   2.47   2.69   (four workgroups a CU)
//   K = 1,537, 6.3e6             0.549  0.557  0.630  0.783   (four from 448 on)
//   K = 2,000, 1.1e7             0.960  1.053  1.279  1.258   (four from 320 on)
// None for few topics of many tokens: the topics' totals are then so large, and a word's least weight so small, that most sums
// are too long to be exact, and rows of so few topics are walked in a pass or two anyway.  Sampling launch, us, by T
// (words 5,000, the generator's topics), shared in tiles of 128 / not shared in tiles of 128 / not shared in tiles of 1,024:
//                       1e6          5e6           1e7           1.5e7         3e7
//   K = 11, n = 150     33 33 41     116 117 123   216 220 219   320 320 315   682 636 614
//           n = 4,800   30 32 39     105 110 113   200 204 203   303 299 296   631 602 578     (8.2e7: 1,750 1,586 1,505)
//   K = 15, n = 4,800   30 32 40     106 111 116   206 209 207   302 304 296   644 603 586
bool few_topics_of_many_tokens(int32_t K, int64_t T) { return K <= 16 && T > 10000000; }
struct KeptSums { int32_t passes, sums; };
KeptSums kept_sums_for(int32_t Kpad, int waves) {
    const size_t budget = (size_t)(128 * waves / 20) * 1280;
    for (int32_t sums = 768; sums > 192; sums -= 64)
        if (mlda::sample_lds_bytes(Kpad, waves, 8, sums / 192 + 1, sums) <= budget) return {sums / 192 + 1, sums};
    return {2, 192};
}
// From this beta on tokens share sums that are up to three bits too long to be exact, too (see kNearlyAll).  8.6e6 tokens in
// documents of 30,000 at K = 299, sampling launch at iteration 90: 0.55 ms without, 0.44 with; 1.28 where every token walks.
constexpr double kSlackBeta = 0.005;
// K > 2048: documents of fewer tokens than these have too few words several times for shared walks, which the
// kernel then leaves out.  1e6 tokens at K = 5,000, sampling launch without / with, us:
//   documents of 15  190/198   30  172/180   50  191/202   80  193/200   120  221/207
//   8e6, K = 3,000, 300 words: of 20  277/287   of 40  320/338
constexpr int kAloneDocs = 90;
// K > 2048: passes whose sums a wave keeps at most.  2 / 8: 5e6 tokens at K = 2,218 358/309 us, 1.5e5 at
// K = 4,983 521/504, 9.9e7 at K = 10,000 22.5/22.2 ms.
constexpr int kMostKeptPasses = 8;
// Tokens from which assignments change their order tile by tile: where the caller's array outgrows the 256 MB
// of last-level cache, in which the plain scatter's lines otherwise meet.  The whole getter, plain / by tiles, ms:
//   1.35e8 tokens 8.6 / 9.8   1.8e8 12.1 / 12.5   2.7e8 20.4 / 18.0   3.8e8 29.8 / 24.8   7.4e8 60.8 / 48.0
// (7.4e8: the scatter itself 24.05 / 11.2, the gather of the setter 12.55 / 7.5; 9.9e7: 1.00 / 1.95 and 1.36 / 1.15.)
constexpr int64_t kReorderByTiles = 200000000;
constexpr int kMaxTimedIters = 1024;
// Words of few tokens whose p* is made from one another's (K > 2048) count in the sampler's bytes as if every
// kRunTiles-th were staged afresh.
constexpr int kRunTiles = 16;
// events of a streamed chunk visit: its uploads have arrived | topics and slots in word-major
// order | theta rebuilt | sampled | phi added to | new topics in document order | theta of the
// new topics (log-likelihood)
constexpr int kVisitEvents = 7;
constexpr int kMaxTimedVisits = 4096;

int tile_tokens_for(int32_t K) { return K <= 2048 ? 1024 : 4096; }
// K <= 2048: the tokens of a sampling tile, and up to how many of them a wave takes the tile alone.  A workgroup
// of four waves keeps three of them idle over a word of few tokens, and on a small corpus the launch takes the time
// of one tile's batches; a wave per tile stages p* of the word by itself, which the longer the column and the smaller
// the tile is the larger part of its work.  Measured, sampling launch (us) by "tile / alone up to", documents of 150:
//                       1024/0  1024/64  256/64  128/128  64/64
//   K = 16,     1e5       24      28       17      15       11
//               3e6      110      99       94      85       86
//               4e7      926     911      961     865      961     (beyond 1e7 see few_topics_of_many_tokens)
//   K = 128,    1e5       34      41       25      22       16
//               1e6      106      92       76      73       67
//               4e7     1538    1439     1507    1427     1518
//   K = 512,    1e6      171     145      117     119      112
//               3e6      321     258      248     244      250      1024/128: 254
//               4e7     2031    1859     1979    1923     2142                1805
//   K = 1,000,  1e5       57      65       39      40       34
//               1e6      188     190      166     183      186
//               4e7     2251    2184     2358    3136     3852
//   K = 2,000,  1e5       66      90       64      62       55
//               1e6      272     338      315     388      415
// (256 < K <= 512, 1024/128 and 128/128: 1e7 tokens at K = 300 in documents of 300, 4,000 and 30,000 567/545, 577/555 and
// 460/440, at K = 500 of 1,500 613/593; 1.2e7 at K = 455 of 20,000 696/711, 3e7 at K = 500 of 10,000 2743/2837.)
// Where a wave per tile of 64 leaves the chip room, tiles are cut smaller, to 16 or 32 tokens, as long as there are no more than
// kFewestTiles (16 a CU) of them: the launch takes the time of one tile, and its passes follow one another.  us by tile size
// 16 / 32 / 64:
//   8e3 tokens, K = 24                6.4   6.4   8.4 (580 tiles of 16)      5e4, K = 32, 3,000 words    8.8   8.1   8.6 (4,600)
//   2e4, K = 100                      7.7   8.1   9.5 (2,300)                5e4, K = 1,500             43.6  38.6  40.3 (4,600)
//   3e4, K = 900, 3,000 words        17.2  21.1  25.2 (3,400)                1e5, K = 32                13.1   9.6  10.1 (8,800)
//   5e4, K = 200, 2,000 words        12.0  14.3  16.2 (4,100)                1e5, K = 900               35.7  27.7  25.1 (7,800)
constexpr int32_t kLeastTile = 16;
constexpr int64_t kFewestTiles = 4096;
struct TileShape { int32_t tokens, alone; };
TileShape tile_shape_for(int32_t K, int64_t T) {
    if (K > 2048) return {4096, 0};
    if (T <= (K <= 512 ? 2000000 : K <= 1024 ? 200000 : 100000)) return {64, 64};
    if (few_topics_of_many_tokens(K, T)) return {1024, 0};
    if (T <= (K <= 256 ? 100000000 : K <= 512 ? 10000000 : 0)) return {128, 128};
    if (K <= 512) return {1024, 128};
    if (K <= 1024) return {T <= 4000000 ? 256 : 1024, 64};
    return {1024, 0};
}
constexpr int kPhiSegment = 16384;    // tokens one workgroup histograms for the phi rebuild
// Up to how many tokens a word's row is changed rather than written anew, K > kPhiDwordTopics: a token costs two lines of memory, a row
// K / 64.  Rebuild of phi and the totals, us, never / up to K / 256 / K / 64 / K / 16 tokens:
//   5e5 tokens, 20,000 words, K = 5,000    40  26  26  26      3e6, 20,000 words, K = 20,000    192  85  86  87
//   4e6, 60,000 words, K = 9,000          263  99  91  92      2e6, 6,000 words, K = 40,000     138  99  99  98
//   2e7, 60,000 words, K = 8,000          289 206 149 145      2e6, 6,000 words, K = 60,000     200 120 123 125
//   9.9e7, 102,000 words, K = 10,000      722 712 618 670      2e4, 100 words, K = 60,000        47  43  42  46
int changed_cells_for(int32_t K) { return K > mlda::kPhiDwordTopics ? K / 64 : 0; }
// Up to how many tokens a wave counts a segment by itself: workgroups are started one in 1.3 ns, and most words have fewer
// tokens than four waves lanes.  All segments where they are so many that the longest does not matter, none where the
// counters of four take a CU's LDS.  Rebuild of phi, us, segments up to 0 / 64 / 256 / 1,024 / 16,384 tokens by a wave each:
//   1e5 tokens, K = 32        5.2   5.1   5.2   5.2   8.5      2e6, K = 2,000        89    70    68    67    66
//   1e6, K = 16, 60,000 words  16    12    11    11    15      2e7, K = 500         131    88    78    74    72
//   1e6, K = 128               21    14    13    12    14      9.9e7, K = 1,000     316   312   296   271   264
//   6.3e6, K = 1,537           59    50    46    45    47      7.4e8, K = 1,000     708   702   682   648   598
//   2e6, K = 4,000            133   119   117   116   115      2e6, K = 8,000       213   213   213   212   212
int solo_segment_for(int32_t K, int64_t T, int64_t n_segs) {
    return K > mlda::kPhiDwordTopics ? 0 : T > 10000000 && n_segs >= 16384 ? kPhiSegment : 1024;
}
constexpr int32_t kHistTopics = 32768; // 32-bit counters of the n_k histogram that share a workgroup's LDS

// A theta row's slot: a header of kRowHeader bytes (the row's number of entries), then the
// entries, filled up to whole 16-byte units.  A document of n tokens needs at most
// min(n, K + n / max_count) entries: one per topic, and one more for every max_count tokens
// that a count exceeds its entry's field by.
size_t slot_bytes_for(int64_t n, int32_t K, int entry_bytes, int max_count) {
    const int64_t cap = std::min<int64_t>(n, (int64_t)K + n / max_count);
    return align_up((size_t)mlda::kRowHeader + align_up((size_t)cap * (size_t)entry_bytes, 16), kSlotAlign);
}

// Layout of the theta rows of D documents over V words (K <= 2048), from their lengths: the rows themselves change
// with every iteration, from spread over many topics at a random start to counts of many tokens.
// 2-byte entries read half the bytes and, eight to a unit, take fewer passes; but a count beyond its
// field takes several of them.  Measured, sampling launch on 5e6 tokens in equal documents, from a random
// start / trained / concentrated (alpha = 0.05), us:
//                               3 bits          5 or 6 bits       4 bytes
//   K = 1,000, 100 tokens    234/ 224/ 219    242/ 228/ 219     285/ 269/ 263
//             400            382/ 343/ 337    392/ 329/ 293     489/ 415/ 387
//             800            613/ 485/ 474    585/ 358/ 348     810/ 449/ 429
//          12,000           6386/5442/5625   1727/ 708/ 645    4214/ 720/ 569
//   K = 300,  4,000          1186/1081/1082    628/ 344/ 267     845/ 385/ 196
//          12,000           5357/5371/5244    623/ 594/ 466     865/ 409/ 206
//   K = 2,000, 12,000        6573/5479/5562   4854/1198/1224    6294/ 854/ 949
//   K = 24,   400             190/ 189/ 154    141/ 139/ 127     137/ 135/ 108
//   K = 44,   400                              172/ 164/ 130     158/ 150/ 111
//   K = 52,   400                              174/ 169/ 133     208/ 154/ 113
// Three bits of count, an instruction less for two entries, where documents are short (what counts is the
// length that a token meets) and few counts can outgrow them.  4 bytes where a row could have so
// many more of the 2-byte entries (of six bits a quarter, of five 0.15 times as many), or where the topics
// are so few that a 4-byte row, too, fits four lanes (twelve units).
// The shortest documents at K >= 1,024, and somewhat longer ones where the words have so few tokens that staging
// p* is most of the work, keep 4-byte entries and fp32 weights (six waves per SIMD instead of five, half
// the LDS, the new topic found in the walk itself).  fp64 walk / this, sampling launch:
//   tokens per word:        62      125      333    1,000
//   K = 2,048,  10 tokens  1.34     1.25     1.20    1.11
//               40         1.29     1.18     1.09    1.03
//               60         1.14     1.07     0.97    0.89
//              200         1.03     0.98     0.88    0.82
//   K = 1,025,  40         1.14     1.10     1.04    1.03
//               60         1.04     0.99     0.92    0.89
constexpr int kShortestDocs = 50, kShortDocs = 400, kFewTopics = 48;
constexpr double kTinyGrowth = 1.25, kTinyGrowth5 = 1.15;
RowKind row_kind_for(const int64_t* doc_ptr, int64_t D, int32_t V, int32_t K) {
    if (sample_waves_for(K) != 4) return RowKind::packed;
    const RowKind tiny = K <= mlda::TinyRows<6>::kMaxK ? RowKind::tiny6 : K <= mlda::TinyRows<5>::kMaxK ? RowKind::tiny5 : RowKind::tiny3;
    const int max_count = with_layout(tiny, [](auto layout) { return layout.kMaxCount; });
    auto most_entries = [&](int64_t n, int max) { return (double)(n <= K ? n : std::min<int64_t>(n, (int64_t)K + n / max)); };
    // sums over the tokens: 1, their document's length, and the most entries its row can have
    double tokens = 0.0, length = 0.0, counted = 0.0, tiny3 = 0.0, wider = 0.0;
    int64_t longest = 0;
    for (int64_t d = 0; d < D; ++d) {
        const int64_t n = doc_ptr[d + 1] - doc_ptr[d];
        const double w = (double)n;
        longest = std::max(longest, n);
        tokens += w;
        length += w * (double)n;
        counted += w * (double)std::min<int64_t>(n, K);
        tiny3 += w * most_entries(n, mlda::TinyRows<3>::kMaxCount);
        wider += w * most_entries(n, max_count);
    }
    if (K > mlda::TinyRows<6>::kMaxK && longest <= mlda::PackedRowsShort::kMaxCount &&
        length <= std::max(kShortestDocs * tokens, std::min(200.0 * tokens, 6.0 * K * V)))
        return RowKind::packed;
    if (length <= kShortDocs * tokens && tiny3 <= kTinyGrowth * counted) return RowKind::tiny3;
    if (K <= kFewTopics) return RowKind::counted;
    return wider > (tiny == RowKind::tiny6 ? kTinyGrowth : kTinyGrowth5) * counted ? RowKind::counted : tiny;
}

// Resident corpora of up to so many tokens and topics: one launch rebuilds phi and theta (the counters of four segments then fit
// 48 KB).  Both rebuilds, us, two launches / one:
//   8e3 tokens, K = 24    8.7/ 5.3     5e5, K = 900    24.8/20.4     5e6, K = 2,000   56/50       2e7, K = 500     163/178
//   1e5, K = 32          11.5/ 6.8     1e6, K = 128    26.2/25.2     6.3e6, K = 1,537 95/96       9.9e7, K = 1,000 922/1063
constexpr int64_t kBothTokens = 5000000;
constexpr int32_t kBothTopics = 3072;
static_assert(kBothTopics <= mlda::kPhiDwordTopics, "a topic has a dword");

constexpr int kLoglikBlocks = 2048;
constexpr int kSmallLoglikBlocks = 256;     // up to so many, the word side's last workgroup adds up
constexpr int kMaxThetaGrid = 4096;    // workgroups of the theta rebuild (each leaves one likelihood partial and one count)
// Up to this K a resident context has a second n_k (in what loglik_word_side_kernel leaves of its partials).
constexpr int32_t kSpareTotals = 2 * kLoglikBlocks;
static_assert(kSpareTotals <= mlda::kPhiDwordTopics, "phi and the totals share a launch's LDS");
constexpr int kEntryRing = 2048;      // per-rebuild counters of theta row entries (> kMaxTimedIters)
// resident: when the four phases of every timed iteration started, and when the last one had ended
constexpr int kPhases = 4;
constexpr size_t kStampBytes = ((size_t)kMaxTimedIters * kPhases + 1) * 8;

// An upper bound of a chunk's layout from the sizes alone.
ChunkLayout chunk_layout_bound(int64_t D, int64_t T, int32_t V, int32_t K, bool streamed) {
    const size_t tile = (size_t)tile_tokens_for(K);
    // (at most one entry of at most 4 bytes per token, a header, a unit's and a slot's rounding)
    const size_t slots = kSlotAlign + (size_t)T * 4 + (size_t)D * (mlda::kRowHeader + 16 + kSlotAlign);
    const size_t n_tiles = (size_t)T / tile + (size_t)V + 1;
    const size_t n_segs = (size_t)T / kPhiSegment + (size_t)V + 1;
    return chunk_layout(D, T, slots, n_tiles, n_segs, (size_t)V, streamed);
}

// Large transfers between the device and the caller's memory, see on_workers.
constexpr int kRingWorkers = 8;
constexpr size_t kRingPiece = (size_t)2 << 20;
constexpr size_t kRingFrom = (size_t)8 << 20;
constexpr int kCopyBlocks = 64;         // workgroups of copy_to_host_kernel (32 to 128: the same)
constexpr size_t kRingFlag = 64;        // bytes from one flag to the next, behind the pieces

// The model and the scratch of the reductions.
// phi[i] is one copy of the model: the 16-bit matrix [V][K], then room for the int32 rows of
// the words with 2^16 tokens or more, of which a corpus of T tokens has at most T / 2^16.
struct ModelLayout {
    size_t phi[2] = {0, 0}, phi_wide = 0, phi_bytes = 0, wide_row = 0, n_k[2] = {0, 0}, ll_partial = 0,
           ll_scalars = 0, lg_table = 0, row_entries = 0, stamps = 0, far_pstar = 0, total = 0;
};

int64_t wide_rows_bound(int32_t V, int64_t T) {
    return std::min<int64_t>((int64_t)V, T / mlda::kNarrowWordLimit);
}

ModelLayout model_layout(int32_t V, int32_t K, int64_t T, bool two_phi) {
    ModelLayout L;
    size_t at = 0;
    auto put = [&](size_t bytes) { const size_t o = at; at += align_up(bytes, kAlign); return o; };
    L.phi_wide = align_up((size_t)V * (size_t)K * 2, kAlign);      // offset of the wide rows inside a copy
    L.phi_bytes = L.phi_wide + align_up((size_t)wide_rows_bound(V, T) * (size_t)K * 4, kAlign);
    L.phi[0] = put(L.phi_bytes);
    L.phi[1] = two_phi ? put(L.phi_bytes) : L.phi[0];
    L.wide_row = put((size_t)V * 4);
    L.n_k[0] = put((size_t)K * 4);
    L.n_k[1] = two_phi ? put((size_t)K * 4) : L.n_k[0];
    L.ll_partial = put((size_t)(2 * kLoglikBlocks + 3 * kMaxThetaGrid) * 8);
    // value, theta sum, document term, the word side's ticket, the sampler's next tile; the workers' counters (copy_to_host_kernel)
    L.ll_scalars = put((size_t)(5 + kRingWorkers) * 8);
    L.lg_table = put((size_t)mlda::kLgTableSize * 8 * 2);   // one for alpha, one for beta
    L.row_entries = put((size_t)kEntryRing * 8);
    L.stamps = put((size_t)kStampBytes);
    L.far_pstar = put(far_bytes_for(K));
    L.total = at;
    return L;
}

// body(0) .. body(n_chunks - 1), each on a thread of its own.  Nothing escapes a thread: an
// exception inside a part (host memory running out) is caught there, every thread that was
// started is joined, and the call returns false.  Parts whose thread could not be started
// run on the calling thread.
template <class F>
bool parallel_chunks(int n_chunks, F&& body) {
    std::vector<std::thread> pool;
    std::vector<char> failed((size_t)std::max(n_chunks, 1), 0);
    auto guarded = [&](int c) {
        try { body(c); } catch (...) { failed[(size_t)c] = 1; }
    };
    int started = 1;
    try {
        pool.reserve((size_t)std::max(n_chunks - 1, 0));
        for (; started < n_chunks; ++started) pool.emplace_back(guarded, started);
    } catch (...) {
        // no more threads (or no memory for them): the rest runs here, below
    }
    guarded(0);
    for (int c = started; c < n_chunks; ++c) guarded(c);
    for (auto& t : pool) t.join();
    for (char f : failed)
        if (f) return false;
    return true;
}

// Documents [d_begin, d_end) of the corpus, preprocessed: the static part of the chunk's
// buffers, laid out as on the device.
struct HostChunk {
    int64_t d_begin = 0, d_end = 0;
    int64_t tok_begin = 0;              // caller's index of the chunk's first token
    int64_t D = 0, T = 0;
    RowKind rows = RowKind::packed;     // layout of the theta rows
    bool wide_counters = false;         // some document has 2^16 tokens or more
    int64_t longest_doc = 0;            // tokens
    int64_t n_unranked = 0, unranked_tokens = 0;        // documents beyond kRankedTokens (they come first), and their tokens
    bool short_docs = true;             // no document has more tokens than a 4-byte entry counts
    size_t slots_bytes = 0;
    int32_t n_tiles = 0, n_segs = 0, n_split = 0;
    int32_t n_shared_segs = 0;          // the segments from this one on are counted by a wave each
    int32_t n_dense_segs = 0;           // from this one on a step writes only the cells of their tokens' topics
    int32_t n_single = 0;               // the tiles from this one on hold whole small words: taken in runs
    int32_t n_shared = 0;               // K <= 2048: the tiles from this one on are taken by a wave each
    int32_t counted_tiles = 0;          // tiles of tile_tokens_for(K) tokens that the words have, as the sampler's bytes count them
    int64_t run_tokens = 0;             // their tokens
    int32_t n_wide_tiles = 0;           // counted tiles of words whose row of phi is int32
    ChunkLayout L;
    unsigned char* arena = nullptr;     // L.static_bytes bytes
    bool pinned = false;

    HostChunk() = default;
    HostChunk(const HostChunk&) = delete;
    HostChunk& operator=(const HostChunk&) = delete;
    ~HostChunk() { release(); }
    void release() {
        if (arena) {
            if (pinned) (void)hipHostFree(arena); else std::free(arena);
            arena = nullptr;
        }
    }
};

// Word-first order (Section 6.1.2), document->token map (Section 6.2), theta row slots, tiles.
// Inside a word the tokens are put in order of falling document length, so that the theta
// rows a wave walks together have similar lengths.  Any order inside a word, and any cut into chunks and tiles,
// draws with the same uniforms (they are keyed by the caller's token index) from the same row sums, added
// up in an order that depends on the other tokens of the batch: those sums that round (row_sums.hpp has the rule for
// those that do not) may differ in their last bit.  So the result is the same but for draws that lie
// within such a rounding; none was seen in any test.
// `accumulate`: the chunk's counts will be added to phi (several chunks) instead of stored.
int prepare_chunk(const int64_t* doc_ptr_all, const int32_t* word_ids_all, int64_t d_begin,
                  int64_t d_end, int32_t V, int32_t K, bool accumulate, bool pinned, bool runs, const TileShape* forced, HostChunk& h) {
    const int64_t D = d_end - d_begin;
    const int64_t tok_begin = doc_ptr_all[d_begin];
    const int64_t T = doc_ptr_all[d_end] - tok_begin;
    const int32_t* word_ids = word_ids_all ? word_ids_all + tok_begin : nullptr;
    auto len_of = [&](int64_t d) { return doc_ptr_all[d_begin + d + 1] - doc_ptr_all[d_begin + d]; };
    auto start_of = [&](int64_t d) { return doc_ptr_all[d_begin + d] - tok_begin; };
    h.d_begin = d_begin; h.d_end = d_end; h.tok_begin = tok_begin; h.D = D; h.T = T;

    int64_t longest_doc = 0;
    for (int64_t d = 0; d < D; ++d) longest_doc = std::max(longest_doc, len_of(d));
    h.longest_doc = longest_doc;
    // a count never exceeds the document's length: 16-bit counters in the theta rebuild if
    // they hold it
    h.wide_counters = longest_doc >= 65536;
    h.short_docs = longest_doc <= mlda::PackedRows::kMaxCount;
    h.rows = row_kind_for(doc_ptr_all + d_begin, D, V, K);
    const int entry_bytes = with_layout(h.rows, [](auto layout) { return layout.kEntryBytes; });
    const int max_count = with_layout(h.rows, [](auto layout) { return layout.kMaxCount; });

    std::vector<int32_t> doc_order;              // documents by falling length
    std::vector<int64_t> order_tokens;           // tokens before each position of doc_order
    std::vector<uint32_t> slot_of;               // slot offset of each document, 16-byte units
    std::vector<int32_t> word_ptr;
    try {
        doc_order.resize((size_t)D);
        order_tokens.resize((size_t)D + 1);
        std::vector<int64_t> len_start((size_t)longest_doc + 2, 0);
        for (int64_t d = 0; d < D; ++d) ++len_start[(size_t)(longest_doc - len_of(d)) + 1];
        for (int64_t l = 0; l <= longest_doc; ++l) len_start[(size_t)l + 1] += len_start[(size_t)l];
        for (int64_t d = 0; d < D; ++d) doc_order[(size_t)len_start[(size_t)(longest_doc - len_of(d))]++] = (int32_t)d;
        order_tokens[0] = 0;
        for (int64_t i = 0; i < D; ++i)
            order_tokens[(size_t)i + 1] = order_tokens[(size_t)i] + len_of(doc_order[(size_t)i]);
        for (h.n_unranked = 0; h.n_unranked < D && len_of(doc_order[(size_t)h.n_unranked]) > mlda::kRankedTokens;) ++h.n_unranked;
        h.unranked_tokens = order_tokens[(size_t)h.n_unranked];
        // theta row slots: fixed capacity, so rows never move; laid out in the
        // order the documents are worked on, so that rows in use together are neighbours.
        // The buffer starts with 64 bytes of padding entries.
        slot_of.resize((size_t)D);
        h.slots_bytes = kSlotAlign;
        for (int64_t i = 0; i < D; ++i) {
            const int64_t d = doc_order[(size_t)i];
            if (h.slots_bytes / 16 > 0xffffffffull) return fail(MLDA_ENOTSUP, "theta rows need more than 64 GiB");
            slot_of[(size_t)d] = (uint32_t)(h.slots_bytes / 16);
            h.slots_bytes += slot_bytes_for(len_of(d), K, entry_bytes, max_count);
        }
        word_ptr.assign((size_t)V + 1, 0);
    } catch (const std::bad_alloc&) {
        return fail(MLDA_ENOMEM, "out of host memory");
    }

    // stable counting sort by word over parts of the length-sorted document sequence
    const int n_parts = (int)std::max<int64_t>(
        1, std::min<int64_t>({(int64_t)std::thread::hardware_concurrency(), 32, T / 65536 + 1}));
    std::vector<std::vector<int32_t>> part_hist(n_parts);
    std::vector<int> part_bad(n_parts, 0);
    // part p holds the documents doc_order[part_lo(p) .. part_lo(p+1)), about T/n_parts tokens
    auto part_lo = [&](int p) -> int64_t {
        if (p >= n_parts) return D;
        const int64_t want = T / n_parts * p;
        return std::lower_bound(order_tokens.begin(), order_tokens.end(), want) - order_tokens.begin();
    };
    const bool counted = parallel_chunks(n_parts, [&](int p) {
        auto& hist = part_hist[p];
        hist.assign((size_t)V, 0);
        for (int64_t i = part_lo(p); i < part_lo(p + 1); ++i) {
            const int64_t d = doc_order[(size_t)i];
            for (int64_t t = start_of(d); t < start_of(d) + len_of(d); ++t) {
                const int32_t w = word_ids[t];
                if (w < 0 || w >= V) { part_bad[p] = 1; return; }
                ++hist[w];
            }
        }
    });
    if (!counted) return fail(MLDA_ENOMEM, "out of host memory");
    for (int p = 0; p < n_parts; ++p)
        if (part_bad[p]) return fail(MLDA_EINVAL, "word id outside [0, V)");

    size_t n_tiles = 0, n_counted = 0, n_segs = 0, n_split = 0;
    for (int32_t v = 0; v < V; ++v) {
        int32_t n = 0;
        for (int p = 0; p < n_parts; ++p) {
            const int32_t c = part_hist[p][v];
            part_hist[p][v] = n;            // becomes the part's offset inside the word
            n += c;
        }
        word_ptr[v + 1] = word_ptr[v] + n;
        n_counted += (size_t)((n + tile_tokens_for(K) - 1) / tile_tokens_for(K));
        n_segs += (size_t)((n + kPhiSegment - 1) / kPhiSegment);
        if (!accumulate && n > kPhiSegment) ++n_split;
    }
    TileShape shape = forced ? *forced : tile_shape_for(K, T);
    auto tiles_of = [&](int32_t tokens) {
        size_t n = 0;
        for (int32_t v = 0; v < V; ++v) n += (size_t)((word_ptr[v + 1] - word_ptr[v] + tokens - 1) / tokens);
        return n;
    };
    if (!forced && shape.alone >= shape.tokens && T <= kFewestTiles * kLeastTile * 4)
        for (int32_t tokens = kLeastTile; tokens < shape.tokens; tokens *= 2)
            if ((int64_t)tiles_of(tokens) <= kFewestTiles) shape = {tokens, tokens};
    for (;;) {
        n_tiles = tiles_of(shape.tokens);
        h.L = chunk_layout(D, T, h.slots_bytes, n_tiles, n_segs, n_split, accumulate);
        // (the bound that a workspace is sized by knows tiles of tile_tokens_for(K))
        if (shape.tokens >= tile_tokens_for(K) || h.L.total <= chunk_layout_bound(D, T, V, K, accumulate).total) break;
        if (shape.tokens < 64) shape = {64, 64};
        else shape.tokens = tile_tokens_for(K);
    }
    const int32_t tile = shape.tokens;
    h.n_tiles = (int32_t)n_tiles; h.n_segs = (int32_t)n_segs; h.n_split = (int32_t)n_split;
    h.counted_tiles = (int32_t)n_counted;

    h.release();
    h.pinned = pinned;
    if (pinned) {
        void* p = nullptr;
        if (hipHostMalloc(&p, std::max<size_t>(h.L.static_bytes, 1), hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return fail(MLDA_ENOMEM, "out of pinned host memory");
        }
        h.arena = (unsigned char*)p;
    } else {
        h.arena = (unsigned char*)std::malloc(std::max<size_t>(h.L.static_bytes, 1));
        if (!h.arena) return fail(MLDA_ENOMEM, "out of host memory");
    }
    int32_t* tok_id = (int32_t*)(h.arena + h.L.tok_id);
    int32_t* doc_ptr32 = (int32_t*)(h.arena + h.L.doc_ptr);
    mlda::DocRec* doc_recs = (mlda::DocRec*)(h.arena + h.L.doc_order);
    uint2* row_rec = (uint2*)(h.arena + h.L.row_rec);
    mlda::Tile* tiles = (mlda::Tile*)(h.arena + h.L.tiles);
    mlda::Tile* segs = (mlda::Tile*)(h.arena + h.L.segs);
    int32_t* split_words = (int32_t*)(h.arena + h.L.split);

    // (the slot of every tile's middle document orders the tiles below)
    std::vector<uint32_t> tile_key;
    std::vector<int32_t> tile_base;
    try {
        tile_key.resize(n_tiles);
        tile_base.resize((size_t)V + 1);
    } catch (const std::bad_alloc&) {
        return fail(MLDA_ENOMEM, "out of host memory");
    }
    tile_base[0] = 0;
    for (int32_t v = 0; v < V; ++v)
        tile_base[v + 1] = tile_base[v] + (word_ptr[v + 1] - word_ptr[v] + tile - 1) / tile;
    const bool placed = parallel_chunks(n_parts, [&](int p) {
        auto& start = part_hist[p];
        for (int64_t i = part_lo(p); i < part_lo(p + 1); ++i) {
            const int64_t d = doc_order[(size_t)i];
            for (int64_t t = start_of(d); t < start_of(d) + len_of(d); ++t) {
                const int32_t w = word_ids[t];
                const int32_t in_word = start[w]++;
                tok_id[word_ptr[w] + in_word] = (int32_t)(tok_begin + t);   // the caller's token index keys the uniforms
                // the tile's middle token names the document whose slot is the tile's sort key
                const int32_t in_tile = in_word % tile;
                const int32_t tile_len = std::min(tile, word_ptr[w + 1] - word_ptr[w] - (in_word - in_tile));
                if (in_tile == tile_len / 2) tile_key[(size_t)(tile_base[w] + in_word / tile)] = slot_of[(size_t)d];
            }
        }
    });
    if (!placed) return fail(MLDA_ENOMEM, "out of host memory");
    part_hist.clear();

    for (int64_t d = 0; d < D; ++d) doc_ptr32[d] = (int32_t)start_of(d);
    doc_ptr32[D] = (int32_t)T;
    for (int64_t d = 0; d < D; ++d) row_rec[d] = make_uint2(slot_of[(size_t)d], 0u);
    for (int64_t i = 0; i < D; ++i) {
        const int64_t d = doc_order[(size_t)i];
        doc_recs[i] = mlda::DocRec{(int32_t)start_of(d), (int32_t)len_of(d), slot_of[(size_t)d], (int32_t)d};
    }
    // tiles and phi segments of one word each
    size_t it = 0, is = 0, ip = 0;
    for (int32_t v = 0; v < V; ++v) {
        const int32_t n = word_ptr[v + 1] - word_ptr[v];
        // a tile's `whole` carries its index until the tiles are sorted, then its word's wide row
        // of phi (mark_wide_tiles)
        for (int32_t b = 0; b < n; b += tile, ++it)
            tiles[it] = mlda::Tile{v, word_ptr[v] + b, std::min(tile, n - b), (int32_t)it};
        if (!accumulate && n > kPhiSegment) split_words[ip++] = v;
        for (int32_t b = 0; b < n; b += kPhiSegment)
            segs[is++] = mlda::Tile{v, word_ptr[v] + b, std::min(kPhiSegment, n - b),
                                    accumulate ? 0 : n <= kPhiSegment ? 1 : b == 0 ? -1 : 0};
    }
    try {
        // Sampling tiles run in the order of their middle document (longest documents first;
        // slot offsets rise in that order), not word by word: tiles of different words that
        // are in flight together then walk the theta rows of the same documents, which are
        // fetched from HBM once instead of once per heavy word.  (The paper issues the tiles
        // of heavy words first, Section 6.1.2; here the long-row tiles come first, which also
        // keeps the tail short.)
        std::stable_sort(tiles, tiles + n_tiles, [&](const mlda::Tile& a, const mlda::Tile& b) {
            return tile_key[(size_t)a.whole] < tile_key[(size_t)b.whole];
        });
        std::stable_sort(segs, segs + n_segs,
                         [](const mlda::Tile& a, const mlda::Tile& b) { return a.count > b.count; });
        h.n_shared_segs = h.n_segs;
        while (h.n_shared_segs > 0 && segs[h.n_shared_segs - 1].count <= solo_segment_for(K, T, h.n_segs)) --h.n_shared_segs;
        const int most_changed = changed_cells_for(K);
        h.n_dense_segs = most_changed == 0 ? h.n_segs
            : (int32_t)(std::stable_partition(segs, segs + n_segs, [&](const mlda::Tile& s) { return !(s.whole > 0 && s.count <= most_changed); }) - segs);
        // tiles that hold a whole word of few tokens go last, to be taken in runs by one
        // workgroup each (their order among themselves stays)
        h.n_single = h.n_shared = h.n_tiles;
        if (shape.alone > 0) {
            mlda::Tile* first_solo = std::stable_partition(tiles, tiles + n_tiles, [&](const mlda::Tile& t) { return t.count > shape.alone; });
            h.n_shared = (int32_t)(first_solo - tiles);
        }
        if (runs) {
            mlda::Tile* first_small = std::stable_partition(tiles, tiles + n_tiles, [&](const mlda::Tile& t) {
                const bool whole_word = word_ptr[t.word + 1] - word_ptr[t.word] == t.count;
                return !(whole_word && t.count <= mlda::kRunTileTokens);
            });
            h.n_single = (int32_t)(first_small - tiles);
            h.run_tokens = 0;
            for (const mlda::Tile* t = first_small; t < tiles + n_tiles; ++t) h.run_tokens += t->count;
        }
    } catch (const std::bad_alloc&) {
        return fail(MLDA_ENOMEM, "out of host memory");
    }
    return MLDA_OK;
}

}  // namespace

struct mlda_ctx {
    // ---- the corpus as a whole and the model
    int64_t D_all = 0, T_all = 0;
    int32_t V = 0, K = 0, Kpad = 0;
    double alpha = 0, beta = 0;
    uint64_t seed = 0;
    int32_t iter = 0;
    hipStream_t stream = nullptr;
    int n_cus = 0, lds_limit = 0;
    bool queued = false;                // the sampler's workgroups take tile after tile (large K)
    bool far_weights = false;           // part of p* in device memory (larger K)
    int64_t reorder_by_tiles = kReorderByTiles;         // MLDA_REORDER_BY_TILES: other tokens than these
    bool wide_slot_offsets = false;     // MLDA_WIDE_SLOT_OFFSETS: 64-bit unit addresses whatever the buffer's size
    TileShape shape = {0, 0};           // MLDA_TILE_SHAPE="tokens,alone": this one whatever the sizes
    const TileShape* forced_shape() const { return shape.tokens > 0 ? &shape : nullptr; }
    float* far_pstar = nullptr;
    int32_t near_topics = 0;            // those of them in LDS
    size_t sample_lds = 0;
    int32_t kept_passes = mlda::kLeastKeptPasses;       // K > 2048: of shared walks, see device_limits
    mlda::PhiView phi[2];                // [model_cur] is the current phi; two copies when streamed
    size_t phi_bytes = 0;                // bytes of one copy
    int32_t n_wide = 0;                  // words with an int32 row
    std::vector<int32_t> wide_row;       // [V] host copy of phi[].wide_row
    int32_t* n_k[2] = {nullptr, nullptr};
    int model_cur = 0;
    // resident, K <= kSpareTotals: two copies of n_k, [n_k_cur] is the current one; the theta rebuild clears the
    // other for the next phi rebuild
    int n_k_cur = 0;
    bool spare_n_k_cleared = false;
    double *ll_partial = nullptr, *ll_scalars = nullptr;   // scalars: value, theta sum, document term
    double* lg_table = nullptr;          // lgG(c + alpha) - lgG(alpha), c < 1024, then lgG(alpha)
    double* lg_table_beta = nullptr;     // the same for beta
    unsigned long long* row_entries = nullptr;   // ring: [r % kEntryRing] belongs to rebuild r
    unsigned long long* visited = nullptr;       // theta rebuilds' row entries, one value per workgroup; see visited_of
    int64_t rebuilds = 0;                        // rebuilds launched so far
    unsigned long long* stamps = nullptr;        // resident: [4 i + phase] of timed iteration i, see stamp_start
    int clock_khz = 0;                           // the rate they count at
    int32_t last_step_iters = 0;
    bool last_step_loglik = false;
    bool has_state = false, ll_fresh = false;
    bool phi_of_z = false;              // resident: phi holds the counts of z[cur] (false while, and if, a rebuild has not gone through)
    std::vector<hipEvent_t> events;     // streamed: kVisitEvents per timed visit
    int32_t timed_iters = 0;            // iterations of the last step that carry events or stamps
    // streamed: what mlda_get_timing and mlda_get_sampler_bytes need of every timed chunk visit
    struct Visit {
        int32_t iter_row;               // row of the step's timed iterations
        int64_t T;
        int32_t n_tiles, n_wide_tiles;
        int64_t rebuild;                // number of the theta rebuild the visit's sampling read
        size_t event0;                  // first of its kVisitEvents events
    };
    std::vector<Visit> visit_log;

    // ---- the chunks (one: attached for good; several: attached in turn, Algorithm 1 WorkSchedule2)
    std::vector<HostChunk> chunks;
    bool streamed = false;
    unsigned char* slot_base[2] = {nullptr, nullptr};   // where an attached chunk's layout begins
    uint16_t* slot_z[2] = {nullptr, nullptr};           // streamed: the assignments in document order, see StreamedSlot
    uint16_t* z_host = nullptr;          // streamed: all assignments in the caller's order (pinned)
    hipStream_t copy_stream = nullptr;   // streamed: uploads run beside the kernels,
    hipStream_t down_stream = nullptr;   // and so do the downloads of new assignments
    hipEvent_t z_ready = nullptr;        // the assignments to be downloaded are in document order
    // what a slot holds has arrived | its visit's kernels are done | and its new assignments have reached the host
    hipEvent_t slot_ready[2] = {nullptr, nullptr}, slot_done[2] = {nullptr, nullptr}, slot_free[2] = {nullptr, nullptr};
    int32_t to_store = -1;               // the chunk whose new assignments are yet to be downloaded, or -1; from
    int to_store_slot = 0;               // this slot
    const uint16_t* to_store_z = nullptr;
    std::vector<hipEvent_t> z_stored;    // per chunk: its assignments have reached z_host
    int64_t visits = 0;                  // chunk visits so far (picks the slot)

    // ---- the attached chunk
    const HostChunk* at = nullptr;
    int64_t D = 0, T = 0;
    uint32_t* tok_slot = nullptr;        // [T] slot of the theta row of each word-major token's document
    int32_t *tok_id = nullptr, *doc_map = nullptr, *doc_ptr = nullptr;
    uint2* doc_pairs = nullptr;          // streamed: {slot of the token's document, its topic}, document order
    mlda::DocRec* doc_order = nullptr;   // documents by falling length, as the theta rebuild walks them
    // a launch of the theta rebuild: D documents of doc_order from `first` on
    struct ThetaLaunch {
        int64_t first = 0, D = 0;
        int ranked = 0;                  // documents per wave of theta_ranked_kernel, 0: theta_rows_kernel
        bool long_docs = false;
        size_t lds = 0;
        int32_t grid = 0;
    };
    ThetaLaunch theta[2];                // documents too long to be ranked, all others (either may have none)
    int32_t theta_grid = 0;              // partials that the last rebuild left
    size_t both_lds = 0;                 // LDS of theta's workgroups where one launch rebuilds phi, too; 0: it does not
    RowKind rows = RowKind::packed;
    bool wide_counters = false, short_docs = true;
    int32_t* split_words = nullptr;
    uint16_t* z[2] = {nullptr, nullptr}; // word-major assignments
    uint16_t* z_doc = nullptr;           // streamed: the same in document order
    int cur = 0;
    uint2* row_rec = nullptr;
    unsigned char* slots = nullptr;
    size_t slots_bytes = 0;
    mlda::Tile* tiles = nullptr;         // sampling tiles
    mlda::Tile* segs = nullptr;          // phi rebuild segments
    int32_t n_tiles = 0, n_segs = 0, n_shared_segs = 0, n_split = 0, n_wide_tiles = 0;
    int32_t n_single = 0;                // the tiles from this one on hold whole small words
    int32_t n_shared = 0;                // tiles taken by workgroups of several waves, the rest by a wave each
    int32_t counted_tiles = 0;           // see HostChunk
    int32_t forced_run = 0;             // MLDA_RUN_TILES: so few workgroups that each takes so many tiles on the whole
    int64_t run_tokens = 0;              // tokens of the tiles that hold whole small words

    // large transfers between the device and the caller's memory (see on_workers): pinned pieces,
    // made by the first of them, one per worker thread
    unsigned char* ring = nullptr;
    std::vector<hipEvent_t> ring_events;
    bool ring_failed = false;

    int static_device = -1;              // >= 0: the workspace is that device's static array
};

// Workspace of contexts made by mlda_create_static: device memory that belongs to the library's
// code object, one copy per GPU, held until the process ends.  In host code the array's name
// is only a handle for hipGetSymbolAddress; kernels and copies take the address it returns.
static __device__ __align__(256) unsigned char scratch[MLDA_STATIC_WORKSPACE_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[kMaxDevices] = {};      // address of `scratch` on each device, once known
const mlda_ctx* g_scratch_user[kMaxDevices] = {};    // the live context that works in it, if any

// The current device's copy of `scratch`, claimed for `user`.  One context per device at a time.
int claim_scratch(const mlda_ctx* user, int* device, unsigned char** ptr) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(MLDA_ENOTSUP, "device index beyond the library's table");
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_user[dev])
        return fail(MLDA_EINVAL, "this device's static workspace is in use by another context: "
                                 "destroy that context first");
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || ((uintptr_t)p) % kAlign != 0) return fail(MLDA_EHIP, "static workspace has no usable address");
        g_scratch_ptr[dev] = (unsigned char*)p;
    }
    g_scratch_user[dev] = user;
    *device = dev;
    *ptr = g_scratch_ptr[dev];
    return MLDA_OK;
}

void release_scratch(const mlda_ctx* user) {
    if (user->static_device < 0) return;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_user[user->static_device] == user) g_scratch_user[user->static_device] = nullptr;
}

int launch_check(const char* what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(MLDA_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    return MLDA_OK;
}

const int32_t* current_n_k(const mlda_ctx* c) { return c->n_k[c->streamed ? c->model_cur : c->n_k_cur]; }

int blocks_for(int64_t n, int per) { return (int)((n + per - 1) / per); }

// Tokens of the longest document that is rebuilt by ranks.
int64_t ranked_longest(const HostChunk& h) { return std::min<int64_t>(h.longest_doc, mlda::kRankedTokens); }

// Point the context at chunk h in workspace part `base` (no data moves).
void point_at(mlda_ctx* c, const HostChunk& h, unsigned char* base) {
    c->at = &h;
    c->D = h.D; c->T = h.T;
    c->rows = h.rows;
    c->wide_counters = h.wide_counters;
    c->short_docs = h.short_docs;
    c->slots_bytes = h.slots_bytes;
    c->n_tiles = h.n_tiles; c->n_segs = h.n_segs; c->n_shared_segs = h.n_shared_segs; c->n_split = h.n_split;
    c->n_wide_tiles = h.n_wide_tiles;
    c->n_single = h.n_single;
    c->n_shared = h.n_shared;
    c->counted_tiles = h.counted_tiles;
    c->run_tokens = h.run_tokens;
    c->tok_slot = (uint32_t*)(base + h.L.tok_slot);
    c->tok_id = (int32_t*)(base + h.L.tok_id);
    c->doc_map = (int32_t*)(base + h.L.doc_map);
    c->doc_pairs = (uint2*)(base + h.L.doc_pairs);
    c->doc_ptr = (int32_t*)(base + h.L.doc_ptr);
    c->doc_order = (mlda::DocRec*)(base + h.L.doc_order);
    c->row_rec = (uint2*)(base + h.L.row_rec);
    c->tiles = (mlda::Tile*)(base + h.L.tiles);
    c->segs = (mlda::Tile*)(base + h.L.segs);
    c->split_words = (int32_t*)(base + h.L.split);
    c->z[0] = (uint16_t*)(base + h.L.z0);
    c->z[1] = (uint16_t*)(base + h.L.z1);
    c->slots = base + h.L.slots;
    c->cur = 0;
    // Ranks, but for 32-bit counters and documents beyond kRankedTokens: few of those are rebuilt with a dense row in a
    // launch of their own, and where documents are long on the whole all of them are.  Two documents per wave where
    // a half-wave suits them: few topics, short documents.
    // Ranks / dense row, rebuild of 3e6 tokens from random topics (trained: alike), us:
    //   tokens       10         40        100       400      1,000     3,000
    //   K = 100   86 / 145   35 / 94    28 / 73   25 / 65   37 / 52   70 / 51
    //     1,000   86 / 128   35 / 82    29 / 72   28 / 66   42 / 61   79 / 57
    //     5,000  150 / 284   47 / 123   30 / 84   28 / 60   54 / 52  155 / 59
    //    30,000  295 / 2753  89 / 1142  49 / 568  38 / 228  65 / 154 203 / 125
    const bool all_long = long_docs_for(h.D, h.T, h.longest_doc, c->n_cus);
    const bool dense = h.wide_counters || all_long || h.T > 1500 * h.D;
    const int64_t n_dense = dense ? h.D : h.n_unranked;
    c->theta[0] = c->theta[1] = mlda_ctx::ThetaLaunch();
    c->theta[0].D = n_dense;
    c->theta[0].long_docs = dense ? all_long : long_docs_for(n_dense, h.unranked_tokens, h.longest_doc, c->n_cus);
    c->theta[0].lds = mlda::theta_lds_bytes(c->K, h.wide_counters);
    c->theta[1].first = n_dense;
    c->theta[1].D = h.D - n_dense;
    c->theta[1].ranked = c->K <= mlda::kPairMaxK && h.T <= 160 * h.D ? 2 : 1;
    c->theta[1].lds = mlda::theta_rank_lds_bytes(c->K, ranked_longest(h), c->theta[1].ranked);
    for (mlda_ctx::ThetaLaunch& l : c->theta) {
        // 16 one-wave workgroups per CU: enough to hide the gathers' latency; more of them
        // touch more lines of z at once than an XCD's L2 holds, and neighbours stop sharing
        const int per_cu = std::max(1, std::min(16, (int)(144 * 1024 / l.lds)));
        l.grid = (int32_t)std::min<int64_t>({l.D, (int64_t)c->n_cus * per_cu, (int64_t)kMaxThetaGrid});
    }
    const size_t both = mlda::theta_rank_lds_bytes(c->K, ranked_longest(h), c->theta[1].ranked, 4);
    c->both_lds = !c->streamed && n_dense == 0 && h.T > 0 && h.T <= kBothTokens && c->K <= kBothTopics && both <= 40 * 1024 ? both : 0;
}

// After the static part of a chunk has arrived: the index arrays that follow from it
// (document->token map, slot of every token's theta row), and what a lane of the sampler
// reads when it has no entries of its own: padding entries (count 0, topic K) in the 64 bytes
// before the first slot.  A streamed chunk arrives with its assignments in document order
// and hands them back so: its theta rebuilds read them directly and it needs no map (building
// one costs as much as a theta rebuild); the tokens' slots come with its assignments (see attach).
void derive_chunk_arrays(mlda_ctx* c) {
    if (!c->streamed && c->T > 0) {
        hipLaunchKernelGGL(mlda::derive_doc_map_kernel, dim3(blocks_for(c->T, 256)), dim3(256), 0, c->stream,
                           c->tok_id, c->T, c->at->tok_begin, c->doc_map);
        const int grid = (int)std::min<int64_t>(c->D, (int64_t)c->n_cus * 32);
        hipLaunchKernelGGL(mlda::derive_tok_slot_kernel, dim3((unsigned)grid), dim3(mlda::kWave), 0, c->stream,
                           c->doc_order, c->D, c->doc_map, c->tok_slot);
        // from here on the map lists a document's tokens by rising place in z
        hipLaunchKernelGGL(mlda::sort_doc_map_kernel, dim3((unsigned)grid), dim3(mlda::kWave), 0, c->stream,
                           c->doc_order, c->D, c->doc_map);
    }
    const uint32_t pad = with_layout(c->rows, [&](auto layout) {
        return (uint32_t)layout.make(0, c->K) * (layout.kEntryBytes == 2 ? 0x10001u : 1u);
    });
    static_assert(kSlotAlign >= (mlda::kKeptUnits + 1) * 16, "the padding units lie before the first slot");
    hipLaunchKernelGGL(mlda::fill_i32_kernel, dim3(1), dim3(256), 0, c->stream, (int32_t*)c->slots,
                       (int64_t)(kSlotAlign / 4), (int32_t)pad);
}

// Streamed: the assignments that are yet to be downloaded are put on their way, on a stream of their own.
int store_z(mlda_ctx* c) {
    if (c->to_store < 0) return MLDA_OK;
    const HostChunk& h = c->chunks[(size_t)c->to_store];
    HIP_TRY(hipStreamWaitEvent(c->down_stream, c->z_ready, 0));
    HIP_TRY(hipMemcpyAsync(c->z_host + h.tok_begin, c->to_store_z, (size_t)h.T * 2, hipMemcpyDeviceToHost, c->down_stream));
    HIP_TRY(hipEventRecord(c->z_stored[(size_t)c->to_store], c->down_stream));
    HIP_TRY(hipEventRecord(c->slot_free[c->to_store_slot], c->down_stream));
    c->to_store = -1;
    return MLDA_OK;
}

// Streamed: bring chunk m into the slot of this visit.  The static part (and with_z: the
// chunk's assignments, caller's order, into z_doc) is copied on the copy stream, so that it
// overlaps the kernels of the chunk before; the context's stream then waits for it and, with_z,
// also puts the assignments in word-major order into z[0].
int attach(mlda_ctx* c, int32_t m, bool with_z, hipEvent_t* ev = nullptr) {
    const HostChunk& h = c->chunks[(size_t)m];
    const int s = (int)(c->visits % 2);
    c->visits += 1;
    point_at(c, h, c->slot_base[s]);
    c->z_doc = c->slot_z[s];
    if (c->to_store >= 0 && (c->to_store == m || c->to_store_slot == s)) RC_TRY(store_z(c));
    // the slot's previous user must be done (its assignments may still be on their way to the host: no chunk's
    // layout reaches them, see StreamedSlot), and this chunk's last assignments stored
    HIP_TRY(hipStreamWaitEvent(c->copy_stream, c->slot_done[s], 0));
    if (h.L.static_bytes > 0)
        HIP_TRY(hipMemcpyAsync(c->slot_base[s], h.arena, h.L.static_bytes, hipMemcpyHostToDevice,
                               c->copy_stream));
    HIP_TRY(hipStreamWaitEvent(c->copy_stream, c->slot_free[s], 0));
    if (with_z && h.T > 0) {
        HIP_TRY(hipStreamWaitEvent(c->copy_stream, c->z_stored[(size_t)m], 0));
        HIP_TRY(hipMemcpyAsync(c->z_doc, c->z_host + h.tok_begin, (size_t)h.T * 2, hipMemcpyHostToDevice,
                               c->copy_stream));
    }
    HIP_TRY(hipEventRecord(c->slot_ready[s], c->copy_stream));
    RC_TRY(store_z(c));         // (of the chunk before, see store_z_and_release)
    HIP_TRY(hipStreamWaitEvent(c->stream, c->slot_ready[s], 0));
    if (ev) HIP_TRY(hipEventRecord(ev[0], c->stream));
    derive_chunk_arrays(c);
    if (with_z && h.T > 0) {
        // every token's topic is paired with the slot of its document's theta row where both
        // are contiguous, and the pairs are then brought to word-major order in one gather
        const int grid = (int)std::min<int64_t>(h.D, (int64_t)c->n_cus * 32);
        hipLaunchKernelGGL(mlda::pair_topics_with_slots_kernel, dim3((unsigned)grid), dim3(mlda::kWave), 0,
                           c->stream, c->doc_order, h.D, c->z_doc, c->doc_pairs);
        hipLaunchKernelGGL(mlda::pairs_to_word_major_kernel, dim3(blocks_for(h.T, 256)), dim3(256), 0,
                           c->stream, c->doc_pairs, c->tok_id, c->z[0], c->tok_slot, h.T, h.tok_begin);
    }
    if (ev) HIP_TRY(hipEventRecord(ev[1], c->stream));
    return launch_check("attaching a chunk");
}

// Streamed: new word-major assignments of the attached chunk, put in document order too.
int to_document_order(mlda_ctx* c, const uint16_t* z_word) {
    if (c->T > 0)
        hipLaunchKernelGGL(mlda::to_doc_major_scatter_kernel, dim3(blocks_for(c->T, 256)), dim3(256), 0,
                           c->stream, z_word, c->tok_id, c->z_doc, c->T, c->at->tok_begin);
    return launch_check("to_doc_major_scatter_kernel");
}

// Streamed: the attached chunk's visit is over.  `store`: its assignments (z_doc) are to go to the host as soon as they are made.  The
// copy is put into its queue by store_z, behind the next chunk's uploads: streams share hardware queues (four in a process: those
// of a second context already), and a copy in front of the uploads that waits for this chunk's kernels would make them wait, too.
// Two iterations with their outputs fetched, ms, the copy queued before the next uploads / after them / after the next theta rebuild:
//   9.9e7 tokens in 4 chunks, first context of a process 31.2/31.2/31.8, second 54.0/34.6/38.7, third 48.4/48.1/48.4
// An iteration as a share of one with the copy queued before the next uploads, in the mean over corpora of 25 to 10,000 tokens a
// document, after them / after the next theta rebuild:
//   tokens a chunk   1e4        5e4        1.5e5      4e5        1.2e6      4e6
//   2 chunks         0.91/0.95  0.90/0.93  0.92/0.95  0.88/0.91  1.00/1.03  1.00/1.04
//   4                0.91/0.95  0.92/0.93  0.95/0.96  0.92/0.96  1.03/1.10  1.01/1.04
//   6                0.92/0.97  0.93/0.95  0.97/0.98  0.94/1.01  1.03/1.17  1.01/1.03
//   12               0.93/0.98  0.96/0.98  0.99/1.00  0.97/1.06  1.00/1.18  1.03/1.17
int store_z_and_release(mlda_ctx* c, int32_t m, bool store) {
    const int s = (int)((c->visits - 1) % 2);
    HIP_TRY(hipEventRecord(c->slot_done[s], c->stream));
    if (store && c->T > 0) {
        RC_TRY(store_z(c));
        HIP_TRY(hipEventRecord(c->z_ready, c->stream));
        c->to_store = m;
        c->to_store_slot = s;
        c->to_store_z = c->z_doc;
    } else {
        HIP_TRY(hipEventRecord(c->slot_free[s], c->stream));
    }
    return MLDA_OK;
}

// The topic totals that a theta rebuild clears.
int32_t* old_totals(const mlda_ctx* c) { return !c->streamed && c->n_k[0] != c->n_k[1] ? c->n_k[c->n_k_cur ^ 1] : nullptr; }

// The counts that theta rebuild number `rebuild` leaves (the next phi rebuild reads them while the next theta rebuild
// may already leave its own).
unsigned long long* visited_of(const mlda_ctx* c, int64_t rebuild) { return c->visited + (rebuild & 1) * kMaxThetaGrid; }

mlda::ThetaRankedArgs ranked_args(const mlda_ctx* c, const mlda_ctx::ThetaLaunch& l, const uint16_t* z, unsigned long long* started,
                                  int32_t n_before) {
    using namespace mlda;
    const int64_t longest = ranked_longest(*c->at);
    const int docs = std::max(l.ranked, 1);         // (0: not ranked, what the ranks need is not read)
    return {c->doc_order + l.first, c->streamed ? nullptr : c->doc_map, z, c->row_rec, c->slots, l.D, c->T, c->K, c->alpha,
            c->lg_table, visited_of(c, c->rebuilds), c->ll_partial + 2 * kLoglikBlocks, old_totals(c), started,
            theta_rank_cells(c->K, longest, docs), theta_rank_stage(longest, docs), n_before,
            (int32_t)theta_rank_wave_bytes(c->K, longest, docs)};
}

// phi (into n_wk[which]) from the attached chunk's assignments z (word-major).  One chunk:
// rows are stored and n_k follows; several: the chunk's counts are added to a phi that was
// zeroed before the first chunk, and n_k is formed after the last (finish_model).
// `with_theta`: theta's rows, too, in the same launch.
// `z_old`: the assignments whose counts phi holds, if it does.
int rebuild_phi(mlda_ctx* c, const uint16_t* z, int which, const uint16_t* z_old = nullptr, unsigned long long* started = nullptr,
                bool with_theta = false, unsigned long long* theta_started = nullptr) {
    using namespace mlda;
    int32_t* n_k = nullptr;
    int32_t n_totals = 0;           // workgroups of the phi launch that count the topic totals
    const bool from_rows = (int64_t)c->V * c->K * 2 < c->T;
    if (!c->streamed) {
        const bool spare = c->n_k[0] != c->n_k[1];
        const bool cleared = spare && c->spare_n_k_cleared;
        if (spare) { c->n_k_cur ^= 1; c->spare_n_k_cleared = false; }
        n_k = c->n_k[c->n_k_cur];
        if (c->n_split > 0 || !cleared) {
            const dim3 grid((unsigned)c->n_split + 1u, (unsigned)blocks_for(c->K, 256));
            hipLaunchKernelGGL(zero_sums_kernel, grid, dim3(256), 0, c->stream, c->split_words, c->phi[which], c->K,
                               cleared ? (int32_t*)nullptr : n_k, started);
            started = nullptr;
        }
        // n_k comes from the fresh n_wk where that is fewer bytes than z (and no LDS atomics); else from z, beside
        // phi while the counters of both leave room for many workgroups per CU
        if (!from_rows && c->K <= kSpareTotals) n_totals = (int32_t)std::min<int64_t>((c->T + 8191) / 8192, (int64_t)c->n_cus * 2);
    }
    unsigned long long* visited_sum =
        !c->streamed && c->rebuilds > 0 ? c->row_entries + ((c->rebuilds - 1) % kEntryRing) : nullptr;
    const int32_t n_segs = z_old ? c->at->n_dense_segs : c->n_segs, n_shared = std::min(c->n_shared_segs, n_segs);
    const int32_t solo_groups = (n_segs - n_shared + kPhiWaves - 1) / kPhiWaves;
    const size_t phi_lds = phi_counter_bytes(c->K) * (solo_groups > 0 ? kPhiWaves : 1);
    const int32_t changed_blocks = std::min(c->n_segs - n_segs, c->n_cus * (int32_t)std::max<size_t>(1, std::min<size_t>(8, kLdsPerWorkgroup / phi_lds)));
    const unsigned blocks = (unsigned)(changed_blocks + n_shared + solo_groups + n_totals + (visited_sum ? 1 : 0));
    const PhiArgs p = {c->segs, n_segs, n_shared, c->n_segs - n_segs, changed_blocks, z_old, z, c->phi[which], c->K, c->T, n_totals, n_k,
                       visited_of(c, c->rebuilds - 1), c->theta_grid, visited_sum, started};
    if (with_theta) {
        const mlda_ctx::ThetaLaunch& l = c->theta[1];
        const ThetaRankedArgs t = ranked_args(c, l, z, theta_started, 0);
        const int32_t n_theta = (l.grid + 3) / 4;
        with_layout(c->rows, [&](auto layout) {
            typedef decltype(layout) Layout;
            hipLaunchKernelGGL((l.ranked == 2 ? rebuild_kernel<Layout, 2> : rebuild_kernel<Layout, 1>), dim3(blocks + (unsigned)n_theta),
                               dim3(256), std::max(phi_lds, c->both_lds), c->stream, p, t, (int32_t)blocks, n_theta);
            return 0;
        });
        RC_TRY(launch_check("rebuild kernel"));         // (a launch that failed has cleared no totals)
        c->spare_n_k_cleared = t.old_n_k != nullptr;
        c->theta_grid = 4 * n_theta;
        c->rebuilds += 1;
    } else if (blocks > 0) {
        hipLaunchKernelGGL((c->K <= kPhiDwordTopics ? phi_tile_kernel<false> : phi_tile_kernel<true>), dim3(blocks), dim3(256),
                           phi_lds, c->stream, p);
    } else if (started) {
        hipLaunchKernelGGL(stamp_kernel, dim3(1), dim3(1), 0, c->stream, started);
    }
    if (!c->streamed && c->T > 0 && n_totals == 0) {        // (streamed: after the last chunk)
        if (from_rows) {
            const int words_per_slice = 64;
            dim3 grid((unsigned)blocks_for(c->K, 256), (unsigned)blocks_for(c->V, words_per_slice));
            hipLaunchKernelGGL(topic_totals_from_rows_kernel, grid, dim3(256), 0, c->stream,
                               c->phi[which], c->V, c->n_wide, c->K, words_per_slice, n_k);
        } else {
            // one counter per topic in LDS; K beyond kHistTopics is counted range by range
            const int32_t span = std::min<int32_t>(c->K, kHistTopics);
            const size_t hist_bytes = (size_t)span * 4;
            const int grid = (int)std::min<int64_t>((c->T + 8191) / 8192, (int64_t)c->n_cus * 2);
            if (c->K <= kHistTopics)
                hipLaunchKernelGGL(topic_totals_kernel<false>, dim3((unsigned)grid), dim3(256), hist_bytes,
                                   c->stream, z, c->T, n_k, c->K, 0, c->K);
            else
                for (int32_t k_lo = 0; k_lo < c->K; k_lo += span)
                    hipLaunchKernelGGL(topic_totals_kernel<true>, dim3((unsigned)grid), dim3(256), hist_bytes,
                                       c->stream, z, c->T, n_k, c->K, k_lo, std::min(span, c->K - k_lo));
        }
    }
    return launch_check("phi rebuild kernels");
}

// Streamed: phi[which] starts at zero before the first chunk adds to it ...
int begin_model(mlda_ctx* c, int which) {
    const int64_t dwords = (int64_t)(c->phi_bytes / 4);
    hipLaunchKernelGGL(mlda::fill_i32_kernel, dim3(blocks_for(dwords, 256)), dim3(256), 0, c->stream,
                       (int32_t*)c->phi[which].narrow, dwords, 0);
    return launch_check("fill_i32_kernel");
}

// ... and n_k[which] is its column sums after the last.
int finish_model(mlda_ctx* c, int which) {
    hipLaunchKernelGGL(mlda::fill_i32_kernel, dim3(blocks_for(c->K, 256)), dim3(256), 0, c->stream,
                       c->n_k[which], (int64_t)c->K, 0);
    const int words_per_slice = 64;
    dim3 grid((unsigned)blocks_for(c->K, 256), (unsigned)blocks_for(c->V, words_per_slice));
    hipLaunchKernelGGL(mlda::topic_totals_from_rows_kernel, grid, dim3(256), 0, c->stream, c->phi[which],
                       c->V, c->n_wide, c->K, words_per_slice, c->n_k[which]);
    return launch_check("topic totals");
}

// theta rows of the attached chunk from its assignments: z word-major, reached through the
// document->token map; streamed: z = z_doc, read directly.  Leaves the rows' part of the
// log-likelihood as one partial per workgroup in ll_partial[2 kLoglikBlocks ..].
int rebuild_theta(mlda_ctx* c, const uint16_t* z, unsigned long long* started = nullptr) {
    using namespace mlda;
    if (c->D == 0 && started) hipLaunchKernelGGL(stamp_kernel, dim3(1), dim3(1), 0, c->stream, started);
    if (c->D > 0) {
        int32_t* old_n_k = old_totals(c);
        int32_t n_before = 0;
        c->theta_grid = 0;
        for (const mlda_ctx::ThetaLaunch& l : c->theta) {
            if (l.D == 0) continue;
            ThetaRankedArgs a = ranked_args(c, l, z, started, n_before);
            void* dense[] = {&a.docs, &a.doc_map, &a.z, &a.row_rec, &a.slots, &a.D, &a.T, &a.K, &a.alpha, &a.lg_table,
                             &a.visited_partial, &a.ll_partial, &a.old_n_k, &a.started};
            void* ranked[] = {&a};
            HIP_TRY(hipLaunchKernel(l.ranked ? theta_ranked_kernel_for(c->rows, l.ranked)
                                             : theta_kernel_for(c->rows, c->wide_counters, l.long_docs),
                                    dim3((unsigned)l.grid), dim3((unsigned)(l.long_docs ? kWave * kLongDocWaves : kWave)),
                                    l.ranked ? ranked : dense, l.lds, c->stream));
            n_before = l.grid;
            c->theta_grid = std::max(c->theta_grid, l.grid);
            started = nullptr;
        }
        c->spare_n_k_cleared = old_n_k != nullptr;
        // (one chunk: the next rebuild_phi adds the counts up; sampler bytes are asked of earlier ones only)
        if (c->streamed)
            hipLaunchKernelGGL(visited_sum_kernel, dim3(1), dim3(256), 0, c->stream, visited_of(c, c->rebuilds), c->theta_grid,
                               c->row_entries + (c->rebuilds % kEntryRing));
    }
    c->rebuilds += 1;
    return launch_check("theta rebuild kernel");
}

int launch_sampler(mlda_ctx* c, const uint16_t* z_cur, uint16_t* z_next, unsigned long long* started = nullptr) {
    if (c->n_tiles == 0) {
        if (started) hipLaunchKernelGGL(mlda::stamp_kernel, dim3(1), dim3(1), 0, c->stream, started);
        return launch_check("stamp_kernel");
    }
    mlda::SampleArgs a;
    a.started = started;
    a.tiles = c->tiles;
    a.tok_slot = c->tok_slot;
    a.tok_id = c->tok_id;
    a.z_cur = z_cur;
    a.z_next = z_next;
    a.slots = c->slots;
    a.phi = c->phi[c->model_cur];
    a.n_k = current_n_k(c);
    a.K = c->K;
    a.Kpad = c->Kpad;
    a.alpha = c->alpha;
    a.beta = c->beta;
    a.beta_V = c->beta * (double)c->V;
    a.seed = c->seed;
    a.iter = (uint32_t)(c->iter + 1);
    a.n_tiles = c->n_shared;
    a.n_single = c->queued ? c->n_single : c->n_shared;
    a.far_pstar = c->far_pstar;
    a.near_topics = c->near_topics;
    a.next_tile = (uint32_t*)(c->ll_scalars + 4);
    // With few tiles the launch takes the time of one tile, and a small tile is done sooner by four waves side
    // by side than by one with a full batch; with more it is the work in all that counts, and later so where
    // rows are long and a pass takes few of a batch's tokens anyway.  Batches of at least 16 / 64 tokens,
    // tiles of 60 tokens (of 300: alike), us:
    //   tiles                              768          1,400        2,040
    //   documents of 40,  K = 100     10.2 / 11.3   14.4 / 12.6   16.6 / 14.2
    //                300, K = 100     10.8 / 12.0   14.7 / 13.6   17.6 / 15.8
    //                300, K = 1,000   13.9 / 18.6   20.3 / 21.8   24.0 / 25.0
    const bool long_rows = c->K >= 200 && c->T >= 200 * c->D;
    a.min_batch = c->n_shared <= (long_rows ? 8 : 4) * c->n_cus ? mlda::kMinBatch * 2 : mlda::kWave;
    const int waves = sample_waves_for(c->K);
    int32_t grid = a.n_tiles;
    if (c->queued) grid = std::min({grid, (waves == 12 ? 2 : 1) * c->n_cus, c->far_weights ? kFarStrips : INT32_MAX});
    if (c->queued && c->forced_run > 0) grid = std::min(grid, (a.n_tiles + c->forced_run - 1) / c->forced_run);
    const bool near = slots_near(c->slots_bytes) && !c->wide_slot_offsets;
    const int weight_bytes = c->rows == RowKind::packed ? 4 : 8;
    const bool shares = !few_topics_of_many_tokens(c->K, c->T);
    const KeptSums kept = shares ? kept_sums_for(c->Kpad, 4) : KeptSums{0, 0};
    const KeptSums kept_solo = shares ? kept_sums_for(c->Kpad, 1) : KeptSums{0, 0};
    a.kept_passes = kept.passes;
    a.kept_sums = kept.sums;
    a.sum_slack = c->beta >= kSlackBeta ? 3u << 20 : 0u;
    const bool alone = c->T < kAloneDocs * c->D;
    if (waves > 4) {
        a.kept_passes = c->kept_passes;
        a.kept_sums = mlda::lane_sums_for(c->kept_passes);
    } else if (weight_bytes != 8) {
        a.kept_passes = a.kept_sums = 0;
    }
    const size_t lds = waves == 4 ? mlda::sample_lds_bytes(c->Kpad, waves, weight_bytes, a.kept_passes, a.kept_sums) : c->sample_lds;
    void* kernel_args[] = {&a};
    if (grid > 0)
        HIP_TRY(hipLaunchKernel(sample_kernel_for(c->K, c->rows, c->short_docs, alone, near), dim3((unsigned)grid),
                                dim3((unsigned)(waves * mlda::kWave)), kernel_args, lds, c->stream));
    const int32_t n_solo = c->n_tiles - c->n_shared;
    if (n_solo > 0) {
        if (grid > 0) a.started = nullptr;
        a.tiles += c->n_shared;
        if (weight_bytes == 8) {
            a.kept_passes = kept_solo.passes;
            a.kept_sums = kept_solo.sums;
        }
        a.n_tiles = a.n_single = n_solo;
        HIP_TRY(hipLaunchKernel(near ? sample_solo_kernel_of<true>(c->rows) : sample_solo_kernel_of<false>(c->rows),
                                dim3((unsigned)n_solo), dim3((unsigned)mlda::kWave), kernel_args,
                                mlda::sample_lds_bytes(c->Kpad, 1, weight_bytes, a.kept_passes, a.kept_sums), c->stream));
    }
    return launch_check("sample_kernel");
}

// The word side of the log-likelihood and the value: with the theta partials that the last
// rebuild_theta left (one chunk), or their sum over all chunks (streamed), and the documents' term.
int launch_loglik(mlda_ctx* c, unsigned long long* started = nullptr) {
    using namespace mlda;
    const int64_t cells = (int64_t)c->V * c->K, wide_cells = (int64_t)c->n_wide * c->K;
    // a thread reads 16 bytes at a time
    const int64_t wanted = std::max(cells / 8, wide_cells / 4) / 256 + 1;
    const bool by_words = !c->streamed && c->at->n_dense_segs < c->n_segs, small = !by_words && wanted <= kSmallLoglikBlocks;
    const int blocks = small ? (int)wanted : kLoglikBlocks;
    const double* theta_partial = c->ll_partial + 2 * kLoglikBlocks;
    const int n_theta = c->streamed ? 0 : c->theta_grid;
    const double* theta_sum = c->streamed ? c->ll_scalars + 1 : nullptr;
    const double* doc_term = c->ll_scalars + 2;
    if (by_words)
        hipLaunchKernelGGL(loglik_word_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, c->stream, c->segs, c->at->n_dense_segs,
                           c->n_segs, c->z[c->cur], c->phi[0], current_n_k(c), c->K, c->beta, (double)c->V * c->beta,
                           c->lg_table_beta, c->ll_partial, started);
    else
        hipLaunchKernelGGL(loglik_word_side_kernel, dim3((unsigned)blocks), dim3(256), 0, c->stream,
                       c->phi[c->model_cur], cells, wide_cells, current_n_k(c), c->K, c->beta,
                       (double)c->V * c->beta, c->lg_table_beta, c->ll_partial, theta_partial, n_theta, theta_sum,
                       doc_term, small ? (unsigned int*)(c->ll_scalars + 3) : (unsigned int*)nullptr, c->ll_scalars, started);
    if (!small)
        hipLaunchKernelGGL(loglik_value_kernel, dim3(1), dim3(256), 0, c->stream, c->ll_partial, blocks, theta_partial,
                           n_theta, theta_sum, doc_term, c->ll_scalars);
    c->ll_fresh = true;
    return launch_check("log-likelihood kernel");
}

// Streamed: the theta partials of the chunk just rebuilt are added to the running sum ...
int add_theta_loglik(mlda_ctx* c, bool first) {
    hipLaunchKernelGGL(mlda::loglik_final_kernel, dim3(1), dim3(256), 0, c->stream,
                       c->ll_partial + 2 * kLoglikBlocks, c->D > 0 ? c->theta_grid : 0, first ? 0 : 1,
                       c->ll_scalars + 1);
    return launch_check("loglik_final_kernel");
}

int need_state(const mlda_ctx* c) {
    if (!c) return fail(MLDA_EINVAL, "null context");
    if (!c->has_state)
        return fail(MLDA_EINVAL, "no topic assignments yet: call mlda_init_random or mlda_set_assignments");
    return MLDA_OK;
}

int check_corpus(const int64_t* doc_ptr, const int32_t* word_ids, bool need_words, int64_t D, int32_t V,
                 int32_t K, double alpha, double beta) {
    if (!doc_ptr) return fail(MLDA_EINVAL, "doc_ptr is null");
    if (D < 0 || V < 1) return fail(MLDA_EINVAL, "need D >= 0 and V >= 1");
    if (K < 1 || K > 65535) return fail(MLDA_EINVAL, "K must be in [1, 65535] (16-bit topic indices)");
    if (!(alpha > 0.0) || !(beta > 0.0) || !std::isfinite(alpha) || !std::isfinite(beta))
        return fail(MLDA_EINVAL, "alpha and beta must be positive and finite");
    if (doc_ptr[0] != 0) return fail(MLDA_EINVAL, "doc_ptr[0] must be 0");
    for (int64_t d = 0; d < D; ++d)
        if (doc_ptr[d + 1] < doc_ptr[d]) return fail(MLDA_EINVAL, "doc_ptr must be non-decreasing");
    if (doc_ptr[D] >= ((int64_t)1 << 31)) return fail(MLDA_EINVAL, "2^31 or more tokens");
    if (need_words && doc_ptr[D] > 0 && !word_ids) return fail(MLDA_EINVAL, "word_ids is null");
    return MLDA_OK;
}

int check_workspace(void* dev_workspace, size_t have, size_t need) {
    if (!dev_workspace) return fail(MLDA_EINVAL, "dev_workspace is null");
    if (((uintptr_t)dev_workspace) % kAlign != 0)
        return fail(MLDA_EINVAL, "dev_workspace must be 256-byte aligned");
    if (have < need)
        return fail(MLDA_ENOMEM, "workspace has " + std::to_string(have) + " bytes, need " +
                                     std::to_string(need));
    return MLDA_OK;
}

int check_device_pointer(void* dev_workspace) {
    hipPointerAttribute_t attr;
    hipError_t e = hipPointerGetAttributes(&attr, dev_workspace);
    if (e != hipSuccess || attr.type != hipMemoryTypeDevice) {
        (void)hipGetLastError();
        return fail(MLDA_EINVAL, "dev_workspace is not device memory");
    }
    return MLDA_OK;
}

size_t streamed_workspace_bound(const int64_t* doc_ptr, int64_t D, int32_t V, int32_t K, int32_t M) {
    size_t chunk = 0;
    int64_t tokens = 0;
    for (int32_t m = 0; m < M; ++m) {
        const int64_t a = chunk_first(doc_ptr, D, M, m), b = chunk_first(doc_ptr, D, M, m + 1);
        tokens = std::max(tokens, doc_ptr[b] - doc_ptr[a]);
        chunk = std::max(chunk, chunk_layout_bound(b - a, doc_ptr[b] - doc_ptr[a], V, K, true).total);
    }
    return model_layout(V, K, doc_ptr[D], true).total + 2 * mlda::streamed_slot(tokens, chunk).total;
}

// Everything mlda_create and mlda_create_streamed share: device limits, the model's buffers
// and tables.  `chunks` are prepared; `base` is the workspace.
int finish_create(mlda_ctx* c, unsigned char* base, const ModelLayout& ML) {
    for (int i = 0; i < 2; ++i) {
        c->phi[i].narrow = (uint16_t*)(base + ML.phi[i]);
        c->phi[i].wide = (int32_t*)(base + ML.phi[i] + ML.phi_wide);
        c->phi[i].wide_row = (const int32_t*)(base + ML.wide_row);
    }
    c->phi_bytes = ML.phi_bytes;
    HIP_TRY(hipMemcpyAsync(base + ML.wide_row, c->wide_row.data(), (size_t)c->V * 4, hipMemcpyHostToDevice,
                           c->stream));
    c->n_k[0] = (int32_t*)(base + ML.n_k[0]);
    c->n_k[1] = (int32_t*)(base + ML.n_k[1]);
    c->ll_partial = (double*)(base + ML.ll_partial);
    if (!c->streamed && c->K <= kSpareTotals) c->n_k[1] = (int32_t*)(c->ll_partial + kLoglikBlocks);
    c->ll_scalars = (double*)(base + ML.ll_scalars);
    c->lg_table = (double*)(base + ML.lg_table);
    c->lg_table_beta = c->lg_table + mlda::kLgTableSize;
    c->row_entries = (unsigned long long*)(base + ML.row_entries);
    c->visited = (unsigned long long*)(c->ll_partial + 2 * kLoglikBlocks + kMaxThetaGrid);
    c->stamps = (unsigned long long*)(base + ML.stamps);
    c->far_pstar = (float*)(base + ML.far_pstar);

    hipLaunchKernelGGL(mlda::lg_table_kernel, dim3(blocks_for(mlda::kLgTableSize, 256)), dim3(256), 0,
                       c->stream, c->lg_table, c->alpha, (double)c->K * c->alpha);
    hipLaunchKernelGGL(mlda::lg_table_kernel, dim3(blocks_for(mlda::kLgTableSize, 256)), dim3(256), 0,
                       c->stream, c->lg_table_beta, c->beta, (double)c->V * c->beta);
    // rows of words without tokens are never written again: start phi at zero
    const int64_t dwords = (int64_t)(c->phi_bytes / 4);
    hipLaunchKernelGGL(mlda::fill_i32_kernel, dim3(blocks_for(dwords, 256)), dim3(256), 0, c->stream,
                       (int32_t*)c->phi[0].narrow, dwords, 0);
    // launch_loglik's ticket, launch_sampler's next tile, copy_to_host_kernel's counters
    hipLaunchKernelGGL(mlda::fill_i32_kernel, dim3(1), dim3(256), 0, c->stream, (int32_t*)(c->ll_scalars + 3),
                       (int64_t)(2 + kRingWorkers) * 2, 0);
    hipLaunchKernelGGL(mlda::fill_i32_kernel, dim3(blocks_for((int64_t)(kStampBytes / 4), 256)), dim3(256), 0, c->stream,
                       (int32_t*)c->stamps, (int64_t)(kStampBytes / 4), 0);
    RC_TRY(launch_check("model set-up kernels"));
    if (c->sample_lds > 48 * 1024)          // (the workgroups of twelve and sixteen waves only)
        for (bool short_docs : {false, true})
            for (int form = 0; form < 4; ++form)
                // (the attribute belongs to the kernel, not to this context: contexts of different
                // needs may live side by side, so it is raised to what the device allows)
                HIP_TRY(hipFuncSetAttribute(sample_kernel_for(c->K, RowKind::packed, short_docs, (form & 1) != 0, (form & 2) != 0),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, c->lds_limit));
    if ((size_t)c->K * 4 > 48 * 1024) {
        const int hist_bytes = std::min<int32_t>(c->K, kHistTopics) * 4;
        for (const void* kernel : {(const void*)mlda::topic_totals_kernel<false>,
                                   (const void*)mlda::topic_totals_kernel<true>})
            HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, hist_bytes));
    }
    if (c->K <= mlda::kPhiDwordTopics && mlda::kPhiWaves * mlda::phi_counter_bytes(c->K) > 48 * 1024)
        HIP_TRY(hipFuncSetAttribute((const void*)mlda::phi_tile_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)(mlda::kPhiWaves * mlda::phi_counter_bytes(mlda::kPhiDwordTopics))));
    if (mlda::phi_counter_bytes(c->K) > 48 * 1024)
        HIP_TRY(hipFuncSetAttribute((const void*)mlda::phi_tile_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)mlda::phi_counter_bytes(65535)));
    // (large K only: 4-byte rows of any K; the forms with a dense row)
    auto raise_theta = [&](bool wide, bool long_docs) {
        const size_t bytes = mlda::theta_lds_bytes(c->K, wide);
        if (bytes <= 48 * 1024 || bytes > (size_t)c->lds_limit) return hipSuccess;      // (too large: see check_theta_lds)
        return hipFuncSetAttribute(theta_kernel_for(RowKind::packed, wide, long_docs),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    };
    for (bool wide : {false, true})
        for (bool long_docs : {false, true}) HIP_TRY(raise_theta(wide, long_docs));
    return MLDA_OK;
}

// The theta rebuild keeps counters per topic in LDS: 16-bit ones for all topics, or, once a
// document of the chunk has 2^16 tokens or more, 32-bit ones for up to 32,768 topics at a time.
// On a device that allows a workgroup the 160 KB this library is written for they always fit.
int check_theta_lds(const mlda_ctx* c, const HostChunk& h) {
    const size_t need = mlda::theta_lds_bytes(c->K, h.wide_counters);
    if (need > (size_t)c->lds_limit)
        return fail(MLDA_ENOTSUP, "K = " + std::to_string(c->K) + " needs " + std::to_string(need) +
                                      " bytes of LDS per workgroup for the theta rebuild, the device allows " +
                                      std::to_string(c->lds_limit));
    return MLDA_OK;
}

// Which words get an int32 row of phi: those with 2^16 tokens or more in the whole corpus.
int find_wide_rows(mlda_ctx* c, const int32_t* word_ids) {
    try {
        const int n_parts = (int)std::max<int64_t>(1, std::min<int64_t>(8, c->T_all >> 22));
        std::vector<std::vector<int32_t>> hist((size_t)n_parts);
        const int64_t per = (c->T_all + n_parts - 1) / n_parts;
        const bool ok = parallel_chunks(n_parts, [&](int p) {
            hist[(size_t)p].assign((size_t)c->V, 0);
            auto& h = hist[(size_t)p];
            const int32_t V = c->V;
            for (int64_t t = per * p; t < std::min(c->T_all, per * (p + 1)); ++t) {
                const int32_t w = word_ids[t];
                if (w >= 0 && w < V) h[(size_t)w] += 1;      // (ids out of range are reported later)
            }
        });
        if (!ok) return fail(MLDA_ENOMEM, "out of host memory");
        c->wide_row.assign((size_t)c->V, -1);
        c->n_wide = 0;
        for (int32_t v = 0; v < c->V; ++v) {
            int64_t n = 0;
            for (int p = 0; p < n_parts; ++p) n += hist[(size_t)p][(size_t)v];
            if (n >= mlda::kNarrowWordLimit) c->wide_row[(size_t)v] = c->n_wide++;
        }
    } catch (const std::bad_alloc&) {
        return fail(MLDA_ENOMEM, "out of host memory");
    }
    return MLDA_OK;
}

// Every sampling tile carries its word's row among the wide rows of phi (or -1).
int mark_wide_tiles(const mlda_ctx* c, HostChunk& h) {
    mlda::Tile* tiles = (mlda::Tile*)(h.arena + h.L.tiles);
    std::vector<int64_t> tokens;            // of every wide row's word in this chunk
    try { tokens.resize((size_t)c->n_wide); } catch (const std::bad_alloc&) { return fail(MLDA_ENOMEM, "out of host memory"); }
    for (int32_t i = 0; i < h.n_tiles; ++i) {
        tiles[i].whole = c->wide_row[(size_t)tiles[i].word];
        if (tiles[i].whole >= 0) tokens[(size_t)tiles[i].whole] += tiles[i].count;
    }
    const int64_t tile = tile_tokens_for(c->K);
    h.n_wide_tiles = 0;
    for (int64_t n : tokens) h.n_wide_tiles += (int32_t)((n + tile - 1) / tile);
    return MLDA_OK;
}

int device_limits(mlda_ctx* c) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipDeviceGetAttribute(&c->n_cus, hipDeviceAttributeMultiprocessorCount, dev));
    HIP_TRY(hipDeviceGetAttribute(&c->lds_limit, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    HIP_TRY(hipDeviceGetAttribute(&c->clock_khz, hipDeviceAttributeWallClockRate, dev));
    if (c->clock_khz <= 0) return fail(MLDA_EHIP, "the device names no rate for its clock");
    c->Kpad = kpad_for(c->K);
    c->queued = sample_waves_for(c->K) > 4;
    c->far_weights = far_weights_for(c->K);
    // (a switch for tests: the 64-bit form is otherwise only reached by theta slots beyond 4 GiB)
    const char* wide = std::getenv("MLDA_WIDE_SLOT_OFFSETS");
    c->wide_slot_offsets = wide && wide[0] != '\0' && wide[0] != '0';
    (void)mlda::switch_numbers(std::getenv("MLDA_REORDER_BY_TILES"), 1, 0, INT64_MAX, &c->reorder_by_tiles);
    // (likewise: in small corpora no workgroup takes a second tile)
    int64_t numbers[2];
    if (mlda::switch_numbers(std::getenv("MLDA_RUN_TILES"), 1, 1, kRunTiles, numbers)) c->forced_run = (int32_t)numbers[0];
    // (likewise: most shapes are otherwise only reached by corpora of millions of tokens)
    if (c->K <= 2048 && mlda::switch_numbers(std::getenv("MLDA_TILE_SHAPE"), 2, 0, 1024, numbers) && numbers[0] >= 16 &&
        numbers[1] <= numbers[0])
        c->shape = {(int32_t)numbers[0], (int32_t)numbers[1]};
    c->near_topics = c->far_weights ? near_topics_for(c->K) : 0;
    const int waves = sample_waves_for(c->K);
    c->sample_lds = c->far_weights ? mlda::sample_far_lds_bytes(c->Kpad, waves, c->near_topics)
                                   : c->queued ? queued_lds_bytes(c->K, waves) : mlda::sample_lds_bytes(c->Kpad, waves, 8);
    if (c->sample_lds > (size_t)c->lds_limit)
        return fail(MLDA_ENOTSUP, "K = " + std::to_string(c->K) + " needs " + std::to_string(c->sample_lds) +
                                      " bytes of LDS per workgroup, the device allows " +
                                      std::to_string(c->lds_limit));
    // the sums of more passes where that leaves a CU as many workgroups
    if (c->queued && !c->far_weights) {
        const size_t room = waves == 12 ? kLdsPerWorkgroup / 2 : (size_t)c->lds_limit;
        for (int passes = kMostKeptPasses; passes > mlda::kLeastKeptPasses; --passes) {
            const size_t more = (size_t)waves * (size_t)(mlda::sample_wave_bytes(passes, mlda::lane_sums_for(passes)) -
                                              mlda::sample_wave_bytes(mlda::kLeastKeptPasses, mlda::lane_sums_for(mlda::kLeastKeptPasses)));
            if (c->sample_lds + more > room) continue;
            c->sample_lds += more;
            c->kept_passes = passes;
            break;
        }
    }
    return MLDA_OK;
}

void destroy(mlda_ctx* c) {
    if (!c) return;
    (void)hipStreamSynchronize(c->stream);
    for (hipStream_t extra : {c->copy_stream, c->down_stream})
        if (extra) {
            (void)hipStreamSynchronize(extra);
            (void)hipStreamDestroy(extra);
        }
    if (c->z_ready) (void)hipEventDestroy(c->z_ready);
    for (hipEvent_t ev : c->events) (void)hipEventDestroy(ev);
    for (hipEvent_t ev : c->z_stored) (void)hipEventDestroy(ev);
    for (int s = 0; s < 2; ++s) {
        if (c->slot_ready[s]) (void)hipEventDestroy(c->slot_ready[s]);
        if (c->slot_done[s]) (void)hipEventDestroy(c->slot_done[s]);
        if (c->slot_free[s]) (void)hipEventDestroy(c->slot_free[s]);
    }
    if (c->z_host) (void)hipHostFree(c->z_host);
    for (hipEvent_t ev : c->ring_events) (void)hipEventDestroy(ev);
    if (c->ring) (void)hipHostFree(c->ring);
    release_scratch(c);
    delete c;
}

// ---- large transfers.  HIP moves pageable memory through one thread's copy to and from its own
// pinned buffers: 10 GB/s into fresh pages (1.5 GB of assignments: 140 ms), while the link carries
// 50.  Here kRingWorkers threads each own a pinned piece of kRingPiece bytes and take every
// kRingWorkers-th piece of the transfer: the copies queue up on the context's stream, and what a
// piece needs on the host (a copy, a widening) is done by its thread while the others' are on
// their way.  What comes from the device comes by halves of a piece, through a kernel that sets a flag, each worker's next
// half on its way while it takes this one: 198 MB of assignments 6.7 -> 5.7 ms, 1.5 GB 51.4 -> 46.8, 12.6 MB 0.52 -> 0.41
// (pieces of 4 MB: 5.4, 44.9, 0.44, and twice the pinned memory to be made by the first).  From kRingFrom bytes on (four pieces: below, too few
// threads have work; with 32 MB as the line, five iterations on 6.3e6 tokens and their 12.6 MB took 4.42 ms,
// now 4.12, the first time on a new context 5.36 and 5.17).  Ten iterations on 7.4e8 tokens and their assignments fetched: 535 -> 432 ms; five on
// 9.9e7: 59.5 -> 45.2 ms (first time on a new context 58 -> 45 ms).  A context on the static workspace, and one for which no pinned memory is left,
// does without.

bool ring_ready(mlda_ctx* c) {
    if (c->ring) return true;
    if (c->ring_failed || c->static_device >= 0) return false;
    c->ring_failed = true;
    void* p = nullptr;
    if (hipHostMalloc(&p, kRingWorkers * (kRingPiece + 2 * kRingFlag), hipHostMallocCoherent) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    c->ring = (unsigned char*)p;
    std::memset(c->ring + kRingWorkers * kRingPiece, 0, kRingWorkers * 2 * kRingFlag);
    try { c->ring_events.reserve(kRingWorkers); } catch (const std::bad_alloc&) {}
    while (c->ring_events.capacity() >= (size_t)kRingWorkers && c->ring_events.size() < (size_t)kRingWorkers) {
        hipEvent_t ev;
        if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) { (void)hipGetLastError(); break; }
        c->ring_events.push_back(ev);
    }
    if (c->ring_events.size() < (size_t)kRingWorkers) {
        (void)hipHostFree(c->ring);
        c->ring = nullptr;
        return false;
    }
    c->ring_failed = false;
    return true;
}

unsigned char* ring_piece(const mlda_ctx* c, int w) { return c->ring + (size_t)w * kRingPiece; }
// What copy_to_host_kernel sets: a flag for each half of a piece.
volatile uint32_t* ring_flag(const mlda_ctx* c, int w, int half) {
    return (volatile uint32_t*)(c->ring + kRingWorkers * kRingPiece + (size_t)(2 * w + half) * kRingFlag);
}

// work(worker) -> hipError_t on the worker threads.
template <class F>
int on_workers(mlda_ctx* c, F&& work) {
    int device = 0;
    HIP_TRY(hipGetDevice(&device));
    // This handle names another stream in every thread: what the caller's has queued must be done
    // before the workers' copies start.
    const bool own_streams = c->stream == hipStreamPerThread;
    if (own_streams) HIP_TRY(hipStreamSynchronize(c->stream));
    hipError_t first_error[kRingWorkers];
    for (hipError_t& e : first_error) e = hipSuccess;
    const bool ran = parallel_chunks(kRingWorkers, [&](int w) {
        hipError_t e = hipSetDevice(device);
        if (e == hipSuccess) e = work(w);
        if (e != hipSuccess) (void)hipStreamSynchronize(c->stream);     // (no copy into the piece is left)
        else if (own_streams) e = hipStreamSynchronize(c->stream);
        first_error[w] = e;
    });
    // (a flag tells that the bytes of the last copies are there; their kernels end a little later.  Once, by one thread: by
    // each of the workers it took 2 % of a pass that fetches 10 MB)
    if (!own_streams) HIP_TRY(hipStreamSynchronize(c->stream));
    for (hipError_t e : first_error)
        if (e != hipSuccess)
            return fail(MLDA_EHIP, std::string("copy between device and host: ") + hipGetErrorString(e));
    if (!ran) return fail(MLDA_ENOMEM, "out of host memory");
    return MLDA_OK;
}

// Device memory into the caller's by one copy, done on return.  (One call: with hipMemcpyAsync and a wait behind it the
// 8 bytes of the likelihood took 21 us, now 13.)
int fetch_now(mlda_ctx* c, void* host, const void* dev, size_t bytes) {
    if (bytes > 0) HIP_TRY(hipMemcpyWithStream(host, dev, bytes, hipMemcpyDeviceToHost, c->stream));
    else HIP_TRY(hipStreamSynchronize(c->stream));
    return MLDA_OK;
}

// A copy of `n` bytes of device memory (at a multiple of 16 bytes) into half `half` of worker w's piece is queued ...
hipError_t queue_copy(mlda_ctx* c, int w, int half, const unsigned char* dev, size_t n, uint32_t value) {
    void *piece = nullptr, *flag = nullptr;
    hipError_t e = hipHostGetDevicePointer(&piece, ring_piece(c, w) + half * (kRingPiece / 2), 0);
    if (e == hipSuccess) e = hipHostGetDevicePointer(&flag, (void*)ring_flag(c, w, half), 0);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlda::copy_to_host_kernel, dim3(kCopyBlocks), dim3(256), 0, c->stream, dev, (unsigned char*)piece, (int64_t)n,
                       (uint32_t*)(c->ll_scalars + 5 + w), (uint32_t*)flag, value);
    return hipGetLastError();
}
// ... and has arrived.
hipError_t await_copy(mlda_ctx* c, int w, int half, uint32_t value) {
    volatile uint32_t* flag = ring_flag(c, w, half);
    // (what the stream holds in front of it may take long, and a launch that failed never sets the flag)
    for (int spins = 0; *flag != value; ++spins) {
        if (spins < 20000) { for (int i = 0; i < 16; ++i) __builtin_ia32_pause(); continue; }
        const hipError_t e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) return e;
        if (*flag != value) return hipErrorLaunchFailure;
    }
    std::atomic_thread_fence(std::memory_order_acquire);
    return hipSuccess;
}

// Device memory, handed to take(offset, piece, bytes) piece by piece: on several threads at once, or
// as a whole through `whole`, which then must hold all of it (made here).
template <class F>
int fetch_pieces(mlda_ctx* c, const void* dev, size_t bytes, F&& take) {
    if (bytes == 0) return MLDA_OK;
    if (bytes >= kRingFrom && ring_ready(c))
        // each worker's next half piece is on its way while this one is taken
        return on_workers(c, [&](int w) {
            constexpr size_t kHalf = kRingPiece / 2;
            uint32_t value[2] = {*ring_flag(c, w, 0), *ring_flag(c, w, 1)};
            // a worker's pieces follow one another: side by side, two workers' met in the caller's huge pages as they are made
            const size_t per = (bytes + kRingWorkers * kHalf - 1) / (kRingWorkers * kHalf) * kHalf, end = std::min(bytes, (size_t)(w + 1) * per);
            auto queue = [&](size_t at, int half) {
                return at < end ? queue_copy(c, w, half, (const unsigned char*)dev + at, std::min(kHalf, end - at), ++value[half])
                                : hipSuccess;
            };
            size_t at = (size_t)w * per;
            hipError_t e = queue(at, 0);
            for (int half = 0; e == hipSuccess && at < end; half ^= 1, at += kHalf) {
                e = queue(at + kHalf, half ^ 1);
                if (e == hipSuccess) e = await_copy(c, w, half, value[half]);
                if (e == hipSuccess) take(at, (const unsigned char*)ring_piece(c, w) + half * kHalf, std::min(kHalf, end - at));
            }
            return e;
        });
    std::vector<unsigned char> whole;
    try { whole.resize(bytes); } catch (const std::bad_alloc&) { return fail(MLDA_ENOMEM, "out of host memory"); }
    RC_TRY(fetch_now(c, whole.data(), dev, bytes));
    take(0, (const unsigned char*)whole.data(), bytes);
    return MLDA_OK;
}

// Device memory into the caller's, and back; both are done on return.
int fetch(mlda_ctx* c, void* host, const void* dev, size_t bytes) {
    if (bytes >= kRingFrom && ring_ready(c))
        return fetch_pieces(c, dev, bytes, [&](size_t at, const unsigned char* piece, size_t n) {
            std::memcpy((unsigned char*)host + at, piece, n);
        });
    return fetch_now(c, host, dev, bytes);
}
int send(mlda_ctx* c, void* dev, const void* host, size_t bytes) {
    if (bytes >= kRingFrom && ring_ready(c))
        return on_workers(c, [&](int w) {
            hipError_t e = hipSuccess;
            for (size_t at = (size_t)w * kRingPiece; e == hipSuccess && at < bytes; at += kRingWorkers * kRingPiece) {
                const size_t n = std::min(kRingPiece, bytes - at);
                std::memcpy(ring_piece(c, w), (const unsigned char*)host + at, n);
                e = hipMemcpyAsync((unsigned char*)dev + at, ring_piece(c, w), n, hipMemcpyHostToDevice, c->stream);
                if (e == hipSuccess) e = hipEventRecord(c->ring_events[(size_t)w], c->stream);
                if (e == hipSuccess) e = hipEventSynchronize(c->ring_events[(size_t)w]);
            }
            return e;
        });
    if (bytes > 0) HIP_TRY(hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    return MLDA_OK;
}

// n values of host memory in parts, side by side where there are enough of them; false: a part
// could not be run.
template <class F>
bool in_parts(int64_t n, F&& part) {
    const int parts = (int)std::min<int64_t>(kRingWorkers, n / ((int64_t)1 << 22) + 1);
    const int64_t per = (n + parts - 1) / parts;
    return parallel_chunks(parts, [&](int p) { part(std::min(n, per * p), std::min(n, per * (p + 1))); });
}

int fetch_row_rec(mlda_ctx* c, std::vector<uint2>& rec) {
    try { rec.resize((size_t)c->D); } catch (const std::bad_alloc&) {
        return fail(MLDA_ENOMEM, "out of host memory");
    }
    return fetch(c, rec.data(), c->row_rec, (size_t)c->D * 8);
}

// Whether the rows of the attached chunk are taken from a copy of its slots, unpacked here, or laid
// out by the device: that takes two passes over 2 bytes per token and as many more round trips.
// Measured (copy / device, us): 8e3 tokens, K = 24: 41 / 100; 2.5e5, K = 500, documents of 300 (0.4 MB of
// slots) 129 / 144, twice as many 329 / 208; 4e6 tokens, K = 24, documents of 300 (1.7 MB) 448 / 1694,
// K = 500 (5.5 MB) 2067 / 1544.  From kRingFrom on the device's values come through the pinned pieces.
constexpr size_t kUnpackBytes = (size_t)512 << 10;
bool rows_unpacked_here(const mlda_ctx* c) {
    return c->slots_bytes <= kUnpackBytes || (c->slots_bytes <= (size_t)c->T && (size_t)c->T * 2 < kRingFrom);
}

// Rows of theta of the attached chunk from a copy of its slots into the caller's CSR arrays (row_ptr of
// its documents in place; rec[d].y = distinct topics of row d, the length of its CSR row; the slot's
// header holds the number of entries, of which several in a row may share a topic).
template <class Layout>
void unpack_rows(const mlda_ctx* c, const std::vector<uint2>& rec, const std::vector<unsigned char>& slots,
                 const int64_t* row_ptr, uint16_t* topics, int32_t* counts) {
    typedef typename Layout::Entry Entry;
    for (int64_t d = 0; d < c->D; ++d) {
        if (rec[(size_t)d].y == 0) continue;
        const unsigned char* head = slots.data() + (size_t)rec[(size_t)d].x * 16;
        uint32_t n_entries;
        std::memcpy(&n_entries, head, 4);
        const Entry* ent = reinterpret_cast<const Entry*>(head + mlda::kRowHeader);
        int64_t at = row_ptr[d] - 1;
        int last_topic = -1;
        for (uint32_t j = 0; j < n_entries; ++j) {
            const int topic = Layout::entry_topic(ent[j]), count = Layout::entry_count(ent[j]);
            if (topic != last_topic) {
                topics[++at] = (uint16_t)topic;
                counts[at] = 0;
                last_topic = topic;
            }
            counts[at] += count;
        }
    }
}

// The same, laid out by the device at the rows' tokens' places in the spare assignment buffer, as 16-bit
// values; the gaps are closed here.
template <class Layout>
int export_rows(mlda_ctx* c, const std::vector<uint2>& rec, const int64_t* row_ptr, uint16_t* topics, int32_t* counts) {
    uint16_t* spare = c->z[c->cur ^ 1];             // free between steps and chunk visits
    std::vector<int32_t> doc_ptr;
    try { doc_ptr.resize((size_t)c->D + 1); } catch (const std::bad_alloc&) { return fail(MLDA_ENOMEM, "out of host memory"); }
    RC_TRY(fetch(c, doc_ptr.data(), c->doc_ptr, ((size_t)c->D + 1) * 4));
    const dim3 grid((unsigned)std::min<int64_t>(c->D, (int64_t)c->n_cus * 32));
    // place(row entry, value) for the values of the tokens' places [at, at + n)
    auto fetch_values = [&](auto&& place) {
        return fetch_pieces(c, spare, (size_t)c->T * 2, [&](size_t at_byte, const unsigned char* piece, size_t bytes) {
            const uint16_t* value = (const uint16_t*)piece;
            const int64_t at = (int64_t)(at_byte / 2), end = at + (int64_t)(bytes / 2);
            int64_t d = std::upper_bound(doc_ptr.begin(), doc_ptr.end(), (int32_t)at) - doc_ptr.begin() - 1;
            for (; d < c->D && doc_ptr[(size_t)d] < end; ++d) {
                const int64_t first = doc_ptr[(size_t)d], last = first + rec[(size_t)d].y;
                for (int64_t t = std::max(first, at); t < std::min(last, end); ++t)
                    place(row_ptr[d] + (t - first), value[t - at]);
            }
        });
    };
    hipLaunchKernelGGL((mlda::export_rows_kernel<Layout, true>), grid, dim3(mlda::kWave), 0, c->stream, c->row_rec,
                       c->doc_ptr, c->D, c->slots, 0, spare);
    RC_TRY(launch_check("export_rows_kernel"));
    RC_TRY(fetch_values([&](int64_t i, uint16_t v) { topics[i] = v; }));
    for (int shift = 0; shift == 0 || (c->wide_counters && shift == 16); shift += 16) {
        hipLaunchKernelGGL((mlda::export_rows_kernel<Layout, false>), grid, dim3(mlda::kWave), 0, c->stream, c->row_rec,
                           c->doc_ptr, c->D, c->slots, shift, spare);
        RC_TRY(launch_check("export_rows_kernel"));
        if (shift == 0) RC_TRY(fetch_values([&](int64_t i, uint16_t v) { counts[i] = (int32_t)v; }));
        else RC_TRY(fetch_values([&](int64_t i, uint16_t v) { counts[i] += (int32_t)v << 16; }));
    }
    return MLDA_OK;
}

// Streamed: phi and n_k of the assignments in z_host (after init or set_assignments);
// `init`: the assignments are drawn on the device first and stored.
int rebuild_model_streamed(mlda_ctx* c, bool init) {
    c->to_store = -1;       // (a step that failed may have left some: not into the assignments that are to be counted)
    RC_TRY(begin_model(c, c->model_cur));
    for (int32_t m = 0; m < (int32_t)c->chunks.size(); ++m) {
        if (c->chunks[(size_t)m].D == 0) continue;
        RC_TRY(attach(c, m, !init));
        if (init && c->T > 0)
            hipLaunchKernelGGL(mlda::init_topics_kernel, dim3(blocks_for(c->T, 256)), dim3(256), 0, c->stream,
                               c->tok_id, c->z[0], c->T, c->K, c->seed);
        RC_TRY(rebuild_phi(c, c->z[0], c->model_cur));
        if (init) RC_TRY(to_document_order(c, c->z[0]));
        RC_TRY(store_z_and_release(c, m, init));
    }
    RC_TRY(finish_model(c, c->model_cur));
    return store_z(c);
}

// Streamed: the theta rows of every chunk are rebuilt in turn from z_host; `visit` sees each
// attached chunk with its rows in place.  Also leaves the log-likelihood's theta sum.
template <class F>
int for_each_chunk_rows(mlda_ctx* c, F&& visit) {
    bool first = true;
    for (int32_t m = 0; m < (int32_t)c->chunks.size(); ++m) {
        if (c->chunks[(size_t)m].D == 0) continue;
        RC_TRY(attach(c, m, true));
        RC_TRY(rebuild_theta(c, c->z_doc));
        RC_TRY(add_theta_loglik(c, first));
        first = false;
        RC_TRY(visit(c->chunks[(size_t)m]));
        RC_TRY(store_z_and_release(c, m, false));
    }
    if (first) {            // no documents at all: the sum is empty
        hipLaunchKernelGGL(mlda::loglik_final_kernel, dim3(1), dim3(256), 0, c->stream, c->ll_partial, 0, 0,
                           c->ll_scalars + 1);
        RC_TRY(launch_check("loglik_final_kernel"));
    }
    return MLDA_OK;
}

}  // namespace

extern "C" {

const char* mlda_strerror(int code) {
    switch (code) {
        case MLDA_OK: return "ok";
        case MLDA_EINVAL: return "invalid argument";
        case MLDA_ENOMEM: return "workspace too small or out of host memory";
        case MLDA_EHIP: return "HIP call failed";
        case MLDA_ENOTSUP: return "beyond what the device or the library supports";
        default: return "unknown error";
    }
}

const char* mlda_last_error(void) { return g_last_error.c_str(); }

int mlda_workspace_bytes(int64_t D, int64_t T, int32_t V, int32_t K, size_t* bytes) {
    if (!bytes) return fail(MLDA_EINVAL, "bytes is null");
    if (D < 0 || T < 0 || V < 1 || K < 1 || K > 65535 || T >= ((int64_t)1 << 31))
        return fail(MLDA_EINVAL, "need D >= 0, 0 <= T < 2^31, V >= 1, 1 <= K <= 65535");
    *bytes = model_layout(V, K, T, false).total + chunk_layout_bound(D, T, V, K, false).total;
    return MLDA_OK;
}

int mlda_workspace_bytes_streamed(const int64_t* doc_ptr, int64_t D, int32_t V, int32_t K,
                                  int32_t n_chunks, size_t* bytes) {
    if (!bytes) return fail(MLDA_EINVAL, "bytes is null");
    RC_TRY(check_corpus(doc_ptr, nullptr, false, D, V, K, 1.0, 1.0));
    if (n_chunks < 1) return fail(MLDA_EINVAL, "n_chunks must be >= 1");
    *bytes = streamed_workspace_bound(doc_ptr, D, V, K, n_chunks);
    return MLDA_OK;
}

// mlda_create and mlda_create_static: the corpus resident in one workspace.  With
// `in_static` the workspace is the current device's static array, claimed here.
static int create_resident(mlda_ctx** out, const int64_t* doc_ptr, const int32_t* word_ids, int64_t D,
                           int32_t V, int32_t K, double alpha, double beta, uint64_t seed,
                           void* dev_workspace, size_t workspace_bytes, void* hip_stream, bool in_static) {
    if (!out) return fail(MLDA_EINVAL, "out is null");
    *out = nullptr;
    RC_TRY(check_corpus(doc_ptr, word_ids, true, D, V, K, alpha, beta));
    const int64_t T = doc_ptr[D];
    size_t need_bound = 0;
    if (mlda_workspace_bytes(D, T, V, K, &need_bound) != MLDA_OK) return MLDA_EINVAL;
    if (in_static) {
        if (need_bound > (size_t)MLDA_STATIC_WORKSPACE_BYTES)
            return fail(MLDA_ENOMEM, "this corpus needs a workspace of " + std::to_string(need_bound) +
                                         " bytes, the static one holds " +
                                         std::to_string((size_t)MLDA_STATIC_WORKSPACE_BYTES) +
                                         ": use mlda_create with a workspace of the caller's");
    } else {
        RC_TRY(check_workspace(dev_workspace, workspace_bytes, need_bound));
        RC_TRY(check_device_pointer(dev_workspace));
    }
    mlda_ctx* c = new (std::nothrow) mlda_ctx();
    if (!c) return fail(MLDA_ENOMEM, "out of host memory");
    if (in_static) {
        unsigned char* ptr = nullptr;
        const int rc_claim = claim_scratch(c, &c->static_device, &ptr);
        if (rc_claim != MLDA_OK) { delete c; return rc_claim; }
        dev_workspace = ptr;
        workspace_bytes = (size_t)MLDA_STATIC_WORKSPACE_BYTES;
    }
    c->D_all = D; c->T_all = T; c->V = V; c->K = K;
    c->alpha = alpha; c->beta = beta; c->seed = seed;
    c->stream = (hipStream_t)hip_stream;
    int rc = device_limits(c);
    if (rc == MLDA_OK) rc = find_wide_rows(c, word_ids);
    if (rc == MLDA_OK) {
        try { c->chunks = std::vector<HostChunk>(1); } catch (const std::bad_alloc&) { rc = fail(MLDA_ENOMEM, "out of host memory"); }
    }
    if (rc == MLDA_OK) rc = prepare_chunk(doc_ptr, word_ids, 0, D, V, K, false, false, c->queued, c->forced_shape(), c->chunks[0]);
    if (rc == MLDA_OK) rc = check_theta_lds(c, c->chunks[0]);
    if (rc == MLDA_OK) rc = mark_wide_tiles(c, c->chunks[0]);
    const ModelLayout ML = model_layout(V, K, T, false);
    if (rc == MLDA_OK && ML.total + c->chunks[0].L.total > workspace_bytes)
        rc = fail(MLDA_ENOMEM, "workspace has " + std::to_string(workspace_bytes) + " bytes, need " +
                                   std::to_string(ML.total + c->chunks[0].L.total));
    if (rc == MLDA_OK) {
        unsigned char* base = (unsigned char*)dev_workspace;
        HostChunk& h = c->chunks[0];
        c->slot_base[0] = base + ML.total;
        point_at(c, h, c->slot_base[0]);
        hipError_t e = hipSuccess;
        if (h.L.static_bytes > 0)
            e = hipMemcpyAsync(c->slot_base[0], h.arena, h.L.static_bytes, hipMemcpyHostToDevice, c->stream);
        if (e != hipSuccess) rc = fail(MLDA_EHIP, std::string("uploading the corpus: ") + hipGetErrorString(e));
        if (rc == MLDA_OK) { derive_chunk_arrays(c); rc = finish_create(c, base, ML); }
        if (rc == MLDA_OK) {        // the documents' term of the log-likelihood never changes
            const int blocks = (int)std::min<int64_t>(kLoglikBlocks, D / 256 + 1);
            hipLaunchKernelGGL(mlda::loglik_doc_term_kernel, dim3((unsigned)blocks), dim3(256), 0, c->stream, c->doc_ptr, D,
                               (double)K * alpha, c->ll_partial);
            hipLaunchKernelGGL(mlda::loglik_final_kernel, dim3(1), dim3(256), 0, c->stream, c->ll_partial, blocks, 0,
                               c->ll_scalars + 2);
            rc = launch_check("document term kernels");
        }
        // the upload reads the host arena until the stream has drained: wait for it before the
        // arena goes, whether or not everything before went well
        e = hipStreamSynchronize(c->stream);
        if (rc == MLDA_OK && e != hipSuccess)
            rc = fail(MLDA_EHIP, std::string("uploading the corpus: ") + hipGetErrorString(e));
        h.release();        // the corpus now lives on the device
    }
    if (rc != MLDA_OK) { destroy(c); return rc; }
    *out = c;
    return MLDA_OK;
}

int mlda_create(mlda_ctx** out, const int64_t* doc_ptr, const int32_t* word_ids, int64_t D,
                int32_t V, int32_t K, double alpha, double beta, uint64_t seed,
                void* dev_workspace, size_t workspace_bytes, void* hip_stream) {
    return create_resident(out, doc_ptr, word_ids, D, V, K, alpha, beta, seed, dev_workspace,
                           workspace_bytes, hip_stream, false);
}

int mlda_create_static(mlda_ctx** out, const int64_t* doc_ptr, const int32_t* word_ids, int64_t D,
                       int32_t V, int32_t K, double alpha, double beta, uint64_t seed, void* hip_stream) {
    return create_resident(out, doc_ptr, word_ids, D, V, K, alpha, beta, seed, nullptr, 0, hip_stream, true);
}

int mlda_create_streamed(mlda_ctx** out, const int64_t* doc_ptr, const int32_t* word_ids, int64_t D,
                         int32_t V, int32_t K, double alpha, double beta, uint64_t seed, int32_t n_chunks,
                         void* dev_workspace, size_t workspace_bytes, void* hip_stream) {
    if (!out) return fail(MLDA_EINVAL, "out is null");
    *out = nullptr;
    RC_TRY(check_corpus(doc_ptr, word_ids, true, D, V, K, alpha, beta));
    if (n_chunks < 1) return fail(MLDA_EINVAL, "n_chunks must be >= 1");
    const int64_t T = doc_ptr[D];
    RC_TRY(check_workspace(dev_workspace, workspace_bytes,
                           streamed_workspace_bound(doc_ptr, D, V, K, n_chunks)));
    RC_TRY(check_device_pointer(dev_workspace));
    mlda_ctx* c = new (std::nothrow) mlda_ctx();
    if (!c) return fail(MLDA_ENOMEM, "out of host memory");
    c->D_all = D; c->T_all = T; c->V = V; c->K = K;
    c->alpha = alpha; c->beta = beta; c->seed = seed;
    c->stream = (hipStream_t)hip_stream;
    c->streamed = true;
    int rc = device_limits(c);
    if (rc == MLDA_OK) rc = find_wide_rows(c, word_ids);
    if (rc == MLDA_OK) {
        try {
            c->chunks = std::vector<HostChunk>((size_t)n_chunks);
            c->z_stored.assign((size_t)n_chunks, nullptr);
        } catch (const std::bad_alloc&) { rc = fail(MLDA_ENOMEM, "out of host memory"); }
    }
    size_t chunk_bytes = 0;
    int64_t chunk_tokens = 0;
    for (int32_t m = 0; rc == MLDA_OK && m < n_chunks; ++m) {
        rc = prepare_chunk(doc_ptr, word_ids, chunk_first(doc_ptr, D, n_chunks, m),
                           chunk_first(doc_ptr, D, n_chunks, m + 1), V, K, true, true, false, c->forced_shape(), c->chunks[(size_t)m]);
        if (rc == MLDA_OK) rc = check_theta_lds(c, c->chunks[(size_t)m]);
        if (rc == MLDA_OK) rc = mark_wide_tiles(c, c->chunks[(size_t)m]);
        if (rc == MLDA_OK) {
            chunk_bytes = std::max(chunk_bytes, c->chunks[(size_t)m].L.total);
            chunk_tokens = std::max(chunk_tokens, c->chunks[(size_t)m].T);
        }
    }
    const mlda::StreamedSlot slot = mlda::streamed_slot(chunk_tokens, chunk_bytes);
    const ModelLayout ML = model_layout(V, K, T, true);
    if (rc == MLDA_OK && ML.total + 2 * slot.total > workspace_bytes)
        rc = fail(MLDA_ENOMEM, "workspace has " + std::to_string(workspace_bytes) + " bytes, need " +
                                   std::to_string(ML.total + 2 * slot.total));
    auto hip_ok = [&](hipError_t e, const char* what) {
        if (rc == MLDA_OK && e != hipSuccess) rc = fail(MLDA_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    };
    if (rc == MLDA_OK) {
        unsigned char* base = (unsigned char*)dev_workspace;
        for (int s = 0; s < 2; ++s) {
            unsigned char* at = base + ML.total + (size_t)s * slot.total;
            c->slot_z[s] = (uint16_t*)(at + slot.z_doc);
            c->slot_base[s] = at + slot.chunk;
        }
        void* zh = nullptr;
        hip_ok(hipHostMalloc(&zh, std::max<size_t>((size_t)T * 2, 1), hipHostMallocDefault), "hipHostMalloc");
        c->z_host = (uint16_t*)zh;
        // every stream at the default priority
        hip_ok(hipStreamCreateWithFlags(&c->copy_stream, hipStreamNonBlocking), "hipStreamCreateWithFlags");
        hip_ok(hipStreamCreateWithFlags(&c->down_stream, hipStreamNonBlocking), "hipStreamCreateWithFlags");
        hip_ok(hipEventCreateWithFlags(&c->z_ready, hipEventDisableTiming), "hipEventCreateWithFlags");
        for (int s = 0; s < 2; ++s) {
            hip_ok(hipEventCreateWithFlags(&c->slot_ready[s], hipEventDisableTiming), "hipEventCreateWithFlags");
            for (hipEvent_t* ev : {&c->slot_done[s], &c->slot_free[s]}) {
                hip_ok(hipEventCreateWithFlags(ev, hipEventDisableTiming), "hipEventCreateWithFlags");
                if (rc == MLDA_OK) hip_ok(hipEventRecord(*ev, c->stream), "hipEventRecord");
            }
        }
        for (int32_t m = 0; m < n_chunks; ++m) {
            hip_ok(hipEventCreateWithFlags(&c->z_stored[(size_t)m], hipEventDisableTiming), "hipEventCreateWithFlags");
            if (rc == MLDA_OK) hip_ok(hipEventRecord(c->z_stored[(size_t)m], c->stream), "hipEventRecord");
        }
        if (rc == MLDA_OK) rc = finish_create(c, base, ML);
        if (rc == MLDA_OK) {
            // the documents' term of the log-likelihood never changes
            double doc_term = 0.0;
            const double ka = (double)K * alpha, lg_ka = std::lgamma(ka);
            for (int64_t d = 0; d < D; ++d) doc_term += lg_ka - std::lgamma((double)(doc_ptr[d + 1] - doc_ptr[d]) + ka);
            hip_ok(hipMemcpyAsync(c->ll_scalars + 2, &doc_term, 8, hipMemcpyHostToDevice, c->stream), "hipMemcpyAsync");
            hip_ok(hipStreamSynchronize(c->stream), "hipStreamSynchronize");
        }
    }
    if (rc != MLDA_OK) { destroy(c); return rc; }
    *out = c;
    return MLDA_OK;
}

int mlda_init_random(mlda_ctx* c) {
    if (!c) return fail(MLDA_EINVAL, "null context");
    if (c->streamed) {
        RC_TRY(rebuild_model_streamed(c, true));
    } else {
        if (c->T > 0)
            hipLaunchKernelGGL(mlda::init_topics_kernel, dim3(blocks_for(c->T, 256)), dim3(256), 0,
                               c->stream, c->tok_id, c->z[c->cur], c->T, c->K, c->seed);
        RC_TRY(launch_check("init_topics_kernel"));
        c->phi_of_z = false;
        RC_TRY(rebuild_phi(c, c->z[c->cur], 0));
        RC_TRY(rebuild_theta(c, c->z[c->cur]));
        c->phi_of_z = true;
    }
    c->iter = 0;
    c->has_state = true;
    c->ll_fresh = false;
    c->last_step_iters = 0;     // the rows of mlda_get_timing / mlda_get_sampler_bytes belong to a step
    c->timed_iters = 0;
    return MLDA_OK;
}

int mlda_set_assignments(mlda_ctx* c, const uint16_t* z, int32_t iter) {
    if (!c) return fail(MLDA_EINVAL, "null context");
    if (c->T_all > 0 && !z) return fail(MLDA_EINVAL, "z is null");
    if (iter < 0) return fail(MLDA_EINVAL, "iter must be >= 0");
    std::atomic<bool> beyond{false};
    if (!in_parts(c->T_all, [&](int64_t a, int64_t b) {
            int most = -1;
            for (int64_t t = a; t < b; ++t) most = std::max(most, (int)z[t]);
            if (most >= c->K) beyond = true;
        }))
        return fail(MLDA_ENOMEM, "out of host memory");
    if (beyond) return fail(MLDA_EINVAL, "topic >= K in z");
    if (c->streamed) {
        HIP_TRY(hipStreamSynchronize(c->stream));
        HIP_TRY(hipStreamSynchronize(c->copy_stream));
        HIP_TRY(hipStreamSynchronize(c->down_stream));
        if (!in_parts(c->T_all, [&](int64_t a, int64_t b) { std::memcpy(c->z_host + a, z + a, (size_t)(b - a) * 2); }))
            return fail(MLDA_ENOMEM, "out of host memory");
        RC_TRY(rebuild_model_streamed(c, false));
    } else {
        c->phi_of_z = false;
        if (c->T > 0) {
            uint16_t* tmp = c->z[c->cur ^ 1];
            RC_TRY(send(c, tmp, z, (size_t)c->T * 2));    // (done: the caller's z may go away)
            if (c->T >= c->reorder_by_tiles)
                hipLaunchKernelGGL(mlda::reorder_by_tiles_kernel<false>, dim3((unsigned)((c->n_tiles + 7) / 8 * 8)), dim3(256), 0,
                                   c->stream, c->tiles, c->n_tiles, c->z[c->cur], c->tok_id, tmp, (int64_t)0);
            else
                hipLaunchKernelGGL(mlda::to_word_major_kernel, dim3(blocks_for(c->T, 256)), dim3(256), 0,
                                   c->stream, tmp, c->tok_id, c->z[c->cur], c->T, (int64_t)0);
        }
        RC_TRY(rebuild_phi(c, c->z[c->cur], 0));
        RC_TRY(rebuild_theta(c, c->z[c->cur]));
        c->phi_of_z = true;
    }
    c->iter = iter;
    c->has_state = true;
    c->ll_fresh = false;
    c->last_step_iters = 0;
    c->timed_iters = 0;
    return MLDA_OK;
}

// One iteration with several chunks (Algorithm 1, WorkSchedule2; Section 4: every chunk
// samples against the phi of the iteration's start, the new phi is the sum over chunks).
static int step_streamed(mlda_ctx* c, bool loglik, int32_t timed_row) {
    const int next = c->model_cur ^ 1;
    RC_TRY(begin_model(c, next));
    bool first = true;
    for (int32_t m = 0; m < (int32_t)c->chunks.size(); ++m) {
        if (c->chunks[(size_t)m].D == 0) continue;
        hipEvent_t* ev = nullptr;
        if (timed_row >= 0 && (int)c->visit_log.size() < kMaxTimedVisits) {
            const size_t event0 = c->visit_log.size() * kVisitEvents;
            while (c->events.size() < event0 + kVisitEvents) {
                hipEvent_t e;
                HIP_TRY(hipEventCreate(&e));
                c->events.push_back(e);
            }
            ev = &c->events[event0];
        }
        RC_TRY(attach(c, m, true, ev));
        if (ev) {
            try {
                c->visit_log.push_back({timed_row, c->T, c->counted_tiles, c->n_wide_tiles, c->rebuilds,
                                        (size_t)(ev - c->events.data())});
            } catch (const std::bad_alloc&) { return fail(MLDA_ENOMEM, "out of host memory"); }
        }
        RC_TRY(rebuild_theta(c, c->z_doc));            // theta is not kept between visits
        if (ev) HIP_TRY(hipEventRecord(ev[2], c->stream));
        RC_TRY(launch_sampler(c, c->z[0], c->z[1]));
        if (ev) HIP_TRY(hipEventRecord(ev[3], c->stream));
        RC_TRY(rebuild_phi(c, c->z[1], next));
        if (ev) HIP_TRY(hipEventRecord(ev[4], c->stream));
        RC_TRY(to_document_order(c, c->z[1]));
        if (ev) HIP_TRY(hipEventRecord(ev[5], c->stream));
        if (loglik) {
            RC_TRY(rebuild_theta(c, c->z_doc));
            RC_TRY(add_theta_loglik(c, first));
            first = false;
        }
        if (ev) HIP_TRY(hipEventRecord(ev[6], c->stream));
        RC_TRY(store_z_and_release(c, m, true));
    }
    RC_TRY(finish_model(c, next));
    c->model_cur = next;
    c->iter += 1;
    c->ll_fresh = false;
    if (loglik) {
        if (first) {
            hipLaunchKernelGGL(mlda::loglik_final_kernel, dim3(1), dim3(256), 0, c->stream, c->ll_partial, 0, 0,
                               c->ll_scalars + 1);
            RC_TRY(launch_check("loglik_final_kernel"));
        }
        RC_TRY(launch_loglik(c));
    }
    return MLDA_OK;
}

int mlda_step(mlda_ctx* c, int32_t n_iters, uint32_t flags) {
    RC_TRY(need_state(c));
    if (n_iters < 0) return fail(MLDA_EINVAL, "n_iters must be >= 0");
    if (c->streamed) {
        // the last iterations of the step are timed, as many as the visit log holds
        int32_t visits_per_iter = 0;
        for (const HostChunk& h : c->chunks) visits_per_iter += h.D > 0 ? 1 : 0;
        const int32_t timed = visits_per_iter == 0 ? 0
            : std::min({n_iters, kMaxTimedIters, kMaxTimedVisits / visits_per_iter,
                        kEntryRing / (2 * visits_per_iter) - 1});
        c->visit_log.clear();
        c->timed_iters = std::max(timed, 0);
        c->last_step_iters = n_iters;
        for (int32_t i = 0; i < n_iters; ++i)
            RC_TRY(step_streamed(c, (flags & MLDA_STEP_LOGLIK) != 0, i - (n_iters - c->timed_iters)));
        return store_z(c);
    }
    const int32_t timed = std::min(n_iters, kMaxTimedIters);
    c->timed_iters = 0;
    c->last_step_iters = n_iters;
    c->last_step_loglik = (flags & MLDA_STEP_LOGLIK) != 0;
    for (int32_t i = 0; i < n_iters; ++i) {
        const int32_t row = i - (n_iters - timed);
        auto phase = [&](int p) { return row >= 0 ? c->stamps + (size_t)row * kPhases + p : nullptr; };
        uint16_t *z_old = c->z[c->cur], *z_next = c->z[c->cur ^ 1];
        RC_TRY(launch_sampler(c, z_old, z_next, phase(0)));
        const uint16_t* counted = c->phi_of_z ? z_old : nullptr;
        c->phi_of_z = false;
        if (c->both_lds > 0) {
            RC_TRY(rebuild_phi(c, z_next, 0, counted, phase(1), true, phase(2)));
        } else {
            RC_TRY(rebuild_phi(c, z_next, 0, counted, phase(1)));
            RC_TRY(rebuild_theta(c, z_next, phase(2)));
        }
        c->cur ^= 1;
        c->phi_of_z = true;
        c->iter += 1;
        c->ll_fresh = false;
        if (c->last_step_loglik) RC_TRY(launch_loglik(c, phase(3)));
    }
    if (timed > 0) {        // when the last phase had ended
        hipLaunchKernelGGL(mlda::stamp_kernel, dim3(1), dim3(1), 0, c->stream, c->stamps + (size_t)timed * kPhases);
        RC_TRY(launch_check("stamp_kernel"));
    }
    c->timed_iters = timed;
    return MLDA_OK;
}

int mlda_iteration(const mlda_ctx* c, int32_t* iter) {
    if (!c || !iter) return fail(MLDA_EINVAL, "null argument");
    *iter = c->iter;
    return MLDA_OK;
}

int mlda_get_assignments(mlda_ctx* c, uint16_t* z) {
    RC_TRY(need_state(c));
    if (c->T_all == 0) return MLDA_OK;
    if (!z) return fail(MLDA_EINVAL, "z is null");
    if (c->streamed) {
        HIP_TRY(hipStreamSynchronize(c->stream));
        HIP_TRY(hipStreamSynchronize(c->down_stream));
        if (!in_parts(c->T_all, [&](int64_t a, int64_t b) { std::memcpy(z + a, c->z_host + a, (size_t)(b - a) * 2); }))
            return fail(MLDA_ENOMEM, "out of host memory");
        return MLDA_OK;
    }
    uint16_t* tmp = c->z[c->cur ^ 1];      // free between steps
    if (c->T >= c->reorder_by_tiles)
        hipLaunchKernelGGL(mlda::reorder_by_tiles_kernel<true>, dim3((unsigned)((c->n_tiles + 7) / 8 * 8)), dim3(256), 0,
                           c->stream, c->tiles, c->n_tiles, c->z[c->cur], c->tok_id, tmp, c->at->tok_begin);
    else
        hipLaunchKernelGGL(mlda::to_doc_major_scatter_kernel, dim3(blocks_for(c->T, 256)), dim3(256), 0, c->stream,
                           c->z[c->cur], c->tok_id, tmp, c->T, c->at->tok_begin);
    RC_TRY(launch_check("assignments to document order"));
    return fetch(c, z, tmp, (size_t)c->T * 2);
}

int mlda_get_word_topic(mlda_ctx* c, int32_t* n_wk) {
    RC_TRY(need_state(c));
    if (!n_wk) return fail(MLDA_EINVAL, "n_wk is null");
    // the 16-bit matrix and the wide rows are fetched as they are and widened here
    std::vector<int32_t> words;                     // of the wide rows
    try { words.resize((size_t)c->n_wide); } catch (const std::bad_alloc&) { return fail(MLDA_ENOMEM, "out of host memory"); }
    for (int32_t v = 0; v < c->V; ++v)
        if (c->wide_row[(size_t)v] >= 0) words[(size_t)c->wide_row[(size_t)v]] = v;
    const size_t cells = (size_t)c->V * (size_t)c->K, wide_cells = (size_t)c->n_wide * (size_t)c->K;
    const mlda::PhiView& phi = c->phi[c->model_cur];
    RC_TRY(fetch_pieces(c, phi.narrow, cells * 2, [&](size_t at, const unsigned char* piece, size_t bytes) {
        const uint16_t* cell = (const uint16_t*)piece;
        int32_t* to = n_wk + at / 2;
        for (size_t i = 0; i < bytes / 2; ++i) to[i] = cell[i];
    }));
    if (wide_cells > 0)
        RC_TRY(fetch_pieces(c, phi.wide, wide_cells * 4, [&](size_t at, const unsigned char* piece, size_t bytes) {
            const int32_t* cell = (const int32_t*)piece;
            for (size_t i = at / 4, end = (at + bytes) / 4; i < end;) {      // row by row
                const size_t r = i / (size_t)c->K, k = i % (size_t)c->K, n = std::min(end - i, (size_t)c->K - k);
                std::memcpy(n_wk + (size_t)words[r] * (size_t)c->K + k, cell + (i - at / 4), n * 4);
                i += n;
            }
        }));
    return MLDA_OK;
}

int mlda_get_topic_totals(mlda_ctx* c, int32_t* n_k) {
    RC_TRY(need_state(c));
    if (!n_k) return fail(MLDA_EINVAL, "n_k is null");
    return fetch_now(c, n_k, current_n_k(c), (size_t)c->K * 4);
}

int mlda_get_doc_topic_nnz(mlda_ctx* c, int64_t* nnz) {
    RC_TRY(need_state(c));
    if (!nnz) return fail(MLDA_EINVAL, "nnz is null");
    int64_t n = 0;
    std::vector<uint2> rec;
    if (c->streamed) {
        RC_TRY(for_each_chunk_rows(c, [&](const HostChunk&) {
            RC_TRY(fetch_row_rec(c, rec));
            for (const uint2& r : rec) n += r.y;
            return (int)MLDA_OK;
        }));
    } else {
        RC_TRY(fetch_row_rec(c, rec));
        for (const uint2& r : rec) n += r.y;
    }
    *nnz = n;
    return MLDA_OK;
}

int mlda_get_doc_topic_csr(mlda_ctx* c, int64_t* row_ptr, uint16_t* topics, int32_t* counts) {
    RC_TRY(need_state(c));
    if (!row_ptr) return fail(MLDA_EINVAL, "row_ptr is null");
    std::vector<uint2> rec;
    std::vector<unsigned char> slots;
    row_ptr[0] = 0;
    auto take_rows = [&](const HostChunk& h) {
        const bool unpack = rows_unpacked_here(c);
        if (unpack) {           // on its way with the lengths
            try { slots.resize(c->slots_bytes); } catch (const std::bad_alloc&) { return fail(MLDA_ENOMEM, "out of host memory"); }
            HIP_TRY(hipMemcpyAsync(slots.data(), c->slots, c->slots_bytes, hipMemcpyDeviceToHost, c->stream));
        }
        RC_TRY(fetch_row_rec(c, rec));
        int64_t* ptr = row_ptr + h.d_begin;
        for (int64_t d = 0; d < c->D; ++d) ptr[d + 1] = ptr[d] + rec[(size_t)d].y;
        if (ptr[c->D] > ptr[0] && (!topics || !counts)) return fail(MLDA_EINVAL, "topics or counts is null");
        if (ptr[c->D] == ptr[0]) return (int)MLDA_OK;
        return with_layout(c->rows, [&](auto layout) {
            if (!unpack) return export_rows<decltype(layout)>(c, rec, ptr, topics, counts);
            unpack_rows<decltype(layout)>(c, rec, slots, ptr, topics, counts);
            return (int)MLDA_OK;
        });
    };
    if (c->streamed) {
        // chunks are visited in document order, so every chunk finds its first row start in place
        RC_TRY(for_each_chunk_rows(c, take_rows));
    } else {
        RC_TRY(take_rows(c->chunks[0]));
    }
    return MLDA_OK;
}

int mlda_get_loglik(mlda_ctx* c, double* ll) {
    RC_TRY(need_state(c));
    if (!ll) return fail(MLDA_EINVAL, "ll is null");
    if (!c->ll_fresh) {
        if (c->streamed) {
            RC_TRY(for_each_chunk_rows(c, [](const HostChunk&) { return (int)MLDA_OK; }));
            RC_TRY(launch_loglik(c));
        } else {
            RC_TRY(launch_loglik(c));
        }
    }
    return fetch_now(c, ll, c->ll_scalars, 8);
}

int mlda_get_timing(mlda_ctx* c, double* ms, int32_t capacity_iters, int32_t* n_iters) {
    if (!c || !ms || !n_iters || capacity_iters < 0) return fail(MLDA_EINVAL, "bad argument");
    HIP_TRY(hipStreamSynchronize(c->stream));
    const int32_t n = std::min(c->timed_iters, capacity_iters);
    const int32_t first = c->timed_iters - n;
    if (c->streamed) {
        // per iteration the sums over its chunk visits: sampling | phi | theta rebuild and the
        // two order changes | the theta rebuild of the new topics (log-likelihood)
        HIP_TRY(hipStreamSynchronize(c->down_stream));
        for (int32_t i = 0; i < 4 * n; ++i) ms[i] = 0.0;
        for (const mlda_ctx::Visit& v : c->visit_log) {
            if (v.iter_row < first) continue;
            hipEvent_t* ev = &c->events[v.event0];
            float t[kVisitEvents - 1];
            for (int j = 0; j + 1 < kVisitEvents; ++j) HIP_TRY(hipEventElapsedTime(&t[j], ev[j], ev[j + 1]));
            double* row = ms + (size_t)(v.iter_row - first) * 4;
            row[0] += t[2];
            row[1] += t[3];
            row[2] += t[0] + t[1] + t[4];
            row[3] += t[5];
        }
        *n_iters = n;
        return MLDA_OK;
    }
    // a phase lasts until the next one that was launched starts
    std::vector<unsigned long long> at;
    try { at.resize((size_t)n * kPhases + 1); } catch (const std::bad_alloc&) { return fail(MLDA_ENOMEM, "out of host memory"); }
    if (n > 0) RC_TRY(fetch(c, at.data(), c->stamps + (size_t)first * kPhases, at.size() * 8));
    for (int32_t i = 0; i < n; ++i)
        for (int j = 0; j < kPhases; ++j) {
            const size_t p = (size_t)i * kPhases + j, next = j == 2 && !c->last_step_loglik ? p + 2 : p + 1;
            ms[p] = j == 3 && !c->last_step_loglik ? 0.0 : (double)(at[next] - at[p]) / c->clock_khz;
        }
    *n_iters = n;
    return MLDA_OK;
}

int mlda_get_sampler_bytes(mlda_ctx* c, double* bytes, int32_t capacity_iters, int32_t* n_iters) {
    RC_TRY(need_state(c));
    if (!bytes || !n_iters || capacity_iters < 0) return fail(MLDA_EINVAL, "bad argument");
    const int32_t n = std::min({c->last_step_iters, capacity_iters, kMaxTimedIters});
    // iteration j of the step (0-based, of last_step_iters) sampled from the state left by
    // rebuild number (rebuilds - last_step_iters + j - 1)
    std::vector<unsigned long long> ring((size_t)kEntryRing);
    HIP_TRY(hipMemcpyAsync(ring.data(), c->row_entries, (size_t)kEntryRing * 8, hipMemcpyDeviceToHost,
                           c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    const double entry_bytes = c->K < 1024 ? 2.0 : 4.0;     // of the nominal entries the rebuild counts
    if (c->streamed) {          // per iteration the sum over its chunk visits
        const int32_t m = std::min(c->timed_iters, capacity_iters), first = c->timed_iters - m;
        for (int32_t i = 0; i < m; ++i) bytes[i] = 0.0;
        for (const mlda_ctx::Visit& v : c->visit_log) {
            if (v.iter_row < first) continue;
            bytes[v.iter_row - first] += 16.0 * (double)v.T +
                entry_bytes * (double)ring[(size_t)(v.rebuild % kEntryRing)] +
                (double)c->K * (2.0 * (double)v.n_tiles + 2.0 * (double)v.n_wide_tiles);
        }
        *n_iters = m;
        return MLDA_OK;
    }
    for (int32_t i = 0; i < n; ++i) {
        const int32_t j = c->last_step_iters - n + i;
        const int64_t r = c->rebuilds - c->last_step_iters + j - 1;
        const double row_entries = c->D > 0 ? (double)ring[(size_t)(r % kEntryRing)] : 0.0;
        // per token: row slot 4, token id 4, old topic 2, new topic 2, row length 4
        // per tile: the word's row of phi, 2 K bytes, or 4 K for a word with 2^16 tokens or more;
        // a tile that follows another one (small words, p* in LDS) reads, instead of a row of phi, the topics of
        // the previous tile's tokens and, for its own tokens, topic and cell of phi: 6 bytes
        // per token, counted as if both tiles had this tile's tokens (and as runs of kRunTiles)
        const bool in_runs = c->queued && !c->far_weights;
        const int32_t n_run_tiles = in_runs ? c->n_tiles - c->n_single : 0;
        const int32_t n_runs = (n_run_tiles + kRunTiles - 1) / kRunTiles;
        const double staged_rows = (double)(c->counted_tiles - n_run_tiles + n_runs);
        bytes[i] = 16.0 * (double)c->T + entry_bytes * row_entries +
                   (double)c->K * (2.0 * staged_rows + 2.0 * (double)c->n_wide_tiles) +
                   (in_runs ? 6.0 * (double)c->run_tokens : 0.0);
    }
    *n_iters = n;
    return MLDA_OK;
}

void mlda_destroy(mlda_ctx* c) { destroy(c); }

int mlda_philox_uniform(uint64_t seed, uint32_t iter, uint64_t token0, int64_t n, double* out_dev,
                        void* hip_stream) {
    if (n < 0) return fail(MLDA_EINVAL, "n must be >= 0");
    if (n == 0) return MLDA_OK;
    if (!out_dev) return fail(MLDA_EINVAL, "out_dev is null");
    hipLaunchKernelGGL(mlda::philox_uniform_kernel, dim3(blocks_for(n, 256)), dim3(256), 0,
                       (hipStream_t)hip_stream, seed, iter, token0, n, out_dev);
    return launch_check("philox_uniform_kernel");
}

}  // extern "C"
