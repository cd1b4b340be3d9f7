// Model update kernels (paper Section 6.2): phi and n_k from the word-sorted
// assignments, theta rows from the document->token map; plus the order changes at
// the boundary and the log-likelihood reductions.
#pragma once
#include "device_util.hpp"
#include "kernels_sample.hpp"

namespace mlda {

// (where no launch of the phase itself stores it)
__global__ void stamp_kernel(unsigned long long* at) { stamp_start(at); }

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// The sum of n values left by the workgroups of a theta rebuild.  256 threads; the first one stores it.
__device__ __forceinline__ void store_visited_sum(const unsigned long long* partial, int n, unsigned long long* out) {
    __shared__ unsigned long long wsum[4];
    unsigned long long acc = 0ull;
    for (int i = (int)threadIdx.x; i < n; i += 256) acc += partial[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
    if (lane_id() == 0) wsum[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) *out = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}
__global__ __launch_bounds__(256) void visited_sum_kernel(const unsigned long long* partial, int n,
                                                          unsigned long long* out) {
    store_visited_sum(partial, n, out);
}

// What the rebuilds of one state add to must start at zero: the rows of words whose tokens span
// several segments, and the topic totals where the theta rebuild before has not cleared them
// (n_k null: it has).  grid = (#split words + 1, ceil(K / blockDim)).
__global__ void zero_sums_kernel(const int32_t* split_words, PhiView phi, int32_t K, int32_t* n_k,
                                 unsigned long long* started) {
    stamp_start(started);
    const int k = (int)(blockIdx.y * blockDim.x + threadIdx.x);
    if (k >= K) return;
    if (blockIdx.x == 0) {
        if (n_k) n_k[k] = 0;
        return;
    }
    const int v = split_words[blockIdx.x - 1], wide_row = phi.wide_row[v];
    if (wide_row >= 0) phi.wide[(size_t)wide_row * (size_t)K + k] = 0;
    else phi.narrow[(size_t)v * (size_t)K + k] = 0;
}

// f(topic) for the tokens [lo, hi) of z, by kThreads threads of which this is number `me`: 16 bytes (eight tokens) per load,
// four loads in flight per thread, single tokens only before the first and after the last aligned eight.
template <int kThreads, class F>
__device__ __forceinline__ void for_topics(const uint16_t* z, int64_t lo, int64_t hi, int me, F&& f) {
    const int64_t lo8 = min((lo + 7) & ~(int64_t)7, hi), hi8 = max(hi & ~(int64_t)7, lo8);
    const int n_head = (int)(lo8 - lo), n_ends = n_head + (int)(hi - hi8);      // at most 14
    int end_topic = -1;
    if (me < n_ends) end_topic = (int)z[me < n_head ? lo + me : hi8 + (me - n_head)];
    auto add_pair = [&](uint32_t two) { f((int)(two & 0xffffu)); f((int)(two >> 16)); };
    auto add_eight = [&](const uint4& v) { add_pair(v.x); add_pair(v.y); add_pair(v.z); add_pair(v.w); };
    const uint4* eights = reinterpret_cast<const uint4*>(z + lo8);
    const int64_t n8 = (hi8 - lo8) / 8;
    int64_t i = me;
    for (; i + 3 * kThreads < n8; i += 4 * kThreads) {
        const uint4 v0 = eights[i], v1 = eights[i + kThreads], v2 = eights[i + 2 * kThreads], v3 = eights[i + 3 * kThreads];
        add_eight(v0); add_eight(v1); add_eight(v2); add_eight(v3);
    }
    for (; i < n8; i += kThreads) add_eight(eights[i]);
    if (end_topic >= 0) f(end_topic);
}

// Topic totals of the tokens [lo, hi) (lo a multiple of 8) added to n_k, through 32-bit counters of the
// topics k_lo .. k_lo + n - 1 in LDS.  (Every workgroup adds each of its topics to the same n_k, 5 ns a time
// for one address: what counts is few workgroups.)
template <bool kRange>
__device__ __forceinline__ void add_topic_totals(int32_t* hist, const uint16_t* z, int64_t lo, int64_t hi, int32_t* n_k,
                                                 int32_t k_lo, int32_t n) {
    const int tid = (int)threadIdx.x;
    for (int k = tid; k < n; k += 256) hist[k] = 0;
    __syncthreads();
    for_topics<256>(z, lo, hi, tid, [&](int k) {
        if (kRange) k -= k_lo;
        if (!kRange || (unsigned)k < (unsigned)n) atomicAdd(&hist[k], 1);
    });
    __syncthreads();
    for (int k = tid; k < n; k += 256) {
        const int c = hist[k];
        if (c != 0) atomicAdd(&n_k[k_lo + k], c);
    }
}

// Update phi (Section 6.2: word by word, atomics with good locality): a workgroup
// histograms one segment (up to 16384 consecutive tokens of one word) in LDS, then stores
// the word's row outright if the segment is the whole word, else adds its non-zero bins
// to the row.  A narrow row is written by dwords of two cells and more, and added to by dwords; the word
// has fewer than 2^16 tokens, so no sum carries into the neighbouring cell.
// Bound by the LDS atomics, 33 to 50 cycles of a CU for a wave's 64 tokens, and small corpora by how fast workgroups
// start: 7.4e8 tokens at K = 1,000 take 0.60 ms with their totals, 1e6 at 128 14 us (0.71 and 21 with a workgroup per segment).
// kPacked: two topics share a dword of LDS (a segment's counts fit 16 bits), so that every K fits at once.
// More atomics then meet at one address: 1e6 to 1e7 tokens at K = 128 ... 1,537 take 3 to 9 % longer than
// with a dword per topic.  Where that takes so much LDS that fewer workgroups fit a CU it is the slower one:
// 2e7 tokens at K = 4,200 90 us (packed 92), 8,000 131 (123), 16,000 158 (147), 30,000 290 (250).
// The segments from n_shared on are counted by a wave each, four of them to a workgroup.
// The workgroups behind those do what else one launch can (each launch costs a small corpus 5 us):
// n_totals of them add the topic totals of a share of the tokens to n_k (which is zero on entry), and the
// last one adds up the counts that the theta rebuild before left (`visited`, to visited_sum; null: none).

// Up to which K a topic has a dword, and the LDS bytes of a segment's counters (the totals' counters are dwords).
constexpr int32_t kPhiDwordTopics = 4096;
__host__ __device__ inline size_t phi_counter_bytes(int32_t K) {
    return ((K <= kPhiDwordTopics ? (size_t)K * 4 : (size_t)((K + 1) / 2) * 4) + 15) & ~(size_t)15;
}
// One segment by kThreads threads, of which this is number `me`; `lds` is theirs, `sync` makes them wait for each other.
template <bool kPacked, int kThreads, class Sync>
__device__ __forceinline__ void phi_segment(unsigned char* lds, const Tile& tl, const uint16_t* z, const PhiView& phi, int32_t K,
                                            int me, Sync&& sync) {
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds);
    const int wide_row = phi.wide_row[tl.word];
    const int n_counters = kPacked ? (K + 1) / 2 : K;
    for (int i = me; i < (n_counters + 3) / 4; i += kThreads) reinterpret_cast<uint4*>(lds)[i] = make_uint4(0u, 0u, 0u, 0u);
    sync();
    for_topics<kThreads>(z, tl.begin, (int64_t)tl.begin + tl.count, me, [&](int k) {
        if (kPacked) atomicAdd(&hist[k >> 1], 1u << ((k & 1) << 4));
        else atomicAdd(&hist[k], 1u);
    });
    sync();
    auto count_of = [&](int k) -> uint32_t {        // (0 outside the row)
        if ((unsigned)k >= (unsigned)K) return 0u;
        return kPacked ? (hist[k >> 1] >> ((k & 1) << 4)) & 0xffffu : hist[k];
    };
    if (wide_row >= 0) {                // (2^16 tokens or more: never a whole word)
        int32_t* row = phi.wide + (size_t)wide_row * (size_t)K;
        for (int k = me; k < K; k += kThreads) {
            const int c = (int)count_of(k);
            if (c != 0) atomicAdd(&row[k], c);
        }
        return;
    }
    const size_t cell0 = (size_t)tl.word * (size_t)K;
    if (tl.whole > 0 && (K & 7) == 0) {     // (every row starts at a multiple of 16 bytes)
        uint4* row = reinterpret_cast<uint4*>(phi.narrow + cell0);
        const uint4* counts = reinterpret_cast<const uint4*>(lds);
        for (int i = me; i < K / 8; i += kThreads) {
            if (kPacked) {
                row[i] = counts[i];
            } else {
                const uint4 a = counts[2 * i], b = counts[2 * i + 1];
                row[i] = make_uint4(a.x | a.y << 16, a.z | a.w << 16, b.x | b.y << 16, b.z | b.w << 16);
            }
        }
        return;
    }
    // The row's dwords: with an odd K every other row starts in the upper half of one, which then holds
    // the row's first cell only (as the last may hold its last only; the other half is another row's).
    const int odd = (int)(cell0 & 1);
    uint32_t* dwords = reinterpret_cast<uint32_t*>(phi.narrow) + (cell0 >> 1);
    for (int i = me; i < (K + odd + 1) / 2; i += kThreads) {
        const int k = 2 * i - odd;
        const uint32_t two = count_of(k) | count_of(k + 1) << 16;
        if (tl.whole <= 0) {
            if (two != 0u) atomicAdd(&dwords[i], two);
        } else if (k < 0) {
            phi.narrow[cell0] = (uint16_t)(two >> 16);
        } else if (k + 1 >= K) {
            phi.narrow[cell0 + k] = (uint16_t)two;
        } else {
            dwords[i] = two;
        }
    }
}
// What the lanes of a wave wrote to LDS is there for all of them.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
constexpr int kPhiWaves = 4;        // waves of a workgroup
// Words of few tokens over many topics (kPacked): their rows hold the counts of z_old, and only the cells of the old and the new topics
// are written.  A workgroup takes every `blocks`-th of the n segments; its counters are zero between them.
// Bound by waiting for each word's topics (the next one's are on their way): 4e6 tokens of 60,000 words at K = 9,000 took 263 us
// with every row written anew, 91 so (changed_cells_for has the line).
__device__ __forceinline__ void phi_changed_cells(unsigned char* lds, const Tile* segs, int32_t n, const uint16_t* z_old,
                                                  const uint16_t* z, const PhiView& phi, int32_t K, int block, int blocks) {
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds);
    const int tid = (int)threadIdx.x;
    for (int i = tid; i < ((K + 1) / 2 + 3) / 4; i += 256) reinterpret_cast<uint4*>(lds)[i] = make_uint4(0u, 0u, 0u, 0u);
    auto count_of = [&](int k) { return (hist[k >> 1] >> ((k & 1) << 4)) & 0xffffu; };
    auto add = [&](int k) { atomicAdd(&hist[k >> 1], 1u << ((k & 1) << 4)); };
    int i = block;
    Tile tl = {0, 0, 0, 0};
    int was = 0, is = 0;            // topics of the thread's first token
    auto ask = [&](int at) {
        if (at < n) tl = segs[at]; else tl.count = 0;
        if (tid < tl.count) { was = (int)z_old[tl.begin + tid]; is = (int)z[tl.begin + tid]; }
    };
    ask(i);
    __syncthreads();
    while (i < n) {
        const Tile cur = tl;
        const int my_was = was, my_is = is;
        uint16_t* row = phi.narrow + (size_t)cur.word * (size_t)K;
        i += blocks;
        ask(i);
        const bool mine = tid < cur.count;
        if (mine) add(my_is);
        for (int t = tid + 256; t < cur.count; t += 256) add((int)z[cur.begin + t]);
        __syncthreads();
        auto write = [&](int before, int now) {
            if (count_of(before) == 0u) row[before] = 0;
            row[now] = (uint16_t)count_of(now);
        };
        if (mine) write(my_was, my_is);
        for (int t = tid + 256; t < cur.count; t += 256) write((int)z_old[cur.begin + t], (int)z[cur.begin + t]);
        __syncthreads();
        if (mine) hist[my_is >> 1] = 0u;
        for (int t = tid + 256; t < cur.count; t += 256) hist[(int)z[cur.begin + t] >> 1] = 0u;
        __syncthreads();
    }
}
struct PhiArgs {
    const Tile* segs;
    int32_t n_segs, n_shared;
    // kPacked: the n_changed segments behind those n_segs are phi_changed_cells's, by this many workgroups
    int32_t n_changed, changed_blocks;
    const uint16_t* z_old;
    const uint16_t* z;
    PhiView phi;
    int32_t K;
    int64_t T;
    int32_t n_totals;
    int32_t* n_k;
    const unsigned long long* visited;
    int32_t n_visited;
    unsigned long long* visited_sum;
    unsigned long long* started;
};
// What workgroup `block` of a phi rebuild does.
template <bool kPacked>
__device__ __forceinline__ void phi_work(unsigned char* lds, const PhiArgs& a, int block) {
    if constexpr (kPacked) {        // (first: they take longest)
        if (block < a.changed_blocks) {
            phi_changed_cells(lds, a.segs + a.n_segs, a.n_changed, a.z_old, a.z, a.phi, a.K, block, a.changed_blocks);
            return;
        }
        block -= a.changed_blocks;
    }
    const int tid = (int)threadIdx.x, n_solo_groups = (a.n_segs - a.n_shared + kPhiWaves - 1) / kPhiWaves;
    if (block < a.n_shared) {
        phi_segment<kPacked, 256>(lds, a.segs[block], a.z, a.phi, a.K, tid, [] { __syncthreads(); });
    } else if (block < a.n_shared + n_solo_groups) {
        const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), i = a.n_shared + (block - a.n_shared) * kPhiWaves + wave;
        if (i < a.n_segs)
            phi_segment<kPacked, kWave>(lds + (size_t)wave * phi_counter_bytes(a.K), a.segs[i], a.z, a.phi, a.K, tid & (kWave - 1),
                                        [] { wave_sync(); });
    } else {
        const int part = block - a.n_shared - n_solo_groups;
        if (part < a.n_totals) {
            const int64_t per = ((a.T + a.n_totals - 1) / a.n_totals + 7) & ~(int64_t)7;
            const int64_t lo = min(per * part, a.T);
            add_topic_totals<false>(reinterpret_cast<int32_t*>(lds), a.z, lo, min(lo + per, a.T), a.n_k, 0, a.K);
        } else if (a.visited_sum) {
            store_visited_sum(a.visited, a.n_visited, a.visited_sum);
        }
    }
}
template <bool kPacked>
__global__ __launch_bounds__(256) void phi_tile_kernel(const PhiArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    stamp_start(a.started);
    phi_work<kPacked>(lds, a, (int)blockIdx.x);
}

// n_k[k] = number of tokens with topic k, as a launch of its own: each workgroup over a contiguous
// share of the tokens; n_k must be zero on entry.
// kRange: K counters do not fit a workgroup's LDS; the launch then covers the topics
// k_lo .. k_lo + kn - 1 only (one launch per such range), else all K.
template <bool kRange>
__global__ __launch_bounds__(256) void topic_totals_kernel(const uint16_t* z, int64_t T, int32_t* n_k,
                                                           int32_t K, int32_t k_lo, int32_t kn) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int64_t per = ((T + gridDim.x - 1) / gridDim.x + 7) & ~(int64_t)7;
    const int64_t lo = min(per * blockIdx.x, T);
    add_topic_totals<kRange>(reinterpret_cast<int32_t*>(lds), z, lo, min(lo + per, T), n_k, kRange ? k_lo : 0,
                             kRange ? kn : K);
}

// The same totals as column sums of n_wk (cheaper than a pass over z when V K is small next to
// T): thread x of a workgroup owns topic blockIdx.x * 256 + x, workgroup row blockIdx.y a
// slice of the words, and the same slice of the wide rows (there are at most V of them); reads
// are coalesced along a word's row.  n_k must be zero on entry.
__global__ __launch_bounds__(256) void topic_totals_from_rows_kernel(PhiView phi, int32_t V, int32_t n_wide,
                                                                     int32_t K, int32_t words_per_slice,
                                                                     int32_t* n_k) {
    const int k = (int)(blockIdx.x * 256 + threadIdx.x);
    if (k >= K) return;
    const int v0 = (int)blockIdx.y * words_per_slice;
    int acc = 0;
    for (int v = v0; v < min(v0 + words_per_slice, V); ++v) acc += (int)phi.narrow[(size_t)v * (size_t)K + k];
    for (int r = v0; r < min(v0 + words_per_slice, n_wide); ++r) acc += phi.wide[(size_t)r * (size_t)K + k];
    if (acc != 0) atomicAdd(&n_k[k], acc);
}

// ------------------------------------------------------------------ log-likelihood helpers
// log p(w,z) = sum_k [lgG(V beta) - lgG(n_k + V beta)] + sum_{v,k} [lgG(n_wk + beta) - lgG(beta)]
//            + sum_d [lgG(K alpha) - lgG(N_d + K alpha)] + sum_{d,k} [lgG(n_dk + alpha) - lgG(alpha)]
// Each workgroup writes one fp64 partial; one workgroup adds them in a fixed order, so the
// value does not depend on scheduling.

// The sum over a workgroup of 256 threads of the n partials each thread takes every 256th of.
// (kShared: the partials come from workgroups of the same launch, and are read past the caches.)
template <bool kShared>
__device__ __forceinline__ double partials_sum(const double* partial, int n) {
    double acc = 0.0;
    for (int i = (int)threadIdx.x; i < n; i += 256)
        acc += kShared ? __hip_atomic_load(partial + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : partial[i];
    return acc;
}
__device__ __forceinline__ double block_sum_256(double acc) {
    __shared__ double buf[256];
    buf[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) buf[threadIdx.x] += buf[threadIdx.x + s];
        __syncthreads();
    }
    return buf[0];
}

// The log-likelihood: the word side's partials, those of the theta rebuild (or, streamed, their
// sum) and the documents' term.
template <bool kShared>
__device__ __forceinline__ void store_loglik(const double* partial, int n, const double* theta_partial, int n_theta,
                                             const double* theta_sum, const double* doc_term, double* out) {
    double sum = partials_sum<kShared>(partial, n) + partials_sum<false>(theta_partial, n_theta);
    if (threadIdx.x == 0) {
        if (theta_sum) sum += *theta_sum;
        sum += *doc_term;
    }
    sum = block_sum_256(sum);
    if (threadIdx.x == 0) *out = sum;
}

// (n_before: so many of the partials are there already, and are added to.  kShared: written past the caches, and there when
// the call returns to the first thread)
template <bool kShared = false>
__device__ __forceinline__ void block_partial_store(double v, double* partial, int n_before = 0) {
    __shared__ double wsum[16];
    const int lane = lane_id(), wave = (int)threadIdx.x / kWave;
    const double s = wave_sum(v);
    if (lane == 0) wsum[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int w = 0; w < (int)blockDim.x / kWave; ++w) tot += wsum[w];
        if constexpr (kShared) {
            __hip_atomic_store(partial + blockIdx.x, tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else {
            partial[blockIdx.x] = (int)blockIdx.x < n_before ? partial[blockIdx.x] + tot : tot;
        }
    }
}

// lgG(c + a) - lgG(a) for the small integer counts c < kLgTable that make up almost all
// cells comes from a table, filled once per context in global memory (kLgTable entries, then
// lgG(a) itself, and lgG(b) of another number b): the kernels that use it call no lgamma and stay register-lean.
constexpr int kLgTable = 1024, kLgTableSize = kLgTable + 2;

__global__ void lg_table_kernel(double* table, double a, double b) {
    const double lg_a = lgamma(a);
    const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (c < kLgTable) table[c] = lgamma((double)c + a) - lg_a;
    if (c == kLgTable) table[c] = lg_a;
    if (c == kLgTable + 1) table[c] = lgamma(b);
}

// lgG(x) for x >= 1024 by Stirling's series; the first omitted term is below 1e-24.
__device__ __forceinline__ double lgamma_large(double x) {
    const double r = 1.0 / x, r2 = r * r;
    return (x - 0.5) * log(x) - x + 0.91893853320467274178 +
           r * (1.0 / 12.0 - r2 * (1.0 / 360.0 - r2 * (1.0 / 1260.0)));
}

// Counts of a theta row are small: the rebuild keeps only this many table entries in LDS
// (occupancy matters more there) and reads the rest of the table from global memory.
constexpr int kThetaLgTable = 128;
constexpr int kXcds = 8;            // accelerator dies of an MI355X, each with its own L2

// Where the topic of the document's token `j` is found in z, or -1 past the document's end:
// its word-major position, through the map; or, without a map (z in document order), the
// token's own index.
__device__ __forceinline__ int doc_token_position(const int32_t* doc_map, const DocRec& r, int j) {
    if (j >= r.n) return -1;
    return doc_map ? doc_map[r.begin + j] : r.begin + j;
}

// The same as loads that every lane makes, from an address that exists: past the document's
// end it is the place of the document's last token (of token 0 of the whole array for an empty
// document).  The loads of a step are then all in flight together and none of them sits
// behind a branch, where what follows would wait for everything in flight.
__device__ __forceinline__ int doc_token_position_any(const int32_t* doc_map, const DocRec& r, int j) {
    const int at = r.n > 0 ? r.begin + min(j, r.n - 1) : 0;
    return doc_map ? doc_map[at] : at;
}
// The topic found at such a position, -1 for a token past the document's end.
__device__ __forceinline__ int doc_token_topic(const uint16_t* z, int position, const DocRec& r, int j) {
    const int k = (int)z[position];
    return j < r.n ? k : -1;
}

// LDS bytes of the rebuild's dense row: the counters (two 16-bit counters per dword, or one
// 32-bit counter per topic when some document has 2^16 tokens or more), then one bit per topic
// that marks the non-zero bins.
// (32-bit counters for more than kThetaWideSpan topics would not fit the LDS: such a document is
// counted once per range of that many topics, and its row grows range by range.)
constexpr int32_t kThetaWideSpan = 32768;
__host__ __device__ inline int32_t theta_span(int32_t K, bool wide) {
    return wide && K > kThetaWideSpan ? kThetaWideSpan : K;
}
__host__ __device__ inline size_t theta_counter_bytes(int32_t K, bool wide) {
    const size_t counters = wide ? (size_t)theta_span(K, wide) * 4 : (size_t)((K + 1) / 2) * 4;
    return (counters + 15) & ~(size_t)15;
}
__host__ __device__ inline size_t theta_hist_bytes(int32_t K, bool wide) {
    const size_t marks = (size_t)((theta_span(K, wide) + 31) / 32) * 4;
    return theta_counter_bytes(K, wide) + ((marks + 15) & ~(size_t)15);
}
// (with 2-byte entries also one counter per 32 topics, see more_entries)
__host__ __device__ inline size_t theta_more_bytes(int32_t K) { return K <= 2048 ? (size_t)((K + 31) / 32) * 4 : 0; }
__host__ __device__ inline size_t theta_lds_bytes(int32_t K, bool wide) {
    return theta_hist_bytes(K, wide) + (size_t)kThetaLgTable * 8 + theta_more_bytes(K);
}

// Entries a count of c > 0 takes in a row whose entries hold at most kMax each.
template <class Layout>
__device__ __forceinline__ int entries_of(int c) {
    return (c + Layout::kMaxCount - 1) / Layout::kMaxCount;
}

// The entries of topic k with count c > 0, written from ent[at] on; returns the next place.
template <class Layout>
__device__ __forceinline__ int write_entries(typename Layout::Entry* ent, int at, int k, int c) {
    while (c > Layout::kMaxCount) {
        ent[at++] = Layout::make(Layout::kMaxCount, k);
        c -= Layout::kMaxCount;
    }
    ent[at++] = Layout::make(c, k);
    return at;
}

// Entries that a count c is taken as in the sampler's algorithmic bytes, whatever the layout in
// use: entries of up to 15 tokens where K < 1024 (2 bytes each), of up to 16,383 (4 bytes) beyond.
__device__ __forceinline__ int nominal_entries(int c, int K) {
    return K < 1024 ? (c + 14) / 15 : (c + 16382) / 16383;
}

// 2-byte entries hold counts up to 7 (31, 63) only, and rows with larger ones are common.  Their entries
// are counted while the tokens are: the token that is one more than a multiple of kMaxCount (of 15
// or 16,383) begins another entry (another nominal one).  Added to the counter of the topic's 32, the
// entries in the lower half, the nominal ones in the upper (fewer than 2^16 tokens: neither
// overflows).  Against looking every bin of such a row up again: 7.2 -> 6.05 ms for 8.2e6 documents
// of 90 tokens at K = 1,000.
// kPlainCount: a count up to which a topic of a row is one entry, and one nominal entry.
template <class Layout> constexpr int kPlainCount = Layout::kEntryBytes == 2 && Layout::kMaxCount > 15 ? 15 : Layout::kMaxCount;
template <class Layout>
__device__ __forceinline__ void more_entries(uint32_t* more, int k, int before, int K) {
    if (before >= kPlainCount<Layout>) {
        const uint32_t another = before % Layout::kMaxCount == 0 ? 1u : 0u;
        const uint32_t nominal = (K < 1024 ? before % 15 : before % 16383) == 0 ? 1u << 16 : 0u;
        if (another | nominal) atomicAdd(&more[k >> 5], another | nominal);
    }
}

// What closes a row: padding entries up to a whole unit (lanes 0 .. 6 of `hl`), the number of
// entries at the head of the slot and a padding entry at the header's very end, so that the
// entry "before the first" is never anybody's topic.
template <class Layout>
__device__ __forceinline__ void close_row(unsigned char* head, int n_entries, int K, int hl, bool real) {
    typedef typename Layout::Entry Entry;
    Entry* ent = reinterpret_cast<Entry*>(head + kRowHeader);
    const int padded = (n_entries + Layout::kUnitEntries - 1) / Layout::kUnitEntries * Layout::kUnitEntries;
    if (real && hl < padded - n_entries) ent[n_entries + hl] = Layout::make(0, K);
    if (real && hl == 0) {
        *reinterpret_cast<uint32_t*>(head) = (uint32_t)n_entries;
        ent[-1] = Layout::make(0, K);
    }
}

// The topic totals that nobody reads any more (null: there are none), for the next phi rebuild to add to.
// (by `threads` threads, of which this is number `me`)
__device__ __forceinline__ void clear_old_totals(int32_t* old_n_k, int32_t K, int me, int threads) {
    if (old_n_k)
        for (int k = me; k < K; k += threads) old_n_k[k] = 0;
}

// Update theta (Section 6.2): document by document, (1) a dense K-long histogram of the
// document's assignments, reached through the document->token map, (2) compaction of the
// non-zero bins into the row (topics ascending).  One wave per document, persistent; the
// dense row lives in LDS and is left all-zero for the next document.  Documents are taken in
// the order the tokens have inside a word (falling length), so that documents in flight
// together gather from neighbouring lines of z.  The walk is a chain of dependent loads
// (record -> map -> z), so it is software-pipelined: while the current document is counted,
// the topics of the wave's next document, the map entries of the one after and the record
// after that are already on their way.  Rows are written in the layout the sampler reads
// (see kernels_sample.hpp).  The compaction visits only the 32-topic
// groups that hold a non-zero bin (one mark bit per topic), so its cost follows the row's
// length rather than K.  While the counts pass through registers the kernel also adds up the
// theta entries' term of the log-likelihood, sum_{d,k} lgG(n_dk + alpha) - lgG(alpha), one
// partial per workgroup.
// kDocWaves: waves that count a document together.  One, but where the documents are too few for
// a wave each to fill the chip and long enough to be counted by many: a wave alone takes
// 0.79 ms for the longest of 311 documents of 30,000 tokens, sixteen take 0.11 ms.
constexpr int kLongDocWaves = 16;
template <class Layout, bool kWide, int kDocWaves = 1>
__global__ __launch_bounds__(kWave * kDocWaves) void theta_rows_kernel(const DocRec* docs,
                                                           const int32_t* doc_map,
                                                           const uint16_t* z, uint2* row_rec,
                                                           unsigned char* slots, int64_t D, int64_t T,
                                                           int32_t K, double alpha,
                                                           const double* lg_table,
                                                           unsigned long long* visited_partial,
                                                           double* ll_partial, int32_t* old_n_k,
                                                           unsigned long long* started) {
    typedef typename Layout::Entry Entry;
    stamp_start(started);
    clear_old_totals(old_n_k, K, (int)(blockIdx.x * blockDim.x + threadIdx.x), (int)(gridDim.x * blockDim.x));
    if (T == 0) {       // no token anywhere: the loads "past a document's end" still need a place that exists
        doc_map = nullptr;
        z = reinterpret_cast<const uint16_t*>(docs);
    }
    extern __shared__ __align__(16) unsigned char lds[];
    uint32_t* hist = reinterpret_cast<uint32_t*>(lds);
    const int span = theta_span(K, kWide);       // topics counted at a time: all, but for kWide and a very large K
    const int n_counters = kWide ? span : (K + 1) / 2;
    const int n_marks = (span + 31) / 32;
    uint32_t* marks = reinterpret_cast<uint32_t*>(lds + theta_counter_bytes(K, kWide));
    double* table = reinterpret_cast<double*>(lds + theta_hist_bytes(K, kWide));
    constexpr bool kMore = sizeof(Entry) == 2 && !kWide;
    // nominal entries: those of the row where the layout is PackedRows; counted with the tokens (kMore), or
    // bin by bin as the row is written
    constexpr bool kNominal = Layout::kDoubleWeights, kNominalByBin = kNominal && !kMore;
    [[maybe_unused]] uint32_t* more = reinterpret_cast<uint32_t*>(table + kThetaLgTable);
    // the document's tokens are dealt to all threads (`me` of `width`); its row is the first wave's
    constexpr int width = kWave * kDocWaves;
    const int me = (int)threadIdx.x, lane = me & (kWave - 1);
    const bool writes_row = kDocWaves == 1 || me < kWave;
    const double lg_alpha = lg_table[kLgTable];
    for (int k = me; k < n_counters; k += width) hist[k] = 0u;
    for (int k = me; k < n_marks; k += width) marks[k] = 0u;
    if constexpr (kMore)
        for (int k = me; k < n_marks; k += width) more[k] = 0u;
    for (int c = me; c < kThetaLgTable; c += width) table[c] = lg_table[c];
    __syncthreads();
    unsigned long long visited = 0;      // sum of N_d * (nominal entries of row d) over this wave's documents
    double ll = 0.0;
    // lgG(c + alpha) - lgG(alpha) added to `ll`; the rare large counts go through a branch the
    // whole wave takes or skips, so that the common case never pays for the logarithm
    auto add_ll = [&](int c) {
        if (c > 0 && c < kThetaLgTable) ll += table[c];
        if (__ballot(c >= kThetaLgTable) != 0) {
            if (c >= kThetaLgTable)
                ll += c < kLgTable ? lg_table[c] : lgamma_large((double)c + alpha) - lg_alpha;
        }
    };
    // one more token of topic k; true if the topic's count has outgrown one entry (kPlainCount)
    auto count_topic = [&](int k) -> bool {
        atomicOr(&marks[k >> 5], 1u << (k & 31));
        if (kWide) return (int)atomicAdd(&hist[k], 1u) >= kPlainCount<Layout>;
        const int before = (int)((atomicAdd(&hist[k >> 1], 1u << ((k & 1) << 4)) >> ((k & 1) << 4)) & 0xffffu);
        if constexpr (kMore) more_entries<Layout>(more, k, before, K);
        return before >= kPlainCount<Layout>;
    };
    // the same for a document too short for that (the atomics then return nothing)
    auto count_topic_short = [&](int k) {
        atomicOr(&marks[k >> 5], 1u << (k & 31));
        if (kWide) atomicAdd(&hist[k], 1u);
        else atomicAdd(&hist[k >> 1], 1u << ((k & 1) << 4));
    };
    auto count_of = [&](int k) -> int {    // (narrow counters: the pair's other half stays)
        return kWide ? (int)hist[k] : (int)((hist[k >> 1] >> ((k & 1) << 4)) & 0xffffu);
    };
    const int64_t step = gridDim.x;
    const DocRec none = {0, 0, 0u, 0};
    // workgroups are dealt to the 8 XCDs round-robin: give each XCD a contiguous run of
    // documents, so that neighbouring gathers meet in the same L2
    const int per_xcd = (int)gridDim.x / kXcds;
    int64_t i = (int)blockIdx.x < per_xcd * kXcds
                    ? (int64_t)((int)blockIdx.x % kXcds) * per_xcd + (int)blockIdx.x / kXcds
                    : (int64_t)blockIdx.x;
    // Three loads deep: the topics of this document's first 128 tokens have been gathered, the
    // positions of the next document's tokens read, and the record after that fetched.
    auto record = [&](int64_t d) {      // (the load is made for every d, from the last record if need be)
        const DocRec r = docs[d < D ? d : D - 1];
        return d < D ? r : none;
    };
    DocRec cur = record(i), nxt = record(i + step), after = record(i + 2 * step);
    int k0, k1;
    {
        const int c0 = doc_token_position_any(doc_map, cur, me);
        const int c1 = doc_token_position_any(doc_map, cur, me + width);
        k0 = doc_token_topic(z, c0, cur, me);
        k1 = doc_token_topic(z, c1, cur, me + width);
    }
    int p0 = doc_token_position_any(doc_map, nxt, me);
    int p1 = doc_token_position_any(doc_map, nxt, me + width);
    for (; i < D; i += step) {
        // on their way while this document is counted: the next document's topics, the
        // positions of the one after, the record after that
        const int n0 = doc_token_topic(z, p0, nxt, me);
        const int n1 = doc_token_topic(z, p1, nxt, me + width);
        const int q0 = doc_token_position_any(doc_map, after, me);
        const int q1 = doc_token_position_any(doc_map, after, me + width);
        const DocRec later = record(i + 3 * step);

        const bool long_doc = cur.n > kPlainCount<Layout>;     // (the same for the whole wave)
        unsigned char* head = slots + (size_t)cur.slot * 16u;
        Entry* ent = reinterpret_cast<Entry*>(head + kRowHeader);
        int filled = 0, distinct = 0, nominal = 0;
        bool any_split = false;
        // (one round, but for 32-bit counters and more topics than they have room for)
        for (int k_lo = 0; k_lo < K; k_lo += span) {
        bool outgrown = false;
        auto count = [&](int k) {
            if (k < 0) return;
            if (kWide) {
                k -= k_lo;
                if ((unsigned)k >= (unsigned)span) return;
            }
            if (long_doc) outgrown |= count_topic(k); else count_topic_short(k);
        };
        count(k0);
        count(k1);
        // the rest of a longer document, four tokens per lane at a time: their positions
        // first, then their topics, each group of loads in flight together
        for (int j = 2 * width + me; j - me < cur.n; j += 4 * width) {
            int at[4], k[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) at[t] = doc_token_position_any(doc_map, cur, j + t * width);
#pragma unroll
            for (int t = 0; t < 4; ++t) k[t] = doc_token_topic(z, at[t], cur, j + t * width);
#pragma unroll
            for (int t = 0; t < 4; ++t) count(k[t]);
        }
        // some count of the document takes several entries
        bool may_split;
        if constexpr (kDocWaves == 1) {
            __syncthreads();
            may_split = __ballot(outgrown) != 0;
        } else {
            may_split = __syncthreads_or(outgrown) != 0;
        }
        any_split |= may_split;
        // Each lane owns one word of marks (32 topics) per round and writes its non-zero bins
        // in ascending order behind those of the lanes below it.
        for (int base = 0; writes_row && base < n_marks; base += kWave) {
            const int wi = base + lane;
            uint32_t w = wi < n_marks ? marks[wi] : 0u;
            if (__ballot(w != 0u) == 0) continue;
            int mine = __popc(w);
            distinct += mine;
            if (may_split && kMore) {
                const uint32_t m = wi < n_marks ? more[wi] : 0u;
                nominal += mine + (int)(m >> 16);
                mine += (int)(m & 0xffffu);
                if (m != 0u) more[wi] = 0u;
            } else if (may_split) {    // the lane's entries, counted one bin at a time
                mine = 0;
                for (uint32_t rest = w; rest != 0u; rest &= rest - 1u)
                    mine += entries_of<Layout>(count_of(wi * 32 + __ffs((int)rest) - 1));
            }
            const int upto = wave_inclusive_sum(mine);
            int at = filled + upto - mine;
            filled += read_lane(upto, kWave - 1);
            if (w != 0u) marks[wi] = 0u;
            if (kWide) {
                while (__ballot(w != 0u) != 0) {
                    int c = 0;
                    if (w != 0u) {
                        const int k = wi * 32 + __ffs((int)w) - 1;
                        w &= w - 1u;
                        c = (int)hist[k];
                        hist[k] = 0u;
                        at = write_entries<Layout>(ent, at, k_lo + k, c);
                        if (kNominalByBin) nominal += nominal_entries(c, K);
                    }
                    add_ll(c);
                }
            } else {
                uint32_t pairs = (w | (w >> 1)) & 0x55555555u;
                while (__ballot(pairs != 0u) != 0) {
                    int lo = 0, hi = 0;
                    if (pairs != 0u) {
                        const int k = wi * 32 + __ffs((int)pairs) - 1;    // even topic of the pair
                        pairs &= pairs - 1u;
                        const uint32_t both = hist[k >> 1];
                        hist[k >> 1] = 0u;
                        lo = (int)(both & 0xffffu);
                        hi = (int)(both >> 16);
                        if (lo != 0) at = write_entries<Layout>(ent, at, k, lo);
                        if (hi != 0) at = write_entries<Layout>(ent, at, k + 1, hi);
                        if (kNominalByBin) nominal += nominal_entries(lo, K) + nominal_entries(hi, K);
                    }
                    add_ll(lo);
                    add_ll(hi);
                }
            }
        }
        if (k_lo + span < K) __syncthreads();
        }
        if (writes_row) {
            close_row<Layout>(head, filled, K, lane, true);
            const int nnz = any_split ? wave_sum(distinct) : filled;
            if (lane == 0) row_rec[cur.doc].y = (uint32_t)nnz;      // distinct topics, for the getters
            visited += (unsigned long long)cur.n * (unsigned long long)(kNominalByBin || (kNominal && any_split) ? wave_sum(nominal) : filled);
        }
        __syncthreads();
        cur = nxt; nxt = after; after = later; k0 = n0; k1 = n1; p0 = q0; p1 = q1;
    }
    // row entries the next sampling pass will read: one row walk per token.  (A value per workgroup:
    // added to one counter by atomics, 4,096 waves took 20 to 40 us for it, 5 ns each.  The rebuild of
    // 1e6 tokens in 20,000 documents 60 -> 20 us, of 6.3e6 in 30,011 87 -> 58.)
    if (me == 0) visited_partial[blockIdx.x] = visited;
    block_partial_store(ll, ll_partial);
}

// The same for documents of up to kRankedTokens tokens, without a dense row.  One bit per topic marks the topics
// of the document; a prefix sum over the mark words tells every marked topic its place among them
// (its rank); the tokens then add to a cell per rank, {topic, count}, and the cells leave as the row,
// one per lane in whole consecutive stores.  Against compacting a dense row of K counters: LDS of K / 4 bytes and a cell per
// topic of a row instead of 2 K (K = 40,000: 17 KB and nine waves per CU instead of 92 KB and one), and every step
// takes all lanes, where the lane that owns 32 topics walked its non-zero bins one by one.
// kDocs = 2 (K <= 1024): lanes 0 .. 31 rebuild one document and lanes 32 .. 63 the next one in the working order
// (of similar length) with the same instructions: a document's mark words are one per lane then.
// n_cells: a row with more topics is made in several rounds of so many; n_stage: so many of the
// topics of the tokens beyond those in registers are kept in LDS, the rest is read again.
// Tokens per lane whose topics are in registers: 128 of each document (256 with one document per wave
// took 6 to 9 % longer on 1e8 tokens in documents of 330: more lines of z in use at once).
// A document much longer than that is read again for every 1,024 of its topics, by one wave: beside 3e6 tokens in documents
// of 300, one of 30,000 took 0.21 ms at K = 500, 0.73 at K = 5,000 and 2.05 at K = 40,000, one of 60,000 0.43, 1.5 and
// 6.7.  Those beyond kRankedTokens are theta_rows_kernel's, in a launch before: 0.04, 0.05 and 0.15 ms, and 0.07, 0.08, 0.2.
// Where the line lies, rebuild with all ranked / with that launch, us (K = 500, 5,000, 40,000):
//   one document of 3,000 beside 3e6 tokens   42/57  51/56   67/100      300 of 3,000 beside 3e7   239/221  260/223
//                   4,100                     51/47  71/51   92/90       300 of 4,000              270/218  301/232
// n_before: an earlier launch left the sums of other documents in so many of the partials; they are added to.
__host__ __device__ constexpr int rank_keep(int docs) { return docs == 1 ? 2 : 4; }
constexpr int kRankStage = 2048;
constexpr int kRankedTokens = 3072;
constexpr int kPairMaxK = 1024;
__host__ __device__ inline int theta_rank_words(int32_t K) { return ((K + 31) / 32 + 3) & ~3; }
__host__ __device__ inline int theta_rank_cells(int32_t K, int64_t longest, int docs) {
    const int64_t most = docs == 1 ? 1024 : 512, n = K < longest ? K : longest;
    return (int)(((n < most ? n : most) + 3) & ~(int64_t)3);
}
__host__ __device__ inline int theta_rank_stage(int64_t longest, int docs) {
    const int64_t most = docs == 1 ? kRankStage : 256, n = longest - rank_keep(docs) * (kWave / docs);
    return n <= 0 ? 0 : (int)(((n < most ? n : most) + 3) & ~(int64_t)3);
}
// (a wave's own, and of a workgroup of so many waves with the table.  Whole 16 bytes: the next wave's words and cells are read and
// written by so many, and one document's stage may end in the middle of them)
__host__ __device__ inline size_t theta_rank_wave_bytes(int32_t K, int64_t longest, int docs) {
    return ((size_t)docs * ((size_t)theta_rank_words(K) * 8 + (size_t)theta_rank_cells(K, longest, docs) * 4 +
                            (size_t)theta_rank_stage(longest, docs) * 2) + 15) & ~(size_t)15;
}
__host__ __device__ inline size_t theta_rank_lds_bytes(int32_t K, int64_t longest, int docs, int waves = 1) {
    return (size_t)waves * theta_rank_wave_bytes(K, longest, docs) + (size_t)kThetaLgTable * 8;
}

struct ThetaRankedArgs {
    const DocRec* docs;
    const int32_t* doc_map;
    const uint16_t* z;
    uint2* row_rec;
    unsigned char* slots;
    int64_t D, T;
    int32_t K;
    double alpha;
    const double* lg_table;
    unsigned long long* visited_partial;    // of every worker
    double* ll_partial;
    int32_t* old_n_k;
    unsigned long long* started;
    int32_t n_cells, n_stage, n_before, wave_bytes;
};
// What worker `worker` of `n_workers`, a wave, does; `lds` is its own, `table` the workgroup's.
template <class Layout, int kDocs>
__device__ __forceinline__ void theta_ranked(unsigned char* lds, const double* table, const ThetaRankedArgs& a, int worker, int n_workers) {
    typedef typename Layout::Entry Entry;
    constexpr int W = kWave / kDocs, kKeep = rank_keep(kDocs);      // lanes per document
    const DocRec* docs = a.docs;
    const int32_t* doc_map = a.doc_map;
    const uint16_t* z = a.z;
    const int64_t D = a.D, T = a.T;
    const int32_t K = a.K, n_cells = a.n_cells, n_stage = a.n_stage;
    const double alpha = a.alpha;
    const double* lg_table = a.lg_table;
    const int lane = (int)threadIdx.x & (kWave - 1), part = lane / W, hl = lane % W;
    clear_old_totals(a.old_n_k, K, worker * kWave + lane, n_workers * kWave);
    if (T == 0) {       // no token anywhere: the loads "past a document's end" still need a place that exists
        doc_map = nullptr;
        z = reinterpret_cast<const uint16_t*>(docs);
    }
    const int n_words = theta_rank_words(K);
    // per document: {marks of 32 topics, topics marked before them}, the cells, the topics of further tokens
    uint2* words = reinterpret_cast<uint2*>(lds) + part * n_words;
    uint32_t* cells = reinterpret_cast<uint32_t*>(lds + (size_t)kDocs * n_words * 8) + part * n_cells;
    uint16_t* stage = reinterpret_cast<uint16_t*>(lds + (size_t)kDocs * (n_words * 8 + n_cells * 4)) + part * n_stage;
    const double lg_alpha = lg_table[kLgTable];
    for (int i = lane; i < kDocs * n_words / 2; i += kWave) reinterpret_cast<uint4*>(lds)[i] = make_uint4(0u, 0u, 0u, 0u);
    wave_sync();
    unsigned long long visited = 0;      // sum of N_d * (nominal entries of row d) over this part's documents
    double ll = 0.0;
    auto add_ll = [&](int c) {
        if (c > 0 && c < kThetaLgTable) ll += table[c];
        if (__ballot(c >= kThetaLgTable) != 0) {
            if (c >= kThetaLgTable)
                ll += c < kLgTable ? lg_table[c] : lgamma_large((double)c + alpha) - lg_alpha;
        }
    };
    // inclusive sum over the lanes of a document, and the last lane's value
    auto part_sums = [](int v) {
        if constexpr (kDocs == 1) return wave_inclusive_sum(v);
        v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
        v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
        return v;
    };
    auto part_last = [&](int sums) {
        if constexpr (kDocs == 1) return read_lane(sums, kWave - 1);
        const int a = read_lane(sums, W - 1), b = read_lane(sums, kWave - 1);
        return part ? b : a;
    };
    auto most_of_parts = [&](int v) {       // (v the same in all lanes of a part)
        if constexpr (kDocs == 1) return v;
        return max(read_lane(v, 0), read_lane(v, W));
    };
    // counts up to this one are one entry, and one nominal entry, each
    constexpr bool kNominal = Layout::kDoubleWeights;
    const int plain = min(Layout::kMaxCount, kNominal && K < 1024 ? 15 : 16383);

    const int64_t n_rounds = (D + kDocs - 1) / kDocs, step = n_workers;
    const DocRec none = {0, 0, 0u, 0};
    auto record = [&](int64_t r) {      // (the load is made for every r, from the last record if need be)
        const int64_t d = r * kDocs + part;
        const DocRec rec = docs[d < D ? d : D - 1];
        return d < D ? rec : none;
    };
    int64_t i = worker;
    // One document per wave: three loads deep, as in theta_rows_kernel, every lane making every load.  Two
    // per wave: the topics of the next two documents are on their way while these are counted (positions and
    // topics of one token after the other: many gathers of a wave in flight at once measured slower).
    auto topic_at = [&](const DocRec& r, int j) {
        const int p = doc_token_position(doc_map, r, j);
        return p >= 0 ? (int)z[p] : -1;
    };
    DocRec cur = record(i), nxt = record(i + step), after = record(i + 2 * step);
    int topic[kKeep], next_at[kKeep];
#pragma unroll
    for (int t = 0; t < kKeep; ++t) {
        if constexpr (kDocs == 1) {
            topic[t] = doc_token_topic(z, doc_token_position_any(doc_map, cur, hl + t * W), cur, hl + t * W);
            next_at[t] = doc_token_position_any(doc_map, nxt, hl + t * W);
        } else {
            topic[t] = topic_at(cur, hl + t * W);
        }
    }
    for (; i < n_rounds; i += step) {
        int next_topic[kKeep], after_at[kKeep];
#pragma unroll
        for (int t = 0; t < kKeep; ++t) {
            if constexpr (kDocs == 1) next_topic[t] = doc_token_topic(z, next_at[t], nxt, hl + t * W);
            else next_topic[t] = topic_at(nxt, hl + t * W);
        }
        if constexpr (kDocs == 1) {
#pragma unroll
            for (int t = 0; t < kKeep; ++t) after_at[t] = doc_token_position_any(doc_map, after, hl + t * W);
        }
        const DocRec later = record(i + 3 * step);

        // ---- mark the topics
        auto mark = [&](int k) {
            if (k >= 0) atomicOr(&words[k >> 5].x, 1u << (k & 31));
        };
#pragma unroll
        for (int t = 0; t < kKeep; ++t) mark(topic[t]);
        const int rest = most_of_parts(cur.n) - kKeep * W;      // tokens beyond those, of the longer document
        for (int s = hl; s - hl < rest; s += 4 * W) {
            int at[4], k[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) at[t] = doc_token_position_any(doc_map, cur, kKeep * W + s + t * W);
#pragma unroll
            for (int t = 0; t < 4; ++t) k[t] = doc_token_topic(z, at[t], cur, kKeep * W + s + t * W);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                mark(k[t]);
                if (s + t * W < n_stage) stage[s + t * W] = (uint16_t)k[t];
            }
        }
        wave_sync();
        // ---- topics marked before every word
        int n_topics;
        if constexpr (kDocs == 2) {
            const int mine = hl < n_words ? __popc(words[hl].x) : 0;
            const int upto = part_sums(mine);
            if (hl < n_words) words[hl].y = (uint32_t)(upto - mine);
            n_topics = part_last(upto);
        } else {
            n_topics = 0;
            for (int base = 0; base < n_words; base += 4 * kWave) {
                const int at = base + 4 * lane;         // four words per lane; n_words is a multiple of four
                uint4* two = reinterpret_cast<uint4*>(words + at);
                uint4 a = make_uint4(0u, 0u, 0u, 0u), b = a;
                if (at < n_words) { a = two[0]; b = two[1]; }
                const int c0 = __popc(a.x), c1 = __popc(a.z), c2 = __popc(b.x), mine = c0 + c1 + c2 + __popc(b.z);
                const int upto = part_sums(mine);
                a.y = (uint32_t)(n_topics + upto - mine);
                a.w = a.y + (uint32_t)c0;
                b.y = a.w + (uint32_t)c1;
                b.w = b.y + (uint32_t)c2;
                if (at < n_words) { two[0] = a; two[1] = b; }
                n_topics += part_last(upto);
            }
        }
        wave_sync();
        auto rank_of = [&](int k) {         // k >= 0, marked
            const uint2 w = words[k >> 5];
            return (int)(w.y + (uint32_t)__popc(w.x & ((1u << (k & 31)) - 1u)));
        };
        int rank[kKeep];
#pragma unroll
        for (int t = 0; t < kKeep; ++t) rank[t] = topic[t] >= 0 ? rank_of(topic[t]) : -1;
        // ---- the row, n_cells topics at a time
        unsigned char* head = a.slots + (size_t)cur.slot * 16u;
        Entry* ent = reinterpret_cast<Entry*>(head + kRowHeader);
        int filled = 0, further = 0;        // entries so far; nominal entries beyond one per topic (this lane's)
        bool any_further = false;
        const int most_topics = most_of_parts(n_topics);
        for (int first = 0; first < most_topics; first += n_cells) {
            const int cleared = min(n_topics - first, n_cells);
            for (int e = 4 * hl; e < cleared; e += 4 * W) *reinterpret_cast<uint4*>(cells + e) = make_uint4(0u, 0u, 0u, 0u);
            // a cell: the count below, the topic above (written by every token of the topic)
            auto add_token = [&](int k, int at) {
                if ((unsigned)at < (unsigned)n_cells) {
                    reinterpret_cast<uint16_t*>(cells + at)[1] = (uint16_t)k;
                    atomicAdd(&cells[at], 1u);
                }
            };
            wave_sync();
#pragma unroll
            for (int t = 0; t < kKeep; ++t) add_token(topic[t], rank[t] < 0 ? -1 : rank[t] - first);
            // the tokens beyond those in registers, four per lane at a time
            const int n_rest = cur.n - kKeep * W;
            for (int s = hl; s - hl < rest; s += 4 * W) {
                int k[4], at[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int j = s + t * W;
                    k[t] = j < n_rest && j < n_stage ? (int)stage[j] : -1;
                }
                if (s - hl + 4 * W > n_stage) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int j = s + t * W;
                        if (j >= n_stage) k[t] = topic_at(cur, kKeep * W + j);
                    }
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) at[t] = k[t] >= 0 ? rank_of(k[t]) - first : -1;
#pragma unroll
                for (int t = 0; t < 4; ++t) add_token(k[t], at[t]);
            }
            wave_sync();
            const int here = min(n_topics - first, n_cells), most_here = min(most_topics - first, n_cells);
            for (int e0 = 0; e0 < most_here; e0 += W) {
                const uint32_t cell = e0 + hl < here ? cells[e0 + hl] : 0u;
                const int c = (int)(cell & 0xffffu), k = (int)(cell >> 16);
                if (__ballot(c > plain) == 0) {
                    if (c > 0) ent[filled + hl] = Layout::make(c, k);
                    filled += max(min(here - e0, W), 0);
                } else {                    // some count takes several entries
                    any_further = true;
                    const int mine = c > 0 ? entries_of<Layout>(c) : 0;
                    const int upto = part_sums(mine);
                    if (c > 0) {
                        write_entries<Layout>(ent, filled + upto - mine, k, c);
                        if (kNominal) further += nominal_entries(c, K) - 1;
                    }
                    filled += part_last(upto);
                }
                add_ll(c);
            }
            wave_sync();
        }
        for (int w = 2 * hl; w < n_words; w += 2 * W) *reinterpret_cast<uint4*>(words + w) = make_uint4(0u, 0u, 0u, 0u);
        const bool real = i * kDocs + part < D;          // the last round may lack its second document
        close_row<Layout>(head, filled, K, hl, real);
        int nominal = filled;
        if (kNominal && any_further) nominal = n_topics + part_last(part_sums(further));
        if (real && hl == 0) {
            a.row_rec[cur.doc].y = (uint32_t)n_topics;     // distinct topics, for the getters
            visited += (unsigned long long)cur.n * (unsigned long long)nominal;
        }
        wave_sync();
        cur = nxt; nxt = after; after = later;
#pragma unroll
        for (int t = 0; t < kKeep; ++t) {
            topic[t] = next_topic[t];
            if constexpr (kDocs == 1) next_at[t] = after_at[t];
        }
    }
    if (kDocs == 2) visited += __shfl_xor(visited, W, kWave);       // the other part's documents
    ll = wave_sum(ll);
    if (lane == 0) {
        const bool more = worker < a.n_before;
        a.visited_partial[worker] = more ? a.visited_partial[worker] + visited : visited;
        a.ll_partial[worker] = more ? a.ll_partial[worker] + ll : ll;
    }
}

// The log-gamma terms of small counts, for the workgroup's waves.
__device__ __forceinline__ void stage_theta_table(double* table, const double* lg_table) {
    for (int c = (int)threadIdx.x; c < kThetaLgTable; c += (int)blockDim.x) table[c] = lg_table[c];
    __syncthreads();
}
// Number of the worker that workgroup `block` of `blocks` is first: workgroups are dealt to the XCDs round-robin, each XCD
// takes a contiguous run of documents (see theta_rows_kernel).
__device__ __forceinline__ int first_worker(int block, int blocks, int waves) {
    const int per_xcd = blocks / kXcds;
    return (block < per_xcd * kXcds ? block % kXcds * per_xcd + block / kXcds : block) * waves;
}

template <class Layout, int kDocs>
__global__ __launch_bounds__(kWave) void theta_ranked_kernel(const ThetaRankedArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    stamp_start(a.started);
    stage_theta_table(reinterpret_cast<double*>(lds), a.lg_table);
    theta_ranked<Layout, kDocs>(lds + kThetaLgTable * 8, reinterpret_cast<const double*>(lds), a,
                                first_worker((int)blockIdx.x, (int)gridDim.x, 1), (int)gridDim.x);
}

// Both rebuilds of a corpus that neither of them fills the chip with, in one launch: the workgroups of phi, then those of
// theta, four waves each, to each its documents.  Bound by the longest chain of waits, which two launches meet one after
// the other: 1e5 tokens, K = 32, 11.5 us in two, 6.8 in one (kBothTokens has the line).
template <class Layout, int kDocs>
__global__ __launch_bounds__(256) void rebuild_kernel(const PhiArgs p, const ThetaRankedArgs t, int32_t n_phi, int32_t n_theta) {
    extern __shared__ __align__(16) unsigned char lds[];
    stamp_start(p.started);
    if ((int)blockIdx.x < n_phi) {
        phi_work<false>(lds, p, (int)blockIdx.x);
        // (theta's time starts when phi's is over, which some of its workgroups tell; earlier steps left earlier times)
        if (t.started && threadIdx.x == 0 && (blockIdx.x % 64 == 0 || (int)blockIdx.x == n_phi - 1))
            atomicMax(t.started, (unsigned long long)wall_clock64());
        return;
    }
    const int block = (int)blockIdx.x - n_phi, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    stage_theta_table(reinterpret_cast<double*>(lds), t.lg_table);
    theta_ranked<Layout, kDocs>(lds + kThetaLgTable * 8 + (size_t)wave * t.wave_bytes, reinterpret_cast<const double*>(lds), t,
                                first_worker(block, n_theta, 4) + wave, 4 * n_theta);
}

// The two per-token index arrays that follow from tok_id and the document records are built
// on the device rather than sent over PCIe.  doc_map (Section 6.2's document->token map) is the
// inverse of tok_id; tokens are numbered from `first` inside a chunk.
__global__ void derive_doc_map_kernel(const int32_t* tok_id, int64_t T, int64_t first, int32_t* doc_map) {
    const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (pos < T) doc_map[(int64_t)tok_id[pos] - first] = (int32_t)pos;
}

// tok_slot[pos] = slot of the theta row of the document that owns word-major token pos.  One
// wave per document, persistent.
__global__ __launch_bounds__(kWave) void derive_tok_slot_kernel(const DocRec* docs, int64_t D,
                                                                const int32_t* doc_map,
                                                                uint32_t* tok_slot) {
    const int lane = (int)threadIdx.x;
    for (int64_t i = blockIdx.x; i < D; i += gridDim.x) {
        const DocRec r = docs[i];
        for (int j = lane; j < r.n; j += kWave) tok_slot[doc_map[r.begin + j]] = r.slot;
    }
}

// The map entries of every document put in rising order, in runs of kMapSortRun entries (a
// whole document if it has no more).  The rebuild counts a document's topics, so the order in
// which it meets them is free; in rising order the tokens that share their document AND their
// word are neighbours in the map as they are in z, neighbouring lanes then read the same line,
// and the gather asks the caches for it once.  After this the map no longer tells a token's
// place inside its document: only the rebuild and derive_tok_slot_kernel read it.
// One wave per document, persistent; a bitonic network over a run held in LDS.
constexpr int kMapSortRun = 256;
__global__ __launch_bounds__(kWave) void sort_doc_map_kernel(const DocRec* docs, int64_t D, int32_t* doc_map) {
    __shared__ int32_t run[kMapSortRun];
    const int lane = (int)threadIdx.x;
    for (int64_t i = blockIdx.x; i < D; i += gridDim.x) {
        const DocRec r = docs[i];
        for (int base = 0; base < r.n; base += kMapSortRun) {
            const int n = min(kMapSortRun, r.n - base);
            if (n < 2) continue;
            // the smallest power of two that holds the run; places past its end sort last
            int width = 2;
            while (width < n) width <<= 1;
            for (int e = lane; e < width; e += kWave)
                run[e] = e < n ? doc_map[r.begin + base + e] : 0x7fffffff;
            __syncthreads();
            for (int k = 2; k <= width; k <<= 1)
                for (int j = k >> 1; j > 0; j >>= 1) {
                    for (int pair = lane; pair < width / 2; pair += kWave) {
                        const int lo = ((pair & ~(j - 1)) << 1) | (pair & (j - 1)), hi = lo | j;
                        const int32_t a = run[lo], b = run[hi];
                        const bool rising = (lo & k) == 0;
                        if ((a > b) == rising) { run[lo] = b; run[hi] = a; }
                    }
                    __syncthreads();
                }
            for (int e = lane; e < n; e += kWave) doc_map[r.begin + base + e] = run[e];
            __syncthreads();
        }
    }
}

// A chunk without a map (its assignments arrive in document order): every token's topic is
// paired with the slot of its document's theta row, one wave per document, persistent, where
// both are contiguous ...
__global__ __launch_bounds__(kWave) void pair_topics_with_slots_kernel(const DocRec* docs, int64_t D,
                                                                       const uint16_t* z_doc, uint2* pairs) {
    const int lane = (int)threadIdx.x;
    for (int64_t i = blockIdx.x; i < D; i += gridDim.x) {
        const DocRec r = docs[i];
        for (int j = lane; j < r.n; j += kWave)
            pairs[r.begin + j] = make_uint2(r.slot, (uint32_t)z_doc[r.begin + j]);
    }
}

// ... and one gather per word-major token brings both along (tok_id counts from the start of
// the whole corpus, the pairs from token `first`).
__global__ void pairs_to_word_major_kernel(const uint2* pairs, const int32_t* tok_id, uint16_t* z_word,
                                           uint32_t* tok_slot, int64_t T, int64_t first) {
    const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (pos >= T) return;
    const uint2 p = pairs[(int64_t)tok_id[pos] - first];
    tok_slot[pos] = p.x;
    z_word[pos] = (uint16_t)p.y;
}

// Boundary order changes.  tok_id[pos] = document-major index of word-major position pos.
// By sampling tiles, in their order, every XCD a run of them: the tiles in flight then hold the same documents,
// and a line of z_doc gathers its tokens in the XCD's L2.  One workgroup per tile; for large corpora
// (kReorderByTiles has both sides).
template <bool kToDocuments>
__global__ __launch_bounds__(256) void reorder_by_tiles_kernel(const Tile* tiles, int32_t n_tiles, uint16_t* z_word,
                                                               const int32_t* tok_id, uint16_t* z_doc, int64_t first) {
    const int per_xcd = (int)gridDim.x / 8;
    const int ti = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (ti >= n_tiles) return;
    const Tile tl = tiles[ti];
    for (int i = (int)threadIdx.x; i < tl.count; i += 4 * 256) {
        int64_t id[4];
        uint16_t z[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = min(i + e * 256, tl.count - 1);
            id[e] = (int64_t)tok_id[(int64_t)tl.begin + j] - first;
            if (kToDocuments) z[e] = z_word[(int64_t)tl.begin + j];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) if (!kToDocuments) z[e] = z_doc[id[e]];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (i + e * 256 >= tl.count) break;
            if (kToDocuments) z_doc[id[e]] = z[e];
            else z_word[(int64_t)tl.begin + i + e * 256] = z[e];
        }
    }
}

__global__ void to_doc_major_scatter_kernel(const uint16_t* z_word, const int32_t* tok_id,
                                            uint16_t* z_doc, int64_t T, int64_t first) {
    const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (pos < T) z_doc[(int64_t)tok_id[pos] - first] = z_word[pos];
}

// (tok_id counts from the start of the whole corpus, z_doc from token `first`: a chunk of
// documents holds the tokens first .. first + T - 1.)
__global__ void to_word_major_kernel(const uint16_t* z_doc, const int32_t* tok_id,
                                     uint16_t* z_word, int64_t T, int64_t first) {
    const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (pos < T) z_word[pos] = z_doc[(int64_t)tok_id[pos] - first];
}

// `bytes` of device memory to pinned host memory, both at multiples of 16 bytes; when all have arrived, `flag` (pinned, too)
// becomes `value`.  `done` counts workgroups, zero before and after.  Bound by the link.  A copy of HIP's with an event
// behind it leaves the link idle for 11 us after every 37 us of copying 2 MB: 32 of them 41 GB/s, of this one 53.
__global__ __launch_bounds__(256) void copy_to_host_kernel(const unsigned char* src, unsigned char* dst, int64_t bytes,
                                                           uint32_t* done, uint32_t* flag, uint32_t value) {
    const int64_t n = bytes / 16, stride = (int64_t)gridDim.x * 256;
    const uint4* from = reinterpret_cast<const uint4*>(src);
    uint4* to = reinterpret_cast<uint4*>(dst);
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (; i + 3 * stride < n; i += 4 * stride) {
        const uint4 a = from[i], b = from[i + stride], c = from[i + 2 * stride], e = from[i + 3 * stride];
        to[i] = a; to[i + stride] = b; to[i + 2 * stride] = c; to[i + 3 * stride] = e;
    }
    for (; i < n; i += stride) to[i] = from[i];
    if (blockIdx.x == 0 && (int)threadIdx.x < (int)(bytes & 15)) dst[16 * n + threadIdx.x] = src[16 * n + threadIdx.x];
    // (a barrier does not wait for the stores of the waves that meet at it: every wave waits for its own, and what all of
    // them have stored is then made visible to the host by one fence.  A fence by every thread: 0.5 GB in 11.2 ms, this 10.4)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence_system();
        if (__hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) {
            __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(flag, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// The rows of theta for the caller: the distinct topics of document d (kTopics), or 16 bits of their
// counts from bit `shift` on, at out[doc_ptr[d] ..].  A document has no more topics than tokens, so the
// rows of all documents fit a buffer of one 16-bit value per token, each at its tokens' place.
// One wave per document, persistent; bound by the slots' bytes.  (A state of 2e7 tokens at K = 1,000
// installed and taken out: 131 ms when the host unpacked the slots entry by entry and all transfers
// went through pageable memory, 12 ms with this and pinned pieces.)
template <class Layout, bool kTopics>
__global__ __launch_bounds__(kWave) void export_rows_kernel(const uint2* row_rec, const int32_t* doc_ptr, int64_t D,
                                                            const unsigned char* slots, int shift, uint16_t* out) {
    typedef typename Layout::Entry Entry;
    const int lane = (int)threadIdx.x;
    for (int64_t d = blockIdx.x; d < D; d += gridDim.x) {
        const uint2 rec = row_rec[d];
        if (rec.y == 0) continue;                       // (the same for the whole wave)
        const unsigned char* head = slots + (size_t)rec.x * 16u;
        const int n = (int)*reinterpret_cast<const uint32_t*>(head);
        const Entry* ent = reinterpret_cast<const Entry*>(head + kRowHeader);
        uint16_t* row = out + doc_ptr[d];
        int before = 0;                                 // distinct topics of the entries so far
        for (int base = 0; base < n; base += kWave) {
            const int e = base + lane;
            int topic = -1;
            bool first = false;
            if (e < n) {
                topic = Layout::entry_topic(ent[e]);
                // (in front of the first entry lies a padding entry, of no topic of the row)
                first = topic != Layout::entry_topic(ent[e - 1]);
            }
            const uint64_t firsts = __ballot(first);
            if (first) {
                const int at = before + __popcll(firsts & (((uint64_t)1 << lane) - 1));
                uint32_t value = (uint32_t)topic;
                if (!kTopics) {
                    value = 0;
                    for (int j = e; j < n && Layout::entry_topic(ent[j]) == topic; ++j)
                        value += (uint32_t)Layout::entry_count(ent[j]);
                    value >>= shift;
                }
                row[at] = (uint16_t)value;
            }
            before += __popcll(firsts);
        }
    }
}

// ------------------------------------------------------------------ log-likelihood kernels

// The topic totals' term, lgG(V beta) - lgG(n_k + V beta), over all threads of the launch.  (One workgroup took 0.2 ms for it
// at K = 60,000.)
__device__ __forceinline__ void add_totals_terms(const int32_t* n_k, int32_t K, double v_beta, double lg_vb, double& acc) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < K; k += (int64_t)gridDim.x * blockDim.x) {
        const double x = (double)n_k[k] + v_beta;
        acc += lg_vb - (x >= 1024.0 ? lgamma_large(x) : lgamma(x));
    }
}

// Word side: sum over all cells of lgG(n_wk + beta) - lgG(beta), plus the topic totals' term.
// The 16-bit cells are read eight at a time, the 32-bit cells of the wide rows four at a time
// (empty cells add nothing, so the unused 16-bit rows of the wide words do not matter); the
// table of small counts comes ready-made from global memory (lg_table: kLgTable entries, then
// lgG(beta) and lgG(V beta)), larger counts use Stirling's series.
__global__ __launch_bounds__(256) void loglik_word_side_kernel(PhiView phi, int64_t n_narrow_cells,
                                                               int64_t n_wide_cells,
                                                               const int32_t* n_k, int32_t K,
                                                               double beta, double v_beta,
                                                               const double* lg_table, double* partial,
                                                               const double* theta_partial, int n_theta,
                                                               const double* theta_sum, const double* doc_term,
                                                               unsigned int* ticket, double* out,
                                                               unsigned long long* started) {
    // (ticket: null if loglik_value_kernel follows)
    stamp_start(started);
    __shared__ double table[kLgTable];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n_octs = n_narrow_cells / 8;
    const uint4* octs = reinterpret_cast<const uint4*>(phi.narrow);
    // (on its way while the table is staged: a small launch has no other)
    uint4 first_oct = make_uint4(0u, 0u, 0u, 0u);
    if (first < n_octs) first_oct = octs[first];
    for (int c = (int)threadIdx.x; c < kLgTable; c += 256) table[c] = lg_table[c];
    const double lg_beta = lg_table[kLgTable];
    __syncthreads();
    double acc = 0.0;
    auto add_cell = [&](int c) {
        if (c > 0 && c < kLgTable) acc += table[c];
        if (__ballot(c >= kLgTable) != 0) {          // rare: taken by the whole wave or not at all
            if (c >= kLgTable) acc += lgamma_large((double)c + beta) - lg_beta;
        }
    };
    auto add_pair = [&](uint32_t two) { add_cell((int)(two & 0xffffu)); add_cell((int)(two >> 16)); };
    auto add_oct = [&](const uint4& v) {
        if (__ballot((v.x | v.y | v.z | v.w) != 0) == 0) return;
        add_pair(v.x); add_pair(v.y); add_pair(v.z); add_pair(v.w);
    };
    {
        add_oct(first_oct);
        int64_t i = first + stride;
        for (; i + 3 * stride < n_octs; i += 4 * stride) {     // four loads in flight per thread
            const uint4 v0 = octs[i], v1 = octs[i + stride], v2 = octs[i + 2 * stride],
                        v3 = octs[i + 3 * stride];
            if (__ballot((v0.x | v0.y | v0.z | v0.w | v1.x | v1.y | v1.z | v1.w | v2.x | v2.y | v2.z | v2.w |
                          v3.x | v3.y | v3.z | v3.w) != 0) == 0)
                continue;
            add_pair(v0.x); add_pair(v0.y); add_pair(v0.z); add_pair(v0.w);
            add_pair(v1.x); add_pair(v1.y); add_pair(v1.z); add_pair(v1.w);
            add_pair(v2.x); add_pair(v2.y); add_pair(v2.z); add_pair(v2.w);
            add_pair(v3.x); add_pair(v3.y); add_pair(v3.z); add_pair(v3.w);
        }
        for (; i < n_octs; i += stride) add_oct(octs[i]);
    }
    {
        const int64_t n_quads = n_wide_cells / 4;
        const int4* quads = reinterpret_cast<const int4*>(phi.wide);
        for (int64_t i = first; i < n_quads; i += stride) {
            const int4 v = quads[i];
            if (__ballot((v.x | v.y | v.z | v.w) != 0) == 0) continue;
            add_cell(v.x); add_cell(v.y); add_cell(v.z); add_cell(v.w);
        }
    }
    if (blockIdx.x == 0) {
        // up to seven 16-bit cells and up to three 32-bit cells are left
        const int64_t i = n_narrow_cells / 8 * 8 + (int64_t)threadIdx.x;
        add_cell(i < n_narrow_cells ? (int)phi.narrow[i] : 0);
        const int64_t j = n_wide_cells / 4 * 4 + (int64_t)threadIdx.x;
        add_cell(j < n_wide_cells ? phi.wide[j] : 0);
    }
    add_totals_terms(n_k, K, v_beta, lg_table[kLgTable + 1], acc);
    if (!ticket) {
        block_partial_store(acc, partial);
        return;
    }
    // A small launch needs no other: the workgroup that finishes last adds up, from partials written and read past
    // the caches.  With fences, which write the caches back, 1.6e5 cells took 9.7 us, now 8.8.  Tickets take their turns at
    // one address: 489 workgroups 13.1 us, with loglik_value_kernel 12.3; 977 19.5 and 12.2.
    block_partial_store<true>(acc, partial);
    __shared__ bool last;
    if (threadIdx.x == 0) last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    if (threadIdx.x == 0) *ticket = 0u;               // for the next launch
    store_loglik<true>(partial, (int)gridDim.x, theta_partial, n_theta, theta_sum, doc_term, out);
}

// The same by words, where most of them have few tokens over many topics: rows of the n_dense segments in front (a word's first
// or only one), and of the words behind them the cells that their tokens' topics z name, each of them for as many of its
// tokens as it counts.  A value per workgroup; bound by the rows' bytes.  All cells / this, us: 4e6 tokens, 60,000 words, K = 9,000
// 282/69, 5e5, 20,000 words, K = 20,000 183/47, 2e6, 6,000 words, K = 40,000 197/79, 9.9e7, 102,000 words, K = 10,000 564/491.
__global__ __launch_bounds__(256) void loglik_word_rows_kernel(const Tile* segs, int32_t n_dense, int32_t n_segs, const uint16_t* z,
                                                               PhiView phi, const int32_t* n_k, int32_t K, double beta,
                                                               double v_beta, const double* lg_table, double* partial,
                                                               unsigned long long* started) {
    stamp_start(started);
    __shared__ double table[kLgTable];
    for (int c = (int)threadIdx.x; c < kLgTable; c += 256) table[c] = lg_table[c];
    const double lg_beta = lg_table[kLgTable];
    __syncthreads();
    double acc = 0.0;
    auto term = [&](int c) { return c < kLgTable ? table[c] : lgamma_large((double)c + beta) - lg_beta; };
    auto add_cell = [&](int c) {
        if (c > 0 && c < kLgTable) acc += table[c];
        if (__ballot(c >= kLgTable) != 0) {
            if (c >= kLgTable) acc += term(c);
        }
    };
    auto add_pair = [&](uint32_t two) { add_cell((int)(two & 0xffffu)); add_cell((int)(two >> 16)); };
    const int tid = (int)threadIdx.x;
    for (int s = (int)blockIdx.x; s < n_dense; s += (int)gridDim.x) {
        const Tile tl = segs[s];
        if (tl.whole == 0) continue;
        const int wide_row = phi.wide_row[tl.word];
        if (wide_row >= 0) {
            const int32_t* row = phi.wide + (size_t)wide_row * (size_t)K;
            for (int i = tid; i - tid < K; i += 256) add_cell(i < K ? row[i] : 0);
            continue;
        }
        const uint16_t* row = phi.narrow + (size_t)tl.word * (size_t)K;
        const int head = min((int)((16 - ((uintptr_t)row & 15)) & 15) / 2, K), n8 = (K - head) / 8, rest = K - head - 8 * n8;
        const uint4* octs = reinterpret_cast<const uint4*>(row + head);
        for (int i = tid; i - tid < n8; i += 512) {
            uint4 a = make_uint4(0u, 0u, 0u, 0u), b = a;
            if (i < n8) a = octs[i];
            if (i + 256 < n8) b = octs[i + 256];
            if (__ballot((a.x | a.y | a.z | a.w | b.x | b.y | b.z | b.w) != 0) == 0) continue;
            add_pair(a.x); add_pair(a.y); add_pair(a.z); add_pair(a.w);
            add_pair(b.x); add_pair(b.y); add_pair(b.z); add_pair(b.w);
        }
        int c = 0;                      // (at most seven cells on either side)
        if (tid < head) c = (int)row[tid];
        else if (tid >= 8 && tid < 8 + rest) c = (int)row[head + 8 * n8 + tid - 8];
        if (tid < kWave) add_cell(c);
    }
    const int waves = (int)gridDim.x * 4, lane = tid & (kWave - 1);
    for (int s = n_dense + (int)blockIdx.x * 4 + tid / kWave; s < n_segs; s += waves) {
        const Tile tl = segs[s];
        const uint16_t* row = phi.narrow + (size_t)tl.word * (size_t)K;
        for (int t = lane; t < tl.count; t += kWave) {
            const int c = (int)row[z[tl.begin + t]];
            if (c > 0) acc += term(c) / (double)c;
        }
    }
    add_totals_terms(n_k, K, v_beta, lg_table[kLgTable + 1], acc);
    block_partial_store(acc, partial);
}

// The value after a large loglik_word_side_kernel.  One workgroup.
__global__ __launch_bounds__(256) void loglik_value_kernel(const double* partial, int n, const double* theta_partial,
                                                           int n_theta, const double* theta_sum,
                                                           const double* doc_term, double* out) {
    store_loglik<false>(partial, n, theta_partial, n_theta, theta_sum, doc_term, out);
}

// The per-document term lgG(K alpha) - lgG(N_d + K alpha), one thread per document (the
// entries of the theta rows are summed by the theta rebuild).  A constant of the corpus.
__global__ __launch_bounds__(256) void loglik_doc_term_kernel(const int32_t* doc_ptr, int64_t D,
                                                              double k_alpha, double* partial) {
    const double lg_ka = lgamma(k_alpha);
    double acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; d < D; d += stride)
        acc += lg_ka - lgamma((double)(doc_ptr[d + 1] - doc_ptr[d]) + k_alpha);
    block_partial_store(acc, partial);
}

// out = (add_to_out ? *out : 0) + sum of the n partials.  One workgroup, fixed order.
__global__ __launch_bounds__(256) void loglik_final_kernel(const double* partial, int n, int add_to_out, double* out) {
    double acc = partials_sum<false>(partial, n);
    if (threadIdx.x == 0 && add_to_out) acc += *out;
    acc = block_sum_256(acc);
    if (threadIdx.x == 0) *out = acc;
}

}  // namespace mlda
