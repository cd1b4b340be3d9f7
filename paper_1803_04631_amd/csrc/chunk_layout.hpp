// Where the documents of a corpus are cut into chunks, and where the buffers of a chunk lie in the workspace.  (Host code only,
// and the records that both sides share.)
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <algorithm>

namespace mlda {

struct Tile {          // consecutive word-major tokens of one word
    int32_t word;
    int32_t begin;     // first word-major token position
    int32_t count;     // 1 .. tile size
    int32_t whole;     // phi segments: 1 if the segment holds every token of its word, -1 if it is the first of several;
                       // sampling tiles: the word's row in PhiView::wide, or -1
};

// One document as the theta rebuild needs it, stored in processing order.
struct alignas(16) DocRec {
    int32_t begin;      // first document-major token
    int32_t n;          // tokens
    uint32_t slot;      // offset of the theta row's slot, 16-byte units
    int32_t doc;        // document id
};

constexpr size_t kAlign = 256;        // workspace sub-buffer alignment

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Chunk m of M covers the documents [chunk_first(m), chunk_first(m + 1)): about T / M tokens each.
inline int64_t chunk_first(const int64_t* doc_ptr, int64_t D, int32_t M, int32_t m) {
    if (m <= 0) return 0;
    if (m >= M) return D;
    const int64_t want = doc_ptr[D] / M * m;
    return std::lower_bound(doc_ptr, doc_ptr + D + 1, want) - doc_ptr;
}

// Where the buffers of one chunk of documents lie inside its part of the workspace (byte
// offsets).  The static part (up to static_bytes) is the preprocessed corpus and is copied
// from the host as one block; two index arrays derived from it on the device, z and the theta
// rows follow.
struct ChunkLayout {
    size_t tok_slot = 0, tok_id = 0, doc_map = 0, doc_ptr = 0, doc_order = 0, row_rec = 0, tiles = 0,
           segs = 0, split = 0, static_bytes = 0, doc_pairs = 0, z0 = 0, z1 = 0, slots = 0, total = 0;
};

// `streamed`: the chunk takes turns on the device with others.  It then needs no
// document->token map: its assignments arrive in document order (see StreamedSlot) and
// are paired with their documents' slots there (doc_pairs) on their way to word-major order.
inline ChunkLayout chunk_layout(int64_t D, int64_t T, size_t slots_bytes, size_t n_tiles, size_t n_segs,
                                size_t n_split, bool streamed) {
    ChunkLayout L;
    size_t at = 0;
    auto put = [&](size_t bytes) { const size_t o = at; at += align_up(bytes, kAlign); return o; };
    L.tok_id = put((size_t)T * 4);
    L.doc_ptr = put((size_t)(D + 1) * 4);
    L.doc_order = put((size_t)D * sizeof(DocRec));
    L.row_rec = put((size_t)D * 8);
    L.tiles = put(n_tiles * sizeof(Tile));
    L.segs = put(n_segs * sizeof(Tile));
    L.split = put(n_split * 4);
    L.static_bytes = at;
    L.tok_slot = put((size_t)T * 4);       // derived on the device from the static part
    L.doc_map = put(streamed ? 0 : (size_t)T * 4);
    L.doc_pairs = put(streamed ? (size_t)T * 8 : 0);
    L.z0 = put((size_t)T * 2);
    L.z1 = put((size_t)T * 2);
    L.slots = put(slots_bytes);
    L.total = at;
    return L;
}

// One of the two parts of the workspace that streamed chunks are attached to in turn (byte offsets): the
// assignments in document order, and behind them the attached chunk's own layout.  The assignments are the one thing
// that outlives a visit: they may be on their way to the host while the static part of the chunk that comes next is on
// its way in.  Their place is therefore common to all chunks, with room for the largest; inside the chunks' layouts,
// which differ, a chunk of more documents, tiles or tokens would be written over the assignments of the one before.
struct StreamedSlot {
    size_t z_doc = 0, chunk = 0, total = 0;
};
// (most_tokens, most_bytes: the largest T and ChunkLayout::total of the chunks)
inline StreamedSlot streamed_slot(int64_t most_tokens, size_t most_bytes) {
    StreamedSlot s;
    s.chunk = align_up((size_t)most_tokens * 2, kAlign);
    s.total = s.chunk + most_bytes;
    return s;
}

}  // namespace mlda
