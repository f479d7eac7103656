// Host build of the rules on the sizes of calls
// (paper_2203_09384_amd/csrc/stream.hpp) for the CPU tests.
#include "stream.hpp"

using namespace mifft;

extern "C" {

int64_t st_chunk_bytes() { return kChunkBytes; }
int64_t st_tail_bytes() { return kTailBytes; }
int64_t st_chunk_units(int64_t each) { return chunk_units(each); }
int64_t st_next_chunk(int64_t left, int64_t per, int64_t each) { return next_chunk(left, per, each); }
}

extern "C" {

int64_t st_bulk_bytes() { return kBulkBytes; }
int64_t st_stream_bytes() { return kStreamBytes; }
int st_fourstep_bulk(int log2n, int64_t bytes) { return fourstep_bulk(log2n, bytes); }
}

extern "C" int st_keep_gradient(int log2n, int64_t bytes, int scaled_next)
{
    return keep_gradient(log2n, bytes, scaled_next != 0);
}

extern "C" int st_feed_next(int log2n, int64_t bytes) { return feed_next(log2n, bytes); }
