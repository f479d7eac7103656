// How passes over memory use MI355X's 256 MiB memory-side cache.
//
// Nontemporal accesses leave the cache to other data; plain ones fill it.
// The rules go by the bytes that one direction of a call moves:
//
// - Streams.  A call whose input and output together exceed the cache can
//   find its input there only by accident, and filling it with data that is
//   not read again costs more than it gives: nontemporal accesses.  A
//   smaller call reads what the kernel before it has just written, and the
//   next one reads its output, at the cache's rate: plain accesses.
//   Measured with 16-column tile copies: 2 x 64 MiB, repeated on the same
//   buffers, 17 us plain against 23 nontemporal; 2 x 512 MiB 205 against 189.
// - One pass.  Batched 1D transforms of a single pass read and store
//   nontemporally at every size.  Plain stores leave an output of up to 256 MiB in the cache,
//   which helps a program that writes one buffer again and again or whose
//   next kernel works on the output in place, and costs the others what
//   the output drives out: N = 64 at 128 MiB, nontemporal -> plain stores, three
//   inputs and one output in turn 0.96 of the time, in-place scaling after it
//   0.94, three outputs 1.07, an input produced just before 1.03; at 250 MiB
//   0.92, 0.86, 1.07 and 1.10.
// - Chunks.  A transform of several passes over memory runs all its passes
//   on one chunk of the batch before the next, so that a later pass reads
//   what the earlier one left in the cache: the first pass reads its input
//   nontemporally and stores plainly.  256 MiB per chunk measured best
//   (four-step 2^16 at 512 MiB: one chunk 386 us, 256 MiB 349, 128 MiB 382):
//   smaller chunks pay more launches, each with its own ramp and drain.
#pragma once
#include <stdint.h>

namespace mifft {

constexpr int64_t kStreamBytes = int64_t(128) << 20;
constexpr int64_t kChunkBytes = int64_t(256) << 20;

// Passes of 128 and 256 points keep 32 points per thread (wide_tile.hpp) in
// calls that fill the chip several times over, for the loads in flight; in
// smaller ones 8 or 16 points per thread make four or two times the
// wavefronts.  MI355X, 8 / 16 -> 32 points per thread, us: four-step 2^16 at
// 64 MiB 51.0 -> 43.0 (three buffer sets in turn 55.9 -> 58.1, at 56 MiB 49.0 ->
// 44.2), at 512 MiB 349 -> 346, at 16 MiB 22.6 -> 23.3, at 2 MiB 10.9 -> 12.0; 2D
// 256 x 256 at 64 MiB 49.2 -> 44.3.
constexpr int64_t kBulkBytes = int64_t(32) << 20;
inline bool is_bulk(int64_t bytes) { return bytes > kBulkBytes; }

// Whether a call that reads `bytes` and writes about as much is a stream.
inline bool is_stream(int64_t bytes) { return bytes > kStreamBytes; }

// The same for the four-step passes (both of 2^15 and 2^16, the row pass of
// 2^17).  2^15 between 64 MiB and a stream does not gain: MiB: us, three buffer
// sets in turn, 72: 60.2 -> 62.5, 96: 76.1 -> 78.2, 128: 101.1 -> 104.1; two sets
// 55.6 -> 58.0, 73.1 -> 76.5, 99.8 -> 103.1; one set 54.4 -> 48.6, 67.8 -> 65.5,
// 88.7 -> 84.4; at 64 one or two sets 49.8 -> 44.1, three 53.1 -> 58.3.
inline bool fourstep_bulk(int log2n, int64_t bytes)
{
    return is_bulk(bytes) && (log2n > 15 || bytes <= (kStreamBytes >> 1) || is_stream(bytes));
}

// Whether the fused loss stores its gradient of `bytes` plainly: small ones, which
// the XCDs' L2 caches take faster than memory does, and larger ones if the next
// kernel scales it (the differentiable loss's backward).  MI355X, us, three inputs
// in turn, nontemporal -> plain: alone N = 512 at 2 MiB 5.2 -> 4.5, N = 2048 at
// 2 MiB 7.0 -> 6.2, N = 256 at 16 MiB 8.9 -> 11.2; forward + backward N = 2048 at
// 0.5 MiB 8.0 -> 7.7, 8: 15.2 -> 16.3, 24: 29.2 -> 29.8, 40: 39.9 -> 39.1, 150: 127.5
// -> 116.8, 250: 206 -> 184, 300: 244 -> 244; N = 128 at 0.5 MiB 6.1 -> 5.8, 16:
// 18.4 -> 19.1, 40: 35.8 -> 33.7, 200: 148.5 -> 142.8, 250: 186 -> 193.
inline bool keep_gradient(int log2n, int64_t bytes, bool scaled_next)
{
    return bytes <= (kStreamBytes >> 6) || (scaled_next && bytes > (kStreamBytes >> 2) &&
                                            bytes <= (log2n >= 9 ? kChunkBytes : kChunkBytes / 8 * 7));
}

// Whether the first pass of a multidimensional transform, along 2^log2n points,
// stores its `bytes` plainly for the next one.  Between 8 and 20 MiB it does not:
// such an output lies in the XCDs' L2 caches (32 MiB together) and is written
// back when the kernel ends, while nothing runs; smaller ones cost little, larger
// ones leave on the way.  The window is a little wider at 128 and at 4096 points.
// MI355X, us, nontemporal -> plain, one buffer set: 16 x 2048 at 1 MiB 6.8 -> 6.5,
// 512 x 512 at 8 MiB 13.3 -> 12.9, 512 x 128 at 16 MiB 17.7 -> 20.2, 128 x 512 at
// 24 MiB 25.9 -> 22.4, at 48 39.3 -> 34.0; 256 x 128 at 8 MiB 13.6 -> 14.1, 128 x
// 4096 at 24 MiB 23.1 -> 24.9.
inline bool feed_next(int log2n, int64_t bytes)
{
    constexpr int64_t MIB = int64_t(1) << 20;
    return bytes <= (log2n == 7 ? 6 : 8) * MIB || bytes > (log2n == 12 ? 28 : 20) * MIB;
}

// Units of `each` bytes in one chunk.
inline int64_t chunk_units(int64_t each) { return each >= kChunkBytes ? 1 : kChunkBytes / each; }

// Units in the next chunk of a multidimensional transform with `left` to go,
// `per` to a chunk: a last chunk of at most kTailBytes joins the one before it,
// whose launches it shares, though the two then take a little more than the
// cache (MI355X, us, whole batch plain -> short last chunk -> joined: 32^3 at
// 136 MiB 109 -> 115 -> 107, at 150 MiB 119 -> 127 -> 115, 64^3 at 150 MiB
// 115 -> 120 -> 111, 512 x 1024 at 280 MiB 238 -> 188 -> 184; but 44 MiB, 512 x 1024
// at 300 MiB 254 -> 197 -> 205).  Chunks of equal size were slower than
// either (32^3 at 136 MiB 121).
constexpr int64_t kTailBytes = int64_t(32) << 20;
inline int64_t next_chunk(int64_t left, int64_t per, int64_t each)
{
    return left > per && (left - per) * each > kTailBytes ? per : left;
}

}  // namespace mifft
