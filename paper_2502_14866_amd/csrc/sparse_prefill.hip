// Block-sparse causal prefill attention (Sec. 3.1, Sec. 3.4) on the gfx950 matrix cores.
//
// Mask tiles are 64 x 64 (query tile x key tile = page).  Dense heads visit every key tile up to
// the diagonal; streaming heads visit only the sink tiles and the local band, so whole tiles
// outside the mask are never loaded.  Only the diagonal tile needs element-wise causal masking.
//
// Mapping to CDNA4: a workgroup of eight wavefronts works on four units, a unit being one mask tile of queries of one
// head; wavefronts 2u and 2u + 1 own the two 32-row halves of unit u.  Units are query heads of a group before they
// are neighbouring query tiles: heads of a group need exactly the same key tiles.  Two wavefronts
// share each SIMD, so the matrix pipe of one overlaps the softmax arithmetic of the other.  K and
// V tiles are brought into LDS once per workgroup by direct-to-LDS loads, double buffered, and
// consumed by all eight wavefronts.  A launch with few query rows has the pairs of wavefronts share out the key tiles
// of fewer units instead (key slices, see sparse_prefill_kernel).  Scores are computed transposed,
//   S^T (keys x queries) = K (keys x d) * Q^T (d x queries)          v_mfma_f32_32x32x16
// so that a lane owns one query column: the softmax reductions over keys stay inside the lane
// (plus one exchange between the two lane halves), and the exponentiated tile is already in the
// register layout of the B operand of the second product
//   O^T (d x queries) += V^T (d x keys) * P^T (keys x queries).
// V stays as it is in memory, one row per key: the V^T operand is read from the row-major tile with the
// transposing LDS read of gfx950 (ds_read_b64_tr_b16), which hands a lane four keys of one channel, so
// there is no transposition pass and no transposed copy of V.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "kernels.h"

namespace lserve {

namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf168_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int kTileLog2 = 6;
constexpr int kTile = 1 << kTileLog2;              // mask tile = key tile = page
constexpr int kPrefillWaves = 8;                   // two per SIMD, each owning 32 query rows
constexpr int kPrefillThreads = kPrefillWaves * kWave;
constexpr int kPairs = kPrefillWaves / 2;          // wavefront pairs; a pair owns the two halves of a mask tile's rows
constexpr int kAhead = 4;                          // operand reads in flight ahead of the score products
constexpr int kKRowBytes = 256;                    // K tile row: 128 x 16 bit = 16 chunks of 16 B
constexpr int kVRowBytes = 256;                    // V tile row (one key): the same
constexpr int kKTileBytes = kTile * kKRowBytes;
constexpr int kVTileBytes = kTile * kVRowBytes;

// Tiles reach LDS through direct-to-LDS loads, which place the 64 lanes of an instruction at 64
// consecutive 16-byte slots, so rows cannot be padded.  Bank conflicts are avoided by permuting the
// chunks inside a row instead.  Chunk c of K row r sits at position c ^ (r % 16): sixteen consecutive rows
// then hit sixteen different 16-byte bank groups for any fixed c, which is what the K operand reads (one
// row per lane) need.  Chunk c of V row r sits at position c ^ 4 (r % 4): a transposing read takes, from
// each of four consecutive rows, the same 64 bytes (32 channels), and the four stretches then fall into
// the four 64-byte quarters of the 256 bytes the banks serve per cycle.
__device__ __forceinline__ int k_chunk_pos(int row, int c) { return c ^ (row % 16); }
__device__ __forceinline__ int v_chunk_pos(int row, int c) { return c ^ (4 * (row % 4)); }

// The load itself is written in assembly: left to the compiler it is treated as an access that may
// touch both memory and LDS, and while one is in flight every LDS operand read in the loop waits with
// lgkmcnt(0), exposing the LDS latency in front of the products.  The source address is a wave-uniform
// 64-bit base (scalar registers) plus a 32-bit lane offset; `lds_base` is the wave-uniform LDS byte
// address of the 1 KiB destination and lane l lands at lds_base + 16 l.  Completion is tracked by
// vmcnt only, which dma_wait() drains before the workgroup barrier.
__device__ __forceinline__ void dma_load16(unsigned long long src_base, unsigned lane_offset, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_offset), "s"(src_base), "s"(lds_base) : "memory");
}
// Tells the compiler that a value every lane agrees on can live in scalar registers.
__device__ __forceinline__ unsigned long long uniform64(unsigned long long x) {
    return ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((unsigned)(x >> 32)) << 32) |
           (unsigned)__builtin_amdgcn_readfirstlane((unsigned)x);
}
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ unsigned lds_address(const void* p) {
    return (unsigned)(size_t)(const __attribute__((address_space(3))) void*)p;
}

constexpr float kLn2 = 0.6931471805599453f;

template <class T> struct Mfma;
template <> struct Mfma<F16> {
    static __device__ __forceinline__ float16_t run(uint4 a, uint4 b, float16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ float4_t run16(uint4 a, uint4 b, float4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
    }
};
template <> struct Mfma<BF16> {
    static __device__ __forceinline__ float16_t run(uint4 a, uint4 b, float16_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf168_t, a), __builtin_bit_cast(bf168_t, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ float4_t run16(uint4 a, uint4 b, float4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf168_t, a), __builtin_bit_cast(bf168_t, b), c, 0, 0, 0);
    }
};

// Chunked prefill over a paged cache (Sec. 2.1, Sec. 3.2).  The cache holds seq_lens[b] tokens of sequence b, in
// any of the forms of PagedParams with 16-bit rows (one pool; dense heads in the main pool and streaming heads in
// their ring of sink + local pages).  With k_new / v_new the queries are n_b new tokens whose K / V arrive
// alongside and have not been written back yet: the cache is their history.  Without, the cache already holds
// the chunk and the queries are its last n_b tokens.
struct PrefillPaged {
    PagedParams kv;
    const uint16_t *k_new, *v_new;  // [total_new][Hkv][D] or null
};

template <class T>
__device__ __forceinline__ uint4 pack8(const float* p) {
    return make_uint4(Elem<T>::pack(p[0], p[1]), Elem<T>::pack(p[2], p[3]), Elem<T>::pack(p[4], p[5]),
                      Elem<T>::pack(p[6], p[7]));
}

// Combine a value with the one held by the same lane of the other 32-lane half of the wave.
// (one swap of the upper half of a register with the lower half of its copy, in the vector ALU)
template <class Op> __device__ __forceinline__ float halves_combine(float x, Op op) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    const swap_pair_t p = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned p0 = p[0], p1 = p[1];
    return op(__builtin_bit_cast(float, p0), __builtin_bit_cast(float, p1));
}
__device__ __forceinline__ float halves_max(float x) {
    return halves_combine(x, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float halves_sum(float x) {
    return halves_combine(x, [](float a, float b) { return a + b; });
}

typedef short short4_t __attribute__((ext_vector_type(4)));
// Transposing LDS read (ds_read_b64_tr_b16).  The sixteen lanes of a row each name four consecutive 16-bit
// elements; lane i receives element i % 4 of the lanes i / 4, i / 4 + 4, i / 4 + 8 and i / 4 + 12.  With lane s
// pointing at channels 4 (s % 4) .. + 3 of key s / 4, lane i ends up with channel i of four consecutive keys.
__device__ __forceinline__ uint2 lds_read_transposed(const unsigned char* p) {
    const short4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) short4_t*)(const __attribute__((address_space(3))) void*)p);
    return __builtin_bit_cast(uint2, v);
}

// Work order of the launch.  Workgroup ids go round-robin over the eight XCDs, each with its own L2, and inside an
// XCD round-robin over its four shader engines.  Dense heads come first, streaming heads after.  When the number of
// heads of a class divides 8, an XCD serves a single KV head of that class at a time, so the
// workgroups resident on it (the query heads of one group, neighbouring query blocks) walk the
// same K / V tiles together and share them in that L2.
constexpr int kXcds = 8;
struct HeadClass {
    int heads;            // KV heads of this class
    int slices;           // XCDs per head (1 when not swizzled)
    int swizzled;         // 8 % heads == 0
    int items_per_xcd;    // workgroups of this class per XCD
    int heads_per_block;  // query heads of a group that share a workgroup (1, 2 or 4)
    int qtiles_log2;      // log2 of the query tiles a workgroup owns
    int fold;             // the key slices of the kernel share a unit (and are folded), or each group of waves has its own
    int blocks_per_seq;   // query blocks of the longest sequence
    int blocks;           // query blocks of the batch, at most
    int ordered;          // blocks are dealt out longest walk first over the whole batch (see block_of)
    unsigned kv_head[16];  // four to a word: a byte of its own is a vector load, one more trip to memory in a start
};
// Dense walks cut into pieces (see PiecePlan); partials is null where blocks are whole.
struct PrefillPieces {
    float* partials;  // kPieceFloats for every piece, pieces of a (KV head, group of query heads) next to each other
    int target;       // pieces of a (KV head, group of query heads) in the launch, at most
    int least;        // of a block
    int short_blocks; // a batch whose sequences have no more blocks than this is left to whole walks (see fold_and_streams_kernel)
};
struct PrefillSchedule {
    HeadClass cls[2];  // dense, streaming
    PrefillPieces pieces;
    int compute_units;  // of the device
};

// Decodes workgroup `li` of XCD `xcd` inside a class of workgroups, `n` of them per (KV head, query block): KV head hk (the
// hidx-th of its class), group of query heads hg, and the position of the query block in the order of blocks.
__device__ __forceinline__ void decode_work(const HeadClass& hc, int n, int xcd, int li, int& hidx, int& hk, int& hg, int& rank) {
    if (hc.swizzled) {
        hidx = xcd % hc.heads;
        hg = li % n;
        rank = (li / n) * hc.slices + xcd / hc.heads;
    } else {
        const int t = li * kXcds + xcd;
        hg = t % n;
        hidx = (t / n) % hc.heads;
        rank = t / (n * hc.heads);
    }
    hk = (int)(hc.kv_head[hidx / 4] >> (8 * (hidx % 4))) & 0xff;
}

// Sum over the wave of a value below 2^24 per lane and in total (exact in fp32).
__device__ __forceinline__ int wave_count(int x) { return __builtin_amdgcn_readfirstlane((int)rows4_sum(row16_sum((float)x))); }

// Batches of up to kOrderedSeqs sequences are dealt out in one order, which a lane's registers hold: four sequences to a lane.
// (Beyond, the blocks of each index follow one another sequence by sequence, gaps and all; up to 64, one to a lane, was too
// few: 128 prompts of 20 .. 2500 tokens, 8 / 2 heads, took 432 us that way.)
constexpr int kSeqGroups = 4, kOrderedSeqs = kSeqGroups * kWave;
struct BlockSpans {
    int lo[kSeqGroups], hi[kSeqGroups];  // blocks [lo, hi) of sequence 64 g + lane
};

// The query blocks of a batch, ordered by their position inside their sequence, farthest first (the
// longest walks start first and the short ones fill in behind them).
// Nothing is left out in this order, and that matters
// beyond the launches it saves: workgroups go to the shader engines of an XCD in strict turn, so an order with gaps
// of a fixed stride (one long sequence among fifteen short ones, each block index of all sixteen in a row) puts the
// real work of a launch on one of the four (sixteen prompts of 77 .. 3001 tokens: 745 us, in this order 214).
struct BlockOrder {
    BlockSpans s;
    int batch, lo0, hi0;  // blocks of the first sequence
    bool alike;           // and of every other

    // calls f(g, blocks of this lane's sequence) for every group in use
    template <class F> __device__ __forceinline__ void each(F f) const {
#pragma unroll
        for (int g = 0; g < kSeqGroups; ++g)
            if (g == 0 || g * kWave < batch) f(g, max(0, s.hi[g] - s.lo[g]));
    }
    // blocks of the batch at position `level` of their sequence or past it
    __device__ __forceinline__ int at_or_past(int level) const {
        if (alike) return batch * max(0, hi0 - max(lo0, level));
        int count = 0;
        each([&](int g, int n) { count += min(max(s.hi[g] - level, 0), n); });
        return wave_count(count);
    }
    // past the last block of any sequence
    __device__ __forceinline__ int top() const {
        if (alike) return hi0;
        int t = 0;
        each([&](int g, int n) { t = max(t, n > 0 ? s.hi[g] : 0); });
        return __builtin_amdgcn_readfirstlane((int)wave_max((float)t));
    }
    // find() for batches of up to sixteen sequences that differ, which a row of lanes holds: each of the four rows counts at a
    // level of its own, so that a round, of half the instructions, leaves a fifth of the levels instead of half of them.  The search is a
    // third of a half workgroup's start (2.4 us of 7 where lengths differ, 1.0 where not): 16 prompts of 77 .. 3001 tokens 173 -> 169 us,
    // six of 100 .. 3000, 64 / 8 heads, 182 -> 177, nine of 108 .. 2283 112 -> 108.
    __device__ __forceinline__ bool find_few(int rank, int& b, int& qblk) const {
        auto everywhere = [](int x) {  // row 0 in all four rows
            const swap_pair_t p = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
            const unsigned u = p[0];
            const swap_pair_t q = __builtin_amdgcn_permlane32_swap(u, u, false, false);
            return (int)q[0];
        };
        const int lo = everywhere(s.lo[0]), hi = everywhere(s.hi[0]), row = threadIdx.x % kWave / 16;
        float t = lo < hi ? (float)hi : 0.f;
        t = fmaxf(t, dpp_f<kDppXor1>(t));
        t = fmaxf(t, dpp_f<kDppXor2>(t));
        t = fmaxf(t, dpp_f<kDppHalfMirror>(t));
        t = fmaxf(t, dpp_f<kDppMirror>(t));
        int below = 0, above = __builtin_amdgcn_readfirstlane((int)t), past = 0;  // past: blocks at `above` or past it
        int step = (above + 3) / 4, at = row * step;
        for (bool begun = false;; begun = true) {
            const float count = row16_sum((float)max(hi - max(lo, at), 0));
            const unsigned long long more = __ballot(count > (float)rank) & 0x0001000100010001ull;
            const int k = __popcll(more);  // levels with more than `rank` blocks at or past them
            if (!begun && k == 0) return false;
            const int first = begun ? below + step : 0;  // the level of row 0
            if (first + k * step < above && k < 4) {
                above = first + k * step;
                past = (int)__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, count), 16 * k));
            }
            if (k > 0) below = first + (k - 1) * step;
            if (above - below <= 1) break;
            step = (above - below + 4) / 5;
            at = below + (row + 1) * step;
        }
        const bool member = threadIdx.x % kWave < 16 && lo <= below && below < hi;
        const unsigned long long members = __ballot(member), lower = (1ull << (threadIdx.x % kWave)) - 1ull;
        b = __builtin_ctzll(__ballot(member && __popcll(members & lower) == rank - past));
        qblk = below;
        return true;
    }
    // The rank-th block of the batch; false past the last one.
    // FEW: see find_few; the other kernels, whose workgroups are fewer and longer, do without the code.
    template <bool FEW = false> __device__ __forceinline__ bool find(int rank, int& b, int& qblk) const {
        if (alike) {
            const int level = batch == 1 ? rank : rank / batch;
            b = rank - level * batch;
            qblk = hi0 - 1 - level;
            return qblk >= lo0;
        }
        if (FEW && batch <= 16) return find_few(rank, b, qblk);
        if (rank >= at_or_past(0)) return false;
        int below = 0, above = top();
        while (above - below > 1) {  // largest level with more than `rank` blocks at or past it
            const int mid = (below + above) / 2;
            if (at_or_past(mid) > rank)
                below = mid;
            else
                above = mid;
        }
        int i = rank - at_or_past(below + 1);
        const unsigned long long lower = (1ull << (threadIdx.x % kWave)) - 1ull;
        int found = -1;
        each([&](int g, int) {
            const bool member = s.lo[g] <= below && below < s.hi[g];
            const unsigned long long members = __ballot(member), hit = __ballot(member && __popcll(members & lower) == i);
            if (found < 0 && hit) found = g * kWave + __builtin_ctzll(hit);
            i -= __popcll(members);
        });
        b = found;
        qblk = below;
        return true;
    }
};

// seq_lens: tokens in the pages, or null without pages; alongside: the batch's new tokens are not among them yet.
__device__ __forceinline__ BlockOrder block_order(const int* cu_seqlens, const int* seq_lens, bool alongside, int batch, int rows_log2) {
    BlockOrder o;
    o.batch = batch;
#pragma unroll
    for (int g = 0; g < kSeqGroups; ++g) {
        o.s.lo[g] = o.s.hi[g] = 0;
        if (g > 0 && g * kWave >= batch) continue;
        const int seq = g * kWave + threadIdx.x % kWave, i = min(seq, batch - 1);
        const int fresh = cu_seqlens[i + 1] - cu_seqlens[i];
        const int past = seq_lens ? seq_lens[i] - (alongside ? 0 : fresh) : 0;
        o.s.lo[g] = past >> rows_log2;
        o.s.hi[g] = seq < batch && fresh > 0 ? ((past + fresh - 1) >> rows_log2) + 1 : 0;
    }
    o.lo0 = __builtin_amdgcn_readfirstlane(o.s.lo[0]);
    o.hi0 = __builtin_amdgcn_readfirstlane(o.s.hi[0]);
    o.alike = true;
    if (batch > 1) {  // all sequences alike: no search
        int n_seq = 0;
        unsigned long long unlike = 0;
        o.each([&](int g, int n) {
            n_seq += __popcll(__ballot(n > 0));
            unlike |= __ballot(n > 0 && (o.s.lo[g] != o.lo0 || o.s.hi[g] != o.hi0));
        });
        o.alike = n_seq == batch && unlike == 0;
    }
    return o;
}

// Pieces of dense walks.  A launch of few blocks with long walks (a chunk over a long history: 32 workgroups of 516 steps on
// 256 compute units) leaves most of the chip idle.  A walk may therefore be cut: block qblk of a sequence, counted from the start of the sequence, is ceil((qblk + 1) / span) pieces of
// nearly equal length, worked on by a workgroup each.  A piece leaves its unnormalised outputs, maxima and sums in
// PrefillPieces::partials, and fold_pieces_kernel puts the pieces of a block together.  The span is the smallest that needs no
// more pieces than the launch has workgroups for; every workgroup works it out from the lengths, which the host does not know.
// Measured, whole walks in the best shape and pieces: 512 tokens over 32768, 32 / 8 heads, 338 and 144 us (8 pieces to a
// block: 65 steps of 1.75 us with every compute unit at work, then 14 us to put 33 MB of pieces together, next to the streaming
// heads, see streams_apart); 17 over 42116, twice, 441 and 79; 108 over 73893, 32 / 16 heads, 982 and 267.  Prompts are not cut: one of 4096
// tokens took 119 us whole and 124 or more in any number of pieces, one of 8192 313 and 340, because what they gained in balance (42
// steps a compute unit where the longest walk has 64) went into the starts of the pieces and into putting them together (with a running
// maximum and a launch of its own for the fold; not measured since, 4096 tokens take 102 us whole).
// No block is fewer pieces than the key slices it has without scratch (PrefillPieces::least), however short its walk: the weights of
// a row are rounded to 16 bits relative to the maximum of their piece or slice, and fewer of these make the error larger.
// A position in the launch stands for a piece: last pieces first (none is shorter than half a span), then the last but one,
// and so on, each kind farthest block first; whole blocks of less than a span come at the end.
constexpr int kLeastSpanTiles = 8;  // key tiles: a piece costs about three steps of its own
constexpr int kPieceFloats = kPrefillWaves * (32 * kHeadDim + 64);  // accumulators as the lanes hold them; (maximum, sum) per row

constexpr int kManyPieces = 1 << 15;  // of a sequence: no launch has as many, and wave_count adds up 256 times that exactly

// x / y for 0 <= x < 2^22, 0 < y, by the reciprocal (a whole division is four times the instructions, and the search below,
// in front of everything else a workgroup does, is a chain of them).
__device__ __forceinline__ int divide(int x, int y, float reciprocal) {
    int k = (int)((float)x * reciprocal);
    const int r = x - k * y;
    k += r >= y;
    return k - (r < 0);
}

struct PiecePlan {
    int span, least, total;  // total: 0 where not even the smallest number of pieces has room (lengths beyond the stated bounds)
    // pieces of block x, and of the x blocks at the start of a sequence
    __device__ __forceinline__ int pieces_of(int x) const { return max(least, divide(x, span, __builtin_amdgcn_rcpf((float)span)) + 1); }
    __device__ __forceinline__ int prefix(int x, float reciprocal) const {
        const int k = divide(x, span, reciprocal), r = x - k * span;
        return k < least ? least * x : span * (k * (k + 1) / 2 + least * (least - 1) / 2) + r * (k + 1);
    }
    // blocks have a piece of this number from here on
    __device__ __forceinline__ int level(int piece) const { return piece < least ? 0 : piece * span; }
    __device__ __forceinline__ int pieces_of_batch(const BlockOrder& o) const {
        const float rec = __builtin_amdgcn_rcpf((float)span);
        if (o.alike) return __builtin_amdgcn_readfirstlane(o.batch * min(prefix(o.hi0, rec) - prefix(o.lo0, rec), kManyPieces));
        int count = 0;
        o.each([&](int g, int n) { count += n > 0 ? min(prefix(o.s.hi[g], rec) - prefix(o.s.lo[g], rec), kManyPieces) : 0; });
        return wave_count(count);
    }
    static __device__ __forceinline__ PiecePlan make(const BlockOrder& o, const PrefillPieces& p, int least_span) {
        // A walk of x is ceil(x / span) pieces, or `least`: with a sum of w over n blocks, at least w / span in all and less than
        // w / span + least n.  (fp32 sums, so one to spare on either side.)
        const int blocks = p.least * o.at_or_past(0);
        float w = 0.f;
        if (o.alike) {
            w = 0.5f * (float)o.batch * (float)(o.hi0 - o.lo0) * (float)(o.hi0 + o.lo0 + 1);
        } else {
            o.each([&](int g, int n) { w += 0.5f * (float)n * (float)(o.s.hi[g] + o.s.lo[g] + 1); });
            w = rows4_sum(row16_sum(w));
        }
        int low = max(least_span, (int)(w * __builtin_amdgcn_rcpf((float)p.target)) - 1) - 1;
        int high = p.target > blocks ? (int)min(1e6f, w * __builtin_amdgcn_rcpf((float)(p.target - blocks))) + 2 : 1 << 20;
        low = __builtin_amdgcn_readfirstlane(low);
        high = __builtin_amdgcn_readfirstlane(max(min(high, max(o.top(), 1)), low + 1));
        PiecePlan plan = {0, p.least, 0};
        while (high - low > 1) {
            plan.span = (low + high) / 2;
            if (plan.pieces_of_batch(o) <= p.target)
                high = plan.span;
            else
                low = plan.span;
        }
        plan.span = high;
        plan.total = plan.pieces_of_batch(o);
        if (plan.total > p.target) plan.total = 0;
        return plan;
    }
    // Position `rank` of the launch, below `total`: which piece it is of which block in the order of blocks, and the slot of
    // the piece.
    __device__ __forceinline__ void find(const BlockOrder& o, int& rank, int& piece, int& slot) const {
        int before = total;  // pieces with numbers up to the one looked at
        for (piece = __builtin_amdgcn_readfirstlane(pieces_of(o.top() - 1)) - 1; piece > 0; --piece) {
            const int n = o.at_or_past(level(piece));
            before -= n;
            if (rank < n) break;
            rank -= n;
        }
        slot = (piece > 0 ? before : 0) + rank;
    }
};

// General block mask (Sec. 3.1, Sec. 3.4): per mask and query tile, the ascending list of kept key
// tiles.  A workgroup of one slice owns four query tiles; a pre-pass merges their rows into one ascending list of
// (key tile, which of the four query tiles keep it) so that the main loop walks a single list.  A workgroup of four
// slices, or half a workgroup, owns one query tile and walks the caller's row as it is (see choose_mask_walk); the last three
// members are then not used.
struct PrefillMask {
    const int* head_mask;     // [H]: mask of query head h, -1 = analytic mask of the layer description
    const int* q_tile_start;  // [batch + 1]: first row of sequence b inside one mask
    const int* row_ptr;       // [num_masks * rows_per_mask + 1]
    const int* cols;          // key tiles, ascending inside a row
    int rows_per_mask;
    int* blk_list;            // merged lists; the list of a workgroup starts at row_ptr[its first row]
    int* blk_count;           // [num_masks][batch][blocks_per_seq]
    int blocks_per_seq;
};
constexpr int kKeepShift = 24;  // list entry = key tile | keep bits << 24

__global__ __launch_bounds__(kWave) void merge_mask_rows_kernel(PrefillMask mk, const int* __restrict__ cu_seqlens,
                                                                int batch) {
    extern __shared__ unsigned char keep_bits[];  // one byte per key tile of the sequence
    const int qblk = blockIdx.x, b = blockIdx.y, m = blockIdx.z, lane = threadIdx.x;
    const int len = cu_seqlens[b + 1] - cu_seqlens[b];
    const int n_tiles = ceil_div(len, kTile);
    int* count = mk.blk_count + ((size_t)m * batch + b) * mk.blocks_per_seq + qblk;
    const int iq0 = qblk * kPairs;
    if (iq0 >= n_tiles) {
        if (lane == 0) *count = 0;
        return;
    }
    const int rows = min(kPairs, n_tiles - iq0);
    const int r0 = m * mk.rows_per_mask + mk.q_tile_start[b] + iq0;
    const int last = min(iq0 + rows, n_tiles);  // key tiles the block can keep: [0, last)
    for (int j = lane; j < last; j += kWave) keep_bits[j] = 0;
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
    for (int t = 0; t < rows; ++t) {  // one row at a time: no two lanes touch the same byte
        const int lo = mk.row_ptr[r0 + t], hi = mk.row_ptr[r0 + t + 1];
        for (int e = lo + lane; e < hi; e += kWave) {
            const int j = mk.cols[e];
            if (j >= 0 && j <= iq0 + t) keep_bits[j] |= (unsigned char)(1u << t);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_wave_barrier();
    }
    int* dst = mk.blk_list + mk.row_ptr[r0];
    int total = 0;
    for (int j0 = 0; j0 < last; j0 += kWave) {
        const int j = j0 + lane;
        const unsigned bits = j < last ? keep_bits[j] : 0u;
        const unsigned long long live = __ballot(bits != 0);
        if (bits) dst[total + __popcll(live & ((1ull << lane) - 1ull))] = j | (int)(bits << kKeepShift);
        total += __popcll(live);
    }
    if (lane == 0) *count = total;
}

// Eight codes of a quantised row -> code * scale + zero -> eight values of the layer's 16-bit type.
template <class T, int BITS> __device__ __forceinline__ uint4 dequantise8(uint2 codes, uint32_t scale_zero) {
    const half2_t sz = __builtin_bit_cast(half2_t, scale_zero);
    const float scale = (float)sz[0], zero = (float)sz[1];
    uint32_t lo = codes.x, hi = codes.y;  // channels 0..3 and 4..7, one byte each
    if constexpr (BITS == 4) {
        hi = (codes.x >> 4) & 0x0f0f0f0fu;
        lo = codes.x & 0x0f0f0f0fu;
    }
    if constexpr (std::is_same<T, F16>::value) {
        // A code under the exponent byte 0x64 is the fp16 number 1024 + code, from which 1024 is taken off exactly; the
        // packed fma then rounds code * scale + zero once, to fp16, at three instructions per two values.
        const half2_t scale2 = {sz[0], sz[0]}, zero2 = {sz[1], sz[1]}, offset = {(_Float16)-1024.f, (_Float16)-1024.f};
        auto pair = [&](uint32_t word, uint32_t select) {
            const half2_t c = __builtin_bit_cast(half2_t, __builtin_amdgcn_perm(0x64646464u, word, select)) + offset;
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(c, scale2, zero2));
        };
        return make_uint4(pair(lo, 0x04010400u), pair(lo, 0x04030402u), pair(hi, 0x04010400u), pair(hi, 0x04030402u));
    }
    float x[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        x[j] = __builtin_fmaf((float)((lo >> (8 * j)) & 0xffu), scale, zero);
        x[4 + j] = __builtin_fmaf((float)((hi >> (8 * j)) & 0xffu), scale, zero);
    }
    return pack8<T>(x);
}

template <class T> struct Ones;
template <> struct Ones<F16> { static constexpr uint32_t pair = 0x3c003c00u; };
template <> struct Ones<BF16> { static constexpr uint32_t pair = 0x3f803f80u; };

enum PrefillMode { kPlain = 0, kMasked = 1, kPaged = 2 };

// BITS: width of the rows in the pages (16, or 8 / 4 for quantised pages, kPaged only).  Quantised tiles cannot take
// the direct-to-LDS path: their codes travel through registers, are turned into the layer's 16-bit type as
// code * scale + zero (fp16: rounded once; bf16: fp32, then rounded) and are stored to the same LDS places the direct loads
// would fill.
//
// SL: key slices.  The four wavefront pairs of a workgroup are (query heads) x (query tiles) x (key slices): with
// one slice all pairs walk the same key tiles; with two or four, slice s of a unit takes every SL-th tile of the walk
// and the slices are folded through LDS at the end.  A launch with few query rows (a short prompt, a chunk over a long
// history) then has SL times the workgroups, each with a walk SL times shorter, for SL times the staging per step
// (see choose_shape).
// KIND: kCut: the dense walks come in pieces (see PiecePlan); kHalf: a workgroup of four wavefronts and two units, two of them to
// a compute unit; kHasty: the same with the first workgroup of every compute unit in front (see longest_walk_decides).
enum WorkgroupKind { kWhole = 0, kCut = 1, kHalf = 2, kHasty = 3 };
template <class T, int MODE, int BITS, int SL, int KIND>
__device__ __forceinline__ void prefill_workgroup(
    const LayerParams& lp, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int* __restrict__ cu_seqlens, int batch, uint16_t* __restrict__ out,
    float* __restrict__ lse_out, int total_tokens, const PrefillSchedule& sched, const PrefillMask& mk, const PrefillPaged& pg,
    int number) {  // of the workgroup in the launch
    constexpr bool MASKED = MODE == kMasked, PAGED = MODE == kPaged, QUANT = BITS != 16;
    constexpr bool CUT = KIND == kCut, HALF = KIND == kHalf || KIND == kHasty, ROWS = MASKED && (SL > 1 || HALF);  // ROWS: lists are the caller's rows
    constexpr int kWaves = HALF ? kPrefillWaves / 2 : kPrefillWaves;
    static_assert(!CUT || (SL == 1 && PAGED), "chunks");
    static_assert(!HALF || SL == 1, "two units share a walk");
    static_assert(!QUANT || PAGED, "quantised rows live in pages");
    static_assert(SL == 1 || SL == 2 || (SL == 4 && !QUANT), "slices");
    // One or two slices: two stages of (K tiles, V tiles).  Four separate arrays, and a loop unrolled over the two
    // stages, so that the compiler can tell the tile being read from the tile being filled and does not wait
    // for the loads in flight before every operand read.  Four slices: 64 KiB of K and 64 KiB of V are one stage;
    // K is refilled while V is in use and the other way round.
    constexpr bool kOneStage = SL == 4;
    constexpr int kSpare = kOneStage ? 16 : SL * kKTileBytes;
    __shared__ __attribute__((aligned(1024))) unsigned char k_lds0[SL * kKTileBytes];
    __shared__ __attribute__((aligned(1024))) unsigned char k_lds1[kSpare];
    __shared__ __attribute__((aligned(1024))) unsigned char v_lds0[SL * kVTileBytes];
    __shared__ __attribute__((aligned(1024))) unsigned char v_lds1[kSpare];
    __shared__ float2 fold_ml[SL == 1 ? 1 : kPrefillWaves][32];  // (maximum, sum) of a wavefront's rows
    __shared__ int walk_len[SL == 1 ? 1 : kPrefillWaves];

    // The arguments fill eight 64-byte lines that the code below wants in dependent rounds, each a miss of the scalar
    // cache in a new workgroup; one word of every line is requested here, together.
#if defined(__HIP_DEVICE_COMPILE__)
    {
        typedef const int __attribute__((address_space(4))) * kernarg_words;
        const kernarg_words args = (kernarg_words)__builtin_amdgcn_kernarg_segment_ptr();
        static_assert(sizeof(LayerParams) + sizeof(PrefillSchedule) + sizeof(PrefillMask) + sizeof(PrefillPaged) + 8 * sizeof(void*) >
                      112 * sizeof(int), "the argument block must reach the last line touched");
        const int a0 = args[0], a1 = args[16], a2 = args[32], a3 = args[48], a4 = args[64], a5 = args[80], a6 = args[96],
                  a7 = args[112];
        asm volatile("" ::"s"(a0), "s"(a1), "s"(a2), "s"(a3), "s"(a4), "s"(a5), "s"(a6), "s"(a7));
    }
#endif

    // heaviest query blocks first; see HeadClass for the XCD-aware order
    const int xcd = number % kXcds;
    int li = number / kXcds, hidx, hk, hg, rank;
    const bool second = li >= sched.cls[0].items_per_xcd;
    if (second) li -= sched.cls[0].items_per_xcd;
    const int heads_per_block = second ? sched.cls[1].heads_per_block : sched.cls[0].heads_per_block;
    const int qtiles_log2 = second ? sched.cls[1].qtiles_log2 : sched.cls[0].qtiles_log2;
    const bool fold = SL > 1 && (second ? sched.cls[1].fold : sched.cls[0].fold);
    const int blocks_per_seq = second ? sched.cls[1].blocks_per_seq : sched.cls[0].blocks_per_seq;
    decode_work(second ? sched.cls[1] : sched.cls[0], lp.group / heads_per_block, xcd, li, hidx, hk, hg, rank);
    int b, qblk = 0;
    const int blocks = second ? sched.cls[1].blocks : sched.cls[0].blocks;
    const bool again = MASKED && HALF && rank >= blocks;  // the second time over the blocks, for heads without a common mask
    if (again) {
        if (heads_per_block == 1) return;
        rank -= blocks;
    }
    int piece = 0, pieces = 1, slot = 0;  // of a cut walk: which piece of how many, and where it goes
    PiecePlan plan = {0x7fffffff, 1, 0};
    if (second ? sched.cls[1].ordered : sched.cls[0].ordered) {
        const BlockOrder order =
            block_order(cu_seqlens, PAGED ? pg.kv.seq_lens : nullptr, PAGED && pg.k_new, batch, kTileLog2 + qtiles_log2);
        if (CUT && !second) {
            if (order.top() <= sched.pieces.short_blocks) return;
            plan = PiecePlan::make(order, sched.pieces, kLeastSpanTiles >> qtiles_log2);
            if (rank >= plan.total) return;
            plan.find(order, rank, piece, slot);
            slot += (hidx * (lp.group / heads_per_block) + hg) * sched.pieces.target;
        }
        if (!order.find<HALF>(rank, b, qblk)) return;
        // All of it comes out of lane arithmetic.  Left in a vector register, the block's position takes the length of the
        // walk, the key tile of every step and the page look-ups there with it, and each branch on them runs under a mask of
        // lanes (a step of one slice 1.71 us, 1.65 with all in scalar registers: 512 tokens over 32768).
        b = __builtin_amdgcn_readfirstlane(b);
        qblk = __builtin_amdgcn_readfirstlane(qblk);
        if (CUT) {
            piece = __builtin_amdgcn_readfirstlane(piece);
            if (!second) pieces = __builtin_amdgcn_readfirstlane(plan.pieces_of(qblk));
            slot = pieces > 1 ? slot : -1;
            asm volatile("" : "+v"(slot));  // wanted at the very end: a vector register, of which there are some left
        }
    } else {
        if (rank >= blocks_per_seq * batch) return;
        b = rank % batch;
    }
    // start: row of the sequence's first query in q / out; len: keys of the sequence; first: position of
    // that first query (0 unless the keys come from a paged cache that already holds earlier tokens)
    const int start = cu_seqlens[b];
    // cached: keys that come from the pages (all of them, or the history of a chunk whose K / V arrive alongside)
    const int cached = PAGED ? pg.kv.seq_lens[b] : 0;
    const int len = PAGED ? (pg.k_new ? cached + (cu_seqlens[b + 1] - start) : cached) : cu_seqlens[b + 1] - start;
    const int first = PAGED ? len - (cu_seqlens[b + 1] - start) : 0;
    const int qtiles = 1 << qtiles_log2;  // query tiles of the workgroup
    if (!(second ? sched.cls[1].ordered : sched.cls[0].ordered))
        qblk = (first >> (kTileLog2 + qtiles_log2)) + blocks_per_seq - 1 - rank / batch;
    const int iq0 = qblk << qtiles_log2;
    if (iq0 * kTile >= len) return;
    if (PAGED && first >= len) return;  // a sequence without queries in this chunk

    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int n = lane % 32, half = lane / 32;
    // This wave's pair: the slice of the staging space it works from, and its (query tile, query head).  Folded, the
    // slices of a workgroup hold different key tiles of the same units; otherwise each slice walks for units of its own.
    constexpr int kSliceUnits = kPairs / SL;
    const int slice = (wave / 2) % SL, unit = wave / 2 / SL;
    const int own = SL > 1 && !fold ? slice * kSliceUnits + unit : unit;
    const int qt = own & (qtiles - 1);
    int h = hk * lp.group + hg * heads_per_block + (own >> qtiles_log2);
    bool idle = false;  // a unit without work
    if (MASKED && HALF) {
        idle = unit > 0;
        h = hk * lp.group + hg;  // of all wavefronts: they walk one list, and meet at its barriers
        if (heads_per_block == 2) {
            // The hg-th two of the group's heads in the order of their masks: one workgroup for both if they have one mask
            // between them, one for each otherwise.
            int head[2] = {0, 0}, mask[2] = {-1, -1};
            const int* ids = mk.head_mask + hk * lp.group;
#pragma unroll
            for (int i = 0; i < kMaxGroup; ++i) {
                if (i >= lp.group) break;
                const int id = ids[i];
                int before = 0;
#pragma unroll
                for (int j = 0; j < kMaxGroup; ++j)
                    if (j < lp.group && j != i) before += j < i ? ids[j] <= id : ids[j] < id;
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    if (before == 2 * hg + u) head[u] = i, mask[u] = id;
            }
            const bool together = mask[0] == mask[1];
            if (together && again) return;
            idle = !together && unit > 0;
            h = hk * lp.group + __builtin_amdgcn_readfirstlane((together ? unit > 0 : again) ? head[1] : head[0]);
        }
    }
    const bool streaming = (lp.streaming_mask >> hk) & 1ull;
    const int iq = iq0 + qt;             // this wave's mask tile; the wave owns one half of its rows
    const int row0 = (wave % 2) * 32;    // first row of the wave inside the mask tile
    const int n_qtiles = ceil_div(len, kTile);
    const bool wave_has_rows = !idle && iq * kTile + row0 < len && iq * kTile + row0 + 32 > first;
    // query tiles that share this wave's walk, and the key tiles it visits: [0, sink_end) and [band_begin, iq_last]
    const int iq_first = iq0 + (SL > 1 && !fold ? (slice * kSliceUnits) & (qtiles - 1) : 0);
    const int iq_last = min(iq_first + (SL > 1 ? min(qtiles, kSliceUnits) : qtiles) - 1, n_qtiles - 1);
    int sink_end, band_begin;
    if (streaming) {
        band_begin = max(0, iq_first - lp.local_pages + 1);
        sink_end = min(lp.sink_pages, band_begin);
    } else {
        band_begin = 0;
        sink_end = 0;
    }
    int n_visit = iq_first <= iq_last ? sink_end + (iq_last - band_begin + 1) : 0;  // 0: past the end of the sequence
    // a listed mask replaces the closed form: the merged list of the query tiles of the walk, or, when it has a single
    // one, the caller's row itself (its entries above the tile's own index are cut off)
    const int* lst = nullptr;
    if (MASKED) {
        const int m = mk.head_mask[h];
        if (m >= 0 && iq_first <= iq_last) {
            const int row = m * mk.rows_per_mask + mk.q_tile_start[b] + iq_first;
            if (!ROWS) {
                lst = mk.blk_list + mk.row_ptr[row];
                n_visit = mk.blk_count[((size_t)m * batch + b) * mk.blocks_per_seq + qblk];
            } else {
                const int lo = mk.row_ptr[row];
                lst = mk.cols + lo;
                n_visit = max(0, mk.row_ptr[row + 1] - lo);
                if (n_visit > 0 && lst[n_visit - 1] > iq) {
                    int below = 0;
                    while (below < n_visit) {
                        const int mid = (below + n_visit) / 2;
                        if (lst[mid] <= iq)
                            below = mid + 1;
                        else
                            n_visit = mid;
                    }
                }
            }
        }
    }

    int it_begin = 0;
    if (CUT && pieces > 1) {
        it_begin = n_visit * piece / pieces;
        n_visit = n_visit * (piece + 1) / pieces;
    }

    float16_t acc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[db][i] = 0.f;
    // Reference of this lane's query row, in units of the unscaled products, and the sum of its weights relative to it.  The
    // reference is a maximum of the row's scores, but not always the latest (see weights_and_values).
    float m_run = -INFINITY, l_run = 0.f;
    const bool first_on_unit = KIND == kHasty && number < sched.compute_units;
    int unset = 1;  // some row of the wave has no reference yet
    // The score products start from -m_run instead of 0 (the accumulator input of the first product), so that scores come
    // relative to it at no cost; 0 while m_run = -inf.
    float16_t neg_m;
#pragma unroll
    for (int i = 0; i < 16; ++i) neg_m[i] = 0.f;

    // ---- staging: the waves of a slice bring in its tile, two direct-to-LDS loads of 1 KiB per wave, operand and slice
    // contiguous keys: tile jt starts jt * 64 rows after the sequence's first row; paged keys: tile jt is the
    // slab of (its page, hk) in the pool the head lives in, rows 256 bytes apart; keys of a chunk that has not
    // been written back: row u - cached of the chunk's own K / V
    const bool ring = PAGED && in_stream_pool(lp, pg.kv, hk);  // a streaming head kept in its bounded pool
    const int heads_in_pool = PAGED ? (ring ? pg.kv.stream_heads : pg.kv.pool_heads) : lp.Hkv;
    constexpr size_t kSlabBytes = slab_chunks(kTile, BITS) * 16;  // one (page, head) of a pool
    const size_t slab_in_page = PAGED ? (size_t)pool_rank(lp, pg.kv, hk, ring) * (kSlabBytes / 2) : 0;  // in 16-bit units
    const uint16_t* kbase = PAGED ? reinterpret_cast<const uint16_t*>(ring ? pg.kv.k_stream : pg.kv.k_pool) + slab_in_page
                                  : k + ((size_t)start * lp.Hkv + hk) * kHeadDim;
    const uint16_t* vbase = PAGED ? reinterpret_cast<const uint16_t*>(ring ? pg.kv.v_stream : pg.kv.v_pool) + slab_in_page
                                  : v + ((size_t)start * lp.Hkv + hk) * kHeadDim;
    const int* page_row = !PAGED ? nullptr
                          : ring ? pg.kv.ring_table + (size_t)b * pg.kv.ring
                                 : pg.kv.page_table + (size_t)b * pg.kv.max_pages;
    // page of key tile jt, for tiles that hold cached keys (0 otherwise: never used)
    auto page_of = [&](int jt) {
        if (!PAGED || jt * kTile >= cached) return 0;
        return page_row[ring ? ring_slot(lp, jt) : jt];
    };
    // The waves of a slice share out its tile: wave w of them takes the n = 64 SL / kWaves rows from n w, four rows per load, and
    // lane `lane` of load i fills position lane % 16 of row n w + 4 i + lane / 16.  Addresses are a wave-uniform
    // 64-bit base (scalar arithmetic) plus a 32-bit lane offset that does not depend on the tile, except in the last
    // tile of a sequence, where rows past the end read the last row again (finite values; their softmax weights
    // are 0).  Sixteen rows on the permutation of K repeats itself, four rows on that of V.
    constexpr int kLoads = SL * 16 / kWaves;  // 1 KiB loads per wave and operand
    constexpr int kOfs = kLoads < 4 ? kLoads : 4;
    const unsigned seq_row_bytes = (unsigned)__builtin_amdgcn_readfirstlane(lp.Hkv * kHeadDim * 2);  // [token][Hkv][D]
    const unsigned k_row_bytes = PAGED ? kHeadDim * 2u : seq_row_bytes;
    const unsigned long long k_page_bytes = (unsigned long long)heads_in_pool * kSlabBytes;
    const int wave_row0 = (unit * 2 + wave % 2) * (kTile * SL / kWaves);
    const int krow0 = wave_row0 + lane / 16;  // row of load 0; load i takes row + 4 i
    unsigned kofs[kOfs];
#pragma unroll
    for (int i = 0; i < kOfs; ++i)
        kofs[i] = (unsigned)(krow0 + 4 * i) * k_row_bytes + k_chunk_pos(krow0 + 4 * i, lane % 16) * 16;  // an involution
    const unsigned vofs = (unsigned)krow0 * k_row_bytes + v_chunk_pos(krow0, lane % 16) * 16;           // likewise
    const unsigned lds_slice = (unsigned)slice * kKTileBytes;
    const unsigned lds_wave = (unsigned)__builtin_amdgcn_readfirstlane(lds_slice + wave_row0 * kKRowBytes);
    const unsigned long long kbase_u = uniform64((unsigned long long)kbase), vbase_u = uniform64((unsigned long long)vbase);
    // the chunk's own rows, addressed from its first token (the row of position `cached`)
    const unsigned long long knew_u =
        uniform64((unsigned long long)(PAGED && pg.k_new ? pg.k_new + ((size_t)start * lp.Hkv + hk) * kHeadDim : nullptr));
    const unsigned long long vnew_u =
        uniform64((unsigned long long)(PAGED && pg.v_new ? pg.v_new + ((size_t)start * lp.Hkv + hk) * kHeadDim : nullptr));
    const int len_u = __builtin_amdgcn_readfirstlane(len), cached_u = __builtin_amdgcn_readfirstlane(cached);
    // quantised rows on their way through registers: per load the codes of this lane's 16-byte place (8 channels), the
    // (scale, zero) pair of the row, and whether the lane's row comes from the pages at all
    constexpr int kRowCodeBytes = kHeadDim * BITS / 8, kPlaceCodeBytes = BITS;  // per row; per 8 channels
    struct Staged {
        uint2 codes[kLoads];
        uint32_t sz[kLoads];
        int from, left;  // of the tile in flight: rows that come from the pages; rows it has
    };
    Staged staged_k, staged_v;
    staged_k.from = staged_v.from = 0;
    staged_k.left = staged_v.left = 1;
    // Requests this wave's share of key tile jt: of K, of V or of both, then in turn (K after K and V after V was 3 % slower
    // on a prompt of 65536 tokens: the first rows of V come before the last rows of K are asked for).  kd, vd: arrays of
    // the stage.
    auto fetch = [&](auto operands, unsigned char* kd, unsigned char* vd, int jt, int phys) {
        constexpr bool K = decltype(operands)::value & 1, V = decltype(operands)::value & 2;
        jt = __builtin_amdgcn_readfirstlane(jt);
        const unsigned lds_k = lds_address(kd) + lds_wave, lds_v = lds_address(vd) + lds_wave;
        // Rows at or past the sequence length must not be read as they are: a page may hold anything there, and
        // although their weights are 0 a non-finite value would still poison the second product.
        const int rows_left = len_u - jt * kTile;
        // rows of the tile below `from_pages` come from the page, the others from the chunk's own K / V: row r of the
        // tile is then the chunk's token jt * 64 + r - cached
        const int from_pages = PAGED ? cached_u - jt * kTile : kTile;
        if (!QUANT && (!PAGED || from_pages >= min(rows_left, kTile))) {
            const unsigned long long ktile =
                PAGED ? kbase_u + (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(phys) * k_page_bytes
                      : kbase_u + (unsigned long long)jt * (kTile * k_row_bytes);
            const unsigned long long vtile = ktile - kbase_u + vbase_u;  // K and V are laid out alike
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const unsigned ldk = __builtin_amdgcn_readfirstlane(lds_k + i * 1024);
                const unsigned ldv = __builtin_amdgcn_readfirstlane(lds_v + i * 1024);
                if (rows_left < kTile) {
                    const int row = krow0 + 4 * i;
                    const unsigned at = (unsigned)min(row, rows_left - 1) * k_row_bytes;
                    if (K) dma_load16(ktile, at + k_chunk_pos(row, lane % 16) * 16, ldk);
                    if (V) dma_load16(vtile, at + v_chunk_pos(row, lane % 16) * 16, ldv);
                } else {
                    if (K) dma_load16(ktile + (unsigned)(i / 4) * (16u * k_row_bytes), kofs[i % 4], ldk);
                    if (V) dma_load16(vtile + (unsigned)i * (4u * k_row_bytes), vofs, ldv);
                }
            }
        } else if (PAGED && from_pages < min(rows_left, kTile)) {
            // the tile holds rows of the chunk; rows of quantised pages come another way (fetch_codes)
            const unsigned long long page = (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(phys) * k_page_bytes;
            const unsigned long long shift = (unsigned long long)((long long)jt * kTile - cached_u) * seq_row_bytes;
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const int row = krow0 + 4 * i, r = min(row, rows_left - 1);
                const unsigned kc = k_chunk_pos(row, lane % 16) * 16, vc = v_chunk_pos(row, lane % 16) * 16;
                const unsigned ldk = __builtin_amdgcn_readfirstlane(lds_k + i * 1024);
                const unsigned ldv = __builtin_amdgcn_readfirstlane(lds_v + i * 1024);
                if (r >= from_pages) {
                    if (K) dma_load16(knew_u + shift, (unsigned)r * seq_row_bytes + kc, ldk);
                    if (V) dma_load16(vnew_u + shift, (unsigned)r * seq_row_bytes + vc, ldv);
                } else if (!QUANT) {  // only in the one tile that straddles the end of the cache
                    if (K) dma_load16(kbase_u + page, (unsigned)r * k_row_bytes + kc, ldk);
                    if (V) dma_load16(vbase_u + page, (unsigned)r * k_row_bytes + vc, ldv);
                }
            }
        }
    };
    constexpr std::integral_constant<int, 1> kOnlyK{};
    constexpr std::integral_constant<int, 2> kOnlyV{};
    constexpr std::integral_constant<int, 3> kBoth{};
    // requests the codes of one operand's share of key tile jt (quantised pages)
    auto fetch_codes = [&](auto operand, Staged& staged, int jt, int phys) {
        constexpr bool K = decltype(operand)::value == 1;
        if constexpr (QUANT) {
            jt = __builtin_amdgcn_readfirstlane(jt);
            staged.left = len_u - jt * kTile;
            staged.from = cached_u - jt * kTile;
            if (staged.from <= 0) return;
            const unsigned char* slab = reinterpret_cast<const unsigned char*>(K ? kbase : vbase) +
                                        (size_t)(unsigned)__builtin_amdgcn_readfirstlane(phys) * k_page_bytes;
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                // a row that does not come from the page reads the page's last valid row, for nothing
                const int row = krow0 + 4 * i, r = min(min(row, staged.left - 1), min(staged.from, kTile) - 1);
                const unsigned char* src =
                    slab + (size_t)r * kRowCodeBytes + (K ? k_chunk_pos(row, lane % 16) : v_chunk_pos(row, lane % 16)) * kPlaceCodeBytes;
                if constexpr (BITS == 8)
                    staged.codes[i] = *reinterpret_cast<const uint2*>(src);
                else
                    staged.codes[i] = make_uint2(*reinterpret_cast<const uint32_t*>(src), 0u);
                staged.sz[i] = reinterpret_cast<const uint32_t*>(slab + kTile * kRowCodeBytes)[r];
            }
        }
    };
    // Entry `it` of the walk: key tile in the low bits; with a listed mask also which query tiles keep it.
    auto entry_of = [&](int it) {
        if (MASKED && lst) {
            const int e = lst[it];
            if (!ROWS) return e;
            const int jt = min(max(e, 0), iq);  // a row of the caller: anything outside the triangle is not kept
            return e == jt ? jt | (1 << kKeepShift) : jt;
        }
        return it < sink_end ? it : band_begin + (it - sink_end);
    };
    constexpr int kTileMask = (1 << kKeepShift) - 1;
    // the wave's entries: first, first + stride, ...
    const int it_first = CUT ? it_begin : fold ? slice : 0, stride = fold ? SL : 1;
    int e_cur = it_first < n_visit ? entry_of(it_first) : 0;
    int e_nxt = it_first + stride < n_visit ? entry_of(it_first + stride) : 0;
    // physical pages of the tiles to come, looked up two steps ahead of the loads that need them
    const int ph_first = it_first < n_visit ? page_of(e_cur & kTileMask) : 0;
    int ph_nxt = it_first + stride < n_visit ? page_of(e_nxt & kTileMask) : 0;
    // quantised pages: the entry after that too, since codes are requested two steps ahead
    int e_nx2 = QUANT && it_first + 2 * stride < n_visit ? entry_of(it_first + 2 * stride) : 0;
    int ph_nx2 = QUANT && it_first + 2 * stride < n_visit ? page_of(e_nx2 & kTileMask) : 0;
    // the first tiles travel while the queries are fetched
    if (it_first < n_visit) {
        if constexpr (kOneStage)
            fetch(kOnlyK, k_lds0, v_lds0, e_cur & kTileMask, ph_first);
        else
            fetch(kBoth, k_lds0, v_lds0, e_cur & kTileMask, ph_first);
        fetch_codes(kOnlyK, staged_k, e_cur & kTileMask, ph_first);
        fetch_codes(kOnlyV, staged_v, e_cur & kTileMask, ph_first);
    }
    // steps of the workgroup: every wave must reach every barrier, so the longest walk counts
    int steps = fold ? ceil_div(n_visit, SL) : n_visit - (CUT ? it_begin : 0);
    if (SL > 1 && !fold) {
        if (lane == 0) walk_len[wave] = n_visit;
        __syncthreads();
        steps = 0;
#pragma unroll
        for (int i = 0; i < kPrefillWaves; ++i) steps = max(steps, walk_len[i]);
        steps = __builtin_amdgcn_readfirstlane(steps);
    }

    // ---- Q^T operand: lane (n, half) holds Q[row][16 kk + 8 half .. + 8]
    uint4 qreg[8];
    {
        // By direct loads into LDS where it has room (the second stage; of a single one V's part, whose first tile comes after), a row
        // to sixteen lanes: 16 bytes of 32 rows to an instruction, as the lanes want them, keep the address path busy twice as long.
        // One prompt of 1024 tokens 21.9 -> 20.5 us, of 3200 80.1 -> 74.7, 16 of 123 12.4 -> 11.3, of 77 .. 3001 177 -> 172.  (Whole
        // workgroups of one slice have half the room, and lose 2 to 3 % on long walks with more.)
        constexpr int kRowsBytes = 32 * kHeadDim * 2, kPerArray = (kOneStage ? SL * kVTileBytes : kSpare) / kRowsBytes;
        if constexpr (kWaves <= (kOneStage ? 1 : 2) * kPerArray) {
            unsigned char* const room = (kOneStage ? v_lds0 : wave < kPerArray ? k_lds1 : v_lds1) + wave % kPerArray * kRowsBytes;
            // rows without a query (in front of the chunk, past the end) read the nearest one
            const int top = min(max(iq * kTile + row0, first), len - 1);
            const unsigned long long rows = uniform64((unsigned long long)(q + ((size_t)(start + top - first) * lp.H + h) * kHeadDim));
            const unsigned q_row_bytes = (unsigned)__builtin_amdgcn_readfirstlane(lp.H * kHeadDim * 2);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int r = 4 * i + lane / 16, at = min(max(iq * kTile + row0 + r, first), len - 1) - top;
                dma_load16(rows, (unsigned)at * q_row_bytes + k_chunk_pos(r, lane % 16) * 16,
                           __builtin_amdgcn_readfirstlane(lds_address(room) + i * 1024));
            }
            dma_wait();
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
                qreg[kk] = *reinterpret_cast<const uint4*>(room + n * kKRowBytes + k_chunk_pos(n, kk * 2 + half) * 16);
        } else {
            const int row = min(max(iq * kTile + row0 + n, first), len - 1) - first;
            const uint4* src = reinterpret_cast<const uint4*>(q + ((size_t)(start + row) * lp.H + h) * kHeadDim);
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) qreg[kk] = src[kk * 2 + half];
        }
        // Pin the loads here.  Left alone the compiler sinks them to the loop entry, and because the
        // memory counter completes in order every tile's first product would then wait for that
        // tile's K / V prefetch.  (And the place in LDS is given to other waves' tiles after the next barrier.)
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
            asm volatile("" : "+v"(qreg[kk].x), "+v"(qreg[kk].y), "+v"(qreg[kk].z), "+v"(qreg[kk].w));
    }

    // loop-invariant operand offsets of this lane inside a stage (its slice's tile)
    int koff[8], voff[4];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) koff[kk] = (int)lds_slice + n * kKRowBytes + k_chunk_pos(n, kk * 2 + half) * 16;
    // V^T operand of (channel block db, 16-key step, half u of the lane's 8 keys): the lane's row of sixteen names
    // keys 16 step + 8 u + 4 half + s / 4 (s = lane % 16) and channels 32 db + 16 (n / 16) + 4 (s % 4) .. + 3, which
    // after the exchange leaves lane (n, half) with channel 32 db + n of keys 16 step + 8 u + 4 half + 0 .. 3: the
    // keys its weights P^T[8 half + 4 u .. + 3] belong to.  Per db the lane part of the address is fixed; step and u
    // add (4 step + 2 u) KiB.
#pragma unroll
    for (int db = 0; db < 4; ++db) {
        const int s16 = lane % 16, rr = s16 / 4;
        const int chunk = 4 * db + 2 * (n / 16) + (s16 % 4) / 2;
        voff[db] = (int)lds_slice + half * 1024 + rr * kVRowBytes + v_chunk_pos(rr, chunk) * 16 + 8 * (s16 % 2);
    }

    auto store_staged = [&](unsigned char* dst, const Staged& staged) {
        if constexpr (QUANT) {
            if (staged.from <= 0) return;
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                if (min(krow0 + 4 * i, staged.left - 1) < staged.from)  // the lanes that fetch() gave codes
                    *reinterpret_cast<uint4*>(dst + lds_wave + i * 1024 + lane * 16) =
                        dequantise8<T, BITS>(staged.codes[i], staged.sz[i]);
            }
        }
    };

    // does this wave's mask tile keep the tile of entry e (entry `it` of the walk)?
    auto keeps = [&](int it, int e) {
        const int jt = e & kTileMask;
        bool keep = wave_has_rows && jt <= iq && (SL == 1 || it < n_visit);
        if (MASKED && lst)
            keep = keep && ((e >> (kKeepShift + iq - iq_first)) & 1);
        else if (streaming)
            keep = keep && (jt < lp.sink_pages || jt > iq - lp.local_pages);
        return keep;
    };
    // S^T for the 64 keys of a tile, two blocks of 32 keys.  All operand reads of a block are issued before its
    // products so that LDS latency is paid once, and the two blocks' accumulation chains alternate in the matrix pipe.
    auto scores = [&](float16_t (&s)[2], const unsigned char* ks, bool diagonal) {
        if (KIND == kHasty && first_on_unit)
            __builtin_amdgcn_s_setprio(3);
        else
            __builtin_amdgcn_s_setprio(2);  // products first: the other wavefront of the SIMD fills in with softmax work
        uint4 ka[8][2];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                ka[kk][kb] = *reinterpret_cast<const uint4*>(ks + kb * 32 * kKRowBytes + koff[kk]);
        s[0] = Mfma<T>::run(ka[0][0], qreg[0], neg_m);
        s[1] = Mfma<T>::run(ka[0][1], qreg[0], neg_m);
#pragma unroll
        for (int kk = 1; kk < 8; ++kk) {
            s[0] = Mfma<T>::run(ka[kk][0], qreg[kk], s[0]);
            s[1] = Mfma<T>::run(ka[kk][1], qreg[kk], s[1]);
        }
        // schedule: operand reads run four ahead of the products that consume them
        __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
        for (int u = 0; u < 16 - kAhead; ++u) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, kAhead, 0);
        if (KIND == kHasty && first_on_unit)
            __builtin_amdgcn_s_setprio(2);
        else
            __builtin_amdgcn_s_setprio(0);
        if (diagonal) {  // causal mask inside the diagonal tile
            // (opaque, or the 32 comparisons are hoisted out of the loop into 64 scalar registers, and what the loop
            // does need is then read back from spilled lanes in every step)
            int last_key = row0 + n - 4 * half;
            asm volatile("" : "+v"(last_key));
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int key = kb * 32 + 8 * (i / 4) + (i % 4);  // less 4 half
                    if (key > last_key) s[kb][i] = -INFINITY;
                }
        }
    };
    // Selects a lane's own row in the sums of weights: see below.
    const uint32_t own_row = ((lane % 16) / 4 - lane / 16) % 2 == 0 ? Ones<T>::pair : 0u;
    // Softmax of this lane's query row (its keys are split between the two lane halves), then O^T += V^T P^T.
    //
    // Weights are exp2(scale (score - reference)), and a row's reference stays what it is until its weights in a tile add up
    // to kMostWeight: below that nothing overflows (fp16 ends at 65504), and weights above 1 have the bits of those below.
    // So no maximum stands between the products and the exponentials, and most tiles need none: a tile is 32 multiplications, 32
    // exponentials and 16 conversions per lane, where a running maximum took a chain of 16 in front of them and, whenever the maximum of
    // one of the wave's 32 rows moved (three of four tiles among a walk's first 64), 112 instructions to rescale.  The scale meets the
    // fp32 products, and the queries stay as they are: scaled and rounded in front of the products they save the multiplications, which
    // gains 0.1 % over 26 prompts and chunks, and lose a quarter of the precision (against 64 bits, 16 of 77 .. 3001 in bf16: 2.00e-3;
    // with rounded queries 2.55e-3, with the running maximum 2.50e-3).  An fma of product, scale and reference instead of the
    // accumulator input and a multiplication: 7 % slower at 65536 tokens.  Running maximum and this, on one box: 65536 tokens 15.68 and 15.08
    // ms, 4096 111 and 105 us, 12345 under a mask 319 and 295, 512 over 32768 174 and 158, two of 2642, 64 / 8 heads, 192 and 177.
    //
    // Each row goes by its own weights, and a sum is taken the same way in every round, so the other rows of the wavefront, which a
    // chunk that begins or ends inside 32 rows has others of, leave no trace in a row's bits (nor in the time: 65536 tokens 15.01 and 14.94
    // ms with one decision for the wavefront and with this, 16 of 77 .. 3001 178.6 and 178.1 us).  What is left of moving references is paid for by loud keys: keys that grow along the sequence to
    // three times their size, running maximum and this, us, 4096 tokens 114.9 and 107.8, 16384 1197 and 1075; to twelve times 113.7 and 121.1
    // in bf16, whose bound is passed once in a while only, 112.7 and 130.0 in fp16.  A row in 37 not a number: 109.9 and 100.0.
    constexpr float kMostWeight = std::is_same<T, F16>::value ? 0x1p15f : 0x1p30f;
    const uint4 own_rows = make_uint4(own_row, own_row, own_row, own_row);
    auto weights_and_values = [&](float16_t (&s)[2], const unsigned char* vs) {
        uint4 pb[2][2];  // P^T packed to 16 bit: [key block][16-key step]
        float sum;
        int moved = unset;
        unsigned long long over = 0;  // lanes of the rows whose weights add up to too much in this tile
        asm volatile("" : "+s"(moved));  // (opaque, or the second round becomes a copy of the first that costs 20 registers)
#pragma clang loop unroll(disable)
        for (;;) {
            if (moved) {  // the reference of rows over the bound, or without one, becomes the maximum so far: subtract and rescale
                float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
                for (int i = 1; i < 16; ++i) mx = __builtin_fmaxf(__builtin_fmaxf(mx, s[0][i]), s[1][i]);  // v_max3_f32
                mx = halves_max(mx);  // relative to the reference (to 0 before the first kept tile)
                const bool first_one = m_run == -INFINITY, stays = !first_one && !__builtin_amdgcn_inverse_ballot_w64(over);
                const float m_base = first_one ? 0.f : m_run;
                const float m_new = stays ? m_run : fmaxf(m_run, m_base + mx);
                const bool none = m_new == -INFINITY;  // nothing but -inf so far
                const float delta = none || stays ? 0.f : m_new - m_base;
                const float alpha = stays ? 1.f : first_one ? 0.f : __builtin_amdgcn_exp2f((m_run - m_new) * lp.sm_scale_log2);
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[db][i] *= alpha;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) s[kb][i] -= delta;
                m_run = m_new;
#pragma unroll
                for (int i = 0; i < 16; ++i) neg_m[i] = none ? 0.f : -m_new;
                unset = __builtin_amdgcn_readfirstlane(__any(none));
            }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                float pf[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) pf[i] = __builtin_amdgcn_exp2f(s[kb][i] * lp.sm_scale_log2);
                pb[kb][0] = pack8<T>(pf);
                pb[kb][1] = pack8<T>(pf + 8);
            }
            // Row sums of the rounded weights, the same values the second product uses, by four products of 16 x 16 x 32 (0.7 %
            // quicker than sixteen dot products).  Read as the 32 x 16 operand of such a product, P^T has query c and query 16 + c in its
            // column c, the one in the first and third eight keys, the other in the second and fourth; ones in those of row r's choice
            // leave every lane with the sum of its own query.
            float4_t sums = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int j = 0; j < 2; ++j) sums = Mfma<T>::run16(own_rows, pb[kb][j], sums);
            sum = sums[0];
            if (__builtin_expect(!__any(!(sum < kMostWeight)), 1)) break;
            // A weight that is infinite or not a number spoils the sum of the other query of its column: once more without the rows
            // that have one.
            if (__any(!(sum < INFINITY))) {
                float own = 0.f;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const uint32_t w[8] = {pb[kb][0].x, pb[kb][0].y, pb[kb][0].z, pb[kb][0].w,
                                           pb[kb][1].x, pb[kb][1].y, pb[kb][1].z, pb[kb][1].w};
#pragma unroll
                    for (int u = 0; u < 8; ++u) own = Elem<T>::dot2(w[u], Ones<T>::pair, own);
                }
                own = halves_sum(own);
                const bool finite = own < INFINITY;
                sums = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        __builtin_amdgcn_sched_barrier(0);  // one at a time, or all four copies are alive together
                        const uint4 w = pb[kb][j];
                        sums = Mfma<T>::run16(own_rows, make_uint4(finite ? w.x : 0u, finite ? w.y : 0u, finite ? w.z : 0u, finite ? w.w : 0u), sums);
                    }
                __builtin_amdgcn_sched_barrier(0);
                sum = finite ? sums[0] : own;
                if (over) {
                    // Not finite by its own maximum either: a row that is not a number, and its sum says so for good.  Its queries give way to
                    // zeros, so that it holds up no more tiles.
                    m_run = finite ? m_run : 0.f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) neg_m[i] = finite ? neg_m[i] : 0.f;
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk)
                        qreg[kk] = make_uint4(finite ? qreg[kk].x : 0u, finite ? qreg[kk].y : 0u, finite ? qreg[kk].z : 0u, finite ? qreg[kk].w : 0u);
                    unset = __builtin_amdgcn_readfirstlane(__any(m_run == -INFINITY));
                }
            }
            if (over) break;
            over = __ballot(!(sum < kMostWeight));
            if (!over) break;
            moved = 1;
            asm volatile("" : "+s"(moved));
        }
        l_run += sum;
        // O^T += V^T * P^T, 16 keys per instruction; operand reads run one step ahead
#pragma unroll
        for (int step = 0; step < 4; ++step) {
            const int kb = step / 2, j = step % 2;
            uint4 va[4];
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                const uint2 lo = lds_read_transposed(vs + (4 * step) * 1024 + voff[db]);
                const uint2 hi = lds_read_transposed(vs + (4 * step + 2) * 1024 + voff[db]);
                va[db] = make_uint4(lo.x, lo.y, hi.x, hi.y);
            }
#pragma unroll
            for (int db = 0; db < 4; ++db) acc[db] = Mfma<T>::run(va[db], pb[kb][j], acc[db]);
        }
        // schedule: operand reads run one step (four products, eight reads) ahead
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
#pragma unroll
        for (int u = 0; u < 12; ++u) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    };

    // One step of two-stage staging: the tiles of the next step are requested, those of this one are worked on.
    auto tile_step = [&](int it, const unsigned char* ks, const unsigned char* vs, unsigned char* kd, unsigned char* vd) {
        const bool more = it + stride < n_visit;
        const int e = e_cur;
        if constexpr (QUANT) {
            // The codes of the next tile were requested a step ago; they are stored first of all, and the registers then take the
            // codes of the tile after it, which have this whole step to arrive.  Two chunks of 698 and 3490 tokens over 28906 of
            // 4 bits, one slice, bf16: 2147 us; with K stored between this tile's products and V after them 2293, with codes
            // requested and stored in the same step 2337, with either half of the waves at either end of the step 2366.
            const bool more2 = it + 2 * stride < n_visit, more3 = it + 3 * stride < n_visit;
            const int e_new = more3 ? entry_of(it + 3 * stride) : 0;
            const int ph_new = more3 ? page_of(e_new & kTileMask) : 0;
            const bool own_rows = more && cached_u - (e_nxt & kTileMask) * kTile < kTile;
            if (own_rows) fetch(kBoth, kd, vd, e_nxt & kTileMask, ph_nxt);
            if (more) {
                store_staged(kd, staged_k);
                store_staged(vd, staged_v);
            }
            if (more2) {
                fetch_codes(kOnlyK, staged_k, e_nx2 & kTileMask, ph_nx2);
                fetch_codes(kOnlyV, staged_v, e_nx2 & kTileMask, ph_nx2);
            }
            if (keeps(it, e)) {
                float16_t s[2];
                scores(s, ks, (e & kTileMask) == iq);
                weights_and_values(s, vs);
            }
            e_cur = e_nxt;
            e_nxt = e_nx2;
            e_nx2 = e_new;
            ph_nxt = ph_nx2;
            ph_nx2 = ph_new;
            if (own_rows) dma_wait();
        } else {
            const int e_new = it + 2 * stride < n_visit ? entry_of(it + 2 * stride) : 0;  // requested two steps ahead of its use
            const int ph_new = it + 2 * stride < n_visit ? page_of(e_new & kTileMask) : 0;
            if (more) fetch(kBoth, kd, vd, e_nxt & kTileMask, ph_nxt);
            ph_nxt = ph_new;
            e_cur = e_nxt;
            e_nxt = e_new;
            if (keeps(it, e)) {
                float16_t s[2];
                scores(s, ks, (e & kTileMask) == iq);
                weights_and_values(s, vs);
            }
            dma_wait();
        }
        __syncthreads();  // the next tiles have landed and these are free
    };

    if (it_first < n_visit) {
        store_staged(k_lds0, staged_k);
        store_staged(v_lds0, staged_v);
    }
    dma_wait();
    if (QUANT && it_first + stride < n_visit) {  // past the wait: these codes have the first step to arrive
        fetch_codes(kOnlyK, staged_k, e_nxt & kTileMask, ph_nxt);
        fetch_codes(kOnlyV, staged_v, e_nxt & kTileMask, ph_nxt);
    }
    __syncthreads();
    if constexpr (!kOneStage) {
        for (int st = 0; st < steps; st += 2) {
            tile_step(it_first + st * stride, k_lds0, v_lds0, k_lds1, v_lds1);
            if (st + 1 >= steps) break;
            tile_step(it_first + (st + 1) * stride, k_lds1, v_lds1, k_lds0, v_lds0);
        }
    } else {
        if (it_first < n_visit) fetch(kOnlyV, k_lds0, v_lds0, e_cur & kTileMask, ph_first);  // the queries have left its place
        // K of the next step is requested once every wave has its scores of this one, V once every wave is done with it
        for (int st = 0; st < steps; ++st) {
            const int it = it_first + st * stride;
            const bool more = it + stride < n_visit;
            const int e_new = it + 2 * stride < n_visit ? entry_of(it + 2 * stride) : 0;
            const int ph_new = it + 2 * stride < n_visit ? page_of(e_new & kTileMask) : 0;
            const bool keep = keeps(it, e_cur);
            float16_t s[2];
            if (keep) scores(s, k_lds0, (e_cur & kTileMask) == iq);
            dma_wait();
            __syncthreads();  // V of this step has landed, K is free
            if (more) fetch(kOnlyK, k_lds0, v_lds0, e_nxt & kTileMask, ph_nxt);
            if (keep) weights_and_values(s, v_lds0);
            dma_wait();
            __syncthreads();  // K of the next step has landed, V is free
            if (more) fetch(kOnlyV, k_lds0, v_lds0, e_nxt & kTileMask, ph_nxt);
            ph_nxt = ph_new;
            e_cur = e_nxt;
            e_nxt = e_new;
        }
    }

    if (CUT) slot = __builtin_amdgcn_readfirstlane(slot);
    // ---- epilogue: lane (n, half) holds O^T[d][q] for d = 32 db + 8 (i / 4) + 4 half + i % 4
    const float lt = l_run;
    m_run *= lp.sm_scale_log2;
    const int pos = iq * kTile + row0 + n;
    const int row = pos - first;
    if (CUT && slot >= 0) {  // a piece: as the lanes hold it, 1 KiB at a time
        if (!wave_has_rows) return;
        float4* dst = reinterpret_cast<float4*>(sched.pieces.partials + (size_t)slot * kPieceFloats) + wave * (kPieceFloats / 4 / kPrefillWaves);
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                dst[(db * 4 + g4) * kWave + lane] =
                    make_float4(acc[db][4 * g4], acc[db][4 * g4 + 1], acc[db][4 * g4 + 2], acc[db][4 * g4 + 3]);
        if (half == 0) reinterpret_cast<float2*>(dst + 16 * kWave)[n] = make_float2(m_run, lt);
        return;
    }
    if (!fold) {
        if (!wave_has_rows) return;
        const float inv = lt > 0.f ? 1.f / lt : 0.f;  // a row that keeps nothing (possible with a listed mask) gives 0
        // The rows go out through LDS (the tiles are done with: the loop ended on a barrier), 8 KiB to a wave, chunks permuted as in a K
        // tile, so that sixteen lanes store a row.  As the lanes hold them, 16 bytes of 32 rows to an instruction, the stores of a
        // workgroup kept the address path, which also brings in the tiles of the compute unit's other workgroup, busy for 1 us: 16
        // prompts of 77 .. 3001 tokens 191 -> 177 us, of 123 14.8 -> 12.9, ten of 105, 32 / 16 heads, 12.2 -> 9.8.
        constexpr int kRowsBytes = 32 * kHeadDim * 2, kPerArray = SL * kKTileBytes / kRowsBytes;
        unsigned char* const arrays[4] = {k_lds0, v_lds0, k_lds1, v_lds1};
        static_assert(kWaves <= (kOneStage ? 2 : 4) * kPerArray, "room for the rows of every wave");
        unsigned char* room = arrays[0];
#pragma unroll
        for (int i = 1; i < ceil_div(kWaves, kPerArray); ++i)
            if (wave / kPerArray == i) room = arrays[i];
        room += wave % kPerArray * kRowsBytes;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                uint2 w;
                w.x = Elem<T>::pack(acc[db][4 * g4] * inv, acc[db][4 * g4 + 1] * inv);
                w.y = Elem<T>::pack(acc[db][4 * g4 + 2] * inv, acc[db][4 * g4 + 3] * inv);
                *reinterpret_cast<uint2*>(room + n * kKRowBytes + k_chunk_pos(n, db * 4 + g4) * 16 + 8 * half) = w;
            }
        asm volatile("" ::: "memory");  // LDS serves a wave in order, if the compiler asks in order
        const int r4 = lane / 16, pos4 = pos - n + r4;  // of the first of the lane's rows, four apart
        uint16_t* dst = out + ((size_t)(start + pos4 - first) * lp.H + h) * kHeadDim + lane % 16 * 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint4 w = *reinterpret_cast<const uint4*>(room + (4 * i + r4) * kKRowBytes + k_chunk_pos(4 * i + r4, lane % 16) * 16);
            if (pos4 + 4 * i < len && pos4 + 4 * i >= first)
                *reinterpret_cast<uint4*>(dst + (ptrdiff_t)(4 * i) * lp.H * kHeadDim) = w;
        }
        if (pos >= len || pos < first) return;
        if (lse_out && half == 0)
            lse_out[(size_t)h * total_tokens + start + row] = lt > 0.f ? (m_run + __builtin_amdgcn_logf(lt)) * kLn2 : -INFINITY;
    } else if constexpr (SL > 1) {
        // The slices of a unit meet in LDS (the tiles are done with: the loop ended on a barrier): every wave leaves
        // its accumulators, 4 KiB per channel block, and then finishes 4 / SL of the four channel blocks for its rows.
        float4* const room[4] = {reinterpret_cast<float4*>(k_lds0),
                                 reinterpret_cast<float4*>(kOneStage ? k_lds0 + kPrefillWaves * 4096 : k_lds1),
                                 reinterpret_cast<float4*>(v_lds0),
                                 reinterpret_cast<float4*>(kOneStage ? v_lds0 + kPrefillWaves * 4096 : v_lds1)};
        static_assert(SL == 1 || SL * kKTileBytes >= kPrefillWaves * 4096, "a channel block of every wave fits an array");
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                room[db][(wave * 4 + g4) * kWave + lane] =
                    make_float4(acc[db][4 * g4], acc[db][4 * g4 + 1], acc[db][4 * g4 + 2], acc[db][4 * g4 + 3]);
        if (half == 0) fold_ml[wave][n] = make_float2(m_run, lt);
        __syncthreads();
        if (!wave_has_rows) return;
        const int peer0 = unit * SL * 2 + wave % 2;  // wave of slice 0 with the same rows; slice i is 2 i waves on
        float2 ml[SL];
        float m_all = -INFINITY;
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            ml[i] = fold_ml[peer0 + 2 * i][n];
            m_all = fmaxf(m_all, ml[i].x);
        }
        float f[SL], l_all = 0.f;
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            f[i] = ml[i].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[i].x - m_all);  // a slice without keys adds nothing
            l_all = __builtin_fmaf(ml[i].y, f[i], l_all);
        }
        const float inv = l_all > 0.f ? 1.f / l_all : 0.f;
        // Finished rows, 64 bytes of a channel block, take the place of the first slice's contribution to the block and are stored
        // from there, four lanes to a row (only this wave reads what the slices left of this block for these rows).
        const int r4 = lane / 4, pos4 = pos - n + r4;
        uint16_t* dst = out + ((size_t)(start + pos4 - first) * lp.H + h) * kHeadDim + lane % 4 * 8;
#pragma unroll
        for (int u = 0; u < 4 / SL; ++u) {
            const int db = slice * (4 / SL) + u;
            float4* from = db == 0 ? room[0] : db == 1 ? room[1] : db == 2 ? room[2] : room[3];
            unsigned char* rows = reinterpret_cast<unsigned char*>(from + peer0 * 4 * kWave);
            uint2 done[4];
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < SL; ++i) {
                    const float4 x = from[((peer0 + 2 * i) * 4 + g4) * kWave + lane];
                    o[0] = __builtin_fmaf(x.x, f[i], o[0]);
                    o[1] = __builtin_fmaf(x.y, f[i], o[1]);
                    o[2] = __builtin_fmaf(x.z, f[i], o[2]);
                    o[3] = __builtin_fmaf(x.w, f[i], o[3]);
                }
                done[g4] = make_uint2(Elem<T>::pack(o[0] * inv, o[1] * inv), Elem<T>::pack(o[2] * inv, o[3] * inv));
            }
            asm volatile("" ::: "memory");
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                *reinterpret_cast<uint2*>(rows + n * 64 + (g4 ^ (n / 4 % 4)) * 16 + 8 * half) = done[g4];
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint4 w = *reinterpret_cast<const uint4*>(rows + (16 * i + r4) * 64 + (lane % 4 ^ (r4 / 4 % 4)) * 16);
                if (pos4 + 16 * i < len && pos4 + 16 * i >= first)
                    *reinterpret_cast<uint4*>(dst + (ptrdiff_t)(16 * i) * lp.H * kHeadDim + db * 32) = w;
            }
        }
        if (pos >= len || pos < first) return;
        if (lse_out && slice == 0 && half == 0)
            lse_out[(size_t)h * total_tokens + start + row] =
                l_all > 0.f ? (m_all + __builtin_amdgcn_logf(l_all)) * kLn2 : -INFINITY;
    }
}

template <class T, int MODE, int BITS, int SL>
__global__ __launch_bounds__(kPrefillThreads, 512 / kPrefillThreads) void sparse_prefill_kernel(
    LayerParams lp, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int* __restrict__ cu_seqlens, int batch, uint16_t* __restrict__ out,
    float* __restrict__ lse_out, int total_tokens, PrefillSchedule sched, PrefillMask mk, PrefillPaged pg) {
    prefill_workgroup<T, MODE, BITS, SL, kWhole>(lp, q, k, v, cu_seqlens, batch, out, lse_out, total_tokens, sched, mk, pg, blockIdx.x);
}
// (a kernel of its own: the search for a piece takes scalar registers from the walk, 2 to 5 % of a launch of whole walks)
template <class T, int BITS>
__global__ __launch_bounds__(kPrefillThreads, 512 / kPrefillThreads) void prefill_pieces_kernel(
    LayerParams lp, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int* __restrict__ cu_seqlens, int batch, uint16_t* __restrict__ out,
    float* __restrict__ lse_out, int total_tokens, PrefillSchedule sched, PrefillMask mk, PrefillPaged pg) {
    prefill_workgroup<T, kPaged, BITS, 1, kCut>(lp, q, k, v, cu_seqlens, batch, out, lse_out, total_tokens, sched, mk, pg, blockIdx.x);
}

// Half workgroups: one does not have a compute unit to itself, so that its start and end, 5 us in which nothing else of it is under
// way, and the time its wavefronts wait for each other at the end of a step go to the other's steps; short walks gain most, and
// where heads of a group keep different tiles (listed masks) two share a walk more often than four.  It stages every tile for half
// as many rows, which long walks pay for (see halves_are_quicker).  Whole and half, us: ten prompts of 327 tokens, 32 / 32 heads, 40.6 and 31.8; 13 of 215, 64 / 8,
// 42.0 and 35.6; one of 4096, 32 / 8, 117 and 111; two of 1024 34.1 and 30.8; 65536, 15500 and 16070.
template <class T, int MODE>
__global__ __launch_bounds__(kPrefillThreads / 2, 2) void prefill_half_kernel(
    LayerParams lp, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int* __restrict__ cu_seqlens, int batch, uint16_t* __restrict__ out,
    float* __restrict__ lse_out, int total_tokens, PrefillSchedule sched, PrefillMask mk, PrefillPaged pg) {
    prefill_workgroup<T, MODE, 16, 1, kHalf>(lp, q, k, v, cu_seqlens, batch, out, lse_out, total_tokens, sched, mk, pg, blockIdx.x);
}

// (a kernel of its own: the choice in every tile, or merely other code in front of the loop, moves the others by 1 to 3 %)
template <class T>
__global__ __launch_bounds__(kPrefillThreads / 2, 2) void prefill_hasty_kernel(
    LayerParams lp, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int* __restrict__ cu_seqlens, int batch, uint16_t* __restrict__ out,
    float* __restrict__ lse_out, int total_tokens, PrefillSchedule sched, PrefillMask mk, PrefillPaged pg) {
    prefill_workgroup<T, kPlain, 16, 1, kHasty>(lp, q, k, v, cu_seqlens, batch, out, lse_out, total_tokens, sched, mk, pg, blockIdx.x);
}

// Puts the pieces of cut walks together: four wavefronts per block and wavefront of its workgroups, one per 32
// channels, which reads 4 KiB of every piece, kBatch pieces at a time.
template <class T>
__device__ __forceinline__ void fold_block(const LayerParams& lp, const BlockOrder& order, const int* __restrict__ cu_seqlens,
                                           const int* __restrict__ seq_lens, int alongside, uint16_t* __restrict__ out,
                                           float* __restrict__ lse_out, int total_tokens, const PrefillSchedule& sched, int wave, int rank, int hidx, int hg, int thread,
                                           unsigned char (&rows)[4][32 * 64]) {
    constexpr int kBatch = 8;
    const HeadClass& hc = sched.cls[0];
    const int hk = (int)(hc.kv_head[hidx / 4] >> (8 * (hidx % 4))) & 0xff;
    const PiecePlan plan = PiecePlan::make(order, sched.pieces, kLeastSpanTiles >> hc.qtiles_log2);
    int b, qblk;
    if (plan.total == 0 || !order.find(rank, b, qblk)) return;
    const int pieces = __builtin_amdgcn_readfirstlane(plan.pieces_of(qblk));
    if (pieces == 1) return;
    const int start = cu_seqlens[b], fresh = cu_seqlens[b + 1] - start;
    const int len = seq_lens[b] + (alongside ? fresh : 0), first = len - fresh;
    const int lane = threadIdx.x % kWave, n = lane % 32, half = lane / 32;
    const int db = __builtin_amdgcn_readfirstlane(thread / kWave);
    const int unit = wave / 2;
    const int h = hk * lp.group + hg * hc.heads_per_block + (unit >> hc.qtiles_log2);
    const int pos = ((qblk << hc.qtiles_log2) + (unit & ((1 << hc.qtiles_log2) - 1))) * kTile + wave % 2 * 32 + n;
    if (pos - n >= len || pos - n + 32 <= first) return;

    const float4* base = reinterpret_cast<const float4*>(sched.pieces.partials) + wave * (kPieceFloats / 4 / kPrefillWaves);
    const size_t slot0 = (size_t)(hidx * (lp.group / hc.heads_per_block) + hg) * sched.pieces.target + rank;
    float m = -INFINITY, l = 0.f, o[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) o[i] = 0.f;
    int before = 0;  // pieces with smaller numbers
    for (int p = 0; p < pieces; p += kBatch) {
        float2 ml[kBatch];
        float4 x[kBatch][4];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const float4* src = base + (slot0 + before) * (kPieceFloats / 4);
            ml[u] = reinterpret_cast<const float2*>(src + 16 * kWave)[n];
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) x[u][g4] = src[(db * 4 + g4) * kWave + lane];
            if (p + u + 1 < pieces) before += order.at_or_past(plan.level(p + u));  // past the end: the last piece again, unused
        }
        float m_new = m;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) m_new = fmaxf(m_new, p + u < pieces ? ml[u].x : -INFINITY);
        const float m_safe = m_new == -INFINITY ? 0.f : m_new;
        const float keep = __builtin_amdgcn_exp2f(m - m_safe);
        l *= keep;
#pragma unroll
        for (int i = 0; i < 16; ++i) o[i] *= keep;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (p + u >= pieces) break;
            const float f = __builtin_amdgcn_exp2f(ml[u].x - m_safe);
            l = __builtin_fmaf(ml[u].y, f, l);
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                o[4 * g4] = __builtin_fmaf(x[u][g4].x, f, o[4 * g4]);
                o[4 * g4 + 1] = __builtin_fmaf(x[u][g4].y, f, o[4 * g4 + 1]);
                o[4 * g4 + 2] = __builtin_fmaf(x[u][g4].z, f, o[4 * g4 + 2]);
                o[4 * g4 + 3] = __builtin_fmaf(x[u][g4].w, f, o[4 * g4 + 3]);
            }
        }
        m = m_new;
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    // 64 bytes of each row, stored by four lanes each
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4)
        *reinterpret_cast<uint2*>(rows[db] + n * 64 + (g4 ^ (n / 4 % 4)) * 16 + 8 * half) =
            make_uint2(Elem<T>::pack(o[4 * g4] * inv, o[4 * g4 + 1] * inv), Elem<T>::pack(o[4 * g4 + 2] * inv, o[4 * g4 + 3] * inv));
    asm volatile("" ::: "memory");
    const int r4 = lane / 4, pos4 = pos - n + r4;
    uint16_t* dst = out + ((size_t)(start + pos4 - first) * lp.H + h) * kHeadDim + db * 32 + lane % 4 * 8;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint4 w = *reinterpret_cast<const uint4*>(rows[db] + (16 * i + r4) * 64 + (lane % 4 ^ (r4 / 4 % 4)) * 16);
        if (pos4 + 16 * i < len && pos4 + 16 * i >= first)
            *reinterpret_cast<uint4*>(dst + (ptrdiff_t)(16 * i) * lp.H * kHeadDim) = w;
    }
    if (pos >= len || pos < first) return;
    const int row = pos - first;
    if (lse_out && db == 0 && half == 0)
        lse_out[(size_t)h * total_tokens + start + row] = l > 0.f ? (m + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY;
}

template <class T>
__global__ __launch_bounds__(256) void fold_pieces_kernel(LayerParams lp, const int* __restrict__ cu_seqlens, const int* __restrict__ seq_lens,
                                                          int alongside, int batch, uint16_t* __restrict__ out, float* __restrict__ lse_out,
                                                          int total_tokens, PrefillSchedule sched) {
    __shared__ __attribute__((aligned(16))) unsigned char rows[4][32 * 64];
    const BlockOrder order = block_order(cu_seqlens, seq_lens, alongside, batch, kTileLog2 + sched.cls[0].qtiles_log2);
    fold_block<T>(lp, order, cu_seqlens, seq_lens, alongside, out, lse_out, total_tokens, sched, blockIdx.x % kPrefillWaves,
                  blockIdx.x / kPrefillWaves, blockIdx.y, blockIdx.z, threadIdx.x, rows);
}

// The same next to the streaming heads of the call, where these are not in the launch of the pieces (see streams_apart): neither
// fills the chip, and both are mostly latency.  First the workgroups of the streaming heads, `uncut` deals them out, then those that fold, two
// of fold_block's side by side.  Two launches of 13 and 11 us were 10 us longer: 512 tokens over 32768
// 154 -> 144 us, 128 over 20000 of 8 bits 78 -> 71.
//
// Pieces are chosen for histories that the page table has room for, and a table may be far wider than its sequences.  Where these are short
// (PrefillPieces::short_blocks), the launch of the pieces ends at once and the workgroups that would fold walk the dense heads, as the
// call without scratch does.
template <class T, int BITS, int SL>
__global__ __launch_bounds__(kPrefillThreads, 512 / kPrefillThreads) void fold_and_streams_kernel(
    LayerParams lp, const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int* __restrict__ cu_seqlens, int batch, uint16_t* __restrict__ out, float* __restrict__ lse_out, int total_tokens,
    PrefillSchedule uncut, PrefillMask mk, PrefillPaged pg, PrefillSchedule sched) {
    const int dense = kXcds * uncut.cls[0].items_per_xcd, i = blockIdx.x - kXcds * uncut.cls[1].items_per_xcd;
    BlockOrder order;
    if (i >= 0) order = block_order(cu_seqlens, pg.kv.seq_lens, pg.k_new != nullptr, batch, kTileLog2 + sched.cls[0].qtiles_log2);
    if (i < 0 || order.top() <= sched.pieces.short_blocks) {
        if (i >= dense) return;
        prefill_workgroup<T, kPaged, BITS, SL, kWhole>(lp, q, k, v, cu_seqlens, batch, out, lse_out, total_tokens, uncut, mk, pg,
                                                       i < 0 ? (int)blockIdx.x + dense : i);
        return;
    }
    __shared__ __attribute__((aligned(16))) unsigned char rows[2][4][32 * 64];
    constexpr int kPerBlock = kPrefillWaves / 2;
    const int side = __builtin_amdgcn_readfirstlane(threadIdx.x / 256), of_head = sched.cls[0].blocks * kPerBlock;
    const int at = i % of_head, head = i / of_head, hg = head / sched.cls[0].heads;
    if (hg * sched.cls[0].heads_per_block >= lp.group) return;
    fold_block<T>(lp, order, cu_seqlens, pg.kv.seq_lens, pg.k_new != nullptr, out, lse_out, total_tokens, sched, at % kPerBlock * 2 + side,
                  at / kPerBlock, head % sched.cls[0].heads, hg, threadIdx.x % 256, rows[side]);
}

// ---- quantised history as 16-bit pages ------------------------------------------------------------
//
// A chunk of many rows has every tile of a quantised history dequantised by every workgroup that walks it, next to the softmax
// in the vector pipe: a step takes 2.21 us where 16-bit pages take 1.75.  With scratch for it the history is dequantised once,
// into pages of the layer's type, and the chunk then walks those: the same values, rounded the same way.  Two chunks of 1500 and
// 2048 tokens over 24001 of 8 bits, 32 / 8 heads: 949 -> 849 us, 27 of them for 98 MB of pages; 859 over 8966, five times, 64 / 8
// heads: 672 -> 573; 1392 over 1055 of 4 bits, twice: 93 -> 83.
struct ExpandedPages {
    uint16_t *k, *v;            // [batch][max_pages][dense heads][64][D]
    uint16_t *k_ring, *v_ring;  // [batch][ring][streaming heads][64][D]: sink and local pages
    int *table, *ring_table;    // page and slot numbers of the above
};

// One workgroup per KV head, sequence and share of its pages; bound by memory (a slab of 8192 codes is 8.5 KB to read and 16 KB to
// write).  Sequences without new tokens are left alone: nobody reads their pages, and their tables need not lead anywhere.
template <class T, int BITS>
__global__ __launch_bounds__(256) void expand_pages_kernel(LayerParams lp, PagedParams kv, const int* __restrict__ cu_new, ExpandedPages to) {
    if (cu_new[blockIdx.z + 1] <= cu_new[blockIdx.z]) return;
    const int hk = blockIdx.y, b = blockIdx.z, cached = kv.seq_lens[b], pages = ceil_div(cached, kTile);
    const bool streaming = (lp.streaming_mask >> hk) & 1ull, ring = in_stream_pool(lp, kv, hk);
    const int heads = streaming ? kv.stream_heads : lp.Hkv - kv.stream_heads;
    const unsigned long long below = (1ull << hk) - 1ull;
    const int rank = __popcll((streaming ? lp.streaming_mask : ~lp.streaming_mask) & below);
    constexpr size_t kSlab = slab_chunks(kTile, BITS) * 16;
    constexpr int kRowBytes = kHeadDim * BITS / 8;
    const size_t page_bytes = (ring ? kv.stream_heads : kv.pool_heads) * kSlab, slab_in_page = pool_rank(lp, kv, hk, ring) * kSlab;
    // pages a query of the chunk can reach: all, or the sink pages and the last local ones
    const int first_local = streaming ? max(lp.sink_pages, pages - lp.local_pages) : 0;
    const int sinks = streaming ? min(lp.sink_pages, pages) : 0, count = sinks + max(0, pages - first_local);
    for (int i = blockIdx.x; i < count; i += gridDim.x) {
        const int p = i < sinks ? i : first_local + i - sinks;
        const int slot = streaming ? b * kv.ring + ring_slot(lp, p) : b * kv.max_pages + p;
        const int from = ring ? kv.ring_table[(size_t)b * kv.ring + ring_slot(lp, p)] : kv.page_table[(size_t)b * kv.max_pages + p];
        if (threadIdx.x == 0 && rank == 0) {
            if (streaming)
                to.ring_table[slot] = slot;
            else
                to.table[slot] = slot;
        }
        const int chunk = threadIdx.x % 16, row0 = threadIdx.x / 16;
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const unsigned char* pool = reinterpret_cast<const unsigned char*>(side ? (ring ? kv.v_stream : kv.v_pool) : (ring ? kv.k_stream : kv.k_pool));
            const unsigned char* slab = pool + (size_t)from * page_bytes + slab_in_page;
            uint16_t* dst = (side ? (streaming ? to.v_ring : to.v) : (streaming ? to.k_ring : to.k)) + ((size_t)slot * heads + rank) * kTile * kHeadDim;
            uint2 codes[4];
            uint32_t sz[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int row = row0 + 16 * u;
                const unsigned char* src = slab + row * kRowBytes + chunk * BITS;
                if constexpr (BITS == 8)
                    codes[u] = *reinterpret_cast<const uint2*>(src);
                else
                    codes[u] = make_uint2(*reinterpret_cast<const uint32_t*>(src), 0u);
                sz[u] = reinterpret_cast<const uint32_t*>(slab + kTile * kRowBytes)[row];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)  // (rows past the end of the cache may hold anything: nobody reads them)
                *reinterpret_cast<uint4*>(dst + (row0 + 16 * u) * kHeadDim + chunk * 8) = dequantise8<T, BITS>(codes[u], sz[u]);
        }
    }
}

// ---- host side -----------------------------------------------------------------------------------

int count_streaming(const LayerParams& lp) {
    int n = 0;
    for (int hk = 0; hk < lp.Hkv; ++hk) n += (int)((lp.streaming_mask >> hk) & 1ull);
    return n;
}

// What a launch is made of: the kernel's key slices, per class of heads whether the slices share a unit, and whether the
// units of a workgroup are query tiles of one head instead of heads of a group.
struct PrefillShape {
    int slices;
    bool fold[2];
    bool one_head;
    bool half;   // workgroups of two units, two to a compute unit
    int pieces;  // of dense walks per (KV head, group of query heads), at most (PrefillPieces::target); 0: whole walks
    int least;   // of a block (PrefillPieces::least)
};

// The queries of a launch as far as the host knows them.
struct PrefillRows {
    int batch, total, longest;
    int history_pages;  // bound of the key tiles in front of them, of every sequence; -1: none (a prompt)
};

// Key ranges, each with a maximum of its own, in which the sums of a row are taken.
int slices_of(const PrefillShape& shape, int cls) { return shape.fold[cls] ? shape.slices : 1; }

int units_of(const PrefillShape& shape, int cls) {
    return shape.half ? kPairs / 2 : shape.fold[cls] ? kPairs / shape.slices : kPairs;
}
// Query heads of a group that share a workgroup: they read the same keys, whole and at the same time, and all end on the
// same diagonal tile, where query tiles side by side would not.  Query tiles make up the rest of the units.
int heads_per_block(const LayerParams& lp, const PrefillShape& shape, int cls) {
    int heads = 1;
    while (!shape.one_head && heads < units_of(shape, cls) && lp.group % (2 * heads) == 0) heads *= 2;
    return heads;
}

// (The constants from here on were fitted to a loop with a running maximum and to rows stored as the lanes hold them.  Since then steps are 4
// to 7 % shorter and starts and ends by up to a third, which these estimates weigh against each other: launches are 4 to 17 % shorter, those of
// many starts by most.  The constants have not been fitted again; over 900 chunks behind tables 1 to 32 times as wide as needed the estimates are
// now 1.01 to 1.04 of the time of whole walks and 1.00 to 1.06 of that of pieces, by geometric mean.)
//
// The estimate behind the choice of a shape: a compute unit holds one workgroup at a time, an XCD deals its workgroups out
// longest walk first, and a workgroup costs a fixed time and its steps.  Constants in microseconds, fitted to 2100 launches
// (211 chunks and 90 prompts of 1 .. 24 sequences in every shape; two thirds of the estimates are within 9 %):
// a step of 64 keys with one / two / four slices takes 1.75 / 2.16 / 2.91, 2.21 / 2.85 over quantised pages (not built for
// four: the codes on their way need more registers than there are); with most wavefronts without rows 22 % less.
constexpr int kMostPieces = 4096;  // per (KV head, group of query heads)
constexpr float kStepUs[2][3] = {{1.75f, 2.16f, 2.91f}, {2.21f, 2.85f, 2.85f}};
constexpr float kStepWithoutRows = 0.78f;
constexpr float kStartUs[2] = {5.2f, 5.8f}, kStartOfSlices[3] = {0.f, 0.5f, 0.55f}, kFoldUs = 0.44f, kLaunchUs = 2.2f;
// past the even share of the work: a part of the last streaming walk, or of the longest dense one
constexpr float kTailOfStream = 0.55f, kTailOfDense = 0.14f;

// Blocks less or more than the mean, where their number is an estimate.
float spread_of(const PrefillRows& rows) { return 0.4f * std::sqrt((float)rows.batch); }

// One class of heads of a launch: workgroups per XCD and what they cost.
struct ClassCost {
    float count, start, step;  // step: of a workgroup's own share of the keys
    int qtiles;
};

// Smallest whole number not below x >= 0.
float whole(float x) {
    const float i = (float)(int)x;
    return i < x ? i + 1.f : i;
}

// side: -1 / 1 for a few blocks less / more than the mean where their number is an estimate, 0 where it is known.
ClassCost class_cost(const LayerParams& lp, const PrefillShape& shape, const PrefillRows& rows, int cls, int heads, bool quant,
                     int side, float spread) {
    ClassCost c = {};
    if (heads == 0) return c;
    const int per_block = heads_per_block(lp, shape, cls);
    c.qtiles = units_of(shape, cls) / per_block;
    const int block = kTile * c.qtiles, log2_slices = shape.slices == 4 ? 2 : shape.slices == 2 ? 1 : 0;
    const float n = (float)rows.batch;
    const bool alike = (long long)rows.batch * rows.longest == rows.total;
    float blocks;
    if (rows.history_pages < 0 ? alike : alike && side < 0 && rows.longest % kTile == 0)
        blocks = n * (float)((rows.longest + block - 1) / block);  // chunks of whole tiles mostly follow others
    else if (rows.history_pages >= 0)  // rows that start anywhere inside a block touch (rows - 1) / block + 1 blocks on average
        blocks = std::max(std::max(n, (float)rows.total / block), (float)(rows.total - rows.batch) / block + n + side * spread);
    else
        blocks = std::max(n, (float)rows.total / block + 0.5f * n + side * spread);
    const int n_per_block = lp.group / per_block;
    c.count = kXcds % heads == 0 ? n_per_block * whole(blocks * heads / kXcds - 1e-4f)
                                 : whole(heads * n_per_block * blocks / kXcds - 1e-4f);
    const float halves = ((float)rows.total + 31.f * n) / 32.f;  // halves of tiles with rows
    const float active = std::min(1.f, halves / (blocks * c.qtiles * 2));
    c.step = kStepUs[quant][log2_slices] * (kStepWithoutRows + (1.f - kStepWithoutRows) * active) / (shape.fold[cls] ? shape.slices : 1);
    c.start = kStartUs[quant] + kStartOfSlices[log2_slices] + (shape.fold[cls] ? kFoldUs : 0.f);
    return c;
}

// Time until the last of n workgroups is through, n dealt out to m units longest first, their times falling evenly from
// `longest` to `shortest`: the unit that ends a round first takes the longest of the next, so every two rounds are even.
float rounds_time(float n, float longest, float shortest, int m) {
    const float fall = (longest - shortest) / std::max(1.f, n - 1.f);
    auto of = [&](float k) { return longest - fall * std::min(k, n - 1.f); };
    const int pairs = (int)(n / (2 * m));
    float t = 0.f;
    if (pairs > 8)
        t = pairs * (longest + shortest);
    else
        for (int i = 0; i < pairs; ++i) t += of(2.f * m * i) + of(2.f * m * i + 2 * m - 1);
    const float done = 2.f * m * pairs, left = n - done;
    if (left < 0.5f) return t;
    return t + (left <= m ? of(done) : std::max(of(done), of(done + m - 1) + of(done + m)));
}

// Key tiles of the walks of one class of heads, and a workgroup's times for them.
struct ClassWalks {
    float hi, lo, mid;
    float longest, shortest, mean;
};
ClassWalks class_walks(const LayerParams& lp, const PrefillRows& rows, float history, const ClassCost& c, int cls) {
    const float longest_tiles = (float)rows.longest / kTile, mean_tiles = (float)rows.total / rows.batch / kTile;
    const float other = rows.batch > 1 ? (float)(rows.total - rows.longest) / (rows.batch - 1) / kTile : longest_tiles;
    ClassWalks w = {};
    if (c.count == 0.f) return w;
    const float qt = (float)c.qtiles;
    if (rows.history_pages >= 0) {
        w.hi = history + longest_tiles + 0.5f;
        w.lo = history + std::min(qt, other + 0.5f);
        w.mid = history + 0.25f * (longest_tiles + mean_tiles) + 0.5f * std::min(qt, longest_tiles);
    } else {
        w.hi = whole(longest_tiles);
        w.lo = std::min(qt, w.hi);
        w.mid = 0.25f * (longest_tiles + mean_tiles) + 0.5f * std::min(qt, other + 0.5f);
    }
    if (cls == 1) {
        const float band = (float)(lp.sink_pages + lp.local_pages) + qt - 1.f;
        w.hi = std::min(w.hi, band);
        w.lo = std::min(w.lo, band);
    }
    w.mid = std::min(w.hi, std::max(w.lo, w.mid));
    w.longest = c.start + c.step * w.hi;
    w.shortest = c.start + c.step * w.lo;
    w.mean = c.start + c.step * w.mid;
    return w;
}

// Estimated time of a launch whose history is `history` key tiles long.
float launch_time(const LayerParams& lp, const PrefillRows& rows, float history, const ClassCost (&c)[2], int units_per_xcd) {
    const ClassWalks w[2] = {class_walks(lp, rows, history, c[0], 0), class_walks(lp, rows, history, c[1], 1)};
    float t = w[1].longest;
    if (c[0].count > 0.f) t = std::max(t, rounds_time(c[0].count, w[0].longest, w[0].shortest, units_per_xcd));
    if (c[0].count + c[1].count > units_per_xcd) {
        const float even = (c[0].count * w[0].mean + c[1].count * w[1].mean) / units_per_xcd;
        t = std::max(t, even + std::max(kTailOfStream * w[1].longest, kTailOfDense * w[0].longest));
    }
    return t + kLaunchUs;
}

// The same with dense walks in up to `pieces` pieces per XCD (see PiecePlan): the time of a piece beside its steps, of
// putting pieces together, and of a step where every compute unit is at work on keys of its own: fitted to 95 drawn chunks with
// streaming heads in the launch.  kStreamsBeside: what streaming heads in the launch that puts pieces together add, as a part of the
// estimate for a launch of theirs, fitted to 152 chunks over 300 .. 131000 tokens of history (130 of them drawn), measured whole and in one to
// four rounds of pieces, behind tables of their length and of eight times as much: the shapes taken cost 4 % over the best ones on average.
// In a launch of its own, which cost 13 us, 9 %: histories of less than some 10000 tokens stayed whole (31 tokens over 5931 of 4 bits, three times, 128 us
// whole and 56 in pieces; 219 over 6972 of 8, twice, 157 and 78; 256 over 20000, four times, 289 and 205).
constexpr float kPieceUs = 0.5f, kFoldLaunchUs = 1.f, kFoldPieceUs = 0.15f, kCutStep = 1.07f, kStreamsBeside = 0.7f;
float cut_launch_time(const LayerParams& lp, const PrefillRows& rows, float history, const ClassCost (&c)[2], int units_per_xcd,
                      float pieces, int least, bool streams_apart) {
    const ClassWalks w[2] = {class_walks(lp, rows, history, c[0], 0), class_walks(lp, rows, history, c[1], 1)};
    const float work = c[0].count * w[0].mid;
    const float alike = w[0].hi / std::max(1.f, (float)(int)(pieces / c[0].count)), apart = work / (pieces - 0.5f * c[0].count);
    const float span = std::min(w[0].hi, std::max((float)kLeastSpanTiles, std::max(apart, apart + (alike - apart) * w[0].lo / w[0].hi)));
    const float count = std::max(least * c[0].count, std::min(pieces, work / span + 0.5f * c[0].count));
    const float longest = c[0].start + kCutStep * c[0].step * span + kPieceUs;
    const float streams = streams_apart ? 0.f : c[1].count, last = streams_apart ? 0.f : w[1].longest;
    float t = std::max(longest, last);
    if (count + streams > units_per_xcd) {
        const float even = (count * (c[0].start + kPieceUs) + work * kCutStep * c[0].step + streams * w[1].mean) / units_per_xcd;
        t = std::max(t, even + std::max(kTailOfStream * last, 0.3f * longest));
    }
    if (streams_apart) t += kStreamsBeside * std::max(w[1].longest, c[1].count * w[1].mean / units_per_xcd);
    return t + kLaunchUs + kFoldLaunchUs + kFoldPieceUs * count;
}

// May it pay to cut the walks of these chunks into pieces?  A first look, for the host's time: not where the history is short
// or whole walks fill the chip.
bool may_cut(const LayerParams& lp, const PrefillRows& rows) {
    const int dense = lp.Hkv - count_streaming(lp);
    return dense > 0 && rows.batch <= kOrderedSeqs && rows.history_pages >= 3 * kLeastSpanTiles &&
           (long long)rows.total * dense * lp.group < (long long)num_compute_units() * kPairs * kTile;
}

// Where dense walks are cut, which is by workgroups of one slice, streaming heads keep the slices that the launch has with whole
// walks, next to the fold, in its launch, if these are several.  Each slice rounds its weights relative to a maximum of its own, so
// that many of the largest weights of a row are exact, which over the few keys of a streaming head tells: against 64 bits 2.78e-3
// with four slices and 2.84e-3 with one (512 tokens over 32768, bf16; dense heads 2.99e-3 whole in four slices and 2.97e-3 in pieces).
bool streams_apart(const LayerParams& lp, const PrefillShape& whole) { return whole.slices > 1 && lp.streaming_mask != 0; }

// Are half workgroups (see prefill_half_kernel) quicker than the whole ones of a shape of one slice?  (Not over quantised pages, which
// every workgroup dequantises for itself: half ones are twice as many.)  Measured over 1000 batches, half as a part of whole: 0.64 to
// 1.08 where a dense walk is up to 60 tiles long on average, 0.92 to 1.03 beyond; and up to 60 whole ones are as quick or quicker
// where (over prompts only but for the first, the second by tiles of one head, and the last)
//   - a dense walk is a single tile and whole workgroups have tiles of one head for units (1.02 to 1.16: 51 tokens, 32 / 16 heads, 6.3 and
//     7.2 us): most of the time is the way of that tile into LDS, on which a half workgroup has half the wavefronts;
//   - whole workgroups of four heads, or of four tiles of one, fill the chip just once with walks of some tiles (1.0 to 1.04: eight of
//     231, 32 / 8 heads, 17.1 and 17.4; 0.96 to 1.1: four of 385, 32 / 32, 20.4 and 22.4, four chunks of 165 over 173 15.8 and 17.6; with walks
//     of up to two tiles 0.87 to 0.95, of seven and more 0.80 to 0.98);
//   - those of four heads fill it twice with walks of two tiles (0.90 to 1.6: 16 of 128, 64 / 8 heads, 30 and 48, of 123 27.6 and 25.8);
//   - they fill it once and a half to twice without a streaming head, whose short walks would fill the gaps (0.98 to 1.06: two of 2000, 32 / 8
//     heads, 82.5 and 87.7);
//   - there are more dense KV heads than XCDs, each of which then works on several heads' keys at a time, in many rounds (0.98 to 1.28: 18 of
//     3001, 32 / 32 heads, 16 of them streaming 1352 and 1447, none 1880 and 2400; 64 of 500, none streaming, 370 and 401; 16 chunks of
//     1000 over 500, none streaming, 458 and 499).
// All of these times are from a loop with a running maximum and rows stored as the lanes hold them.  Steps, starts and ends are shorter
// now, starts and ends of half workgroups by most, and the lines have not been drawn again.  Over 3100 more batches, half as a part of whole: 0.89
// on average where half ones are taken (2 % slower or more in 41 of 2551); in the exceptions 0.96 for single tiles, 0.92 for one full round,
// 0.95 without a streaming head, 1.03 in many rounds of many heads; 0.98 beyond 60 tiles.  So whole ones are kept in the first three
// exceptions at a loss of 4 to 8 %, and in many rounds of many heads the line lies too far out (21 of 1888, 32 / 32 heads, 632 whole
// and 691 half).
bool halves_are_quicker(const LayerParams& lp, const PrefillRows& rows, const PrefillShape& whole) {
    const int n_stream = count_streaming(lp), heads[2] = {lp.Hkv - n_stream, n_stream};
    const PrefillShape half = {1, {false, false}, false, true, 0, 1};
    const int cls = heads[0] > 0 ? 0 : 1;  // (of the dense heads, if there are any)
    const ClassWalks walks =
        class_walks(lp, rows, (float)std::max(0, rows.history_pages), class_cost(lp, half, rows, cls, heads[cls], false, 0, 0.f), cls);
    if (walks.mid > 60.f) return false;
    const bool prompt = rows.history_pages < 0, fours = lp.group % 4 == 0, single = lp.group % 2 != 0;
    if (walks.hi <= 1.f && whole.one_head) return false;
    float rounds = 0.f;
    for (int c = 0; c < 2; ++c) rounds += class_cost(lp, whole, rows, c, heads[c], false, 0, 0.f).count;
    rounds /= std::max(1, num_compute_units() / kXcds);
    if (single && rounds > 0.8f && rounds <= 1.f && walks.mid >= 2.9f && walks.mid <= 6.5f) return false;
    const float together = heads[0] > kXcds ? rounds * (float)heads[0] : 0.f;
    if (!prompt) return together <= 280.f;
    if (fours && rounds > 0.875f && rounds <= 1.f && walks.mid >= 2.2f && walks.mid <= 6.f) return false;
    if (fours && rounds > 1.75f && rounds <= 2.f && walks.mid >= 1.4f && walks.hi <= 2.f) return false;
    if (n_stream == 0 && rounds > 1.4f && rounds <= 2.05f && walks.mid >= 12.f && walks.mid <= 32.f) return false;
    return together <= 256.f || (together <= 400.f && walks.mid <= 20.f);
}

// Key tiles of history up to which whole walks, after a launch of pieces that ends at once (4 to 6 us), are quicker than the pieces of
// `shape`, by these estimates.  Up to some kWholeUs only: in a longer call that launch is little, and a wrong estimate much (one call in 60
// was slower, by up to 1.7 times).  Measured, 900 chunks over 300 .. 131000 tokens that go in pieces, tables 1, 2, 4, 8 and 32 times as wide
// as needed, time as a part of whole walks', always in pieces and now: 0.33, 0.42, 0.495, 0.53, 0.64 and 0.33, 0.42, 0.49, 0.51, 0.59, at worst
// 2.2 and 1.4.  Seven of 2 to 17 tokens over 1214 of 8 bits, 64 / 8 heads, table eight times as wide: 78 and 62 us, whole 57.
float whole_walks_until(const LayerParams& lp, const PrefillRows& rows, bool quant, const PrefillShape& uncut, const PrefillShape& shape) {
    constexpr float kSkippedUs = 4.f, kCutShort = 1.1f, kWholeUs = 80.f;
    const int n_stream = count_streaming(lp), heads[2] = {lp.Hkv - n_stream, n_stream}, units_per_xcd = std::max(1, num_compute_units() / kXcds);
    const float spread = spread_of(rows), per_xcd = (float)(shape.pieces * heads[0] * (lp.group / heads_per_block(lp, shape, 0))) / kXcds;
    const ClassCost whole[2] = {class_cost(lp, uncut, rows, 0, heads[0], quant, 0, spread), class_cost(lp, uncut, rows, 1, heads[1], quant, 0, spread)};
    const ClassCost cut[2] = {class_cost(lp, shape, rows, 0, heads[0], quant, 0, spread), whole[1]};
    float until = 0.f;
    for (float history = 4.f; history <= (float)rows.history_pages; history *= 1.2f) {
        const float t = launch_time(lp, rows, history, whole, units_per_xcd);
        if (t > kWholeUs) break;
        if (t + kSkippedUs < kCutShort * cut_launch_time(lp, rows, history, cut, units_per_xcd, per_xcd, shape.least, true)) until = history;
    }
    return until;
}

constexpr float kWeight[4] = {4.f, 1.f, 1.f, 1.f};  // of the guesses

// The shape of a launch.  Measured with one / two / four slices: 512 new tokens over a history of 32768, 849 / 520 / 363 us;
// 2635 over 45405, 1229 / 1480 / 1513 us (one round of workgroups, or two of half the length at more per step); one prompt of
// 4096 tokens, 119 / 116 / 146 us; of 65536, 15.4 / 17.6 / 21.6 ms.  Heads or query tiles as units of one slice: 5 sequences of
// 7 .. 123 tokens, 12.4 and 9.3 us (fewer wavefronts at work on a compute unit); 8 of 100 .. 1500, 60 and 73 us.
// The history of a chunk is not known on the host.  It may be as long as the page table allows, which a caller that
// allocates what it needs sees to, or far shorter, in a table as wide as the longest context: the shape is the one that on
// average costs least over what it could have been for histories of that length (counted four times), a quarter, a
// sixteenth and a sixty-fourth of it (490 chunks: 1.5 % over the best shape with a tight table and 2.2 % with one 32 times as
// wide; by the length of the table alone 1.1 and 3.3 %, and up to half the speed lost).  Where the number of blocks is an
// estimate, near the end of a round of workgroups, so is the time: the mean of a few blocks less and a few more.
// cut: pieces too, so many that the workgroups of the launch are about one, two ... rounds of the chip.
// uncut: the shape of the same call without scratch.  Streaming heads keep it where dense walks are cut, and no row's sums are taken in
// fewer key ranges than there.
PrefillShape choose_shape(const LayerParams& lp, const PrefillRows& rows, bool quant, const PrefillShape* uncut = nullptr, bool cut = false,
                          bool halves = true, float* times = nullptr) {
    constexpr PrefillShape kShapes[] = {{1, {false, false}, false, false, 0, 1}, {1, {false, false}, true, false, 0, 1},
                                        {2, {true, true}, true, false, 0, 1},    {2, {true, true}, false, false, 0, 1},
                                        {2, {true, false}, false, false, 0, 1},  {4, {true, true}, false, false, 0, 1}};
    constexpr int kCount = (int)(sizeof(kShapes) / sizeof(kShapes[0])), kRounds = 4;
    const int n_stream = count_streaming(lp), heads[2] = {lp.Hkv - n_stream, n_stream};
    const int units_per_xcd = std::max(1, num_compute_units() / kXcds);
    const bool prompt = rows.history_pages < 0, exact = prompt && (long long)rows.batch * rows.longest == rows.total;
    // a walk of one or two tiles leaves nothing to share out; quantised pages are not built for four slices
    const int count = prompt && rows.longest <= 2 * kTile ? 2 : quant ? kCount - 1 : kCount;
    const int guesses = prompt ? 1 : 4;
    const float spread = spread_of(rows);
    // pieces per (KV head, group of query heads), and per XCD, of launches of one, two ... rounds (0: not to be had)
    int pieces[kRounds] = {};
    float per_xcd[kRounds] = {};
    const bool apart = cut && streams_apart(lp, *uncut);
    const int least = cut ? slices_of(*uncut, 0) : 1;
    if (cut) {
        const ClassCost dense = class_cost(lp, kShapes[0], rows, 0, heads[0], quant, 0, 0.f), stream = class_cost(lp, kShapes[0], rows, 1, heads[1], quant, -1, 0.f);
        const int per_block = lp.group / heads_per_block(lp, kShapes[0], 0), block = kTile * dense.qtiles;
        const long long blocks = least * std::min((long long)rows.batch * ((rows.longest + block - 1) / block + 1), (long long)rows.total / block + 2LL * rows.batch);
        for (int r = 0; r < kRounds; ++r) {
            const int room = (r + 1) * units_per_xcd - (apart ? 0 : (int)stream.count);
            const int n = kXcds % heads[0] == 0 ? room / per_block * (kXcds / heads[0]) : room * kXcds / (heads[0] * per_block);
            if (room <= 0 || n < blocks + blocks / 4 || n > kMostPieces) continue;
            pieces[r] = n;
            per_xcd[r] = (float)(n * heads[0] * per_block) / kXcds;
        }
    }
    auto allowed = [&](int i) {
        if (i >= kCount) return pieces[i - kCount] > 0;
        if (i >= count) return false;
        for (int c = 0; c < 2; ++c)
            if (uncut && heads[c] > 0 && slices_of(kShapes[i], c) < slices_of(*uncut, c)) return false;
        return true;
    };
    float time[kCount + kRounds][4] = {};
    for (int side = exact ? 0 : -1; side <= 1; side += 2) {
        for (int i = 0; i < kCount + kRounds; ++i) {
            if (i < kCount ? i >= count : pieces[i - kCount] == 0) continue;
            const PrefillShape& shape = kShapes[i < kCount ? i : 0];
            const ClassCost c[2] = {class_cost(lp, shape, rows, 0, heads[0], quant, exact ? 0 : side, spread),
                                    class_cost(lp, i >= kCount && apart ? *uncut : shape, rows, 1, heads[1], quant, exact ? 0 : side, spread)};
            float history = prompt ? 0.f : (float)rows.history_pages;
            for (int g = 0; g < guesses; ++g, history *= 0.25f)
                time[i][g] += i < kCount ? launch_time(lp, rows, history, c, units_per_xcd)
                                         : cut_launch_time(lp, rows, history, c, units_per_xcd, per_xcd[i - kCount], least, apart);
        }
    }
    int best = -1;
    float best_score = 0.f;
    for (int i = 0; i < kCount + kRounds; ++i) {
        if (!allowed(i)) continue;
        float score = 0.f;
        for (int g = 0; g < guesses; ++g) {
            float fastest = time[0][g];
            for (int k = 1; k < count; ++k) fastest = std::min(fastest, time[k][g]);
            score += kWeight[g] * time[i][g] / fastest;
        }
        if (best < 0 || score < best_score) best = i, best_score = score;
    }
    if (times)
        for (int g = 0; g < guesses; ++g) times[g] = time[best][g] / (exact ? 1 : 2);
    PrefillShape shape = kShapes[best < kCount ? best : 0];
    if (best >= kCount) {
        shape.pieces = pieces[best - kCount];
        shape.least = least;
    } else if (halves && shape.slices == 1 && !quant && halves_are_quicker(lp, rows, shape)) {
        // the same walks by half workgroups: the same sums in the same order, so the results are of the shape they were
        shape = {1, {false, false}, false, true, 0, 1};
    }
    return shape;
}

// Scratch of a launch in pieces.
size_t pieces_bytes(const LayerParams& lp, const PrefillShape& shape) {
    return (size_t)shape.pieces * (lp.Hkv - count_streaming(lp)) * (lp.group / heads_per_block(lp, shape, 0)) * kPieceFloats * sizeof(float);
}

// Rows of a chunk in front of which up to `pages` pages of keys may lie, its own among them.
PrefillRows chunk_rows(int batch, int total_new, int max_new_per_seq, int pages) {
    return {batch, total_new, max_new_per_seq, std::max(0, pages - max_new_per_seq / kTile)};
}

// Bytes of ExpandedPages, each array on a multiple of 256.
constexpr size_t kMostExpanded = (size_t)1 << 30;
size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
struct ExpandedSizes {
    size_t pool, ring, table, ring_table;
    size_t all() const { return 2 * pool + 2 * ring + table + ring_table; }
};
ExpandedSizes expanded_sizes(const LayerParams& lp, int batch, int max_pages) {
    const size_t slab = (size_t)kTile * kHeadDim * 2, n_stream = count_streaming(lp), ring = lp.sink_pages + lp.local_pages;
    return {align256((size_t)batch * max_pages * (lp.Hkv - n_stream) * slab), align256((size_t)batch * ring * n_stream * slab),
            align256((size_t)batch * max_pages * sizeof(int)), align256((size_t)batch * ring * sizeof(int))};
}

// How a launch over pages goes about its work, and the scratch it takes.
struct ChunkPlan {
    bool expand;  // quantised pages are turned into 16-bit ones first
    PrefillShape shape;
    size_t bytes;
    PrefillShape uncut;  // without scratch; also of the streaming heads, if dense walks are cut
};
// width: of the page table (and of the table of the expanded pages).
ChunkPlan plan_chunk(const LayerParams& lp, const PrefillRows& rows, int width, bool quant, bool scratch) {
    const PrefillShape uncut = choose_shape(lp, rows, quant);
    if (!scratch) return {false, uncut, 0, uncut};
    const bool cut = may_cut(lp, rows);
    const int dense = lp.Hkv - count_streaming(lp);
    // Dequantising once takes the whole chip 13 ns a tile and head, doing it in the walk 1.8 ns a workgroup of it: eight workgroups.
    const bool many = quant && dense > 0 && rows.history_pages >= 2 * kLeastSpanTiles && (long long)rows.total * lp.group >= 8LL * kPairs * kTile * rows.batch &&
                      expanded_sizes(lp, rows.batch, width).all() <= kMostExpanded;
    if (!cut && !many) return {false, uncut, 0, uncut};
    float times[2][4];
    const PrefillShape as_is = choose_shape(lp, rows, quant, &uncut, cut, true, times[0]);
    const ChunkPlan plan = {false, as_is, pieces_bytes(lp, as_is), uncut};
    if (!many) return plan;
    const PrefillShape expanded = choose_shape(lp, rows, false, &uncut, cut, true, times[1]);
    constexpr float kTileUs = 0.013f, kExpandUs = 3.f;
    float score[2] = {0.f, 0.f}, history = (float)rows.history_pages;
    for (int g = 0; g < 4; ++g, history *= 0.25f) {
        score[0] += kWeight[g];
        score[1] += kWeight[g] * (times[1][g] + kExpandUs + kTileUs * history * rows.batch * dense) / times[0][g];
    }
    if (score[1] >= score[0]) return plan;
    return {true, expanded, expanded_sizes(lp, rows.batch, width).all() + pieces_bytes(lp, expanded), uncut};
}

// How a listed mask is walked: by merged lists of four query tiles of a head, or by the caller's rows as they are, for a head
// and a query tile at a time in four key slices, or by half workgroups, for two heads of a group where they have a mask in common.
enum MaskWalk { kMergedRows = 0, kRowSlices = 1, kRowHalves = 2 };

// `row`: mean number of tiles kept by a row of the lists.  How much neighbouring rows have in common is not known here: merged
// lists are taken half way between a row and the union of four random ones, and a walk of single rows has to be quicker by a
// margin.  Nor is it known which heads have a mask in common: in the order of their masks a group's heads make pairs, of which all
// but one fewer than there are masks are of one mask, whoever has which.  (Merged, slices, halves: 12345 tokens at density 0.3, 32 / 8
// heads, two masks in turn, 473, 530 and 329 us; 6330 tokens, twice, at 0.08, 64 / 8 heads, 466, 702 and 399; 5101 tokens at 0.35,
// 8 / 2 heads, slices 54 where merged lists take 119; 519 tokens, twice, at 0.4, 32 and 28; a pattern of 65536 tokens whose rows
// agree, 24 and 16 ms: times of a loop with a running maximum, as are the constants below; 12345 tokens in halves take 295 now.  A second launch that walked blocks of little common row by row gained 2 to 9 % over merged lists above 10000
// tokens and lost up to 30 % below.  Two heads to a row in two slices: 392 us at 12345 tokens, but 41 where halves take 47 at 2907,
// twice, 8 / 2 heads; not kept for that.)
MaskWalk choose_mask_walk(const LayerParams& lp, double tiles, double longest, double row, int masks) {
    constexpr double kFixedUs = 7., kFoldedUs = 8., kStepUs = 2., kSlicedStepUs = 3., kHalfStartUs = 5.5, kHalfStepUs = 1.9,
                     kAloneStepUs = 1.5, kNothingUs = 1.;  // of a workgroup, rounded up
    const double units = num_compute_units();
    auto launch_time = [&](double work, double last) { return std::max(last, work / units + 0.35 * last); };
    const int n_stream = count_streaming(lp);
    const double dense = tiles * (lp.Hkv - n_stream) * lp.group, stream = tiles * n_stream * lp.group;
    const double band = std::min<double>(lp.sink_pages + lp.local_pages, longest);
    const double keep = std::min(1., row / (0.5 * longest)), drop = 1. - keep, joint = 1. - drop * drop * drop * drop;
    const double walk = 0.5 * (row + 0.5 * longest * joint), merge_us = 5.;
    const double merged = merge_us + launch_time((dense * (kFixedUs + kStepUs * walk) + stream * (kFixedUs + kStepUs * (band + 3))) / kPairs,
                                                 kFixedUs + kStepUs * longest * joint);
    const double sliced = launch_time(dense * (kFoldedUs + kSlicedStepUs * row / 4) + stream * (kFoldedUs + kSlicedStepUs * band / 4),
                                      kFoldedUs + kSlicedStepUs * std::min(2 * row, longest) / 4);
    // two half workgroups to a compute unit; in groups of even size the second of a pair finds nothing to do where the first has both
    const bool even = lp.group % 2 == 0;
    const double pairs = even ? std::max(0., 1. - 2. * (masks - 1) / lp.group) : 0.;
    auto halves_of = [&](double n, double joined, double steps) {
        return n * (0.5 * joined * (kHalfStartUs + kHalfStepUs * steps) + (1. - joined) * (kHalfStartUs + kAloneStepUs * steps)) +
               (even ? 0.5 * n * kNothingUs : 0.);
    };
    const double halves = launch_time(0.5 * (halves_of(dense, pairs, row) + halves_of(stream, even ? 1. : 0., band)),
                                      kHalfStartUs + kAloneStepUs * std::min(2 * row, longest));
    // Where slices are clearly quicker than merged lists they are taken, also over half workgroups that are quicker still: each
    // slice rounds its weights relative to a maximum of its own, and in one slice the error against 64 bits is some 1 % larger
    // (1342 tokens at density 0.42, 32 / 8 heads; merged lists are one slice as well).
    if (1.15 * sliced < merged) return kRowSlices;
    return 1.15 * halves < merged ? kRowHalves : kMergedRows;
}
MaskWalk choose_mask_walk(const LayerParams& lp, int batch, int total_tokens, int max_seqlen, int masks, int rows_per_mask, int nnz) {
    const double row = (double)nnz / ((double)masks * rows_per_mask);
    const double tiles = (double)total_tokens / kTile + 0.5 * batch;  // half a tile of padding per sequence
    return choose_mask_walk(lp, tiles, (max_seqlen + kTile - 1) / kTile, row, masks);
}

// max_rows: rows of the longest sequence; any_start: they may start anywhere inside a block; single_rows: a workgroup has one
// query tile, whatever units that leaves without work.
PrefillSchedule make_schedule(const LayerParams& lp, const PrefillShape& shape, int max_rows, int total_rows, bool any_start,
                              int batch, bool single_rows = false) {
    PrefillSchedule sched;
    sched.pieces = {nullptr, shape.pieces, shape.least, 0};
    sched.compute_units = num_compute_units();
    for (int c = 0; c < 2; ++c) {
        HeadClass& hc = sched.cls[c];
        hc.fold = shape.fold[c];
        const int units = units_of(shape, c), heads = heads_per_block(lp, shape, c);
        hc.heads_per_block = heads;
        hc.qtiles_log2 = 0;
        while (!single_rows && (heads << hc.qtiles_log2) < units) ++hc.qtiles_log2;
        const int rows = kTile << hc.qtiles_log2;
        // rows that start anywhere inside a block reach into one block more than their number needs
        hc.blocks_per_seq = (max_rows + rows - 1) / rows + (any_start ? 1 : 0);
        hc.ordered = batch <= kOrderedSeqs;
        long long blocks = (long long)hc.blocks_per_seq * batch;
        // n rows fill floor(n / rows) blocks and touch at most one more, two more if they start anywhere
        if (hc.ordered) blocks = std::min(blocks, (long long)total_rows / rows + (any_start ? 2LL : 1LL) * batch);
        hc.blocks = (int)std::min(blocks, 0x7fffffffLL);
        if (c == 0 && shape.pieces) blocks = shape.pieces;
        if (single_rows && shape.half && heads == 2) blocks *= 2;  // `again`
        hc.heads = 0;
        for (unsigned& w : hc.kv_head) w = 0;
        for (int hk = 0; hk < lp.Hkv; ++hk)
            if ((int)((lp.streaming_mask >> hk) & 1ull) == c) {
                hc.kv_head[hc.heads / 4] |= (unsigned)hk << (8 * (hc.heads % 4));
                ++hc.heads;
            }
        hc.swizzled = hc.heads > 0 && kXcds % hc.heads == 0;
        hc.slices = hc.swizzled ? kXcds / hc.heads : 1;
        const int per_block = lp.group / heads;
        if (hc.heads == 0)
            hc.items_per_xcd = 0;
        else if (hc.swizzled)
            hc.items_per_xcd = (int)(per_block * ((blocks + hc.slices - 1) / hc.slices));
        else
            hc.items_per_xcd = (int)((hc.heads * per_block * blocks + kXcds - 1) / kXcds);
    }
    return sched;
}

size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

// merged lists of a listed mask, one per block of four query tiles, of a sequence
int mask_blocks(int max_seqlen) { return (max_seqlen + kPairs * kTile - 1) / (kPairs * kTile); }

struct PrefillLaunch {
    const LayerParams* lp;
    const uint16_t *q, *k, *v;
    const int* cu_seqlens;
    int batch, total_tokens, max_rows;
    PrefillRows rows;  // (of chunks)
    uint16_t* out;
    float* lse_out;
    PrefillSchedule sched;
    PrefillMask mk;
    PrefillPaged pg;
    hipStream_t stream;
};

template <class T, int MODE, int BITS>
hipError_t launch_slices(const PrefillLaunch& a, int slices) {
    const int grid = kXcds * (a.sched.cls[0].items_per_xcd + a.sched.cls[1].items_per_xcd);
#define LSERVE_PREFILL_SLICES(SL)                                                                                       \
    hipLaunchKernelGGL((sparse_prefill_kernel<T, MODE, BITS, SL>), dim3(grid), dim3(kPrefillThreads), 0, a.stream, *a.lp, \
                       a.q, a.k, a.v, a.cu_seqlens, a.batch, a.out, a.lse_out, a.total_tokens, a.sched, a.mk, a.pg)
    if constexpr (BITS == 16) {
        if (slices == 4) {
            LSERVE_PREFILL_SLICES(4);
            return hipGetLastError();
        }
    }
    if constexpr (MODE != kMasked) {  // listed masks: one or four
        if (slices == 2) {
            LSERVE_PREFILL_SLICES(2);
            return hipGetLastError();
        }
    }
    LSERVE_PREFILL_SLICES(1);
#undef LSERVE_PREFILL_SLICES
    return hipGetLastError();
}

template <class T, int MODE>
hipError_t launch_half(const PrefillLaunch& a) {
    hipLaunchKernelGGL((prefill_half_kernel<T, MODE>), dim3(kXcds * (a.sched.cls[0].items_per_xcd + a.sched.cls[1].items_per_xcd)),
                       dim3(kPrefillThreads / 2), 0, a.stream, *a.lp, a.q, a.k, a.v, a.cu_seqlens, a.batch, a.out, a.lse_out, a.total_tokens,
                       a.sched, a.mk, a.pg);
    return hipGetLastError();
}

// A launch of whole walks over pages.
template <class T, int BITS>
hipError_t launch_whole(const PrefillLaunch& a, const PrefillShape& shape) {
    if constexpr (BITS == 16) {
        if (shape.half) return launch_half<T, kPaged>(a);
    }
    return launch_slices<T, kPaged, BITS>(a, shape.slices);
}

// A launch over pages, in pieces if that is the shape.
template <class T, int BITS>
hipError_t launch_chunk(PrefillLaunch& a, const ChunkPlan& plan, void* scratch) {
    if (!plan.shape.pieces) return launch_whole<T, BITS>(a, plan.shape);
    a.sched.pieces.partials = reinterpret_cast<float*>(scratch);
    const bool apart = streams_apart(*a.lp, plan.uncut);
    const HeadClass& dense = a.sched.cls[0];
    if (apart) {
        a.sched.cls[1].items_per_xcd = 0;
        const int until = (int)whole_walks_until(*a.lp, a.rows, BITS != 16, plan.uncut, plan.shape);
        if (until > 0) a.sched.pieces.short_blocks = (until + ceil_div(a.max_rows, kTile)) >> dense.qtiles_log2;
    }
    hipLaunchKernelGGL((prefill_pieces_kernel<T, BITS>), dim3(kXcds * (dense.items_per_xcd + a.sched.cls[1].items_per_xcd)),
                       dim3(kPrefillThreads), 0, a.stream, *a.lp, a.q, a.k, a.v, a.cu_seqlens, a.batch, a.out, a.lse_out, a.total_tokens,
                       a.sched, a.mk, a.pg);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int heads = dense.heads * (a.lp->group / dense.heads_per_block);
    if (!apart) {
        hipLaunchKernelGGL((fold_pieces_kernel<T>), dim3(dense.blocks * kPrefillWaves, dense.heads, a.lp->group / dense.heads_per_block), dim3(256),
                           0, a.stream, *a.lp, a.cu_seqlens, a.pg.kv.seq_lens, a.pg.k_new != nullptr, a.batch, a.out, a.lse_out, a.total_tokens,
                           a.sched);
        return hipGetLastError();
    }
    const PrefillSchedule uncut = make_schedule(*a.lp, plan.uncut, a.max_rows, a.total_tokens, true, a.batch);
    const int grid = kXcds * uncut.cls[1].items_per_xcd + std::max(dense.blocks * (kPrefillWaves / 2) * heads, kXcds * uncut.cls[0].items_per_xcd);
    auto launch = [&](auto slices) {
        hipLaunchKernelGGL((fold_and_streams_kernel<T, BITS, decltype(slices)::value>), dim3(grid), dim3(kPrefillThreads), 0, a.stream, *a.lp, a.q,
                           a.k, a.v, a.cu_seqlens, a.batch, a.out, a.lse_out, a.total_tokens, uncut, a.mk, a.pg, a.sched);
        return hipGetLastError();
    };
    if constexpr (BITS == 16) {
        if (plan.uncut.slices == 4) return launch(std::integral_constant<int, 4>{});
    }
    return launch(std::integral_constant<int, 2>{});
}

// Does a launch of half workgroups last as long as its longest walk?  With about two dense workgroups to a compute unit, dealt out
// longest first, the longest walk of all shares its unit from beginning to end, with one half as long and then with streaming heads, at 1.7
// us a step where it would take 1.0 alone, and the chip runs empty around it (one prompt of 4096 tokens: 64 steps where an even share is
// 42).  The first workgroup of every unit then has a higher wave priority throughout.  4096 tokens 103 -> 98 us, 4300 110 -> 104, 4200 of 32 / 16
// heads 105 -> 100, 3900 of 32 / 32 94 -> 91.  Walks of fewer tiles lose 1 to 3 % (1600 tokens, 64 / 8 heads: 44.2 and 45.3), and so do launches
// of more workgroups, whose units have other long walks to fill up with (4900 of 32 / 32, 2.4 to a unit, 123 and 126).  At the edges, time
// with priority as a part of that without, 28 prompts and batches of 32 query heads, half of the KV heads streaming: 55 tiles, 1.7
// workgroups to a unit 0.96, 63 to 72 tiles, 2.25 to a unit 0.95 to 0.99; just outside 47 tiles, 2.2 1.02, 32 tiles, 2.0 1.00 to 1.01, 74 tiles, 2.3 0.97
// to 0.98, 77 tiles, 2.4 0.98 and 1.015, 2.5 and more 1.01 to 1.04.  (Fewer than 1.7 to a unit go in key slices.)
bool longest_walk_decides(const PrefillSchedule& sched, int tiles) {
    const long long n = (long long)kXcds * sched.cls[0].items_per_xcd, units = sched.compute_units;
    return tiles >= 48 && 4 * n > 5 * units && 4 * n <= 9 * units;
}

template <class T>
hipError_t launch_prefill(const LayerParams& lp, const void* q, const void* k, const void* v, const int* cu_seqlens,
                          int batch, int total_tokens, int max_seqlen, void* out, float* lse_out, void* workspace,
                          const PrefillMaskArgs* mask, hipStream_t stream) {
    const int max_tiles = (max_seqlen + kTile - 1) / kTile;
    PrefillLaunch a = {};
    a.lp = &lp;
    a.q = reinterpret_cast<const uint16_t*>(q);
    a.k = reinterpret_cast<const uint16_t*>(k);
    a.v = reinterpret_cast<const uint16_t*>(v);
    a.cu_seqlens = cu_seqlens;
    a.batch = batch;
    a.total_tokens = total_tokens;
    a.out = reinterpret_cast<uint16_t*>(out);
    a.lse_out = lse_out;
    a.stream = stream;
    if (!mask) {
        const PrefillShape shape = choose_shape(lp, {batch, total_tokens, max_seqlen, -1}, false);
        a.sched = make_schedule(lp, shape, max_seqlen, total_tokens, false, batch);
        if (shape.half && longest_walk_decides(a.sched, max_tiles)) {
            hipLaunchKernelGGL((prefill_hasty_kernel<T>), dim3(kXcds * (a.sched.cls[0].items_per_xcd + a.sched.cls[1].items_per_xcd)),
                               dim3(kPrefillThreads / 2), 0, stream, lp, a.q, a.k, a.v, cu_seqlens, batch, a.out, lse_out, total_tokens,
                               a.sched, a.mk, a.pg);
            return hipGetLastError();
        }
        if (shape.half) return launch_half<T, kPlain>(a);
        return launch_slices<T, kPlain, 16>(a, shape.slices);
    }
    PrefillMask& mk = a.mk;
    mk.head_mask = mask->head_mask;
    mk.q_tile_start = mask->q_tile_start;
    mk.row_ptr = mask->row_ptr;
    mk.cols = mask->cols;
    mk.rows_per_mask = mask->rows_per_mask;
    const MaskWalk walk = choose_mask_walk(lp, batch, total_tokens, max_seqlen, mask->num_masks, mask->rows_per_mask, mask->nnz);
    if (walk == kRowHalves) {
        a.sched = make_schedule(lp, {1, {false, false}, false, true, 0, 1}, max_seqlen, total_tokens, false, batch, true);
        return launch_half<T, kMasked>(a);
    }
    if (walk == kRowSlices) {
        a.sched = make_schedule(lp, {4, {true, true}, true, false, 0, 1}, max_seqlen, total_tokens, false, batch);
        return launch_slices<T, kMasked, 16>(a, 4);
    }
    mk.blocks_per_seq = mask_blocks(max_seqlen);
    mk.blk_list = reinterpret_cast<int*>(workspace);
    mk.blk_count = reinterpret_cast<int*>(reinterpret_cast<unsigned char*>(workspace) + align16((size_t)mask->nnz * sizeof(int)));
    hipLaunchKernelGGL(merge_mask_rows_kernel, dim3(mk.blocks_per_seq, batch, mask->num_masks), dim3(kWave),
                       (size_t)align16(max_tiles), stream, mk, cu_seqlens, batch);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    a.sched = make_schedule(lp, {1, {false, false}, true, false, 0, 1}, max_seqlen, total_tokens, false, batch);
    return launch_slices<T, kMasked, 16>(a, 1);
}

template <class T>
hipError_t launch_prefill_paged(const LayerParams& lp, const PagedParams& kv, const void* q, const void* k_new,
                                const void* v_new, const int* cu_q, int total_new, int max_new_per_seq, int max_seqlen,
                                void* out, float* lse_out, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    PrefillLaunch a = {};
    a.lp = &lp;
    a.q = reinterpret_cast<const uint16_t*>(q);
    a.cu_seqlens = cu_q;
    a.batch = kv.batch;
    a.total_tokens = total_new;
    a.max_rows = max_new_per_seq;
    a.out = reinterpret_cast<uint16_t*>(out);
    a.lse_out = lse_out;
    a.pg.kv = kv;
    a.pg.k_new = reinterpret_cast<const uint16_t*>(k_new);
    a.pg.v_new = reinterpret_cast<const uint16_t*>(v_new);
    a.stream = stream;
    const int pages = max_seqlen > 0 ? std::min(kv.max_pages, (max_seqlen - 1) / kTile + 1) : kv.max_pages;
    const PrefillRows rows = a.rows = chunk_rows(kv.batch, total_new, max_new_per_seq, pages);
    ChunkPlan plan = plan_chunk(lp, rows, kv.max_pages, kv.kv_bits != 16, workspace && workspace_bytes > 0);
    if (plan.bytes > workspace_bytes) plan = plan_chunk(lp, rows, kv.max_pages, kv.kv_bits != 16, false);
    a.sched = make_schedule(lp, plan.shape, max_new_per_seq, total_new, true, kv.batch);
    if (plan.expand) {
        const ExpandedSizes size = expanded_sizes(lp, kv.batch, kv.max_pages);
        unsigned char* at = reinterpret_cast<unsigned char*>(workspace);
        auto take = [&](size_t bytes) {
            unsigned char* p = at;
            at += bytes;
            return p;
        };
        ExpandedPages to;
        to.k = reinterpret_cast<uint16_t*>(take(size.pool));
        to.v = reinterpret_cast<uint16_t*>(take(size.pool));
        to.k_ring = reinterpret_cast<uint16_t*>(take(size.ring));
        to.v_ring = reinterpret_cast<uint16_t*>(take(size.ring));
        to.table = reinterpret_cast<int*>(take(size.table));
        to.ring_table = reinterpret_cast<int*>(take(size.ring_table));
        workspace = at;
        const dim3 grid(std::min(pages, 64), lp.Hkv, kv.batch);
        if (kv.kv_bits == 8)
            hipLaunchKernelGGL((expand_pages_kernel<T, 8>), grid, dim3(256), 0, stream, lp, kv, cu_q, to);
        else
            hipLaunchKernelGGL((expand_pages_kernel<T, 4>), grid, dim3(256), 0, stream, lp, kv, cu_q, to);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        PagedParams& pages16 = a.pg.kv;
        pages16.k_pool = to.k;
        pages16.v_pool = to.v;
        pages16.page_table = to.table;
        pages16.pool_heads = lp.Hkv - kv.stream_heads;
        pages16.k_stream = kv.stream_heads ? to.k_ring : nullptr;
        pages16.v_stream = kv.stream_heads ? to.v_ring : nullptr;
        pages16.ring_table = to.ring_table;
        pages16.kv_bits = 16;
        return launch_chunk<T, 16>(a, plan, workspace);
    }
    if (kv.kv_bits == 8) return launch_chunk<T, 8>(a, plan, workspace);
    if (kv.kv_bits == 4) return launch_chunk<T, 4>(a, plan, workspace);
    return launch_chunk<T, 16>(a, plan, workspace);
}

}  // namespace

hipError_t preload_prefill_kernels() {
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&merge_mask_rows_kernel));
}

void prefill_shape(const LayerParams& lp, int batch, int total_rows, int max_rows, int pages, int kv_bits, int (&out)[4]) {
    const PrefillRows rows = pages > 0 ? chunk_rows(batch, total_rows, max_rows, pages) : PrefillRows{batch, total_rows, max_rows, -1};
    const PrefillShape shape = choose_shape(lp, rows, pages > 0 && kv_bits != 16, nullptr, false, false);
    out[0] = shape.slices;
    out[1] = shape.fold[0];
    out[2] = shape.fold[1];
    out[3] = shape.one_head;
}

void prefill_plan(const LayerParams& lp, int batch, int total_rows, int max_rows, int pages, int kv_bits, bool scratch, int (&out)[6]) {
    ChunkPlan plan = {};
    if (pages > 0)
        plan = plan_chunk(lp, chunk_rows(batch, total_rows, max_rows, pages), pages, kv_bits != 16, scratch);
    else
        plan.shape = plan.uncut = choose_shape(lp, {batch, total_rows, max_rows, -1}, false);
    const bool apart = plan.shape.pieces && streams_apart(lp, plan.uncut);
    out[0] = plan.shape.pieces ? plan.shape.least : slices_of(plan.shape, 0);
    out[1] = slices_of(apart ? plan.uncut : plan.shape, 1);
    out[2] = plan.shape.half;
    out[3] = plan.shape.pieces;
    out[4] = apart;
    out[5] = plan.expand;
}

bool prefill_longest_first(const LayerParams& lp, int batch, int total_rows, int max_rows) {
    const PrefillShape shape = choose_shape(lp, {batch, total_rows, max_rows, -1}, false);
    return shape.half && longest_walk_decides(make_schedule(lp, shape, max_rows, total_rows, false, batch), ceil_div(max_rows, kTile));
}

int mask_walk(const LayerParams& lp, int batch, int total_tokens, int max_seqlen, int masks, int rows_per_mask, int nnz) {
    return choose_mask_walk(lp, batch, total_tokens, max_seqlen, masks, rows_per_mask, nnz);
}

size_t chunk_scratch_bytes(const LayerParams& lp, int batch, int total_rows, int max_rows, int pages, int kv_bits) {
    return plan_chunk(lp, chunk_rows(batch, total_rows, max_rows, pages), pages, kv_bits != 16, true).bytes;
}

size_t paged_prefill_workspace_bytes(const LayerParams& lp, int batch, int max_pages) {
    (void)lp;
    (void)batch;
    (void)max_pages;
    return 0;  // keys and values are read from the pages as they are
}

hipError_t launch_sparse_prefill_paged(int dtype, const LayerParams& lp, const PagedParams& kv, const void* q,
                                       const void* k_new, const void* v_new, const int* cu_q, int total_new,
                                       int max_new_per_seq, int max_seqlen, void* out, float* lse_out, void* workspace,
                                       size_t workspace_bytes, hipStream_t stream) {
    return dtype == 0 ? launch_prefill_paged<F16>(lp, kv, q, k_new, v_new, cu_q, total_new, max_new_per_seq, max_seqlen,
                                                  out, lse_out, workspace, workspace_bytes, stream)
                      : launch_prefill_paged<BF16>(lp, kv, q, k_new, v_new, cu_q, total_new, max_new_per_seq, max_seqlen,
                                                   out, lse_out, workspace, workspace_bytes, stream);
}

size_t prefill_workspace_bytes(const LayerParams& lp, int total_tokens, int batch) {
    (void)lp;
    (void)total_tokens;
    (void)batch;
    return 0;  // Q, K and V are read where they are
}

// The merged tile lists (at most one entry per mask entry), then one count per (mask, sequence, workgroup of
// query rows).
size_t masked_prefill_workspace_bytes(const LayerParams& lp, int total_tokens, int batch, int max_seqlen, int num_masks,
                                      int nnz) {
    const int blocks_per_seq = mask_blocks(max_seqlen);
    (void)lp;
    (void)total_tokens;
    return align16((size_t)nnz * sizeof(int)) +
           align16((size_t)num_masks * batch * blocks_per_seq * sizeof(int));
}

hipError_t launch_sparse_prefill(int dtype, const LayerParams& lp, const void* q, const void* k, const void* v,
                                 const int* cu_seqlens, int batch, int total_tokens, int max_seqlen, void* out,
                                 float* lse_out, void* workspace, const PrefillMaskArgs* mask, hipStream_t stream) {
    return dtype == 0 ? launch_prefill<F16>(lp, q, k, v, cu_seqlens, batch, total_tokens, max_seqlen, out, lse_out,
                                            workspace, mask, stream)
                      : launch_prefill<BF16>(lp, q, k, v, cu_seqlens, batch, total_tokens, max_seqlen, out, lse_out,
                                             workspace, mask, stream);
}

}  // namespace lserve
