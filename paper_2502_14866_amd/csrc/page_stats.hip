// Key statistics for hierarchical paging (Sec. 3.5.2): channel-wise max / min of the keys of
// every logical page of the non-streaming KV heads.  Pure streaming work: one wavefront reads one
// logical page with 16-byte loads (16 lanes cover one 256-byte token row, the four rows of the
// wave cover four tokens per load) and folds the rows together at the end.
#include "kernels.h"

namespace lserve {

template <class T>
__global__ __launch_bounds__(kWave* kMaxLogical) void page_stats_kernel(LayerParams lp, PagedParams kv,
                                                                         const int* __restrict__ start_pos,
                                                                         HeadList heads) {
    const int b = blockIdx.z;
    const int hk = heads.idx[blockIdx.y];
    const int j = threadIdx.x / kWave;  // logical page inside the physical page
    const int lane = threadIdx.x % kWave;
    const int L = kv.seq_lens[b];
    const int start = start_pos ? start_pos[b] : 0;
    const int P = ceil_div(L, lp.NP);
    const int p = P - 1 - (int)blockIdx.x;  // pages are visited from the tail
    if (p < 0 || p < start / lp.NP) return;
    const int lo = p * lp.NP + j * lp.NL;
    const int hi = min(lo + lp.NL, L);
    if (lo >= L || hi <= start) return;

    const int phys = kv.page_table[(size_t)b * kv.max_pages + p];
    const int r = lane / 16, c = lane % 16;
    const size_t ph = (size_t)phys * kv.pool_heads + pool_rank(lp, kv, hk, false);  // (page, head) index inside the main pool
    const uint4* slab = reinterpret_cast<const uint4*>(kv.k_pool) + ph * lp.NP * (kHeadDim / 8);

    float vmax[8], vmin[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        vmax[i] = -INFINITY;
        vmin[i] = INFINITY;
    }
    for (int t = lo + r; t < hi; t += 4) {
        uint4 x = slab[(size_t)(t - p * lp.NP) * (kHeadDim / 8) + c];
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float a = Elem<T>::lo(w[i]), bb = Elem<T>::hi(w[i]);
            vmax[2 * i] = fmaxf(vmax[2 * i], a);
            vmin[2 * i] = fminf(vmin[2 * i], a);
            vmax[2 * i + 1] = fmaxf(vmax[2 * i + 1], bb);
            vmin[2 * i + 1] = fminf(vmin[2 * i + 1], bb);
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        vmax[i] = rows4_max(vmax[i]);
        vmin[i] = rows4_min(vmin[i]);
    }
    if (r == 0) {
        uint4* dst = reinterpret_cast<uint4*>(kv.stats) + ((ph * lp.g + j) * 2) * (kHeadDim / 8);
        // max / min of stored values are stored values: the conversion back is exact
        dst[c] = make_uint4(Elem<T>::pack(vmax[0], vmax[1]), Elem<T>::pack(vmax[2], vmax[3]),
                            Elem<T>::pack(vmax[4], vmax[5]), Elem<T>::pack(vmax[6], vmax[7]));
        dst[kHeadDim / 8 + c] = make_uint4(Elem<T>::pack(vmin[0], vmin[1]), Elem<T>::pack(vmin[2], vmin[3]),
                                           Elem<T>::pack(vmin[4], vmin[5]), Elem<T>::pack(vmin[6], vmin[7]));
    }
}

// Smaller and larger of two pairs of fp16, and a pair with its signalling not-a-numbers quieted.  The first two return the other
// operand for a quiet not-a-number, but the quieted one itself for a signalling one, which would drop what the range held before:
// what comes from memory goes through quiet() first.  (Written out: ahead of the compiler's own forms goes such an instruction per
// operand, results of the forms themselves among them, where one per loaded pair will do.)
__device__ __forceinline__ half2_t pk_min(half2_t a, half2_t b) {
    half2_t r;
    asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ half2_t pk_max(half2_t a, half2_t b) {
    half2_t r;
    asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ half2_t quiet(uint32_t w) {
    const half2_t x = __builtin_bit_cast(half2_t, w);
    return pk_max(x, x);
}

// Smallest and largest of eight values (f: the same as numbers).
template <class T> __device__ __forceinline__ void range8(const uint32_t (&)[4], const float (&f)[8], float& lo, float& hi) {
    lo = hi = f[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) {
        lo = fminf(lo, f[i]);
        hi = fmaxf(hi, f[i]);
    }
}
template <> __device__ __forceinline__ void range8<F16>(const uint32_t (&w)[4], const float (&)[8], float& lo, float& hi) {
    half2_t l = quiet(w[0]), h = l;
#pragma unroll
    for (int i = 1; i < 4; ++i) {
        const half2_t x = quiet(w[i]);
        l = pk_min(l, x);
        h = pk_max(h, x);
    }
    lo = fminf((float)l[0], (float)l[1]);
    hi = fmaxf((float)h[0], (float)h[1]);
}

// Running channel-wise maximum and minimum of rows, eight channels to a lane.
template <class T> struct RowRange {
    float hi[8], lo[8];
    __device__ __forceinline__ RowRange() {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            hi[i] = -INFINITY;
            lo[i] = INFINITY;
        }
    }
    __device__ __forceinline__ void add(const uint4& x) {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            hi[2 * i] = fmaxf(hi[2 * i], Elem<T>::lo(w[i]));
            lo[2 * i] = fminf(lo[2 * i], Elem<T>::lo(w[i]));
            hi[2 * i + 1] = fmaxf(hi[2 * i + 1], Elem<T>::hi(w[i]));
            lo[2 * i + 1] = fminf(lo[2 * i + 1], Elem<T>::hi(w[i]));
        }
    }
    __device__ __forceinline__ float largest(int i) const { return hi[i]; }
    __device__ __forceinline__ float smallest(int i) const { return lo[i]; }
};
template <> struct RowRange<F16> {
    half2_t hi[4], lo[4];
    __device__ __forceinline__ RowRange() {
        const _Float16 inf = (_Float16)INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            hi[i] = half2_t{(_Float16)-inf, (_Float16)-inf};
            lo[i] = half2_t{inf, inf};
        }
    }
    __device__ __forceinline__ void add(const uint4& x) {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const half2_t v = quiet(w[i]);
            hi[i] = pk_max(hi[i], v);
            lo[i] = pk_min(lo[i], v);
        }
    }
    __device__ __forceinline__ float largest(int i) const { return (float)hi[i / 2][i % 2]; }
    __device__ __forceinline__ float smallest(int i) const { return (float)lo[i / 2][i % 2]; }
};

// Asymmetric quantisation of one token row held by the 16 lanes of a DPP row, eight features per lane
// (Sec. 3.2: scale factor and zero point of a token are stored next to its features), to codes 0 .. levels = 2^BITS - 1:
//   zero = fp16(min), scale = fp16((max - zero) / levels), code = clamp(rint((x - zero) / scale), 0, levels),
// every step rounded as IEEE fp32 does, divisions too, so that the codes do not depend on the machine.
// Yields the lane's eight codes and the token's (scale, zero) pair as two fp16 in one word.
// The codes come packed as the pages keep them: 8 bits, one byte each, channels in order; 4 bits, byte j of the word holding
// channel j in its low and channel 4 + j in its high half, so that masking out either half leaves four codes in the byte lanes
// the 8-bit path uses.
template <class T, int BITS>
__device__ __forceinline__ void quantize_row(const uint4& x, uint2& packed, uint32_t& scale_zero) {
    constexpr float kLevels = (float)((1 << BITS) - 1);
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
    float f[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = Elem<T>::lo(w[i]);
        f[2 * i + 1] = Elem<T>::hi(w[i]);
    }
    float lo, hi;
    range8<T>(w, f, lo, hi);
    lo = fminf(lo, dpp_f<kDppXor1>(lo));
    hi = fmaxf(hi, dpp_f<kDppXor1>(hi));
    lo = fminf(lo, dpp_f<kDppXor2>(lo));
    hi = fmaxf(hi, dpp_f<kDppXor2>(hi));
    lo = fminf(lo, dpp_f<kDppHalfMirror>(lo));
    hi = fmaxf(hi, dpp_f<kDppHalfMirror>(hi));
    lo = fminf(lo, dpp_f<kDppMirror>(lo));
    hi = fmaxf(hi, dpp_f<kDppMirror>(hi));
    constexpr float kBig = 65504.f;  // largest finite fp16
    const _Float16 zero_h = (_Float16)fminf(fmaxf(lo, -kBig), kBig);
    const float zero = (float)zero_h;
    // (hi - zero) / levels: the product with the rounded reciprocal, corrected by its remainder, is the correctly rounded quotient
    // (for 15 and 255 with every one of the 2^23 significands); an infinite range, whose remainder is not a number, is its own
    // quotient (of either sign: rows of nothing but -inf have -inf - zero).
    constexpr float kInverse = 1.f / kLevels;
    const float range = hi - zero, q = range * kInverse;
    const float quotient = fabsf(range) == INFINITY ? range : __builtin_fmaf(__builtin_fmaf(-q, kLevels, range), kInverse, q);
    const _Float16 scale_h = (_Float16)fminf(quotient, kBig);
    const float scale = (float)scale_h;
    // code = rint of the fp32 quotient.  An IEEE division is some ten instructions, and eight of them per lane and row were
    // most of the write-back of quantised pages.  The product with the reciprocal is within 3 units in the last place of
    // the quotient, which for quotients up to 256 is less than 1e-4, so the two round to the same whole number unless the
    // product lies that close to a half.  That is two quotients in ten thousand, one lane in 600 (of eight quotients) and
    // one wavefront in ten (of 512), which then divides.  (Where the product is not a number or not finite, neither is the
    // quotient.)
    const float inv = __builtin_amdgcn_rcpf(scale);
    float t[8], off = 0.f;
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        const float a = (f[i] - zero) * inv, b = (f[i + 1] - zero) * inv;
        t[i] = __builtin_rintf(a);
        t[i + 1] = __builtin_rintf(b);
        off = fmaxf(fmaxf(off, fabsf(a - t[i])), fabsf(b - t[i + 1]));
    }
    if (off >= 0.4999f) {
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = __builtin_rintf((f[i] - zero) / scale);
    }
    const float top = scale > 0.f ? kLevels : 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = __builtin_amdgcn_fmed3f(t[i], 0.f, top);  // 0 where there is no number
    auto bytes4 = [](float a, float b, float c, float d) {
        uint32_t u = __builtin_amdgcn_cvt_pk_u8_f32(a, 0, 0u);
        u = __builtin_amdgcn_cvt_pk_u8_f32(b, 1, u);
        u = __builtin_amdgcn_cvt_pk_u8_f32(c, 2, u);
        return (uint32_t)__builtin_amdgcn_cvt_pk_u8_f32(d, 3, u);
    };
    if constexpr (BITS == 8)
        packed = make_uint2(bytes4(t[0], t[1], t[2], t[3]), bytes4(t[4], t[5], t[6], t[7]));
    else
        packed = make_uint2(bytes4(__builtin_fmaf(t[4], 16.f, t[0]), __builtin_fmaf(t[5], 16.f, t[1]),
                                   __builtin_fmaf(t[6], 16.f, t[2]), __builtin_fmaf(t[7], 16.f, t[3])), 0u);
    const half2_t sz = {scale_h, zero_h};
    scale_zero = __builtin_bit_cast(uint32_t, sz);
}

// KV write-back with the statistics updated in the same pass (Sec. 3.2, Sec. 3.5.2): one workgroup per
// (physical page touched by the new tokens, KV head, sequence), one wavefront per logical page.  New
// rows are copied into both pools with 16-byte accesses; for non-streaming heads the wave folds the
// new keys into max / min rows and, when the logical page already held tokens, combines them with the
// stored rows instead of re-reading the old keys.  BITS = 8 or 4 stores the rows quantised (one byte or half
// a byte per feature, then the page's (scale, zero) pairs); the statistics are still those of the 16-bit
// keys handed in.
template <class T, int BITS>
__global__ __launch_bounds__(kWave* kMaxLogical) void append_kv_kernel(LayerParams lp, PagedParams kv,
                                                                        const uint4* __restrict__ k_new,
                                                                        const uint4* __restrict__ v_new,
                                                                        const int* __restrict__ cu_new,
                                                                        const int* __restrict__ start_pos) {
    const int b = blockIdx.z, hk = blockIdx.y;
    const int j = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int r = lane / 16, c = lane % 16;
    const int s = start_pos[b], src0 = cu_new[b];
    const int e = s + (cu_new[b + 1] - src0);  // new tokens occupy positions [s, e)
    const int p = s / lp.NP + (int)blockIdx.x;
    const int lo = p * lp.NP + j * lp.NL, hi = lo + lp.NL;  // this wave's logical page
    const int t0 = max(lo, s), t1 = min(hi, e);
    if (t0 >= t1) return;
    const bool streaming = (lp.streaming_mask >> hk) & 1ull;
    size_t ph;  // (page, head) index inside the pool that stores this head
    uint4 *kdst, *vdst;
    if (in_stream_pool(lp, kv, hk)) {
        // bounded pool: only sink pages and the pages that are still local once all new tokens are in
        // are stored; a local page lands on the ring slot of the page w positions before it
        if (p >= lp.sink_pages && p < ceil_div(e, lp.NP) - lp.local_pages) return;
        const int phys = kv.ring_table[(size_t)b * kv.ring + ring_slot(lp, p)];
        ph = (size_t)phys * kv.stream_heads + pool_rank(lp, kv, hk, true);
        kdst = reinterpret_cast<uint4*>(const_cast<void*>(kv.k_stream));
        vdst = reinterpret_cast<uint4*>(const_cast<void*>(kv.v_stream));
    } else {
        const int phys = kv.page_table[(size_t)b * kv.max_pages + p];
        ph = (size_t)phys * kv.pool_heads + pool_rank(lp, kv, hk, false);
        kdst = reinterpret_cast<uint4*>(const_cast<void*>(kv.k_pool));
        vdst = reinterpret_cast<uint4*>(const_cast<void*>(kv.v_pool));
    }
    kdst += ph * slab_chunks(lp.NP, BITS);
    vdst += ph * slab_chunks(lp.NP, BITS);

    RowRange<T> range;
    // Rows to be quantised sixteen (a logical page, as a rule) at a time, all of them requested before the first is worked on: the
    // work on a row is some 140 vector instructions.  16-bit rows, which are only copied, four at a time: 16 sequences of 100 to 300
    // tokens, fp16, 5.8 us and with sixteen at a time 6.15, one of 4000 6.4 and 6.7, of 65536 113 and 115.
    constexpr int kRows = BITS == 16 ? 1 : 4;  // per lane row
    for (int tb = t0; tb < t1; tb += 4 * kRows) {
        uint4 x[kRows], y[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int t = min(tb + 4 * u + r, t1 - 1);
            const size_t src = ((size_t)(src0 + t - s) * lp.Hkv + hk) * (kHeadDim / 8) + c;
            x[u] = k_new[src];
            y[u] = v_new[src];
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int t = tb + 4 * u + r;
            if (t >= t1) continue;
            const int slot = t - p * lp.NP;
            const size_t dst = (size_t)slot * (kHeadDim / 8) + c;
            if constexpr (BITS == 16) {
                kdst[dst] = x[u];
                vdst[dst] = y[u];
            } else {
                uint32_t ksz, vsz;
                uint2 kc, vc;
                quantize_row<T, BITS>(x[u], kc, ksz);
                quantize_row<T, BITS>(y[u], vc, vsz);
                if constexpr (BITS == 8) {
                    reinterpret_cast<uint2*>(kdst)[dst] = kc;
                    reinterpret_cast<uint2*>(vdst)[dst] = vc;
                } else {
                    reinterpret_cast<uint32_t*>(kdst)[dst] = kc.x;
                    reinterpret_cast<uint32_t*>(vdst)[dst] = vc.x;
                }
                if (c == 0) {  // the pairs follow the page's code rows
                    reinterpret_cast<uint32_t*>(kdst + lp.NP * (kHeadDim * BITS / 128))[slot] = ksz;
                    reinterpret_cast<uint32_t*>(vdst + lp.NP * (kHeadDim * BITS / 128))[slot] = vsz;
                }
            }
            range.add(x[u]);
        }
    }
    if (streaming) return;  // streaming heads are never scored
    float vmax[8], vmin[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        vmax[i] = rows4_max(range.largest(i));
        vmin[i] = rows4_min(range.smallest(i));
    }
    if (r == 0) {
        uint4* st = reinterpret_cast<uint4*>(kv.stats) + ((ph * lp.g + j) * 2) * (kHeadDim / 8);
        if (lo < s) {  // the logical page already held tokens: fold the stored rows in
            const uint4 om = st[c], on = st[kHeadDim / 8 + c];
            const uint32_t wm[4] = {om.x, om.y, om.z, om.w}, wn[4] = {on.x, on.y, on.z, on.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                vmax[2 * i] = fmaxf(vmax[2 * i], Elem<T>::lo(wm[i]));
                vmax[2 * i + 1] = fmaxf(vmax[2 * i + 1], Elem<T>::hi(wm[i]));
                vmin[2 * i] = fminf(vmin[2 * i], Elem<T>::lo(wn[i]));
                vmin[2 * i + 1] = fminf(vmin[2 * i + 1], Elem<T>::hi(wn[i]));
            }
        }
        st[c] = make_uint4(Elem<T>::pack(vmax[0], vmax[1]), Elem<T>::pack(vmax[2], vmax[3]),
                           Elem<T>::pack(vmax[4], vmax[5]), Elem<T>::pack(vmax[6], vmax[7]));
        st[kHeadDim / 8 + c] = make_uint4(Elem<T>::pack(vmin[0], vmin[1]), Elem<T>::pack(vmin[2], vmin[3]),
                                          Elem<T>::pack(vmin[4], vmin[5]), Elem<T>::pack(vmin[6], vmin[7]));
    }
}

// The same for at most one new token per sequence (a decode step).  Nothing but latency and launch: the general kernel
// starts a workgroup per (page, KV head, sequence) and a wavefront per logical page to move 512 bytes.  Here sixteen
// lanes own the K row of a (sequence, KV head) and the next sixteen its V row, eight such pairs to a workgroup, and all
// loads that depend on nothing but the position go out together (64 sequences, 8 KV heads, 4-bit pages: 7.2 -> 4.6 us).
template <class T, int BITS>
__global__ __launch_bounds__(256) void append_token_kernel(LayerParams lp, PagedParams kv, const uint4* __restrict__ k_new,
                                                           const uint4* __restrict__ v_new, const int* __restrict__ cu_new,
                                                           const int* __restrict__ start_pos) {
    const int row = threadIdx.x / 16, c = threadIdx.x % 16;
    const int pair = blockIdx.x * 8 + row / 2;
    const bool is_v = row % 2;
    if (pair >= kv.batch * lp.Hkv) return;
    const int b = pair / lp.Hkv, hk = pair - b * lp.Hkv;
    const int s = start_pos[b], src0 = cu_new[b], src1 = cu_new[b + 1];
    if (src1 <= src0) return;  // no new token
    const int p = s / lp.NP, slot = s - p * lp.NP, j = slot / lp.NL;
    const bool streaming = (lp.streaming_mask >> hk) & 1ull, ring = in_stream_pool(lp, kv, hk);
    // the one new token is the last of its sequence, so its page is a local one: a bounded pool always keeps it
    const int phys = ring ? kv.ring_table[(size_t)b * kv.ring + ring_slot(lp, p)] : kv.page_table[(size_t)b * kv.max_pages + p];
    const uint4 x = (is_v ? v_new : k_new)[((size_t)src0 * lp.Hkv + hk) * (kHeadDim / 8) + c];
    const size_t ph = (size_t)phys * (ring ? kv.stream_heads : kv.pool_heads) + pool_rank(lp, kv, hk, ring);
    const bool with_stats = !streaming && !is_v, first = slot - j * lp.NL == 0;
    uint4* st = reinterpret_cast<uint4*>(kv.stats) + ((ph * lp.g + j) * 2) * (kHeadDim / 8) + c;
    uint4 om = x, on = x;
    if (with_stats && !first) {  // the logical page already holds tokens
        om = st[0];
        on = st[kHeadDim / 8];
    }
    uint4* dst = reinterpret_cast<uint4*>(const_cast<void*>(is_v ? (ring ? kv.v_stream : kv.v_pool) : (ring ? kv.k_stream : kv.k_pool))) +
                 ph * slab_chunks(lp.NP, BITS);
    if (BITS == 16) {
        dst[(size_t)slot * (kHeadDim / 8) + c] = x;
    } else {
        uint32_t sz;
        uint2 code;
        quantize_row<T, BITS == 16 ? 8 : BITS>(x, code, sz);
        if (BITS == 8)
            reinterpret_cast<uint2*>(dst)[(size_t)slot * (kHeadDim / 8) + c] = code;
        else
            reinterpret_cast<uint32_t*>(dst)[(size_t)slot * (kHeadDim / 8) + c] = code.x;
        if (c == 0) reinterpret_cast<uint32_t*>(dst + lp.NP * (kHeadDim * BITS / 128))[slot] = sz;
    }
    if (!with_stats) return;
    const uint32_t w[4] = {x.x, x.y, x.z, x.w}, wm[4] = {om.x, om.y, om.z, om.w}, wn[4] = {on.x, on.y, on.z, on.w};
    uint32_t mx[4], mn[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        mx[i] = Elem<T>::pack(fmaxf(fmaxf(-INFINITY, Elem<T>::lo(w[i])), Elem<T>::lo(wm[i])),
                              fmaxf(fmaxf(-INFINITY, Elem<T>::hi(w[i])), Elem<T>::hi(wm[i])));
        mn[i] = Elem<T>::pack(fminf(fminf(INFINITY, Elem<T>::lo(w[i])), Elem<T>::lo(wn[i])),
                              fminf(fminf(INFINITY, Elem<T>::hi(w[i])), Elem<T>::hi(wn[i])));
    }
    st[0] = make_uint4(mx[0], mx[1], mx[2], mx[3]);
    st[kHeadDim / 8] = make_uint4(mn[0], mn[1], mn[2], mn[3]);
}

template <class T>
void launch_append_token(const LayerParams& lp, const PagedParams& kv, const uint4* k4, const uint4* v4, const int* cu_new,
                         const int* start_pos, hipStream_t stream) {
    const dim3 grid((kv.batch * lp.Hkv + 7) / 8), block(256);
    if (kv.kv_bits == 8)
        hipLaunchKernelGGL((append_token_kernel<T, 8>), grid, block, 0, stream, lp, kv, k4, v4, cu_new, start_pos);
    else if (kv.kv_bits == 4)
        hipLaunchKernelGGL((append_token_kernel<T, 4>), grid, block, 0, stream, lp, kv, k4, v4, cu_new, start_pos);
    else
        hipLaunchKernelGGL((append_token_kernel<T, 16>), grid, block, 0, stream, lp, kv, k4, v4, cu_new, start_pos);
}

hipError_t launch_append_kv(int dtype, const LayerParams& lp, const PagedParams& kv, const void* k_new, const void* v_new,
                            const int* cu_new, const int* start_pos, int max_new_per_seq, hipStream_t stream) {
    if (max_new_per_seq == 1) {
        if (dtype == 0)
            launch_append_token<F16>(lp, kv, reinterpret_cast<const uint4*>(k_new), reinterpret_cast<const uint4*>(v_new), cu_new,
                                     start_pos, stream);
        else
            launch_append_token<BF16>(lp, kv, reinterpret_cast<const uint4*>(k_new), reinterpret_cast<const uint4*>(v_new), cu_new,
                                      start_pos, stream);
        return hipGetLastError();
    }
    // the new tokens of a sequence touch at most ceil(n / N_P) + 1 physical pages
    dim3 grid((max_new_per_seq + lp.NP - 1) / lp.NP + 1, lp.Hkv, kv.batch);
    dim3 block(kWave * lp.g);
    const uint4* k4 = reinterpret_cast<const uint4*>(k_new);
    const uint4* v4 = reinterpret_cast<const uint4*>(v_new);
    if (kv.kv_bits == 8) {
        if (dtype == 0)
            hipLaunchKernelGGL((append_kv_kernel<F16, 8>), grid, block, 0, stream, lp, kv, k4, v4, cu_new, start_pos);
        else
            hipLaunchKernelGGL((append_kv_kernel<BF16, 8>), grid, block, 0, stream, lp, kv, k4, v4, cu_new, start_pos);
    } else if (kv.kv_bits == 4) {
        if (dtype == 0)
            hipLaunchKernelGGL((append_kv_kernel<F16, 4>), grid, block, 0, stream, lp, kv, k4, v4, cu_new, start_pos);
        else
            hipLaunchKernelGGL((append_kv_kernel<BF16, 4>), grid, block, 0, stream, lp, kv, k4, v4, cu_new, start_pos);
    } else if (dtype == 0) {
        hipLaunchKernelGGL((append_kv_kernel<F16, 16>), grid, block, 0, stream, lp, kv, k4, v4, cu_new, start_pos);
    } else {
        hipLaunchKernelGGL((append_kv_kernel<BF16, 16>), grid, block, 0, stream, lp, kv, k4, v4, cu_new, start_pos);
    }
    return hipGetLastError();
}

hipError_t preload_stats_kernels() {
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&page_stats_kernel<F16>));
}

hipError_t launch_page_stats(int dtype, const LayerParams& lp, const PagedParams& kv, const int* start_pos,
                             int tail_pages, const HeadList& heads, hipStream_t stream) {
    if (heads.count == 0) return hipSuccess;
    dim3 grid(tail_pages, heads.count, kv.batch);
    dim3 block(kWave * lp.g);
    if (dtype == 0)
        hipLaunchKernelGGL(page_stats_kernel<F16>, grid, block, 0, stream, lp, kv, start_pos, heads);
    else
        hipLaunchKernelGGL(page_stats_kernel<BF16>, grid, block, 0, stream, lp, kv, start_pos, heads);
    return hipGetLastError();
}

}  // namespace lserve
