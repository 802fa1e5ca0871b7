// Paged sparse decode attention (Sec. 3.6): one query token per sequence attends only the pages of
// its index table -- the selector's list (plus pages newer than the selection) for dense heads,
// sink + local pages for streaming heads.  Both kinds run in one launch.
//
// The work is GEMV-shaped (n <= 8 query rows per KV head) and bound by HBM bandwidth: each page is a 2 * N_P * 256-byte
// contiguous K / V slab read with 16-byte loads (16 lanes per token row).  Scores come from small matrix products or, without a
// group and over small pages, from packed 16-bit dot instructions (see scores_by_matrix), values are weighted in fp32, and the
// softmax is kept online per wavefront.
//
// Work distribution: a launch is only a few thousand pages, far too few for the hardware scheduler
// to even out, so the page lists of all (sequence, KV head) pairs are laid end to end and cut into
// G equal ranges, G = resident workgroups of the whole chip.  A workgroup resolves the table entries
// of its pages in one go (one lane per page) and then streams its pages, the next page's slabs in
// flight while it works on the current one; its four wavefronts each take a quarter of a page's
// tokens.  A range may cross list boundaries; every (workgroup, list) piece yields either the final
// result (the list lies inside the range) or a partial (max, sum, unnormalised output) at slot
// workgroup + list index; the workgroup that delivers the last piece of a list folds them in slot order.
// Reduction orders are fixed, so results are deterministic.
//
// Pages may also hold quantised rows (Sec. 3.2: 8- or 4-bit codes with one fp16 scale and zero point per
// token, stored after the page's rows).  The kernel is the same with the slab loads and the per-page
// arithmetic swapped (template parameter BITS); see quantised_quarter_page.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace lserve {

namespace {

constexpr int kDecodeThreads = 256;
constexpr int kDecodeWaves = kDecodeThreads / kWave;
constexpr int kMaxBlocksPerCU = 4;       // upper bound used to size the workspace
constexpr int kBlocksPerCU = 2;          // measured best on MI355X: more resident workgroups only queue up in the fabric
constexpr int kSlackFromEntries = 8;     // ranges at least this long model the cost of a list boundary (see make_plan)
constexpr float kLn2 = 0.6931471805599453f;

// ---- index tables --------------------------------------------------------------------------------

struct PageList {
    int len;          // number of pages attended
    int head;         // entries [0, head) come from `first`, the rest are consecutive from `tail_start`
    int tail_start;
    const int* first; // selected pages (NULL for streaming heads: entry i is page i)
};

// Index table of KV head hk (Sec. 3.6): streaming heads list sink and local pages, dense heads the
// selection followed by every page created after it.
__device__ __forceinline__ PageList make_page_list(const LayerParams& lp, int b, int hk, int L,
                                                   const int* sel_pages, const int* sel_count,
                                                   const int* sel_seq_len, int sel_stride) {
    PageList pl;
    const int P = ceil_div(L, lp.NP);
    if ((lp.streaming_mask >> hk) & 1ull) {
        pl.head = min(lp.sink_pages, P);
        pl.tail_start = max(pl.head, P - lp.local_pages);
        pl.first = nullptr;
    } else {
        pl.head = sel_count[b * lp.Hkv + hk];
        pl.tail_start = ceil_div(sel_seq_len[b], lp.NP);
        pl.first = sel_pages + ((size_t)b * lp.Hkv + hk) * sel_stride;
    }
    pl.len = pl.head + max(0, P - pl.tail_start);
    return pl;
}

__device__ __forceinline__ int page_of(const PageList& pl, int i) {
    if (i < pl.head) return pl.first ? pl.first[i] : i;
    return pl.tail_start + (i - pl.head);
}

// ---- per-wave online softmax over quarter pages --------------------------------------------------
//
// A wave owns NP / 4 consecutive tokens of every page.  Keys and values use different lane maps:
//   keys  : LPT lanes per token; lane l reads 16-byte chunks LPT * j + l % LPT of token l / LPT, so a
//           dot product over the 128 channels needs only log2(LPT) cross-lane steps (LPT = 4 for
//           N_P >= 64: every 4 lanes read 64 contiguous bytes);
//   values: 16 lanes per token row, lane (r, c) reads chunk c of tokens 4 it + r, so the output
//           accumulators stay at 8 channels per lane and head.
// The softmax weights cross from one map to the other through a few hundred bytes of LDS.

template <int NP> struct KeyMap {
    static constexpr int LPT = NP >= 64 ? 4 : (NP == 32 ? 8 : 16);  // lanes per token
    static constexpr int TPP = kWave / LPT;                          // tokens per pass of the wave
    static constexpr int PASSES = (NP / 4) / TPP;                    // 2 for N_P = 128, else 1
    static constexpr int KLOADS = 16 / LPT;                          // 16-byte chunks per lane and token
    static constexpr int ITS = NP / 16;                              // 16-byte loads per lane and slab
};

// 16-bit rows: are the scores taken on the matrix cores (matrix_quarter_page)?  Not without a group, where the vector form is as quick
// (32 sequences of 4096 .. 131072, 32 / 32 heads, 657 and 671 us a pass), nor for two heads over pages of 128 tokens (30 of 300 .. 9000,
// 32 / 16 heads, 302 and 308); a quarter of a smaller page has fewer tokens than a product has columns.
constexpr bool scores_by_matrix(int n, int np) { return np == 64 ? n >= 2 : np == 128 && n >= 3; }

template <int NP, int BITS> struct Slabs;
template <int NP> struct Slabs<NP, 16> {
    uint4 k[KeyMap<NP>::ITS], v[KeyMap<NP>::ITS];
};
// Quantised pages (N_P = 64 only): a token row is 128 one-byte codes.  Lane (t, g) = (lane % 16, lane / 16) reads, as
// the matrix instructions take their operands, two 16-byte chunks of the key row of token t, and eight codes (its
// t-th eight channels) of the value rows of tokens 4 g .. 4 g + 3.  The (scale, zero) pairs of both the K and the V
// row of token t travel with it.
template <> struct Slabs<64, 8> {
    uint4 k[2];
    uint2 v[4];
    uint32_t ksz, vsz;
};
// 4-bit codes: a token row is 64 bytes, byte j of every 4-byte word holding channel 8 g + j in its low and
// channel 8 g + 4 + j in its high half (g = index of the word).  One 16-byte chunk per key lane, one word per
// value lane.
template <> struct Slabs<64, 4> {
    uint4 k[1];
    uint32_t v[4];
    uint32_t ksz, vsz;
};

// Slab loads: a wave-uniform slab address plus a 32-bit lane offset (and a constant), which is the form the load
// instruction takes as it is; with 64-bit lane addresses the additions were a third of the vector instructions of the
// quantised kernels.  live: all ones, or 0 for a request that only keeps the count of loads in flight what it is (see
// the page loop): every lane then reads the slab's first bytes.
template <class V> __device__ __forceinline__ V load_at(const uint4* slab, unsigned lane_bytes, unsigned constant_bytes) {
    return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(slab) + lane_bytes + constant_bytes);
}

template <int N, int NP>
__device__ __forceinline__ void load_k(Slabs<NP, 16>& s, const uint4* kslab, int tok0, int lane, unsigned live) {
    using M = KeyMap<NP>;
    if constexpr (scores_by_matrix(N, NP)) {  // lane (t, g): the chunks g, g + 4 ... of token t, as the products take them
        const unsigned at = (unsigned)((tok0 + lane % 16) * (kHeadDim / 8) + lane / 16) * 16u & live;
#pragma unroll
        for (int ps = 0; ps < M::PASSES; ++ps)
#pragma unroll
            for (int j = 0; j < 4; ++j) s.k[4 * ps + j] = load_at<uint4>(kslab, at, (ps * 16 * (kHeadDim / 8) + 4 * j) * 16u);
        return;
    }
    const unsigned at = (unsigned)((tok0 + lane / M::LPT) * (kHeadDim / 8) + lane % M::LPT) * 16u & live;
#pragma unroll
    for (int ps = 0; ps < M::PASSES; ++ps)
#pragma unroll
        for (int j = 0; j < M::KLOADS; ++j)
            s.k[ps * M::KLOADS + j] = load_at<uint4>(kslab, at, (ps * M::TPP * (kHeadDim / 8) + M::LPT * j) * 16u);
}

template <int NP>
__device__ __forceinline__ void load_v(Slabs<NP, 16>& s, const uint4* vslab, int tok0, int r, int c, int, unsigned live) {
    const unsigned at = (unsigned)((tok0 + r) * (kHeadDim / 8) + c) * 16u & live;
#pragma unroll
    for (int it = 0; it < KeyMap<NP>::ITS; ++it) s.v[it] = load_at<uint4>(vslab, at, 4 * it * kHeadDim * 2u);
}

template <int N> __device__ __forceinline__ void load_k(Slabs<64, 4>& s, const uint4* kslab, int tok0, int lane, unsigned live) {
    const int tok = tok0 + lane % 16;
    s.k[0] = load_at<uint4>(kslab, (unsigned)(tok * (kHeadDim / 32) + lane / 16) * 16u & live, 0);
    s.ksz = load_at<uint32_t>(kslab + 64 * (kHeadDim / 32), (unsigned)tok * 4u & live, 0);
}
__device__ __forceinline__ void load_v(Slabs<64, 4>& s, const uint4* vslab, int tok0, int r, int c, int lane, unsigned live) {
    const unsigned at = (unsigned)((tok0 + 4 * r) * (kHeadDim / 8) + c) * 4u & live;
#pragma unroll
    for (int it = 0; it < 4; ++it) s.v[it] = load_at<uint32_t>(vslab, at, it * kHeadDim / 2u);
    s.vsz = load_at<uint32_t>(vslab + 64 * (kHeadDim / 32), (unsigned)(tok0 + lane % 16) * 4u & live, 0);
}
template <int N> __device__ __forceinline__ void load_k(Slabs<64, 8>& s, const uint4* kslab, int tok0, int lane, unsigned live) {
    const int tok = tok0 + lane % 16;
    const unsigned at = (unsigned)(tok * (kHeadDim / 16) + lane / 16) * 16u & live;
#pragma unroll
    for (int j = 0; j < 2; ++j) s.k[j] = load_at<uint4>(kslab, at, 4 * j * 16u);
    s.ksz = load_at<uint32_t>(kslab + 64 * (kHeadDim / 16), (unsigned)tok * 4u & live, 0);
}
__device__ __forceinline__ void load_v(Slabs<64, 8>& s, const uint4* vslab, int tok0, int r, int c, int lane, unsigned live) {
    const unsigned at = (unsigned)((tok0 + 4 * r) * (kHeadDim / 8) + c) * 8u & live;
#pragma unroll
    for (int it = 0; it < 4; ++it) s.v[it] = load_at<uint2>(vslab, at, it * kHeadDim);
    s.vsz = load_at<uint32_t>(vslab + 64 * (kHeadDim / 16), (unsigned)(tok0 + lane % 16) * 4u & live, 0);
}

typedef float floatx4_t __attribute__((ext_vector_type(4)));

// Factor of weight * scale on its way to fp16: clear of the subnormals, and below 65504 for scales up to 1023.  The quantiser
// makes larger ones (4-bit rows that span more than 15350, 8-bit ones more than 260000): from the first weight that would
// not fit on, the wave does without the factor, which fits any weight (at most 1) times any scale.
constexpr float kWeightScale = 64.f, kMaxWeight = 65504.f;

template <int N, int BITS> struct WaveState {
    // Quantised pages: lane (t, g) keeps the softmax of query heads g and g + 4 (the latter for groups above four): their
    // running maxima (equal over the sixteen lanes of g), and its token's share of the sums of weights and of weight *
    // zero point.  acc[m][j] is the output of head g + 4 j in channel 8 t + m, in units of the stored weights and codes
    // (see quantised_quarter_page); acc[m][2], acc[m][3] belong to no head.  q: the queries as matrix operands.
    static constexpr int kHeadsPerLane = (N + 3) / 4;
    // weight_scale: the factor the weights are stored with, one for the wave (kWeightScale or 1).
    float m[kHeadsPerLane], l[kHeadsPerLane], z[kHeadsPerLane], q_sum[kHeadsPerLane], weight_scale;
    floatx4_t acc[8];
    uint4 q[4];
    __device__ __forceinline__ void reset() {
        weight_scale = kWeightScale;
#pragma unroll
        for (int j = 0; j < kHeadsPerLane; ++j) {
            m[j] = -INFINITY;
            l[j] = 0.f;
            z[j] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    }
};
template <int N> struct WaveState<N, 16> {
    float m[N], l[N], o[N][8];
    __device__ __forceinline__ void reset() {
#pragma unroll
        for (int hh = 0; hh < N; ++hh) {
            m[hh] = -INFINITY;
            l[hh] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) o[hh][i] = 0.f;
        }
    }
};

// 16-bit rows with scores from the matrix cores: lane (t, g) keeps the softmax of heads g and g + 4 as over quantised pages, the
// outputs are those of the vector form.
template <int N> struct MatrixState {
    static constexpr int kHeadsPerLane = (N + 3) / 4;
    float m[kHeadsPerLane], l[kHeadsPerLane], o[N][8];
    uint4 q[4];
    __device__ __forceinline__ void reset() {
#pragma unroll
        for (int j = 0; j < kHeadsPerLane; ++j) {
            m[j] = -INFINITY;
            l[j] = 0.f;
        }
#pragma unroll
        for (int hh = 0; hh < N; ++hh)
#pragma unroll
            for (int i = 0; i < 8; ++i) o[hh][i] = 0.f;
    }
};
template <int N, int NP, int BITS>
using StateOf = std::conditional_t<BITS == 16 && scores_by_matrix(N, NP), MatrixState<N>, WaveState<N, BITS>>;

constexpr int p_row(int n) { return n <= 4 ? 4 : 8; }  // floats per token row of the weight buffer

// Sum over the LPT lanes that share a token; every one of them receives the total.
template <int LPT> __device__ __forceinline__ float token_sum(float x) {
    x += dpp_f<kDppXor1>(x);
    x += dpp_f<kDppXor2>(x);
    if (LPT >= 8) x += dpp_f<kDppHalfMirror>(x);
    if (LPT >= 16) x += dpp_f<kDppMirror>(x);
    return x;
}

// Maximum over the wave of a value that is already equal inside every group of four lanes.
__device__ __forceinline__ float wave_max_of_quads(float x) {
    x = fmaxf(x, dpp_f<kDppHalfMirror>(x));
    x = fmaxf(x, dpp_f<kDppMirror>(x));
    return rows4_max(x);
}

// Adds weights * values of a quarter page to the outputs: four rows to a pass, sixteen lanes to a row.
template <class T, int N, int NP>
__device__ __forceinline__ void add_values(float (&o)[N][8], const float* p_lds, const Slabs<NP, 16>& cur, int valid, int tok0, int r) {
    using M = KeyMap<NP>;
    constexpr int PR = p_row(N);
    const bool tail = valid < NP;
#pragma unroll
    for (int it = 0; it < M::ITS; ++it) {
        uint4 vv = cur.v[it];
        if (tail && tok0 + 4 * it + r >= valid) vv = make_uint4(0, 0, 0, 0);  // slots past the end may hold anything
        const uint32_t vw[4] = {vv.x, vv.y, vv.z, vv.w};
        float pv[PR];
#pragma unroll
        for (int x4 = 0; x4 < PR / 4; ++x4) {
            const float4 t4 = *reinterpret_cast<const float4*>(p_lds + (4 * it + r) * PR + 4 * x4);
            pv[4 * x4] = t4.x;
            pv[4 * x4 + 1] = t4.y;
            pv[4 * x4 + 2] = t4.z;
            pv[4 * x4 + 3] = t4.w;
        }
#pragma unroll
        for (int hh = 0; hh < N; ++hh) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                o[hh][2 * i] = __builtin_fmaf(pv[hh], Elem<T>::lo(vw[i]), o[hh][2 * i]);
                o[hh][2 * i + 1] = __builtin_fmaf(pv[hh], Elem<T>::hi(vw[i]), o[hh][2 * i + 1]);
            }
        }
    }
}

// One quarter page.  q_lds: [N][16] 16-byte chunks of the group's queries; p_lds: this wave's
// [NP / 4][p_row(N)] weight buffer.  `valid` = tokens of the page below the sequence length.
template <class T, int N, int NP>
__device__ __forceinline__ void process_quarter_page(WaveState<N, 16>& st, const uint4* q_lds, float* p_lds,
                                                     Slabs<NP, 16>& cur, int valid, int tok0, int lane,
                                                     float scale_log2) {
    using M = KeyMap<NP>;
    constexpr int PR = p_row(N);
    const int r = lane / 16;
    float s[M::PASSES][N];
#pragma unroll
    for (int ps = 0; ps < M::PASSES; ++ps)
#pragma unroll
        for (int hh = 0; hh < N; ++hh) s[ps][hh] = 0.f;
#pragma unroll
    for (int j = 0; j < M::KLOADS; ++j) {
#pragma unroll
        for (int hh = 0; hh < N; ++hh) {
            const uint4 qv = q_lds[hh * 16 + M::LPT * j + lane % M::LPT];
            const uint32_t qw[4] = {qv.x, qv.y, qv.z, qv.w};
#pragma unroll
            for (int ps = 0; ps < M::PASSES; ++ps) {
                const uint4 kv4 = cur.k[ps * M::KLOADS + j];
                const uint32_t kw[4] = {kv4.x, kv4.y, kv4.z, kv4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) s[ps][hh] = Elem<T>::dot2(qw[i], kw[i], s[ps][hh]);
            }
        }
    }
    const bool tail = valid < NP;
#pragma unroll
    for (int ps = 0; ps < M::PASSES; ++ps) {
        const bool dead = tail && tok0 + ps * M::TPP + lane / M::LPT >= valid;
#pragma unroll
        for (int hh = 0; hh < N; ++hh) {
            const float x = token_sum<M::LPT>(s[ps][hh]) * scale_log2;
            s[ps][hh] = dead ? -INFINITY : x;
        }
    }
#pragma unroll
    for (int hh = 0; hh < N; ++hh) {
        float pm = s[0][hh];
#pragma unroll
        for (int ps = 1; ps < M::PASSES; ++ps) pm = fmaxf(pm, s[ps][hh]);
        pm = wave_max_of_quads(pm);
        if (pm > st.m[hh]) {  // wave-uniform: rescale only when the running maximum moves
            const float alpha = __builtin_amdgcn_exp2f(st.m[hh] - pm);
            st.m[hh] = pm;
            st.l[hh] *= alpha;
#pragma unroll
            for (int i = 0; i < 8; ++i) st.o[hh][i] *= alpha;
        }
        const float m_safe = st.m[hh] == -INFINITY ? 0.f : st.m[hh];
#pragma unroll
        for (int ps = 0; ps < M::PASSES; ++ps) {
            s[ps][hh] = __builtin_amdgcn_exp2f(s[ps][hh] - m_safe);
            st.l[hh] += s[ps][hh];  // counted once per lane of the token: divided by LPT at the end
        }
    }
    if (lane % M::LPT == 0) {
#pragma unroll
        for (int ps = 0; ps < M::PASSES; ++ps) {
            float* dst = p_lds + (ps * M::TPP + lane / M::LPT) * PR;
#pragma unroll
            for (int hh = 0; hh < N; ++hh) dst[hh] = s[ps][hh];
        }
    }
    __builtin_amdgcn_wave_barrier();
    add_values<T, N, NP>(st.o, p_lds, cur, valid, tok0, r);
    __builtin_amdgcn_wave_barrier();
}

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf168_t __attribute__((ext_vector_type(8)));
template <class T> __device__ __forceinline__ floatx4_t mfma_16x16x32(uint4 a, uint4 b, floatx4_t c) {
    if constexpr (std::is_same<T, F16>::value)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf168_t, a), __builtin_bit_cast(bf168_t, b), c, 0, 0, 0);
}

// One quarter page of 16-bit rows under a group of heads, scores from the matrix cores: Q (heads x 128) * K^T (128 x tokens), four
// v_mfma_f32_16x16x32 per sixteen tokens, with the heads in the rows that quantised_quarter_page has them in.  A lane then has the
// score of one token under one head in four instead of a quarter of it under every head: an exponential, a maximum over sixteen lanes
// and a sum per four heads, where packed dot products took 16 instructions and three cross-lane sums and maxima per head, and the queries are
// operands in registers.  Weights stay in fp32 and meet the values in the vector pipe as before, so sums are as exact as they were.
// The vector instructions bounded this path under large groups and the latency of a page under small ones.  Passes of four steps, us: 16
// sequences of 32768, 32 / 8 heads, 155.6 -> 152.0; of 16384, 64 / 8 heads, 186 -> 154, over pages of 128 tokens (eight of 20000) 167 -> 133; four
// of 262144 108 -> 104, one of 4000 59.3 -> 57.4; 57 of 290 .. 6691 337 -> 282.
template <class T, int N, int NP>
__device__ __forceinline__ void matrix_quarter_page(MatrixState<N>& st, float* p_lds, Slabs<NP, 16>& cur, int valid, int tok0,
                                                    int lane, float scale_log2) {
    constexpr int HPL = MatrixState<N>::kHeadsPerLane, PASSES = NP / 64, PR = p_row(N);
    const int t = lane % 16, g = lane / 16;
    floatx4_t s[PASSES];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        s[ps] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) s[ps] = mfma_16x16x32<T>(st.q[j], cur.k[4 * ps + j], s[ps]);
    }
    const bool tail = valid < NP;
    float x[HPL][PASSES], pm[HPL];
    bool moved = false;
#pragma unroll
    for (int j = 0; j < HPL; ++j) {
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            x[j][ps] = tail && tok0 + 16 * ps + t >= valid ? -INFINITY : s[ps][j] * scale_log2;
            pm[j] = ps == 0 ? x[j][ps] : fmaxf(pm[j], x[j][ps]);
        }
        pm[j] = fmaxf(pm[j], dpp_f<kDppXor1>(pm[j]));
        pm[j] = fmaxf(pm[j], dpp_f<kDppXor2>(pm[j]));
        pm[j] = fmaxf(pm[j], dpp_f<kDppHalfMirror>(pm[j]));
        pm[j] = fmaxf(pm[j], dpp_f<kDppMirror>(pm[j]));
        moved |= pm[j] > st.m[j];
    }
    if (__any(moved)) {
        float alpha[HPL];
#pragma unroll
        for (int j = 0; j < HPL; ++j) {
            const float m_new = fmaxf(st.m[j], pm[j]);
            alpha[j] = m_new > st.m[j] ? __builtin_amdgcn_exp2f(st.m[j] - m_new) : 1.f;
            st.m[j] = m_new;
            st.l[j] *= alpha[j];
        }
#pragma unroll
        for (int hh = 0; hh < N; ++hh) {
            const float a = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha[hh / 4]), 16 * (hh % 4)));
#pragma unroll
            for (int i = 0; i < 8; ++i) st.o[hh][i] *= a;
        }
    }
#pragma unroll
    for (int j = 0; j < HPL; ++j) {
        const float m_safe = st.m[j] == -INFINITY ? 0.f : st.m[j];
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const float p = __builtin_amdgcn_exp2f(x[j][ps] - m_safe);
            st.l[j] += p;
            p_lds[(16 * ps + t) * PR + 4 * j + g] = p;
        }
    }
    __builtin_amdgcn_wave_barrier();
    add_values<T, N, NP>(st.o, p_lds, cur, valid, tok0, g);
    __builtin_amdgcn_wave_barrier();
}

constexpr float kCodeUnit = 0x1p-24f;  // value of the fp16 number whose bits are 1

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));

// The same over a quantised quarter page, on the matrix cores.  With k = code * scale + zero the logit of a token is
//   q . k = scale * (q . code) + zero * sum(q),
// and with the weight folded into the scale of a value row,
//   sum_t p_t v_t = sum_t (p_t scale_t) code_t + sum_t p_t zero_t,
// whose second sum no channel distinguishes: one number per query head.  Both first sums are products of small
// matrices over the sixteen tokens of a wavefront's quarter page,
//   scores (heads x tokens) = Q (heads x 128) * codes (128 x tokens)    v_mfma_f32_16x16x32_f16, four of them
//   out (heads x channels) += weights (heads x 16) * codes (16 x 128)   v_mfma_f32_16x16x16_f16, one per 16 channels
// with query head g + 4 j in row 4 g + j, so that lane (t, g) receives the scores of its own heads g and g + 4 and, later,
// their outputs; the other rows hold copies whose results nobody reads.
// A code needs no conversion: a byte (or nibble) alone in the low bits of a 16-bit half is the fp16 subnormal
// code * 2^-24, which the matrix instructions of gfx950 take at its value, so one byte permute (or mask) yields two operands
// and the unit is folded into factors that are there anyway.  Nibbles four bits up stand for 16 * code: they get products
// (keys) or output channels (values) of their own.  Weights are rounded to fp16 (2^-11 relative), times kWeightScale, before
// they meet the codes, and cross lanes through LDS; the denominator keeps the unrounded weights.
// The instruction count, not the memory system, bounds this path (a page is half or a quarter of the bytes for the same
// number of tokens): with packed dot products it took about 215 vector instructions per quarter page and four heads, now
// about 90.  64 sequences of 9K .. 24K tokens, 32 / 8 heads, 4096-token budget: 60.0 -> 40 us over 4-bit pages, 65.3 ->
// 58 us over 8-bit ones (324 MB: 5.6 TB/s); eight heads per group at batch 16: 31.7 -> 19.6 and 40.1 -> 21.9 us.
// p_lds is read as fp16 [heads][16 tokens].
template <int N, int BITS>
__device__ __forceinline__ void quantised_quarter_page(WaveState<N, BITS>& st, float* p_lds, Slabs<64, BITS>& cur, int valid,
                                                       int tok0, int lane, float scale_log2) {
    static_assert(BITS == 8 || BITS == 4, "quantised pages");
    constexpr int HPL = WaveState<N, BITS>::kHeadsPerLane;
    const int t = lane % 16, g = lane / 16;
    auto mfma_k = [](uint4 a, uint4 b, floatx4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
    };
    floatx4_t s = {0.f, 0.f, 0.f, 0.f};
    if constexpr (BITS == 8) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t w[4] = {cur.k[j].x, cur.k[j].y, cur.k[j].z, cur.k[j].w};
#pragma unroll
            for (int u = 0; u < 2; ++u) {  // selector byte 0x0c: zero
                const uint4 c = make_uint4(__builtin_amdgcn_perm(0u, w[2 * u], 0x0c010c00u), __builtin_amdgcn_perm(0u, w[2 * u], 0x0c030c02u),
                                           __builtin_amdgcn_perm(0u, w[2 * u + 1], 0x0c010c00u), __builtin_amdgcn_perm(0u, w[2 * u + 1], 0x0c030c02u));
                s = mfma_k(st.q[2 * j + u], c, s);
            }
        }
    } else {
        const uint32_t w[4] = {cur.k[0].x, cur.k[0].y, cur.k[0].z, cur.k[0].w};
        floatx4_t s16 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint32_t a = w[2 * u], b = w[2 * u + 1], a8 = a >> 8, b8 = b >> 8;
            s = mfma_k(st.q[2 * u], make_uint4(a & 0x000f000fu, a8 & 0x000f000fu, b & 0x000f000fu, b8 & 0x000f000fu), s);
            s16 = mfma_k(st.q[2 * u + 1], make_uint4(a & 0x00f000f0u, a8 & 0x00f000f0u, b & 0x00f000f0u, b8 & 0x00f000f0u), s16);
        }
#pragma unroll
        for (int j = 0; j < HPL; ++j) s[j] = __builtin_fmaf(0.0625f, s16[j], s[j]);
    }
    const bool dead = valid < 64 && tok0 + t >= valid;
    const half2_t ksz = __builtin_bit_cast(half2_t, cur.ksz), vsz = __builtin_bit_cast(half2_t, cur.vsz);
    const float k_scale = (float)ksz[0] * (scale_log2 / kCodeUnit), k_zero = (float)ksz[1] * scale_log2;
    // slots past the end may hold anything
    const float v_scale = dead ? 0.f : (float)vsz[0] * st.weight_scale, v_zero = dead ? 0.f : (float)vsz[1];
    _Float16* w_lds = reinterpret_cast<_Float16*>(p_lds);
    float w[HPL];
#pragma unroll
    for (int j = 0; j < HPL; ++j) {
        const float x = dead ? -INFINITY : __builtin_fmaf(k_scale, s[j], k_zero * st.q_sum[j]);
        float pm = x;  // maximum over the sixteen tokens
        pm = fmaxf(pm, dpp_f<kDppXor1>(pm));
        pm = fmaxf(pm, dpp_f<kDppXor2>(pm));
        pm = fmaxf(pm, dpp_f<kDppHalfMirror>(pm));
        pm = fmaxf(pm, dpp_f<kDppMirror>(pm));
        const bool moved = pm > st.m[j];
        if (__any(moved)) {  // rare after the first pages: some head's running maximum moves
            const float alpha = moved ? __builtin_amdgcn_exp2f(st.m[j] - pm) : 1.f;
            st.m[j] = moved ? pm : st.m[j];
            st.l[j] *= alpha;
            st.z[j] *= alpha;
#pragma unroll
            for (int i = 0; i < 8; ++i) st.acc[i][j] *= alpha;
        }
        const float m_safe = st.m[j] == -INFINITY ? 0.f : st.m[j];
        const float p = dead ? 0.f : __builtin_amdgcn_exp2f(x - m_safe);
        st.l[j] += p;
        st.z[j] = __builtin_fmaf(p, v_zero, st.z[j]);
        w[j] = p * v_scale;
    }
    // Hardly ever: a value row of a very large scale (known before the weights are), and a weight for it that does not fit.
    if (__any(v_scale > kMaxWeight) && __any(HPL == 1 ? w[0] > kMaxWeight : fmaxf(w[0], w[HPL - 1]) > kMaxWeight)) {
        const float down = 1.f / kWeightScale;  // (a second time cannot be: without the factor every weight fits)
        st.weight_scale = 1.f;
#pragma unroll
        for (int j = 0; j < HPL; ++j) {
            w[j] *= down;
#pragma unroll
            for (int i = 0; i < 8; ++i) st.acc[i][j] *= down;
        }
    }
#pragma unroll
    for (int j = 0; j < HPL; ++j) w_lds[(4 * j + g) * 16 + t] = (_Float16)w[j];
    __builtin_amdgcn_wave_barrier();
    // row t of the operand: query head t / 4 + 4 (t % 4), tokens 4 g .. 4 g + 3 (rows without a head repeat one)
    const int head = t / 4 + 4 * (t % 4 < HPL ? t % 4 : 0);
    const half4_t weights = __builtin_bit_cast(half4_t, *reinterpret_cast<const uint2*>(w_lds + head * 16 + 4 * g));
    auto mfma_v = [&](uint32_t lo, uint32_t hi, floatx4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x16f16(weights, __builtin_bit_cast(half4_t, make_uint2(lo, hi)), c, 0, 0, 0);
    };
    if constexpr (BITS == 8) {
        const uint32_t v[4][2] = {{cur.v[0].x, cur.v[0].y}, {cur.v[1].x, cur.v[1].y}, {cur.v[2].x, cur.v[2].y}, {cur.v[3].x, cur.v[3].y}};
        constexpr uint32_t pick[4] = {0x0c040c00u, 0x0c050c01u, 0x0c060c02u, 0x0c070c03u};  // byte i of two tokens
#pragma unroll
        for (int i = 0; i < 8; ++i)
            st.acc[i] = mfma_v(__builtin_amdgcn_perm(v[1][i / 4], v[0][i / 4], pick[i % 4]),
                               __builtin_amdgcn_perm(v[3][i / 4], v[2][i / 4], pick[i % 4]), st.acc[i]);
    } else {
        constexpr uint32_t pick[4] = {0x0c040c00u, 0x0c050c01u, 0x0c060c02u, 0x0c070c03u};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t lo = __builtin_amdgcn_perm(cur.v[1], cur.v[0], pick[i]), hi = __builtin_amdgcn_perm(cur.v[3], cur.v[2], pick[i]);
            st.acc[i] = mfma_v(lo & 0x000f000fu, hi & 0x000f000fu, st.acc[i]);
            st.acc[4 + i] = mfma_v(lo & 0x00f000f0u, hi & 0x00f000f0u, st.acc[4 + i]);
        }
    }
    __builtin_amdgcn_wave_barrier();
}

// The queries of a list as this lane's matrix operands, from the fp16 rows stage_query() left in LDS: row t holds query
// head t / 4 + 4 (t % 4) (rows without a head repeat one), channels in the order in which the codes of a key row come.
template <int N, int BITS>
__device__ __forceinline__ void load_query_operands(WaveState<N, BITS>& st, const uint4* q_lds, const float* q_sum, int lane) {
    constexpr int HPL = WaveState<N, BITS>::kHeadsPerLane;
    const int t = lane % 16, g = lane / 16;
    const int head = min(t / 4 + 4 * (t % 4 < HPL ? t % 4 : 0), N - 1);
    if constexpr (BITS == 8) {
#pragma unroll
        for (int m = 0; m < 4; ++m) st.q[m] = q_lds[head * 16 + 2 * (4 * (m / 2) + g) + m % 2];
    } else {
        auto low = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); };   // even elements of two words
        auto high = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); };  // odd ones
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint4 a = q_lds[head * 16 + 4 * g + 2 * u], b = q_lds[head * 16 + 4 * g + 2 * u + 1];
            st.q[2 * u] = make_uint4(low(a.x, a.y), high(a.x, a.y), low(b.x, b.y), high(b.x, b.y));
            st.q[2 * u + 1] = make_uint4(low(a.z, a.w), high(a.z, a.w), low(b.z, b.w), high(b.z, b.w));
        }
    }
#pragma unroll
    for (int j = 0; j < HPL; ++j) st.q_sum[j] = q_sum[min(g + 4 * j, N - 1)];
}

template <int N>
__device__ __forceinline__ void load_query_operands(MatrixState<N>& st, const uint4* q_lds, const float*, int lane) {
    constexpr int HPL = MatrixState<N>::kHeadsPerLane;
    const int t = lane % 16, g = lane / 16;
    const int head = min(t / 4 + 4 * (t % 4 < HPL ? t % 4 : 0), N - 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) st.q[j] = q_lds[head * 16 + 4 * j + g];
}

template <class T, int N, int NP, int BITS>
__device__ __forceinline__ void process_quarter(StateOf<N, NP, BITS>& st, const uint4* q_lds, float* p_lds,
                                                Slabs<NP, BITS>& cur, int valid, int tok0, int lane, float scale_log2) {
    if constexpr (BITS == 16 && scores_by_matrix(N, NP))
        matrix_quarter_page<T, N, NP>(st, p_lds, cur, valid, tok0, lane, scale_log2);
    else if constexpr (BITS == 16)
        process_quarter_page<T, N, NP>(st, q_lds, p_lds, cur, valid, tok0, lane, scale_log2);
    else
        quantised_quarter_page<N, BITS>(st, p_lds, cur, valid, tok0, lane, scale_log2);
}

// Shared memory of a decode workgroup.
template <int N, int NP> struct DecodeShared {
    alignas(16) float o[kDecodeWaves][N][kHeadDim];   // cross-wave merge
    float m[kDecodeWaves][N], l[kDecodeWaves][N], z[kDecodeWaves][N];
    uint4 q[N * 16];                      // queries of the current group
    float q_sum[kMaxGroup];               // quantised pages only: sum over the channels of each query
    alignas(16) float p[kDecodeWaves][(NP / 4) * p_row(N)];
    unsigned arrived;                     // pieces of a cut list that were in before this workgroup's
};

// Loads the n queries of KV head hk into shared memory.  Called by the whole workgroup.
// For quantised pages the queries are converted to fp16 (exact for every bf16 value of magnitude between
// 2^-14 and 65504; larger ones saturate) and their channel sums are taken, from the converted values.
// A workgroup's range starts inside a list that is known from the launch plan alone, so the queries of that
// list and of the one after it are requested at the very start of the kernel, in parallel with the table
// look-ups, and are at hand when the first page (or the first page after a list boundary) arrives: the load
// would otherwise sit exposed between two workgroup barriers.
struct QueryAhead {
    int list;      // first list of the range; list + 1 is held too
    uint4 x[2];    // this thread's 16-byte chunk of the group's queries (threads below N * 16)
};

template <class T, int N, int NP, int BITS>
__device__ __forceinline__ void stage_query(DecodeShared<N, NP>& sm, const uint4* q, int b, int H, int hk, int list,
                                            const QueryAhead& ahead) {
    static_assert(N * 16 <= kDecodeThreads, "one pass");
    const int i = threadIdx.x;  // chunk i of the group: the 16 chunks of a query are the 16 lanes of a DPP row
    uint4 x = ahead.x[0];
    if (list == ahead.list + 1) x = ahead.x[1];
    if ((list < ahead.list || list > ahead.list + 1) && i < N * 16) x = q[((size_t)b * H + hk * N) * (kHeadDim / 8) + i];
    __syncthreads();  // earlier readers of sm.q are done
    if (BITS == 16) {
        if (i < N * 16) sm.q[i] = x;
    } else {
        float part = 0.f;
        if (i < N * 16) {
            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
            uint32_t o[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float a = fminf(fmaxf(Elem<T>::lo(w[u]), -65504.f), 65504.f);
                const float c = fminf(fmaxf(Elem<T>::hi(w[u]), -65504.f), 65504.f);
                o[u] = Elem<F16>::pack(a, c);
                part += Elem<F16>::lo(o[u]) + Elem<F16>::hi(o[u]);
            }
            sm.q[i] = make_uint4(o[0], o[1], o[2], o[3]);
        }
        part = row16_sum(part);
        if (i < N * 16 && i % 16 == 0) sm.q_sum[i / 16] = part;
    }
    __syncthreads();
}

// Partial results travel between workgroups that may sit on different XCDs, each with an L2 of its own.  They are
// written and read with agent-scope accesses (write-through stores, loads that are not served from a stale line),
// which costs those few hundred kilobytes nothing, instead of fences that write back and invalidate whole caches.
// Two floats per access (8-byte aligned).
__device__ __forceinline__ void store_shared_across_chip(float* p, float a, float b) {
    const float2 v = make_float2(a, b);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), __builtin_bit_cast(unsigned long long, v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_shared_across_chip(const float* p) {
    return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT));
}

// Leaves a wave's maxima, sums and outputs in shared memory.  16-bit pages: the four token rows of the wave are folded
// on the way, four values at a time so that row r ends up with the total of the r-th.
template <int N, int NP>
__device__ __forceinline__ void deposit_wave(WaveState<N, 16>& st, DecodeShared<N, NP>& sm, int wave, int lane) {
    const int r = lane / 16, c = lane % 16;
    constexpr int kQuads = (N + 3) / 4;
    float lrow[4 * kQuads];
#pragma unroll
    for (int hh = 0; hh < 4 * kQuads; ++hh)
        lrow[hh] = hh < N ? row16_sum(st.l[hh]) : 0.f;  // every lane of a token added the token's weight: LPT copies of the sum
#pragma unroll
    for (int q = 0; q < kQuads; ++q) {
        const float lsum = rows4_sum_scatter(lrow[4 * q], lrow[4 * q + 1], lrow[4 * q + 2], lrow[4 * q + 3]);
        if (c == 0 && 4 * q + r < N) sm.l[wave][4 * q + r] = lsum * (1.0f / KeyMap<NP>::LPT);
    }
#pragma unroll
    for (int hh = 0; hh < N; ++hh) {
#pragma unroll
        for (int q = 0; q < 2; ++q)  // lane (r, c) receives channel 8 c + 4 q + r
            sm.o[wave][hh][8 * c + 4 * q + r] =
                rows4_sum_scatter(st.o[hh][4 * q], st.o[hh][4 * q + 1], st.o[hh][4 * q + 2], st.o[hh][4 * q + 3]);
        if (lane == 0) sm.m[wave][hh] = st.m[hh];
    }
}
template <int N, int NP>
__device__ __forceinline__ void deposit_wave(MatrixState<N>& st, DecodeShared<N, NP>& sm, int wave, int lane) {
    const int t = lane % 16, g = lane / 16;
#pragma unroll
    for (int j = 0; j < MatrixState<N>::kHeadsPerLane; ++j) {
        const float l = row16_sum(st.l[j]);
        if (t == 0 && g + 4 * j < N) {
            sm.m[wave][g + 4 * j] = st.m[j];
            sm.l[wave][g + 4 * j] = l;
        }
    }
#pragma unroll
    for (int hh = 0; hh < N; ++hh)
#pragma unroll
        for (int q = 0; q < 2; ++q)  // lane (r, c) receives channel 8 c + 4 q + r
            sm.o[wave][hh][8 * t + 4 * q + g] =
                rows4_sum_scatter(st.o[hh][4 * q], st.o[hh][4 * q + 1], st.o[hh][4 * q + 2], st.o[hh][4 * q + 3]);
}
// Quantised pages: the outputs are whole already and take their unit here, the sums are added over the sixteen tokens.
template <int N, int NP, int BITS>
__device__ __forceinline__ void deposit_wave(WaveState<N, BITS>& st, DecodeShared<N, NP>& sm, int wave, int lane) {
    const int t = lane % 16, g = lane / 16;
    const float unit = st.weight_scale == kWeightScale ? 1.f / (kCodeUnit * kWeightScale) : 1.f / kCodeUnit;
    const float upper = BITS == 4 ? unit * 0.0625f : unit;
#pragma unroll
    for (int j = 0; j < WaveState<N, BITS>::kHeadsPerLane; ++j) {
        const float l = row16_sum(st.l[j]), z = row16_sum(st.z[j]);
        const int hh = g + 4 * j;
        if (hh < N) {
            if (t == 0) {
                sm.m[wave][hh] = st.m[j];
                sm.l[wave][hh] = l;
                sm.z[wave][hh] = z;
            }
            float4* dst = reinterpret_cast<float4*>(&sm.o[wave][hh][8 * t]);
            dst[0] = make_float4(st.acc[0][j] * unit, st.acc[1][j] * unit, st.acc[2][j] * unit, st.acc[3][j] * unit);
            dst[1] = make_float4(st.acc[4][j] * upper, st.acc[5][j] * upper, st.acc[6][j] * upper, st.acc[7][j] * upper);
        }
    }
}

// Folds the four waves of the workgroup, and writes either
// the final rows (out / lse) or a partial (part_o / part_ml).  Must be called by all 256 threads.
template <class T, int N, int NP, int BITS>
__device__ __forceinline__ void flush_block(StateOf<N, NP, BITS>& st, DecodeShared<N, NP>& sm, bool final_result, int H,
                                            int b, int hk, uint16_t* out, float* lse_out, float* part_o,
                                            float* part_ml, size_t part_slot) {
    deposit_wave(st, sm, threadIdx.x / kWave, threadIdx.x % kWave);
    __syncthreads();
    // one thread per (query head, four channels): N * 32 <= 256 work items
    if (threadIdx.x < N * (kHeadDim / 4)) {
        const int hh = threadIdx.x / (kHeadDim / 4), ch = threadIdx.x % (kHeadDim / 4) * 4;
        float M = sm.m[0][hh];
#pragma unroll
        for (int w = 1; w < kDecodeWaves; ++w) M = fmaxf(M, sm.m[w][hh]);
        float lt = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kDecodeWaves; ++w) {
            const float f = sm.m[w][hh] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sm.m[w][hh] - M);
            lt += sm.l[w][hh] * f;
            const float4 o4 = *reinterpret_cast<const float4*>(&sm.o[w][hh][ch]);
            const float z = BITS != 16 ? sm.z[w][hh] : 0.f;
            acc[0] += (o4.x + z) * f;
            acc[1] += (o4.y + z) * f;
            acc[2] += (o4.z + z) * f;
            acc[3] += (o4.w + z) * f;
        }
        const int h = hk * N + hh;
        if (final_result) {
            const uint2 packed = make_uint2(Elem<T>::pack(acc[0] / lt, acc[1] / lt), Elem<T>::pack(acc[2] / lt, acc[3] / lt));
            *reinterpret_cast<uint2*>(out + ((size_t)b * H + h) * kHeadDim + ch) = packed;
            if (lse_out && ch == 0) lse_out[b * H + h] = (M + __builtin_amdgcn_logf(lt)) * kLn2;
        } else {
            const size_t pi = part_slot * N + hh;
            store_shared_across_chip(part_o + pi * kHeadDim + ch, acc[0], acc[1]);
            store_shared_across_chip(part_o + pi * kHeadDim + ch + 2, acc[2], acc[3]);
            if (ch == 0) store_shared_across_chip(part_ml + pi * 2, M, lt);
        }
    }
    __syncthreads();
}

// ---- balanced kernel over the nominal page space -------------------------------------------------
//
// Launch shape and work split must not depend on device data, and a prefix sum over the real list
// lengths would put two more dependent memory round trips in front of the first K/V load of every
// workgroup.  The split is therefore done over *nominal* list lengths the host knows: s + w pages
// for a streaming head, sel_stride + 1 for a dense head (the selection plus one page created since).
// Nominal entry x of the launch maps to (sequence, KV head, entry) by arithmetic alone.  Entries
// past a list's real length are skipped; real entries past the nominal length (a selection reused
// for more than one new page) are handled by the workgroup that owns the list's last nominal entry.

struct DecodePlan {
    int per_seq;                 // nominal entries per sequence
    int total;                   // batch * per_seq
    int quot, rem;               // total = G * quot + rem: the first `rem` ranges hold quot + 1 entries
    int stream_len, select_len;  // nominal entries of a streaming head's list and of a selecting head's
};

// First nominal entry of KV head hk inside a sequence (hk = Hkv gives per_seq).  The lists of a sequence follow
// each other in head order, so the start is a count of the streaming heads below hk: plain arithmetic on two
// launch constants, with nothing to fetch before the first table look-up can be issued.
__device__ __forceinline__ int first_entry(const DecodePlan& plan, unsigned long long streaming_mask, int hk) {
    const unsigned long long below = hk >= 64 ? ~0ull : (1ull << hk) - 1ull;
    const int ns = __popcll(streaming_mask & below);
    return ns * plan.stream_len + (hk - ns) * plan.select_len;
}
__device__ __forceinline__ int nominal_len(const DecodePlan& plan, unsigned long long streaming_mask, int hk) {
    return ((streaming_mask >> hk) & 1ull) ? plan.stream_len : plan.select_len;
}

// Range of workgroup j is [range_begin(j), range_begin(j + 1)); no division on the device.
__device__ __forceinline__ int range_begin(const DecodePlan& plan, int j) { return j * plan.quot + min(j, plan.rem); }

// Workgroup whose range holds nominal entry x.
__device__ __forceinline__ int range_of(const DecodePlan& plan, int x) {
    const int big = plan.rem * (plan.quot + 1);
    return x < big ? x / (plan.quot + 1) : plan.rem + (x - big) / plan.quot;
}

// KV head of nominal entry y of a sequence: the number of heads whose list starts at or before y, less one.
__device__ __forceinline__ int head_of_entry(const DecodePlan& plan, unsigned long long streaming_mask, int Hkv, int y) {
    int hk = 0;
    for (int h = 1; h < Hkv; ++h) hk += y >= first_entry(plan, streaming_mask, h);
    return hk;
}

// Maximum, sum and four channels `ch .. ch + 3` of query head `hh`, folded over pieces ja .. jb of a list, in slot order,
// kBatch at a time so that their loads are in flight together.  Every range between a list's first and last holds a
// real entry of the list and wrote a piece (empty ranges come after all others).
struct Folded {
    float m, l, acc[4];
};
template <int N, int kBatch>
__device__ __forceinline__ Folded fold_pieces(int list, int ja, int jb, int hh, int ch, const float* part_o,
                                              const float* part_ml) {
    Folded f = {-INFINITY, 0.f, {0.f, 0.f, 0.f, 0.f}};
    for (int j = ja; j <= jb; j += kBatch) {
        float2 ml[kBatch], lo[kBatch], hi[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const size_t pi = ((size_t)min(j + u, jb) + list) * N + hh;  // past the end: the last piece again, unused
            ml[u] = load_shared_across_chip(part_ml + pi * 2);
            lo[u] = load_shared_across_chip(part_o + pi * kHeadDim + ch);
            hi[u] = load_shared_across_chip(part_o + pi * kHeadDim + ch + 2);
        }
        float bm = -INFINITY;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) bm = fmaxf(bm, j + u <= jb ? ml[u].x : -INFINITY);
        if (bm == -INFINITY) continue;  // only if every logit of these pieces was -inf
        const float m_new = fmaxf(f.m, bm);
        const float keep = __builtin_amdgcn_exp2f(f.m - m_new);  // 0 for the first batch (m = -inf)
        f.l *= keep;
#pragma unroll
        for (int i = 0; i < 4; ++i) f.acc[i] *= keep;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const float w = j + u <= jb ? __builtin_amdgcn_exp2f(ml[u].x - m_new) : 0.f;
            f.l += ml[u].y * w;
            f.acc[0] += lo[u].x * w;
            f.acc[1] += lo[u].y * w;
            f.acc[2] += hi[u].x * w;
            f.acc[3] += hi[u].y * w;
        }
        f.m = m_new;
    }
    return f;
}

// Folds pieces j0 .. j1 of a list and writes its rows.  Called by all threads.  Up to eight pieces (the lists of a large
// batch) are one round of loads by one thread per (query head, four channels).  A small batch cuts its lists into as many
// as sixty: eight at a time they were seven rounds, one after the other (6 of the call's 15 us at one sequence of 4000
// tokens); then the pieces are shared out over all threads, sixteen at a time, and met in shared memory.  Pages of 128 tokens
// make half as many pieces and fill the registers: sixteen at a time left room for one workgroup to a compute unit instead
// of two (57 sequences of 290 .. 6691 tokens, 32 / 8 heads: 440 us for four steps, eight at a time 298).
template <class T, int N, int NP>
__device__ __forceinline__ void fold_list(DecodeShared<N, NP>& sm, int list, int j0, int j1, int H, int b, int hk,
                                          uint16_t* out, float* lse_out, const float* part_o, const float* part_ml) {
    constexpr int kItems = N * (kHeadDim / 4), kParts = N <= 2 ? 4 : N <= 4 ? 2 : 1;
    const int item = threadIdx.x % kItems, part = threadIdx.x / kItems;
    const int hh = item / (kHeadDim / 4), ch = item % (kHeadDim / 4) * 4;
    Folded f;
    if (NP == 128 || j1 - j0 < 8) {
        if (part == 0) f = fold_pieces<N, 8>(list, j0, j1, hh, ch, part_o, part_ml);
    } else {
        const int share = (j1 - j0 + kParts) / kParts, ja = j0 + part * share;
        if (part < kParts) f = fold_pieces<N, 16>(list, ja, min(ja + share - 1, j1), hh, ch, part_o, part_ml);
        if (kParts > 1) {
            if (part > 0 && part < kParts) {
                *reinterpret_cast<float4*>(&sm.o[part][hh][ch]) = make_float4(f.acc[0], f.acc[1], f.acc[2], f.acc[3]);
                if (ch == 0) sm.m[part][hh] = f.m, sm.l[part][hh] = f.l;
            }
            __syncthreads();
            if (part == 0) {
                float m_all = f.m;
#pragma unroll
                for (int i = 1; i < kParts; ++i) m_all = fmaxf(m_all, sm.m[i][hh]);
                const float w0 = f.m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(f.m - m_all);
                f.l *= w0;
#pragma unroll
                for (int i = 0; i < 4; ++i) f.acc[i] *= w0;
#pragma unroll
                for (int i = 1; i < kParts; ++i) {  // a part without pieces, or without a finite logit, adds nothing
                    const float w = sm.m[i][hh] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sm.m[i][hh] - m_all);
                    const float4 o = *reinterpret_cast<const float4*>(&sm.o[i][hh][ch]);
                    f.l += sm.l[i][hh] * w;
                    f.acc[0] += o.x * w;
                    f.acc[1] += o.y * w;
                    f.acc[2] += o.z * w;
                    f.acc[3] += o.w * w;
                }
                f.m = m_all;
            }
        }
    }
    if (part > 0) return;
    const int h = hk * N + hh;
    const uint2 packed = make_uint2(Elem<T>::pack(f.acc[0] / f.l, f.acc[1] / f.l), Elem<T>::pack(f.acc[2] / f.l, f.acc[3] / f.l));
    *reinterpret_cast<uint2*>(out + ((size_t)b * H + h) * kHeadDim + ch) = packed;
    if (lse_out && ch == 0) lse_out[b * H + h] = (f.m + __builtin_amdgcn_logf(f.l)) * kLn2;
}

// Ends a (workgroup, list) piece.  `len` is the real length of the list, so its real entries occupy the nominal
// entries [n0, n_end) and exactly the workgroups whose ranges meet that stretch hold a piece of it.  A list that
// lies inside this workgroup's range is written out directly.  Otherwise the piece goes to the workspace, the
// workgroup counts itself in on the list's arrival counter, and the one that finds every other piece already in
// folds them all, in slot order (so the result does not depend on which workgroup folds), writes the rows and
// puts the counter back to zero for the next launch.  Nobody waits for anybody.  Stores, counter and loads are
// agent-scope accesses with a wait for the stores in between; no cache-wide fence (a device-scope fence here was
// measured at three times the whole kernel: it writes back and invalidates the L2).  Called by all threads.
template <class T, int N, int NP, int BITS>
__device__ __forceinline__ void end_piece(StateOf<N, NP, BITS>& st, DecodeShared<N, NP>& sm, const DecodePlan& plan, int blk,
                                          int lo, int hi, int list, int len, int H, int Hkv,
                                          unsigned long long streaming_mask, uint16_t* out,
                                          float* lse_out, float* part_o, float* part_ml, unsigned* arrivals) {
    const int b = list / Hkv, hk = list % Hkv;
    const int n0 = b * plan.per_seq + first_entry(plan, streaming_mask, hk);
    const int n_end = n0 + min(len, nominal_len(plan, streaming_mask, hk));
    const bool whole = n0 >= lo && n_end <= hi;
    flush_block<T, N, NP, BITS>(st, sm, whole, H, b, hk, out, lse_out, part_o, part_ml, (size_t)blk + list);
    if (whole) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's part of the piece has reached memory
    __syncthreads();
    if (threadIdx.x == 0)
        sm.arrived = __hip_atomic_fetch_add(arrivals + list, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int j0 = range_of(plan, n0), j1 = range_of(plan, n_end - 1);
    if ((int)sm.arrived != j1 - j0) return;  // somebody else will fold
    fold_list<T, N, NP>(sm, list, j0, j1, H, b, hk, out, lse_out, part_o, part_ml);
    if (threadIdx.x == 0) __hip_atomic_store(arrivals + list, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Visits entry IDX of the current batch, whose slabs are in CUR: when the (wave-uniform) list changes the
// piece of the previous list is ended and the new list's queries are staged; then the quarter page is
// folded in; real entries beyond the nominal length of a list (rare) are fetched and folded in on the spot,
// without prefetch (only dense heads outgrow their nominal list, so they are always in the main pool).
// A macro, not a lambda: with the state captured by reference the compiler keeps 70 more registers live in
// the 16-bit kernel.
#define LSERVE_DECODE_VISIT(IDX, CUR)                                                                                \
    {                                                                                                                \
        const int list = __builtin_amdgcn_readlane(my_list, (IDX));                                                  \
        if (list != cur_list) {                                                                                      \
            if (cur_list >= 0)                                                                                       \
                end_piece<T, N, NP, BITS>(st, sm, plan, blk, lo, hi, cur_list, cur_len, lp.H, lp.Hkv,                \
                                          lp.streaming_mask, out, lse_out, part_o, part_ml, arrivals);               \
            cur_list = list;                                                                                         \
            cur_len = __builtin_amdgcn_readlane(my_len, (IDX));                                                      \
            cur_b = list / lp.Hkv;                                                                                   \
            cur_hk = list % lp.Hkv;                                                                                  \
            stage_query<T, N, NP, BITS>(sm, q, cur_b, lp.H, cur_hk, list, q_ahead);                                  \
            if constexpr (BITS != 16 || scores_by_matrix(N, NP)) load_query_operands(st, sm.q, sm.q_sum, lane);            \
            st.reset();                                                                                              \
        }                                                                                                            \
        process_quarter<T, N, NP, BITS>(st, sm.q, sm.p[wave], CUR, __builtin_amdgcn_readlane(my_left, (IDX)), tok0, lane, lp.sm_scale_log2); \
        if ((outgrown >> (IDX)) & 1) {                                                                               \
            const int extra = __builtin_amdgcn_readlane(my_extra, (IDX)), L = __builtin_amdgcn_readlane(my_L, (IDX)); \
            const int nominal = nominal_len(plan, lp.streaming_mask, cur_hk);                                        \
            const int tail = __builtin_amdgcn_readlane(my_tail, (IDX));                                              \
            for (int e = 0; e < extra; ++e) {                                                                        \
                const int epos = tail + nominal + e;                                                                 \
                const int ephys = kv.page_table[(size_t)cur_b * kv.max_pages + epos];                                \
                const uint4 *ke, *ve;                                                                                \
                slab_of(ephys, cur_hk, ke, ve);                                                                      \
                load_k<N>(CUR, ke, tok0, lane, ~0u);                                                                     \
                load_v(CUR, ve, tok0, r, c, lane, ~0u);                                                                \
                process_quarter<T, N, NP, BITS>(st, sm.q, sm.p[wave], CUR, L - epos * NP, tok0, lane, lp.sm_scale_log2);\
            }                                                                                                        \
        }                                                                                                            \
    }

// The pointer that lane `lane` holds, wave-uniform.
__device__ __forceinline__ const uint4* pointer_of_lane(const uint4* p, int lane) {
    const unsigned long long x = reinterpret_cast<unsigned long long>(p);
    return reinterpret_cast<const uint4*>(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(x >> 32), lane) << 32) |
                                          (unsigned)__builtin_amdgcn_readlane((int)x, lane));
}

// Quantised pages: two wavefronts to a SIMD is what the compiler is told to plan for, and what the launch has (kBlocksPerCU).  Left alone
// it keeps registers down for more, and puts the unpacking of codes and their products in an order that takes longer: 64 sequences of 9K
// .. 24K over 4-bit pages, four steps, 209 -> 193 us, 57 of 290 .. 6691 over 8-bit ones 193 -> 171, eight heads to a group, 16 of 30000,
// 116 -> 105.  16-bit rows gain nothing and over pages of 32 tokens lose 4 %; for three wavefronts the quantised kernels spill.
// Pages of 128 tokens take a few registers more than there are for two wavefronts, which the compiler only gives up if told (57 of
// 290 .. 6691 tokens 360 and 288 us); under six and more heads it would have to spill.
template <class T, int N, int NP, int BITS>
__global__ __launch_bounds__(kDecodeThreads, BITS != 16 || (NP == 128 && N >= 3 && N <= 5) ? 2 : 1) void sparse_decode_kernel(
    LayerParams lp, PagedParams kv, DecodePlan plan, const uint4* __restrict__ q, const int* __restrict__ sel_pages,
    const int* __restrict__ sel_count, const int* __restrict__ sel_seq_len, int sel_stride,
    uint16_t* __restrict__ out, float* __restrict__ lse_out, float* __restrict__ part_o, float* __restrict__ part_ml,
    unsigned* __restrict__ arrivals) {
    __shared__ DecodeShared<N, NP> sm;

    // The launch constants fill four 64-byte lines of the kernel argument block, and the code below wants them in
    // half a dozen dependent rounds; fetched as needed, each round missed the scalar cache and the first table
    // look-up left 2.2 us after the start of the kernel.  One word of every line is requested here, together.
#if defined(__HIP_DEVICE_COMPILE__)
    {
        typedef const int __attribute__((address_space(4))) * kernarg_words;
        const kernarg_words args = (kernarg_words)__builtin_amdgcn_kernarg_segment_ptr();
        static_assert(sizeof(LayerParams) + sizeof(PagedParams) + sizeof(DecodePlan) + 9 * sizeof(void*) > 48 * sizeof(int),
                      "the argument block must reach the last line touched");
        const int a0 = args[0], a1 = args[16], a2 = args[32], a3 = args[48];
        asm volatile("" ::"s"(a0), "s"(a1), "s"(a2), "s"(a3));
    }
#endif

    const int blk = blockIdx.x;
    const int lo = range_begin(plan, blk), hi = range_begin(plan, blk + 1);
    if (lo >= hi) return;

    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int r = lane / 16, c = lane % 16;
    const int tok0 = wave * (NP / 4);
    const size_t slab = slab_chunks(NP, BITS);  // uint4 per (page, head)
    const uint4* kpool = reinterpret_cast<const uint4*>(kv.k_pool);
    const uint4* vpool = reinterpret_cast<const uint4*>(kv.v_pool);
    const uint4* kstream = reinterpret_cast<const uint4*>(kv.k_stream);
    const uint4* vstream = reinterpret_cast<const uint4*>(kv.v_stream);
    // slab of (physical page, KV head): streaming heads may live in their own bounded pool (Sec. 3.2)
    auto slab_of = [&](int phys, int hk, const uint4*& kslab, const uint4*& vslab) {
        const bool ring = in_stream_pool(lp, kv, hk);
        const size_t o = ((size_t)phys * (ring ? kv.stream_heads : kv.pool_heads) + pool_rank(lp, kv, hk, ring)) * slab;
        kslab = (ring ? kstream : kpool) + o;
        vslab = (ring ? vstream : vpool) + o;
    };

    // Only where the eight registers do not cost a resident workgroup (measured: 128-token pages and the
    // quantised kernels lose more than the early queries gain).
    constexpr bool kQueriesAhead = BITS == 16 && NP <= 64;
    QueryAhead q_ahead;
    q_ahead.list = -4;  // matches no list
    q_ahead.x[0] = q_ahead.x[1] = make_uint4(0, 0, 0, 0);

    StateOf<N, NP, BITS> st;
    int cur_list = -1, cur_b = 0, cur_hk = 0, cur_len = 0;
    // with every head streaming there is no selection: the loads below then read a valid word of the lengths
    const int* sel_table = sel_pages ? sel_pages : kv.seq_lens;
    const int* sel_counts = sel_pages ? sel_count : kv.seq_lens;
    const int* sel_lens = sel_pages ? sel_seq_len : kv.seq_lens;
    const int has_sel = sel_pages != nullptr;  // a factor, not a condition: the loads must not sit behind a branch

    for (int base = lo; base < hi; base += kWave) {
        // One lane per nominal entry.  Every load that depends on nothing loaded goes out first and together (the
        // length; for a selecting head its selection entry, count and selection-time length), then the page
        // table, then the slabs: three round trips before the first byte of K / V, and no more.  Lanes past the
        // end of the range repeat its last entry, so that every lane forms valid addresses without a branch.
        const int cnt = min(kWave, hi - base);
        const int x = base + min(lane, cnt - 1);
        const int b = x / plan.per_seq, y = x - b * plan.per_seq;
        const int hk = head_of_entry(plan, lp.streaming_mask, lp.Hkv, y);
        const int i = y - first_entry(plan, lp.streaming_mask, hk), nominal = nominal_len(plan, lp.streaming_mask, hk);
        const bool streaming = (lp.streaming_mask >> hk) & 1ull;
        const int my_list = b * lp.Hkv + hk;
        // no branch between these loads and their first use, or the wait for them could not be counted exactly
        // and would take in the query loads as well; lanes of streaming heads read valid words they ignore
        const int my_L = kv.seq_lens[b];
        const int sel_word = sel_table[has_sel * ((size_t)my_list * sel_stride + min(i, sel_stride - 1))];
        const int sel_head = sel_counts[has_sel * my_list];
        const int sel_len = sel_lens[has_sel * b];
        // The queries of the first two lists of these entries go out behind the table loads (in front of them they
        // would be waited for first: loads complete in order).  Thread t holds chunk t % (N * 16) of the group.
        if constexpr (kQueriesAhead) {
            q_ahead.list = __builtin_amdgcn_readfirstlane(my_list);
            const int last = kv.batch * lp.Hkv - 1;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int list = min(q_ahead.list + u, last);
                q_ahead.x[u] = q[((size_t)(list / lp.Hkv) * lp.H + (list % lp.Hkv) * N) * (kHeadDim / 8) +
                                 threadIdx.x % (N * 16)];
            }
        }
        __builtin_amdgcn_sched_barrier(0);  // all of the above is requested before any of it is used
        const int P = ceil_div(my_L, NP);
        const int stream_head = min(lp.sink_pages, P);
        const int head = streaming ? stream_head : sel_head;
        const int tail_start = streaming ? max(stream_head, P - lp.local_pages) : ceil_div(sel_len, NP);
        const int sel_entry = streaming ? i : sel_word;
        const int my_len = head + max(0, P - tail_start);
        const bool my_valid = lane < cnt && i < my_len;
        const int my_pos = i < head ? sel_entry : tail_start + (i - head);
        const int my_tail = tail_start - head;  // position of entry i >= head is my_tail + i
        const int my_extra = (i == nominal - 1 && my_len > nominal) ? my_len - nominal : 0;
        int my_phys = 0;
        if (my_valid)
            my_phys = in_stream_pool(lp, kv, hk) ? kv.ring_table[(size_t)b * kv.ring + ring_slot(lp, my_pos)]
                                                 : kv.page_table[(size_t)b * kv.max_pages + my_pos];
        unsigned long long todo = __ballot(my_valid);
        if (todo == 0) continue;
        // Everything the page loop needs of an entry is worked out here, by its lane, for all entries at once: in the
        // loop the same arithmetic (a remainder by the head count, head ranks, 64-bit products) is a chain of scalar
        // instructions per page.  Pages of 128 tokens are four times the work, and have no registers left for addresses.
        const uint4 *my_k, *my_v;
        slab_of(my_phys, hk, my_k, my_v);
        auto slabs_of = [&](int idx, const uint4*& k, const uint4*& v) {
            if constexpr (NP == 128) {
                slab_of(__builtin_amdgcn_readlane(my_phys, idx), __builtin_amdgcn_readlane(my_list, idx) % lp.Hkv, k, v);
            } else {
                k = pointer_of_lane(my_k, idx);
                v = pointer_of_lane(my_v, idx);
            }
        };
        const int my_left = my_L - my_pos * NP;  // tokens of the page below the sequence length (or more than a page)
        const unsigned long long outgrown = __ballot(my_valid && my_extra > 0);
        // The two workgroups of a compute unit take turns at the higher wave priority, page by page
        // (workgroups j and j + G / 2 share a unit); measured 0.4 us per call on the 32K benchmark shape.
        auto take_turn = [&] {
            if ((__builtin_popcountll(todo) + (blk >= (int)gridDim.x / 2)) & 1)
                __builtin_amdgcn_s_setprio(1);
            else
                __builtin_amdgcn_s_setprio(0);
        };
        if constexpr (BITS == 16) {
            // one page in flight behind the one being worked on
            Slabs<NP, BITS> cur, nxt;
            {
                const uint4 *k0, *v0;
                slabs_of(__builtin_ctzll(todo), k0, v0);
                load_k<N>(cur, k0, tok0, lane, ~0u);
                load_v(cur, v0, tok0, r, c, lane, ~0u);
            }
            while (todo) {
                const int idx = __builtin_ctzll(todo);
                todo &= todo - 1;
                if (todo) {
                    const uint4 *k1, *v1;
                    slabs_of(__builtin_ctzll(todo), k1, v1);
                    load_k<N>(nxt, k1, tok0, lane, ~0u);
                    load_v(nxt, v1, tok0, r, c, lane, ~0u);
                }
                take_turn();
                LSERVE_DECODE_VISIT(idx, cur)
                cur = nxt;
            }
        } else {
            // One page in flight here too (two to six changed nothing over 4-bit pages and cost up to a quarter over 8-bit
            // ones); the stages rotate by name (a copy of a register whose load is in flight would wait for it).  Over
            // 4-bit pages a request goes out with every page, past the last one too: the wait for a page's slabs is a
            // count of the loads behind them, and where a request may or may not have been made the compiler can only
            // wait for all of them (batch 16, no groups: 40.4 us without, 39.1 with; 8-bit pages lose 2 to 5 % instead).
            constexpr bool kAlways = BITS == 4;
            unsigned long long ahead = todo;  // entries whose slabs have not been requested yet
            auto request = [&](Slabs<NP, BITS>& dst, int current) {
                if (!kAlways && !ahead) return;
                const unsigned live = ahead ? ~0u : 0u;
                const int nx = ahead ? __builtin_ctzll(ahead) : current;
                ahead &= ahead - 1;
                const uint4 *k1, *v1;
                slabs_of(nx, k1, v1);
                load_k<N>(dst, k1, tok0, lane, live);
                load_v(dst, v1, tok0, r, c, lane, live);
            };
            constexpr int kStages = 2;
            Slabs<NP, BITS> stage[kStages];
            request(stage[0], __builtin_ctzll(todo));
            while (todo) {
#pragma unroll
                for (int u = 0; u < kStages; ++u) {
                    if (!todo) break;
                    const int idx = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    request(stage[(u + 1) % kStages], idx);
                    take_turn();
                    LSERVE_DECODE_VISIT(idx, stage[u])
                }
            }
        }
    }
    if (cur_list < 0) return;  // no real entry in this range
    end_piece<T, N, NP, BITS>(st, sm, plan, blk, lo, hi, cur_list, cur_len, lp.H, lp.Hkv, lp.streaming_mask, out, lse_out,
                              part_o, part_ml, arrivals);
}

#undef LSERVE_DECODE_VISIT

// ---- host side -----------------------------------------------------------------------------------

// `slack`: nominal entries added to a streaming head's list beyond its s + w pages.  They are never real, so they
// cost the workgroup that holds them nothing, which makes up for what a list boundary inside a range costs it
// (the piece of the list that ends there is folded and delivered, the next list's queries are staged: about
// 0.7 of a page's time, measured).  A selecting head's list has such an entry already, since its "+ 1" page is
// real only after the sequence has grown into a new page.
DecodePlan make_plan(const LayerParams& lp, int batch, int sel_stride, int G, int slack) {
    DecodePlan plan;
    plan.stream_len = lp.sink_pages + lp.local_pages + slack;
    plan.select_len = sel_stride + 1;
    int n_stream = 0;
    for (int hk = 0; hk < lp.Hkv; ++hk) n_stream += (int)((lp.streaming_mask >> hk) & 1ull);
    plan.per_seq = n_stream * plan.stream_len + (lp.Hkv - n_stream) * plan.select_len;
    plan.total = batch * plan.per_seq;
    plan.quot = plan.total / G;
    plan.rem = plan.total % G;
    return plan;
}

struct DecodeScratch {
    float *part_o, *part_ml;  // pieces: unnormalised outputs, (max, sum) pairs
    unsigned* arrivals;       // per list: pieces that have arrived
};

size_t arrival_bytes(const LayerParams& lp, int batch) {
    return ((size_t)batch * lp.Hkv * sizeof(unsigned) + 255) & ~(size_t)255;
}

size_t partial_slots(const LayerParams& lp, int batch) {
    return (size_t)num_compute_units() * kMaxBlocksPerCU + (size_t)batch * lp.Hkv;
}

template <class T, int N, int NP, int BITS>
hipError_t launch_decode_kernels(const LayerParams& lp, const PagedParams& kv, const void* q, const int* sel_pages,
                                 const int* sel_count, const int* sel_seq_len, int sel_stride, void* out,
                                 float* lse_out, const DecodeScratch& ws, hipStream_t stream) {
    const uint4* q4 = reinterpret_cast<const uint4*>(q);
    uint16_t* o16 = reinterpret_cast<uint16_t*>(out);
    // Resident workgroups per compute unit of this instantiation: a property of the binary and the device, asked
    // once (thread-safe initialisation of a function-local static); a failed query counts as one.
    static const int per_cu = [] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, sparse_decode_kernel<T, N, NP, BITS>, kDecodeThreads, 0) !=
            hipSuccess) {
            (void)hipGetLastError();
            return 1;
        }
        return nb < 1 ? 1 : (nb > kBlocksPerCU ? kBlocksPerCU : nb);
    }();
    // two workgroups per compute unit, unless that leaves fewer than four entries each: a small launch is all
    // start-up and fold, and half as many workgroups with twice the pages do less of each (measured).  A very small one
    // whose lists are long (no list is longer than the page table) gives every workgroup two entries, so that half as
    // many pieces are counted in and folded (one sequence of 4000 tokens: 12.9 us with one entry each, 11.2 with two,
    // 12.8 with three); short lists take one (1000 tokens: 8.9 us with one entry, 10.1 with two).
    const int cus = num_compute_units();
    int G = cus * per_cu;
    DecodePlan plan = make_plan(lp, kv.batch, sel_stride, G, 0);
    if (per_cu > 1 && plan.quot < 4) {
        G = std::min(plan.select_len, kv.max_pages) > 32 && plan.total < 2 * cus ? (plan.total + 1) / 2 : cus;
        plan = make_plan(lp, kv.batch, sel_stride, G, 0);
    } else if (plan.quot >= kSlackFromEntries) {
        plan = make_plan(lp, kv.batch, sel_stride, G, 1);
    }
    hipLaunchKernelGGL((sparse_decode_kernel<T, N, NP, BITS>), dim3(G), dim3(kDecodeThreads), 0, stream, lp, kv, plan, q4,
                       sel_pages, sel_count, sel_seq_len, sel_stride, o16, lse_out, ws.part_o, ws.part_ml, ws.arrivals);
    return hipGetLastError();
}

template <class T, int N>
hipError_t launch_decode_np(const LayerParams& lp, const PagedParams& kv, const void* q, const int* sel_pages,
                            const int* sel_count, const int* sel_seq_len, int sel_stride, void* out, float* lse_out,
                            const DecodeScratch& ws, hipStream_t stream) {
#define LSERVE_DECODE_NP(NPV)                                                                                       \
    case NPV:                                                                                                       \
        return launch_decode_kernels<T, N, NPV, 16>(lp, kv, q, sel_pages, sel_count, sel_seq_len, sel_stride, out,   \
                                                    lse_out, ws, stream);
    if (kv.kv_bits == 8)  // quantised pages are always 64 tokens (checked by the caller)
        return launch_decode_kernels<T, N, 64, 8>(lp, kv, q, sel_pages, sel_count, sel_seq_len, sel_stride, out, lse_out,
                                                  ws, stream);
    if (kv.kv_bits == 4)
        return launch_decode_kernels<T, N, 64, 4>(lp, kv, q, sel_pages, sel_count, sel_seq_len, sel_stride, out, lse_out,
                                                  ws, stream);
    switch (lp.NP) {
        LSERVE_DECODE_NP(16)
        LSERVE_DECODE_NP(32)
        LSERVE_DECODE_NP(64)
        LSERVE_DECODE_NP(128)
        default:
            return hipErrorInvalidValue;
    }
#undef LSERVE_DECODE_NP
}

template <class T>
hipError_t launch_decode(const LayerParams& lp, const PagedParams& kv, const void* q, const int* sel_pages,
                         const int* sel_count, const int* sel_seq_len, int sel_stride, void* out, float* lse_out,
                         void* workspace, hipStream_t stream) {
    // arrival counters (one per list, zero between launches), then the pieces
    DecodeScratch ws;
    ws.arrivals = reinterpret_cast<unsigned*>(workspace);
    ws.part_o = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + arrival_bytes(lp, kv.batch));
    ws.part_ml = ws.part_o + partial_slots(lp, kv.batch) * lp.group * kHeadDim;
#define LSERVE_DECODE_N(NV)                                                                                          \
    case NV:                                                                                                         \
        return launch_decode_np<T, NV>(lp, kv, q, sel_pages, sel_count, sel_seq_len, sel_stride, out, lse_out,       \
                                       ws, stream);
    switch (lp.group) {
        LSERVE_DECODE_N(1)
        LSERVE_DECODE_N(2)
        LSERVE_DECODE_N(3)
        LSERVE_DECODE_N(4)
        LSERVE_DECODE_N(5)
        LSERVE_DECODE_N(6)
        LSERVE_DECODE_N(7)
        LSERVE_DECODE_N(8)
        default:
            return hipErrorInvalidValue;
    }
#undef LSERVE_DECODE_N
}

// Measurement aid, not part of the attention path: reads the K and V slabs a decode call with the same arguments
// would read, one short workgroup per index-table entry, folds the words together and throws the result away.  The
// time of this launch is what the memory system charges for the decode call's access pattern alone.
__global__ __launch_bounds__(kDecodeThreads) void decode_read_probe_kernel(LayerParams lp, PagedParams kv,
                                                                           const int* __restrict__ sel_pages,
                                                                           const int* __restrict__ sel_count,
                                                                           const int* __restrict__ sel_seq_len,
                                                                           int sel_stride, int slab_u4,
                                                                           unsigned* __restrict__ sink) {
    const int list = blockIdx.y, i = blockIdx.x;
    const int b = list / lp.Hkv, hk = list % lp.Hkv;
    const PageList pl = make_page_list(lp, b, hk, kv.seq_lens[b], sel_pages, sel_count, sel_seq_len, sel_stride);
    if (i >= pl.len) return;
    const int pos = page_of(pl, i);
    const bool ring = in_stream_pool(lp, kv, hk);
    const int phys = ring ? kv.ring_table[(size_t)b * kv.ring + ring_slot(lp, pos)] : kv.page_table[(size_t)b * kv.max_pages + pos];
    const size_t o = ((size_t)phys * (ring ? kv.stream_heads : kv.pool_heads) + pool_rank(lp, kv, hk, ring)) * slab_u4;
    const uint4* k = reinterpret_cast<const uint4*>(ring ? kv.k_stream : kv.k_pool) + o;
    const uint4* v = reinterpret_cast<const uint4*>(ring ? kv.v_stream : kv.v_pool) + o;
    unsigned acc = 0;
    for (int j0 = 0; j0 < slab_u4; j0 += 4 * kDecodeThreads) {  // four 16-byte loads of K and of V in flight per thread
        uint4 a[4], c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int j = min(j0 + u * kDecodeThreads + (int)threadIdx.x, slab_u4 - 1);
            a[u] = k[j];
            c[u] = v[j];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc ^= a[u].x ^ a[u].y ^ a[u].z ^ a[u].w ^ c[u].x ^ c[u].y ^ c[u].z ^ c[u].w;
    }
    if (sink && acc == 0x9e3779b9u) *sink = acc;  // keeps the loads alive
}

}  // namespace

hipError_t launch_decode_read_probe(const LayerParams& lp, const PagedParams& kv, const int* sel_pages,
                                    const int* sel_count, const int* sel_seq_len, int sel_stride, hipStream_t stream) {
    // entries of the longest list the launch looks at: the nominal length plus eight pages created since the selection
    const int entries = std::max(sel_stride, lp.sink_pages + lp.local_pages) + 8;
    hipLaunchKernelGGL(decode_read_probe_kernel, dim3(entries, kv.batch * lp.Hkv), dim3(kDecodeThreads), 0, stream, lp, kv,
                       sel_pages, sel_count, sel_seq_len, sel_stride, (int)slab_chunks(lp.NP, kv.kv_bits), (unsigned*)nullptr);
    return hipGetLastError();
}

long long decode_nominal_entries(const LayerParams& lp, int sel_stride) {
    long long acc = 0;
    for (int hk = 0; hk < lp.Hkv; ++hk)
        acc += ((lp.streaming_mask >> hk) & 1ull) ? (long long)lp.sink_pages + lp.local_pages + 1  // with the slack entry
                                                  : (long long)sel_stride + 1;
    return acc;
}

size_t decode_workspace_bytes(const LayerParams& lp, int batch, int sel_stride) {
    (void)sel_stride;
    return arrival_bytes(lp, batch) + partial_slots(lp, batch) * lp.group * (kHeadDim + 2) * sizeof(float);
}

hipError_t preload_decode_kernels() {
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(&sparse_decode_kernel<F16, 1, 64, 16>));
}

hipError_t launch_sparse_decode(int dtype, const LayerParams& lp, const PagedParams& kv, const void* q,
                                const int* sel_pages, const int* sel_count, const int* sel_seq_len,
                                int sel_stride, void* out, float* lse_out, void* workspace, hipStream_t stream) {
    return dtype == 0 ? launch_decode<F16>(lp, kv, q, sel_pages, sel_count, sel_seq_len, sel_stride, out, lse_out,
                                           workspace, stream)
                      : launch_decode<BF16>(lp, kv, q, sel_pages, sel_count, sel_seq_len, sel_stride, out, lse_out,
                                            workspace, stream);
}

}  // namespace lserve
