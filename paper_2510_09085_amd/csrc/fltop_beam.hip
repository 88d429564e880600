// CTC prefix beam search over the survivor lists (paper Sec. 3, Algorithm 1: the
// loop over beam entries and kept tokens, the set-insert that merges equal
// prefixes, SelectTopK and GetHighestScorePrefix).
//
// One workgroup decodes one utterance and stays resident for all its frames.
// The beam (prefix hash, parent hash, last token, p_b, p_nb, trie node) lives in
// LDS.  A candidate is either "entry j stays" or "entry i extended by survivor
// k"; candidates are held in registers (or recomputed when there are more than
// the registers hold), never written to memory.  An extension i+s can only
// coincide with a prefix that is already in the beam (a prefix has one parent),
// so merging is done from the side of that beam entry: it knows its parent's
// place in the beam and adds the parent's extension mass to its own p_nb; the
// extension itself is then skipped.  Every log-sum-exp has two operands.  The
// parent links are carried from frame to frame through a map "old place -> new
// place" of the entries that stay; only a prefix whose parent was absent looks
// it up in a small LDS hash table of the prefixes that entered in this frame.
//
// Top-`beam` selection works on an order-preserving 64-bit image of the fp64
// score: a two-level histogram over the distance to an upper bound locates the
// bucket holding the beam-th best candidate, buckets are refined until the
// boundary bucket is small, and its members are ranked exactly by (score, hash).
//
// Latency is what matters here (frames of one utterance are strictly serial):
//  - frame headers (which carry the first six survivors) are staged through LDS
//    32 frames at a time, one chunk ahead, and barriers wait for LDS traffic only,
//    so global loads and trie stores stay in flight across them;
//  - frames whose only survivor is blank change no prefix and no order: every entry's
//    total takes the frame's log-prob (the thread that owns the entry adds it in a
//    register, in the order a plain implementation adds them) and a flag says that
//    p_b = total, p_nb = -inf holds for every entry; a run of such frames is consumed at
//    once (the frames of a chunk are classified together) and costs one LDS round trip
//    and one barrier for the whole run;
//  - frames with at most six survivors keep them in registers; what the prune
//    stage can say about a frame by itself (blank kept?, the division constant
//    that maps a candidate index to its beam entry) comes with the header;
//  - "stay" candidates (which need the log-sum-exps) and extension candidates are
//    mapped to different wavefronts so that they are evaluated side by side, and
//    the end-of-frame clean-up is done by the wavefronts that have no links to set.
//
// The kernel is built several times over (workgroup size, beam capacity, register budget, and
// the length of the survivor lists it is to expect):
// four wavefronts for the frames of a pruned small vocabulary, eight with an entry-major
// candidate mapping where frames hold hundreds to thousands of candidates, and two with a
// tighter register budget for batches that fill the chip, where instruction issue and
// residency count instead of one frame's latency (see launch_beam).
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "fltop_internal.h"
#include "fltop_light.h"

namespace fltop {
namespace {

constexpr int kThreadsSmall = 256;  // workgroup size for small vocabularies
constexpr int kThreadsLarge = 512;  // and for large ones (see launch_beam)
constexpr int kThreadsHuge = 1024;  // beams beyond 512 entries: still one thread per entry
constexpr int kThreadsDense = 128;  // small frames, batches larger than the chip holds at once
constexpr int kWave = 64;
// The beam lives in LDS, so its capacity is a compile-time size: kernels are built for a
// small one (which keeps several workgroups per CU for large batches) and for the largest.
constexpr int kBeamSmall = 128;
constexpr int kBeamTiny = 64;  // one-shot decodes of dense batches (20 KB of LDS)
constexpr int kBeamLarge = 512;
constexpr int kBeamHuge = FLTOP_MAX_BEAM;  // 1000-entry beams (paper Sec. 4: beam-size 1000)
static_assert(kBeamHuge == 1024, "the LDS budget below is worked out for 1024 entries");
constexpr int kFine = 1024;  // histogram bins
constexpr int kCoarse = 64;  // one per lane; a coarse bin covers 16 fine bins
constexpr int kExactCap = 64;
constexpr int kMaxShift = 54;  // kFine << kMaxShift covers all 64-bit distances
constexpr int kRegK = kInlineSurvivors;  // survivors kept in registers
constexpr int kRegCand = 1;              // extension candidates kept in registers per thread
// Candidates per thread from which a frame gets a score floor (times at 2 / 3 / 4 / 8, us, with the list of
// tokens below: 64 utterances x 500 frames, V = 32, beam 32, every token kept: 2358 / 2282 / 2282 / 2284;
// 150 frames, beam 100: 1030 / 1019 / 1019 / 1801; 128 x 400, V = 1024, beam 64, R = 0.01: 763 / 751 / 752 /
// 812; 64 x 400, V = 100, beam 32, R = 0.001: 1160 / 1148 / 1156 / 1175).
constexpr int kFlooredFrom = 4;
// Tokens that can reach the floor are listed up to this many (1 KB of LDS); beyond it a frame's whole
// list is gone through.  (128 utterances, V = 1024, every token kept, beam 64: a floor without the list
// 11.1 ms, with it 2.75 ms: 65 k candidates per frame were scored one by one, now ~1.5 k.)
constexpr int kListCap = 512;
constexpr int kChunk = 32;               // frame headers staged per chunk
constexpr int kWaypoints = 256;
constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kAllOnes = ~0ull;

// Two generations of a 1024-entry beam with everything in LDS would take 219 KB of the 160 KB
// a workgroup can have.  For that capacity the fields that only the trie bookkeeping needs
// (parent hash, trie node, length, skip ancestor: read once per emitted entry, never by the
// candidate evaluation) live in global memory instead (ColdSlab, in the workspace; L2-resident),
// the children lists are left out (builds with 512 threads and more use the pair table) and the
// two open-addressing tables are half as large per entry.
template <int MB>
struct SlabTraits {
    static constexpr bool kColdGlobal = MB > 512;
    static constexpr int kColdInLds = kColdGlobal ? 1 : MB;   // places of the cold fields in LDS
    static constexpr int kKidLists = kColdGlobal ? 4 : MB;    // places of the children lists
    static constexpr int kHashSlots = kColdGlobal ? 2 * MB : 4 * MB;
};

template <int MB>
struct BeamSlab {
    uint64_t h[MB];   // prefix hash
    uint64_t hp[SlabTraits<MB>::kColdInLds];  // parent prefix hash (unused when plen == 0)
    double pb[MB];
    double pnb[MB];
    double ptot[MB];
    int32_t last[MB];  // last token, -1 for the empty prefix
    int32_t node[SlabTraits<MB>::kColdInLds];  // trie node of the prefix
    int32_t plen[SlabTraits<MB>::kColdInLds];  // prefix length
    int32_t xanc[SlabTraits<MB>::kColdInLds];  // trie node of the ancestor at depth 8*floor(plen/8)
};

// The same four fields of one beam generation in global memory (kColdGlobal builds).
template <int MB>
struct ColdSlab {
    uint64_t hp[MB];
    int32_t node[MB];
    int32_t plen[MB];
    int32_t xanc[MB];
};
static_assert(sizeof(ColdSlab<FLTOP_MAX_BEAM>) == kColdBytesPerGeneration,
              "the workspace reserves two of these per utterance");

// One generation's trie bookkeeping fields, wherever they live.
template <int MB>
struct ColdRef {
    BeamSlab<MB>* lds;
    ColdSlab<MB>* glb;
    __device__ __forceinline__ uint64_t hp(int i) const {
        if constexpr (SlabTraits<MB>::kColdGlobal) return glb->hp[i];
        else return lds->hp[i];
    }
    __device__ __forceinline__ int32_t node(int i) const {
        if constexpr (SlabTraits<MB>::kColdGlobal) return glb->node[i];
        else return lds->node[i];
    }
    __device__ __forceinline__ int32_t plen(int i) const {
        if constexpr (SlabTraits<MB>::kColdGlobal) return glb->plen[i];
        else return lds->plen[i];
    }
    __device__ __forceinline__ int32_t xanc(int i) const {
        if constexpr (SlabTraits<MB>::kColdGlobal) return glb->xanc[i];
        else return lds->xanc[i];
    }
    __device__ __forceinline__ void set(int i, uint64_t hp_, int32_t node_, int32_t plen_,
                                        int32_t xanc_) const {
        if constexpr (SlabTraits<MB>::kColdGlobal) {
            glb->hp[i] = hp_;
            glb->node[i] = node_;
            glb->plen[i] = plen_;
            glb->xanc[i] = xanc_;
        } else {
            lds->hp[i] = hp_;
            lds->node[i] = node_;
            lds->plen[i] = plen_;
            lds->xanc[i] = xanc_;
        }
    }
};

// parent / children links of one beam generation
template <int MB>
struct alignas(16) Links {
    int32_t par[MB];
    int32_t first_kid[SlabTraits<MB>::kKidLists];
    int32_t next_kid[SlabTraits<MB>::kKidLists];
    uint32_t kidmask[MB];  // bit (token & 31) set for every child in the beam
    int32_t ht[SlabTraits<MB>::kHashSlots];  // open addressing: slot -> beam index of a prefix that
                                             // entered in this generation's frame, keyed by prefix hash
};

// One beam generation.
template <int MB>
struct Generation {
    BeamSlab<MB> slab;
    Links<MB> links;
};

// What the last wavefront says of the next light frame, and of the state that the others do not follow.
struct alignas(16) LightLine {
    uint32_t what, live;      // see fltop_beam_reach.inc; entries of the beam
    float lpb, scale;         // log-prob of the blank (-inf: pruned); bins per nat
    double ref, kmax;         // above every candidate's score; above every total
    float spread, margin;
    int32_t next_t, sure;     // frame that follows; whether the spread is a bound
};

// What a streaming (chunked) decode carries from one call to the next, per utterance: the
// beam and its links as they stand after the last frame seen, plus the scalars the frame
// loop keeps in registers.  The prefix trie lives behind the array of these records.
template <int MB>
struct StreamState {
    int32_t frames_done;  // frames decoded so far (= trie frame index of the next one)
    int32_t n_live;
    int32_t collapsed;    // bit 0: the blank-run flag; bit 1: kmin is a bound
    int32_t out_len;      // length of the transcript as last written
    double kmax, kmin;
    // where the transcript and its entry frames were last written: the record of trie nodes
    // behind the written tokens holds for those rows only
    uint64_t out_tokens_at, out_frames_at;
    BeamSlab<MB> slab;
    int32_t par[MB];
    int32_t first_kid[MB];
    int32_t next_kid[MB];
    uint32_t kidmask[MB];
};
static_assert(sizeof(StreamState<kBeamSmall>) % 8 == 0 && sizeof(StreamState<kBeamLarge>) % 8 == 0,
              "records sit in an array: doubles stay aligned");
static_assert(offsetof(Links<kBeamSmall>, ht) == 4 * kBeamSmall * sizeof(int32_t) &&
                  offsetof(Links<kBeamLarge>, ht) == 4 * kBeamLarge * sizeof(int32_t),
              "the four link arrays are the head of Links (streaming copies them as one block)");

struct BeamArgs {
    const int32_t* lengths;
    const FrameHdr* hdr;
    const Survivor* rec;
    TrieNode* trie;
    int64_t trie_stride;
    void* cold;             // kColdGlobal builds: [B][2] ColdSlab, else unused
    const float* lm_table;  // global copy (always valid when LM is on)
    const float* lm_bound;
    double lm_alpha, lm_beta;
    int32_t B, T, V, beam;
    int32_t lm_in_lds;  // 1: table staged into LDS
    int32_t dcache_off;   // dynamic LDS: byte offset of the distance cache ...
    int32_t dcache_rows;  // ... and its size in rows of one distance per thread (0: none)
    int32_t light_off;    // dynamic LDS: survivors of light frames
    void* stream;          // streaming decode: array of StreamState<MB> (NULL for a one-shot decode)
    int32_t* out_nodes;    // streaming: [B, t_total] trie node behind each written token
    int32_t t_total;       // streaming: frames the trie and the output rows are sized for
    int32_t out_stride;    // row length of out_tokens and of the traces
    double beam_window;  // SelectTopK's score window below the frame's best candidate; <= 0: off
    int32_t* frame_beam;        // optional trace: entries kept after each frame
    int32_t* out_token_frames;  // optional trace: frame at which each output token was appended
    int32_t* out_tokens;
    int32_t* out_lengths;
    float* out_scores;
    fltop_stats* stats;
    int32_t* nbest_count;
    int32_t* nbest_tokens;
    int32_t* nbest_lengths;
    double* nbest_pb;
    double* nbest_pnb;
};

__device__ inline uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ inline uint64_t child_hash(uint64_t h, int32_t tok) {
    return mix64(h + kGolden * (uint64_t)((int64_t)tok + 1));
}

// Order-preserving map fp64 -> u64 (larger score, larger key); -0.0 is folded into +0.0.
__device__ inline uint64_t order_key(double x) {
    if (x == 0.0) x = 0.0;
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__device__ inline double key_value(uint64_t k) {
    const uint64_t b = (k >> 63) ? (k & 0x7FFFFFFFFFFFFFFFull) : ~k;
    return __longlong_as_double((long long)b);
}

// ---- log-sum-exp of two log-masses ------------------------------------------------------
// hi + log1p(exp(lo - hi)).  The general-purpose exp and log1p of the device math library
// take about 250 instructions for this, and two of these sit on every frame's critical path;
// the argument ranges here are narrow (exp of a non-positive number, log1p of a number in
// [0,1]), so both are written out for just that: exp by n ln2 + r reduction and the Taylor
// series to r^13, log1p(u) as log(w) + c/w with w = fl(1+u), c its rounding error, log(w)
// = k ln2 + 2 atanh(s), s = f/(2+f), series to s^25.  The quotient is a reciprocal with two
// Newton steps, times f, its rounding error carried along.  The term is within 2.5 ulp of the
// exact one (measured against 80-bit arithmetic), i.e. far below half an ulp of the sum it is
// added to.
// REGS says only where the series' coefficients are kept; every build of the search rounds alike,
// so an utterance's scores do not depend on how many others are decoded with it.  In vector
// registers (40 of them) the multiply-adds read them directly; the compiler's own choice for a
// polynomial copies every coefficient into the accumulator first.  They are taken by light frames
// and by the builds that leave a thread 256 registers (unpruned V = 1024, beam 64: 11.30 -> 11.16
// ms; V = 32, beam 32: 2275 -> 2244 us); in the frames of the builds with fewer they cost 2% (beam
// 1000: 2257 -> 2309 us).
template <bool REGS>
__device__ __forceinline__ double fma_coeff(double x, double y, double coeff) {
    if constexpr (!REGS) return fma(x, y, coeff);
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(x), "v"(y), "v"(coeff));
    return d;
}

// Without branches: an operand may be -inf, or both.
template <bool REGS>
__device__ __forceinline__ double lse2_any(double a, double b) {
    const double hi = fmax(a, b);
    // exp(-800) is 0, and nothing below gets into the reduction (masses of masked tokens lie up to 1e42
    // apart, for which n is no integer any more); the difference is NaN for two operands of -inf
    const double x = fmax(fmin(a, b) - hi, -800.0);
    const double n = rint(x * 1.4426950408889634);  // log2(e)
    // ln2 in two pieces; the upper one has 21 trailing zero bits, so n * upper is exact
    double r = fma(-n, 0.6931471803691238, x);
    r = fma(-n, 1.9082149292705877e-10, r);
    double p = 1.6059043836821613e-10;  // 1/13!, then 1/12! ... 1/2!, 1, 1
    p = fma_coeff<REGS>(p, r, 2.08767569878681e-09);
    p = fma_coeff<REGS>(p, r, 2.505210838544172e-08);
    p = fma_coeff<REGS>(p, r, 2.755731922398589e-07);
    p = fma_coeff<REGS>(p, r, 2.7557319223985893e-06);
    p = fma_coeff<REGS>(p, r, 2.48015873015873e-05);
    p = fma_coeff<REGS>(p, r, 0.0001984126984126984);
    p = fma_coeff<REGS>(p, r, 0.001388888888888889);
    p = fma_coeff<REGS>(p, r, 0.008333333333333333);
    p = fma_coeff<REGS>(p, r, 0.041666666666666664);
    p = fma_coeff<REGS>(p, r, 0.16666666666666666);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    const double u = ldexp(p, (int)n);
    const double w = 1.0 + u;
    const double c = u - (w - 1.0);  // what the addition lost
    const bool upper = w > 1.4142135623730951;
    const double f = upper ? fma(w, 0.5, -1.0) : w - 1.0;  // exact; w / 2^k = 1 + f
    const double den = 2.0 + f;
    double y = __builtin_amdgcn_rcp(den);
    y = fma(fma(-den, y, 1.0), y, y);
    y = fma(fma(-den, y, 1.0), y, y);
    const double s = f * y;
    const double s_lo = fma(-s, den, f) * y;
    const double z = s * s;
    double q = 0.08;  // 2/25, then 2/23 ... 2/3
    q = fma_coeff<REGS>(q, z, 0.08695652173913043);
    q = fma_coeff<REGS>(q, z, 0.09523809523809523);
    q = fma_coeff<REGS>(q, z, 0.10526315789473684);
    q = fma_coeff<REGS>(q, z, 0.11764705882352941);
    q = fma_coeff<REGS>(q, z, 0.13333333333333333);
    q = fma_coeff<REGS>(q, z, 0.15384615384615385);
    q = fma_coeff<REGS>(q, z, 0.18181818181818182);
    q = fma_coeff<REGS>(q, z, 0.2222222222222222);
    q = fma_coeff<REGS>(q, z, 0.2857142857142857);
    q = fma_coeff<REGS>(q, z, 0.4);
    q = fma_coeff<REGS>(q, z, 0.6666666666666666);
    const double cw = (upper ? 0.5 * c : c) * __builtin_amdgcn_rcp(1.0 + f);  // c / w
    double tail = fma(s * z, q, 2.0 * s_lo + cw);
    if constexpr (!REGS) {  // (the same, for builds short of registers)
        if (upper) tail += 1.9082149292705877e-10;
        const double body = 2.0 * s + tail;
        return hi + (upper ? 0.6931471803691238 + body : body);
    }
    tail += upper ? 1.9082149292705877e-10 : 0.0;
    const double body = 2.0 * s + tail;
    return hi + (body + (upper ? 0.6931471803691238 : 0.0));
}

// The same, skipped by wavefronts in which no lane has two operands.
template <bool REGS>
__device__ __forceinline__ double lse2(double a, double b) {
    if (a == -INFINITY) return b;
    if (b == -INFINITY) return a;
    return lse2_any<REGS>(a, b);
}

// number of set bits of `mask` below this lane's own position
__device__ inline int lanes_below(uint64_t mask, int lane) {
    (void)lane;
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ inline uint64_t sat_add(uint64_t a, uint64_t b) {
    const uint64_t s = a + b;
    return s < a ? kAllOnes : s;
}

// top of bucket `b` of a window starting at lo with bucket width 2^sh (inclusive, saturating)
__device__ inline uint64_t bucket_top(uint64_t lo, int b, int sh) {
    const uint64_t nb = (uint64_t)(b + 1);
    if (sh > 0 && (nb >> (64 - sh)) != 0) return kAllOnes;  // nb << sh overflows
    return sat_add(lo, (nb << sh) - 1ull);
}

// Workgroup barrier that orders LDS traffic only: global loads and stores issued
// earlier (header chunks, survivor records, trie nodes) stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Value of `v` in the lane selected by a DPP control word, 0 where that lane does
// not exist or the row is masked off.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_or_zero(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}

// Inclusive prefix sum inside each row of 16 lanes (row_shr 1,2,3 then 4 and 8).
__device__ __forceinline__ int row_inclusive_scan(int v0) {
    int v1 = v0 + dpp_or_zero<0x111, 0xf>(v0);
    v1 += dpp_or_zero<0x112, 0xf>(v0);
    v1 += dpp_or_zero<0x113, 0xf>(v0);
    v1 += dpp_or_zero<0x114, 0xf>(v1);
    v1 += dpp_or_zero<0x118, 0xf>(v1);
    return v1;
}

// Inclusive prefix sum over the 64 lanes: row scans, then lane 15 of a row is
// broadcast into the next row (rows 1 and 3), then lane 31 into rows 2 and 3.
__device__ __forceinline__ int wave_inclusive_scan(int v0) {
    int v1 = row_inclusive_scan(v0);
    v1 += dpp_or_zero<0x142, 0xa>(v1);
    v1 += dpp_or_zero<0x143, 0xc>(v1);
    return v1;
}

// Inclusive prefix sum of floats over lanes 0..31 (the same over lanes 32..63).
__device__ __forceinline__ float row32_inclusive_sum(float v) {
    v += __int_as_float(dpp_or_zero<0x111, 0xf>(__float_as_int(v)));
    v += __int_as_float(dpp_or_zero<0x112, 0xf>(__float_as_int(v)));
    v += __int_as_float(dpp_or_zero<0x114, 0xf>(__float_as_int(v)));
    v += __int_as_float(dpp_or_zero<0x118, 0xf>(__float_as_int(v)));
    v += __int_as_float(dpp_or_zero<0x142, 0xa>(__float_as_int(v)));
    return v;
}

// Minimum of an unsigned value over the wavefront, returned in every lane: pairwise
// exchanges inside a row of 16 lanes, then lane 15 / lane 31 carried into the next rows
// (the last lane then holds the result).
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xf, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xa, 0xf, false));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xc, 0xf, false));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

// The same for a 64-bit value: high words first, then the low words of the lanes that
// hold the smallest high word.
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) {
    const uint32_t hi = wave_min_u32((uint32_t)(v >> 32));
    const uint32_t lo = wave_min_u32((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0xFFFFFFFFu);
    return ((uint64_t)hi << 32) | lo;
}

// dynamic LDS: dense_lp[V] fp32, s_tok[V] u16, in the 512-thread builds s_lp[V] fp32, then
// (optionally) the LM table
__host__ __device__ inline size_t s_lp_lds_offset(int V) {
    return (((size_t)V * (sizeof(float) + sizeof(uint16_t))) + 15) / 16 * 16;
}
__host__ __device__ inline size_t lm_lds_offset(int V, bool with_s_lp) {
    return s_lp_lds_offset(V) + (with_s_lp ? ((size_t)V * sizeof(float) + 15) / 16 * 16 : 0);
}

// Optional per-phase cycle accounting, compiled in only with -DFLTOP_PHASE_CLOCKS; the default
// build carries none of it.  The wavefronts of a workgroup form four groups (group 0 holds the
// stay candidates, group 2 the first extension candidates); lane 0 of each group's first
// wavefront keeps the clocks, so the table shows which group a barrier waits for.
#ifdef FLTOP_PHASE_CLOCKS
#define PHASE_MARK(idx)                      \
    do {                                     \
        if (ph_rec) {                        \
            const uint64_t now_ = clock64(); \
            ph_clk[idx] += now_ - ph_last;   \
            ph_last = now_;                  \
        }                                    \
    } while (0)
#else
#define PHASE_MARK(idx) \
    do {                \
    } while (0)
#endif

// What a frame header holds besides survivors 2..5 (one 32-byte LDS read).
struct HdrHead {
    int32_t count;
    uint32_t rec_base;
    float best;
    uint32_t div_magic;
    Survivor s0, s1;
};

// An LDS-typed pointer: reads through it are LDS reads, not generic (flat) ones, which
// would wait on the global-memory counter as well.
typedef const __attribute__((address_space(3))) float* LdsFloatPtr;

// Uniform per-frame values the candidate evaluation needs.  Only ever read through
// constant field names, so it dissolves into registers after inlining.
template <int MB>
struct FrameCtx {
    const BeamSlab<MB>* cur;
    const Links<MB>* lk;
    const float* dense_lp;   // LDS, K > 6 only: log-prob by token, -inf if pruned
    const uint16_t* s_tok;   // LDS, K > 6 only: surviving tokens, ascending
    const float* s_lp;       // LDS, K > 6 only, 512-thread builds: their log-probs, same order
    LdsFloatPtr lm_lds;      // LM table staged in LDS (kernel variant kLmLds)
    const float* lm_glb;     // LM table in global memory (kernel variant kLmGlobal)
    double lm_alpha, lm_beta;
    int V;
    bool big;                // survivors staged through LDS
    bool collapsed;          // blank-only frames came last: read p_b as total, p_nb as -inf
    int nb0;                 // 1 if blank survived (it is record 0 then)
    int Knb;                 // non-blank survivors
    uint32_t div_magic;      // from the frame header: umulhi(e, div_magic) is e / Knb, or one
                             // more when e is large (Knb > 1)
    uint64_t Rk;             // key of an upper bound of every candidate score
    // survivors 0..5 as plain scalars (an indexed private array would live in scratch)
    int32_t t0, t1, t2, t3, t4, t5;
    float l0, l1, l2, l3, l4, l5;
};

// Selection window: bucket(x) = (x - lo) >> sh over score distances (mode 0) or over
// prefix hashes of the candidates whose distance is exactly Dfix (mode 1).
struct Window {
    uint64_t lo, Dfix;
    int sh, mode;
};

// The register-resident survivors travel by value (twelve scalars): selecting among
// fields read through a pointer would be turned into an indexed load, i.e. scratch.
__device__ __forceinline__ float pick_lp(int32_t tok, int32_t t0, int32_t t1, int32_t t2,
                                         int32_t t3, int32_t t4, int32_t t5, float l0, float l1,
                                         float l2, float l3, float l4, float l5) {
    float r = -INFINITY;
    r = (t0 == tok) ? l0 : r;
    r = (t1 == tok) ? l1 : r;
    r = (t2 == tok) ? l2 : r;
    r = (t3 == tok) ? l3 : r;
    r = (t4 == tok) ? l4 : r;
    r = (t5 == tok) ? l5 : r;
    return r;
}

// (token, log-prob) of survivor k in one pass: the index compares serve both selections
template <int MB>
__device__ __forceinline__ int32_t surv_tok_lp(const FrameCtx<MB>& f, int k, double& lp) {
    if (f.big) {
        const int32_t s = (int32_t)f.s_tok[k];
        lp = (double)f.dense_lp[s];
        return s;
    }
    const int32_t t0 = f.t0, t1 = f.t1, t2 = f.t2, t3 = f.t3, t4 = f.t4, t5 = f.t5;
    const float l0 = f.l0, l1 = f.l1, l2 = f.l2, l3 = f.l3, l4 = f.l4, l5 = f.l5;
    int32_t r = t0;
    float l = l0;
    r = (k == 1) ? t1 : r;
    l = (k == 1) ? l1 : l;
    r = (k == 2) ? t2 : r;
    l = (k == 2) ? l2 : l;
    r = (k == 3) ? t3 : r;
    l = (k == 3) ? l3 : l;
    r = (k == 4) ? t4 : r;
    l = (k == 4) ? l4 : l;
    r = (k == 5) ? t5 : r;
    l = (k == 5) ? l5 : l;
    lp = (double)l;
    return r;
}

// log-prob of a token in this frame, -inf when it did not survive (or tok < 0)
template <int MB>
__device__ __forceinline__ double lp_of(const FrameCtx<MB>& f, int32_t tok) {
    if (tok < 0) return -INFINITY;
    if (f.big) return (double)f.dense_lp[tok];
    const int32_t t0 = f.t0, t1 = f.t1, t2 = f.t2, t3 = f.t3, t4 = f.t4, t5 = f.t5;
    const float l0 = f.l0, l1 = f.l1, l2 = f.l2, l3 = f.l3, l4 = f.l4, l5 = f.l5;
    return (double)pick_lp(tok, t0, t1, t2, t3, t4, t5, l0, l1, l2, l3, l4, l5);
}

// What the kernel is built for, as to the survivor lists of the frames it will meet (512 and
// 1024 threads; see launch_beam): short ones, as a threshold leaves them, every token of a
// vocabulary that gives a thread up to three candidates, or lists long enough for a score floor.
// and those whose floor few of the tokens can reach (kListsLongest).
enum : int { kListsShort = 0, kListsWhole = 1, kListsLong = 2, kListsLongest = 3 };
// ... and, added to that, that most of the frames' tokens cannot reach the beam (fltop_beam_reach.inc)
constexpr int kReachFlag = 8;

// The LM flavour is a kernel template parameter: with one kernel serving all three, the
// LDS read and the global read would meet at a joint wait on both memory counters.
enum : int { kLmNone = 0, kLmLds = 1, kLmGlobal = 2 };

template <int LM, int MB>
__device__ __forceinline__ double lm_term(const FrameCtx<MB>& f, int32_t prev, int32_t tok) {
    if (LM == kLmNone) return 0.0;
    const int32_t row = prev < 0 ? 0 : prev;
    const int64_t at = (int64_t)row * f.V + tok;
    const float v = (LM == kLmLds) ? f.lm_lds[at] : f.lm_glb[at];
    return f.lm_alpha * (double)v + f.lm_beta;
}

// Extension candidate e = i * Knb + k (entry i, non-blank survivor k): distance of its
// score below the reference, or ~0 when it has no mass or coincides with a beam entry
// (that entry's own update absorbs it).
// Extension candidate number e names entry i = e / Knb and non-blank survivor k = e % Knb.
template <int MB>
__device__ __forceinline__ void cand_of(const FrameCtx<MB>& f, int e, int& entry, int32_t& tok,
                                        double& lp) {
    // the reciprocal is rounded up, so for large e the quotient can come out one too large
    // (never more): a negative remainder says so
    int i = f.Knb > 1 ? (int)__umulhi((uint32_t)e, f.div_magic) : e;
    int k = e - i * f.Knb;
    if (k < 0) {
        --i;
        k += f.Knb;
    }
    entry = i;
    tok = surv_tok_lp(f, f.nb0 + k, lp);
}

// What a new prefix takes over from the entry it extends.  Builds with four wavefronts read it
// together with that entry's masses when the thread's first extension is evaluated, so that
// entering the beam does not begin with a round trip to LDS.
struct ExtSource {
    uint64_t h;  // the entry's prefix hash
    int32_t node, plen, xanc;
};

template <int LM, int MB, bool WITH_SOURCE = false>
__device__ __forceinline__ uint64_t eval_ext(const FrameCtx<MB>& f, int e, int& src_entry,
                                             int32_t& tok, const ColdRef<MB>* cold = nullptr,
                                             ExtSource* source = nullptr) {
    int i;
    int32_t s;
    double lps;
    cand_of(f, e, i, s, lps);
    src_entry = i;
    tok = s;
    // the four reads go out together; the children list is walked only on a mask hit
    const int32_t li = f.cur->last[i];
    const uint32_t km = f.lk->kidmask[i];
    const double pti = f.cur->ptot[i];
    const double pbi = f.collapsed ? pti : f.cur->pb[i];
    if constexpr (WITH_SOURCE) {
        source->h = f.cur->h[i];
        source->node = cold->node(i);
        source->plen = cold->plen(i);
        source->xanc = cold->xanc(i);
    }
    if ((km >> (s & 31)) & 1u) {  // maybe a child i+s is in the beam
        int guard = 0;
        for (int kid = f.lk->first_kid[i]; kid >= 0 && guard < MB;
             kid = f.lk->next_kid[kid], ++guard)
            if (f.cur->last[kid] == s) return kAllOnes;
    }
    const double src = (s == li) ? pbi : pti;
    const double sc = src + lps + lm_term<LM>(f, li, s);
    if (!(sc > -INFINITY)) return kAllOnes;
    return f.Rk - order_key(sc);
}

// ---- 512-thread builds: entry-major candidates --------------------------------------------
// Frames of a large vocabulary (or a large beam) have thousands of candidates, dozens per
// thread.  There a thread takes all its candidates from ONE beam entry, which it reads once
// per frame, and "is entry i extended by token s already in the beam?" is one probe of a
// table of (parent place, token) pairs, whatever the number of children (with lanes on
// different entries, walking the children lists would cost every lane the longest list).

// What an extension candidate needs of its beam entry.
struct EntryView {
    int32_t last;      // the entry's last token
    uint32_t kidmask;  // bit (token & 31) of every child in the beam
    double ptot, pb;   // total mass, and the mass of alignments ending in blank
};

template <int MB>
__device__ __forceinline__ EntryView view_entry(const FrameCtx<MB>& f, int i) {
    EntryView v;
    v.last = f.cur->last[i];
    v.kidmask = f.lk->kidmask[i];
    v.ptot = f.cur->ptot[i];
    v.pb = f.collapsed ? v.ptot : f.cur->pb[i];
    return v;
}

__device__ __forceinline__ uint32_t kid_key(int parent, int32_t tok) {
    return ((uint32_t)parent << 16) | ((uint32_t)tok & 0xffffu);
}
static_assert(FLTOP_MAX_VOCAB <= 65536 && FLTOP_MAX_BEAM <= 32768, "a (place, token) pair is 32 bits");
constexpr uint32_t kNoKid = 0xffffffffu;

// kidset: open addressing over `slots` (a power of two) words, kNoKid = empty
__device__ __forceinline__ void kidset_insert(uint32_t* kidset, int slots, int parent, int32_t tok) {
    const uint32_t key = kid_key(parent, tok);
    uint32_t hs = (key * 2654435761u >> 12) & (slots - 1);
    for (int probe = 0; probe < slots; ++probe) {
        if (atomicCAS(&kidset[hs], kNoKid, key) == kNoKid) break;
        hs = (hs + 1) & (slots - 1);
    }
}

__device__ __forceinline__ bool kidset_has(const uint32_t* kidset, int slots, int parent, int32_t tok) {
    const uint32_t key = kid_key(parent, tok);
    uint32_t hs = (key * 2654435761u >> 12) & (slots - 1);
    bool found = false, done = false;  // (one way out of the loop)
    for (int probe = 0; probe < slots && !done; ++probe) {
        const uint32_t v = kidset[hs];
        found = v == key;
        done = found || v == kNoKid;
        hs = (hs + 1) & (slots - 1);
    }
    return found;
}

// (token, log-prob) of survivor k, the staged ones by rank
template <int MB>
__device__ __forceinline__ int32_t surv_by_rank(const FrameCtx<MB>& f, int k, double& lp) {
    if (f.big) {
        lp = (double)f.s_lp[k];
        return (int32_t)f.s_tok[k];
    }
    return surv_tok_lp(f, k, lp);
}

// Extension of entry i (seen as `v`) by non-blank survivor k: distance of its score below
// the reference, or ~0 when it has no mass, lies below `floor` or coincides with a beam entry.
template <int LM, int MB>
__device__ __forceinline__ uint64_t eval_ext_of(const FrameCtx<MB>& f, const EntryView& v, int i,
                                                int k, const uint32_t* kidset, int kid_slots,
                                                double floor, int32_t& tok) {
    double lps;
    const int32_t s = surv_by_rank(f, f.nb0 + k, lps);
    tok = s;
    if ((v.kidmask >> (s & 31)) & 1u) {  // maybe a child i+s is in the beam
        if (kidset_has(kidset, kid_slots, i, s)) return kAllOnes;
    }
    const double src = (s == v.last) ? v.pb : v.ptot;
    const double sc = src + lps + lm_term<LM>(f, v.last, s);
    if (!(sc > -INFINITY) || sc < floor) return kAllOnes;
    return f.Rk - order_key(sc);
}

// Token of non-blank survivor k alone (for a candidate whose distance is already known).
template <int MB>
__device__ __forceinline__ int32_t ext_token(const FrameCtx<MB>& f, int k) {
    double lp_unused;
    return surv_by_rank(f, f.nb0 + k, lp_unused);
}

template <int MB>
__device__ __forceinline__ uint64_t cand_hash(const FrameCtx<MB>& f, int src_entry, int32_t tok) {
    const uint64_t h = f.cur->h[src_entry];
    return tok < 0 ? h : child_hash(h, tok);
}

__device__ __forceinline__ int window_bin(const Window& w, uint64_t x) {
    const uint64_t q = (x - w.lo) >> w.sh;
    return q > (uint64_t)(kFine - 1) ? (kFine - 1) : (int)q;
}

// One candidate into the two-level histogram of the current window.
template <int MB>
__device__ __forceinline__ void hist_add(const FrameCtx<MB>& f, const Window& w, uint64_t D, int se,
                                         int32_t tk, uint32_t* hfine, uint32_t* hcoarse) {
    uint64_t x = D;
    if (w.mode != 0) {
        if (D != w.Dfix) return;
        x = cand_hash(f, se, tk);
    }
    if (x < w.lo) return;
    const int bin = window_bin(w, x);
    atomicAdd(&hfine[bin], 1u);
    atomicAdd(&hcoarse[bin >> 4], 1u);
}

// The same for the candidates beyond the register cache, of which a frame may have thousands
// (and for all of a thread's, see kCountAll).  All that lie beyond the window share the last
// bin, and one LDS word cannot take that many atomics quickly: those are counted in a register
// (`n_clamp`) instead.
template <int MB>
__device__ __forceinline__ void hist_add_many(const FrameCtx<MB>& f, const Window& w, uint64_t D,
                                              int se, int32_t tk, uint32_t* hfine,
                                              uint32_t* hcoarse, int& n_clamp) {
    uint64_t x = D;
    if (w.mode != 0) {
        if (D != w.Dfix) return;
        x = cand_hash(f, se, tk);
    }
    if (x < w.lo) return;
    const int bin = window_bin(w, x);
    if (bin == kFine - 1) {
        ++n_clamp;
        return;
    }
    atomicAdd(&hfine[bin], 1u);
    atomicAdd(&hcoarse[bin >> 4], 1u);
}

// One candidate into the boundary list if it falls into bucket `bstar`.
template <int MB>
__device__ __forceinline__ void boundary_add(const FrameCtx<MB>& f, const Window& w, int bstar,
                                             uint64_t D, int se, int32_t tk, int32_t* count,
                                             uint64_t* bl_D, uint64_t* bl_h) {
    uint64_t x = D;
    uint64_t hh = 0;
    bool have_h = false;
    if (w.mode != 0) {
        if (D != w.Dfix) return;
        hh = cand_hash(f, se, tk);
        have_h = true;
        x = hh;
    }
    if (x < w.lo) return;
    if (window_bin(w, x) != bstar) return;
    if (!have_h) hh = cand_hash(f, se, tk);
    const int pos = atomicAdd(count, 1);
    if (pos < kExactCap) {
        bl_D[pos] = D;
        bl_h[pos] = hh;
    }
}

// Kept iff (D, hash) <= (selD, selH) lexicographically; the hash is computed only on
// a distance tie.
template <int MB>
__device__ __forceinline__ bool is_selected(const FrameCtx<MB>& f, uint64_t selD, uint64_t selH,
                                            uint64_t D, int se, int32_t tk, uint64_t& hh,
                                            bool& have_h) {
    if (D < selD) return true;
    if (D != selD) return false;
    hh = cand_hash(f, se, tk);
    have_h = true;
    return hh <= selH;
}

template <int MB>
__device__ __forceinline__ void publish_hash(Links<MB>* lkn, uint64_t hh, int slot) {
    constexpr int kHashSlots = SlabTraits<MB>::kHashSlots;
    uint32_t hs = (uint32_t)hh & (kHashSlots - 1);
    if (atomicCAS(&lkn->ht[hs], -1, slot) == -1) return;  // the usual case: the first place is free
    for (int probe = 1; probe < kHashSlots; ++probe) {
        hs = (hs + 1) & (kHashSlots - 1);
        if (atomicCAS(&lkn->ht[hs], -1, slot) == -1) break;
    }
}

// What an entry that stays in the beam carries over unchanged.  It is read together with the
// entry's masses when the stay candidate is evaluated, so that the copy into the next beam
// does not begin with a round trip to wherever these fields live.
struct StayFields {
    uint64_t h, hp;
    int32_t par, last, node, plen, xanc;
};

// Entry `se` keeps its prefix: copy it into `slot` of the next beam with its new masses.
template <int MB, bool PREFETCHED>
__device__ __forceinline__ void emit_stay(const FrameCtx<MB>& f, BeamSlab<MB>* nxt, Links<MB>* lkn,
                                          const ColdRef<MB>& ccur, const ColdRef<MB>& cnxt,
                                          int32_t* newslot, int slot, int beam, int se, double pb,
                                          double pnb, double tot, const StayFields& sf) {
    if (slot >= beam) return;  // only after a hash collision
    // where this entry went, and where its parent was (or -2: the parent was not in the
    // beam, so it can only be in the new one as a fresh extension)
    if constexpr (PREFETCHED) {
        newslot[se] = slot;
        lkn->par[slot] = sf.par >= 0 ? sf.par : -2;
        nxt->h[slot] = sf.h;
        nxt->pb[slot] = pb;
        nxt->pnb[slot] = pnb;
        nxt->ptot[slot] = tot;
        nxt->last[slot] = sf.last;
        cnxt.set(slot, sf.hp, sf.node, sf.plen, sf.xanc);
    } else {
        const BeamSlab<MB>* cur = f.cur;
        const uint64_t hh = cur->h[se];
        const int32_t par_old = f.lk->par[se];
        newslot[se] = slot;
        lkn->par[slot] = par_old >= 0 ? par_old : -2;
        nxt->h[slot] = hh;
        nxt->pb[slot] = pb;
        nxt->pnb[slot] = pnb;
        nxt->ptot[slot] = tot;
        nxt->last[slot] = cur->last[se];
        cnxt.set(slot, ccur.hp(se), ccur.node(se), ccur.plen(se), ccur.xanc(se));
    }
}

// Entry `se` extended by token `tk` becomes a new prefix in `slot`; its trie node id is
// fixed by (frame, slot), so no counter is needed.
template <int MB>
__device__ __forceinline__ void emit_ext(const FrameCtx<MB>& f, BeamSlab<MB>* nxt, Links<MB>* lkn,
                                         const ColdRef<MB>& ccur, const ColdRef<MB>& cnxt, int slot,
                                         int beam, int t, uint64_t D, int se, int32_t tk,
                                         uint64_t hh, bool have_h, TrieNode* trie,
                                         int64_t trie_stride) {
    if (slot >= beam) return;
    const BeamSlab<MB>* cur = f.cur;
    if (!have_h) hh = cand_hash(f, se, tk);
    const double sc = key_value(f.Rk - D);
    const int node = 1 + t * beam + slot;
    const int depth = ccur.plen(se) + 1;
    const int32_t xa = ccur.xanc(se);
    nxt->h[slot] = hh;
    nxt->pb[slot] = -INFINITY;
    nxt->pnb[slot] = sc;
    nxt->ptot[slot] = sc;
    nxt->last[slot] = tk;
    cnxt.set(slot, cur->h[se], node, depth, (depth & 7) == 0 ? node : xa);
    TrieNode tn;
    tn.parent = ccur.node(se);
    tn.xup = xa;
    tn.tok = tk;
    tn.depth = depth;
    if ((int64_t)node < trie_stride) trie[node] = tn;
    lkn->par[slot] = se;  // the parent's place in the old beam
    publish_hash(lkn, hh, slot);
}

// The same with what the new prefix takes over from entry `se` already in registers.
template <int MB>
__device__ __forceinline__ void emit_ext_prefetched(const FrameCtx<MB>& f, BeamSlab<MB>* nxt, Links<MB>* lkn,
                                         const ColdRef<MB>& ccur, const ColdRef<MB>& cnxt, int slot,
                                         int beam, int t, uint64_t D, int se, int32_t tk,
                                         uint64_t hh, bool have_h, TrieNode* trie,
                                         int64_t trie_stride, const ExtSource* source) {
    constexpr bool WITH_SOURCE = true;
    if (slot >= beam) return;
    const BeamSlab<MB>* cur = f.cur;
    if (!have_h) {
        if constexpr (WITH_SOURCE) hh = child_hash(source->h, tk);
        else hh = cand_hash(f, se, tk);
    }
    const double sc = key_value(f.Rk - D);
    const int node = 1 + t * beam + slot;
    const int depth = (WITH_SOURCE ? source->plen : ccur.plen(se)) + 1;
    const int32_t xa = WITH_SOURCE ? source->xanc : ccur.xanc(se);
    nxt->h[slot] = hh;
    nxt->pb[slot] = -INFINITY;
    nxt->pnb[slot] = sc;
    nxt->ptot[slot] = sc;
    nxt->last[slot] = tk;
    cnxt.set(slot, WITH_SOURCE ? source->h : cur->h[se], node, depth, (depth & 7) == 0 ? node : xa);
    TrieNode tn;
    tn.parent = WITH_SOURCE ? source->node : ccur.node(se);
    tn.xup = xa;
    tn.tok = tk;
    tn.depth = depth;
    if ((int64_t)node < trie_stride) trie[node] = tn;
    lkn->par[slot] = se;  // the parent's place in the old beam
    publish_hash(lkn, hh, slot);
}

// Light frames (fltop_beam_light.inc).
typedef unsigned short Ushort2 __attribute__((ext_vector_type(2)));
// Their tables, one per generation: the bins, then a bitmap over the hashes of the prefixes that entered.
// They take the place of the general path's hash tables, which light frames do not need: with tables of
// their own (2.5 KB in the 64-entry state) a batch with a table in LDS had 5 workgroups per CU instead
// of 6 (1536 utterances x 100 frames, V = 32, beam 64, R = 0.001: 816 -> 1169 us).
template <int THREADS, int MB>
struct LightTables {
    static constexpr int kWords = SlabTraits<MB>::kHashSlots;
    static constexpr int kFresh = THREADS == kThreadsDense ? 128 : 256;
    static_assert(kLightBins / 2 + kFresh <= kWords, "bins and bitmap");
    static __device__ __forceinline__ int fresh_word(uint64_t h) {
        return kLightBins / 2 + ((int)((uint32_t)h >> 5) & (kFresh - 1));
    }
    static __device__ __forceinline__ uint32_t* of(Links<MB>& lk) { return reinterpret_cast<uint32_t*>(lk.ht); }
    // where, from there, a word per lane lies that nobody reads (light frames have no children lists)
    static constexpr int kUnread = -(int)((offsetof(Links<MB>, ht) - offsetof(Links<MB>, next_kid)) / 4);
    static_assert(MB >= kWave, "one per lane");
};

// Value of another lane, the same one for the whole wavefront.
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int from) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, from);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), from);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ double lane_value(double v, int from) {
    return __longlong_as_double((long long)lane_value((uint64_t)__double_as_longlong(v), from));
}

// Selection of both kinds of light frames.  Both halves of a word:
__device__ __forceinline__ uint32_t sum16(uint32_t two, uint32_t acc) {
    return __builtin_amdgcn_udot2(__builtin_bit_cast(Ushort2, two), Ushort2{1, 1}, acc, false);
}
// Counts a candidate in; what its bin held before.  (What is not alive counts into words that nobody reads, one per
// lane.)
template <typename Tables>
__device__ __forceinline__ uint32_t count_in(uint32_t* hist, uint32_t bin, bool live, int lane) {
    const uint32_t sh = (bin & 1u) * 16u;
    const int word = live ? (int)(bin >> 1) : Tables::kUnread + lane;
    return __builtin_amdgcn_ubfe(atomicAdd(&hist[word], 1u << sh), sh, 16u);
}
// The row of four bins (row = lane) that a bin lies in; with the candidates before its rows, one per lane, those in better
// bins than this one, and in this one.
__device__ __forceinline__ uint64_t row_of(const uint32_t* hist, uint32_t bin) {
    return reinterpret_cast<const uint64_t*>(hist)[bin >> 2];
}
__device__ __forceinline__ int better_than(uint32_t bin, uint64_t row, int before_row, int& same) {
    const int before = __builtin_amdgcn_ds_bpermute((int)(bin & ~3u), before_row);
    const uint32_t sh = (bin & 3u) * 16u;
    const uint64_t lower = row & ~(~0ull << sh);
    same = (int)((uint32_t)(row >> sh) & 0xFFFFu);
    return before + (int)sum16((uint32_t)lower, sum16((uint32_t)(lower >> 32), 0u));
}
// Place in the new beam, which takes `limit` entries of `most`, of a candidate whose bin fits it (else `most`); `split`: its
// bin fits only in part.  (What is not alive counts as far behind.)
__device__ __forceinline__ int place_of(bool live, int ahead, int same, uint32_t number, int limit, int most,
                                        bool& split) {
    ahead = live ? ahead : 4 * most;
    const int end = ahead + same;
    split = ((ahead - limit) & (limit - end)) < 0;
    return end <= limit ? ahead + (int)number : most;
}
// Score window: only what scores at least the best score less the window is kept.  That is an upper part of the
// candidates' order like the beam's, so it is enough to know how many.
__device__ __forceinline__ int kept_by_window(const double* scores, int n, double window, int lane) {
    uint64_t nearest = kAllOnes;
    for (int c = lane; c < n; c += kWave) nearest = min(nearest, ~order_key(scores[c]));
    const double floor = key_value(~wave_min_u64(nearest)) - window;
    int kept = 0;
    for (int c = lane; c < n; c += kWave) {
        const double o = scores[c];
        kept += __popcll(__builtin_amdgcn_ballot_w64(o >= floor && o > -INFINITY));
    }
    return kept;
}

// State of a beam's parent links between frames: places of the parents, and the children lists that
// the general path needs; or what a light frame leaves: the parents' places in the beam before, -2
// for a parent that was not there.
enum : int { kLinksBuilt = 0, kLinksCoded = 1 };

// WAVES = wavefronts per SIMD the register budget is cut for: 2 leaves the allocator all it
// asks for (no spills: the fastest single workgroup); 3 and 4 spill a few registers (each
// frame some per cent slower) so that more utterances are resident when the batch has more
// workgroups than the chip can hold at 2.
// LISTS: the survivor lists it is made for.
template <int LM, int THREADS, int MB, int WAVES, int LISTS_AND_REACH>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(WAVES, WAVES)))
void beam_kernel(BeamArgs a) {
    constexpr int LISTS = LISTS_AND_REACH & ~kReachFlag;
    constexpr int kThreads = THREADS;
    constexpr int kWalkers = kThreads < kWaypoints ? kThreads : kWaypoints;  // back-walk batch
    static_assert(THREADS >= 4 * kChunk, "a chunk of headers is staged 16 bytes per thread");
    constexpr int kMaxBeam = MB;
    constexpr int kHashSlots = SlabTraits<MB>::kHashSlots;
    constexpr bool kColdGlobal = SlabTraits<MB>::kColdGlobal;
    static_assert(THREADS >= MB, "one thread per beam entry");
    // builds with 512 threads or more take a thread's candidates from one entry (see EntryView)
    constexpr bool kEntryMajor = THREADS >= kThreadsLarge;
    static_assert(kEntryMajor || LISTS < kListsLong, "the floor is made for the entry-major mapping");
    constexpr bool FLOOR = LISTS >= kListsLong;  // with the score floor (see `floored_frame`)
    // ... and a list of the tokens that can reach it
    constexpr bool LISTED = LISTS == kListsLongest;
    static_assert(kEntryMajor || !kColdGlobal, "the largest capacity has no children lists");
    // Builds with four wavefronts read what a staying entry carries over together with its
    // masses (measured: cfg 3 -1.7%); the larger builds, shorter of registers, read it when the
    // entry is copied (measured there: +0.4% to +1.4% otherwise).
    constexpr bool kPrefetchStay = !kEntryMajor;
    constexpr bool kLseRegs = WAVES == 2;
    // Whether a thread counts all its candidates of the last bin in a register, its stay and first
    // extension included: hundreds of a frame's candidates may lie beyond the histogram's window,
    // and atomics on one word queue up (64 utterances x 500 frames, V = 32, every token kept: 2354
    // -> 2270 us).  Frames of short lists have few there and pay for the wavefront's sum (64 x 500
    // frames, V = 32, beam 200, R = 0.1: 609 -> 623 us; V = 100, beam 8, table in memory: 605 -> 627).
    constexpr bool kCountAll = kEntryMajor && LISTS != kListsShort;
    // Where the last bin's count is handed over: inside the block of a thread's later candidates,
    // which the usual frame of a pruned small vocabulary jumps over, or behind it, which is one
    // more branch for that frame (measured when all of these calls' frames took the general path).  It costs the 256- and 128-thread builds without a table 2-3% (64
    // utterances x 500 frames, V = 32, beam 32: 625 against 644 us; 4096 of them: 2287 against
    // 2327); with a table in LDS they are 0.2-2% faster with it (128 x 500, beam 64: 692 against
    // 690 us; 1500 x 60, beam 100, R = 0.001: 1238 against 1213).  The 256-thread build for batches
    // of large vocabularies beyond the chip, whose frames mostly have later candidates, is faster
    // with it (600 x 100, V = 1024: 698 against 668 us), with a table in memory slower (740
    // against 748).
    constexpr bool kClampApart =
        kCountAll || (!kEntryMajor && LM == kLmLds) ||
        (THREADS == kThreadsSmall && WAVES == 4 && LM == kLmNone);
    // Which way a uniform branch of the frame loop usually goes, for the block layout of the
    // four-wavefront builds: a lone wavefront per SIMD pays for every taken branch, and with the
    // usual path laid out straight a frame is 2-4% shorter (the set below was chosen by timing
    // builds with each hint on and off; the builds with 512 and 1024 threads gained nothing from
    // any of them and are left to the compiler's own guesses).
#define FLTOP_RARE(c) (kEntryMajor ? !!(c) : __builtin_expect(!!(c), 0))
#define FLTOP_USUAL(c) (kEntryMajor ? !!(c) : __builtin_expect(!!(c), 1))
    constexpr int kKidSlots = kEntryMajor ? (kColdGlobal ? 2 * MB : 4 * MB) : 4;
    __shared__ uint32_t kidset2[2][kKidSlots];  // (parent place, token) pairs, per generation
    // The two generations of the beam.  Both parts of one at the same offset from the other's takes fewer registers for
    // their addresses; the builds cut for four wavefronts per SIMD are faster with the parts apart (555 utterances x
    // 100 frames, V = 32, beam 77, R = 0: 2833 us, together 3154; the others together: 64 x 200, V = 73, table, beam 79,
    // R = 0.01 318 us, apart 342; 128 x 400, V = 1024, beam 64, R = 0 2654 and 2704; 2527 x 92, beam 20, Top-4, window
    // 25 599 and 632).  (What is not used takes no room.)
    constexpr bool kTogether = WAVES < 4 || THREADS == kThreadsHuge;
    __shared__ Generation<MB> both_parts[2];
    __shared__ BeamSlab<MB> slabs[2];
    __shared__ Links<MB> all_links[2];
    auto slab_of = [&](int g) __attribute__((always_inline)) -> BeamSlab<MB>& {
        if constexpr (kTogether) return both_parts[g].slab;
        else return slabs[g];
    };
    auto links_of = [&](int g) __attribute__((always_inline)) -> Links<MB>& {
        if constexpr (kTogether) return both_parts[g].links;
        else return all_links[g];
    };
    __shared__ __align__(16) uint32_t hfine[kFine];
    __shared__ __align__(16) uint32_t hcoarse[kCoarse];
    __shared__ uint64_t bl_D[kExactCap], bl_h[kExactCap];
    __shared__ FrameHdr ring[kChunk];
    __shared__ uint64_t sh_selD, sh_selH, sh_kbest;
    __shared__ uint64_t sh_minD;  // smallest distance (= best score) among a frame's candidates
    // frames with a score floor (see `floored_frame`)
    __shared__ uint64_t sh_floor;  // complement of the largest of the entries' own distances
    __shared__ int32_t sh_toptok;  // non-blank token with the frame's top emission, if there is one
    __shared__ int32_t sh_below;   // candidates below the floor
    __shared__ uint16_t s_list[LISTED ? kListCap : 2];  // non-blank survivors that can reach it
    __shared__ int32_t sh_nlist, sh_nout;  // how many those are, and the others with mass
    __shared__ int32_t sh_nnew, sh_blcount, sh_best;
    __shared__ unsigned long long sh_stat[8];
    __shared__ __align__(16) int32_t newslot[kMaxBeam];  // old beam index -> new beam index of an entry that stays
    // (the builds for more utterances than that have no LDS and registers to spare for them)
    // ... of the tokens that can reach the beam only, however long the lists are (kReach), or of all that frames
    // with few of them keep
    constexpr bool kReach = (LISTS_AND_REACH & kReachFlag) != 0;
    static_assert(!kReach || (WAVES == 2 && MB == kBeamSmall), "LDS and registers to spare");
    constexpr bool kLight =
        kReach || (LISTS == kListsShort && !kReach && ((THREADS == kThreadsSmall && WAVES == 2) || (THREADS == kThreadsDense && MB == kBeamTiny)));
    using Tables = LightTables<THREADS, MB>;
    // light frame in which entry i's extension by non-blank survivor k was last merged, at
    // (k << light_lg) + i
    __shared__ uint32_t light_kill[kLight && !kReach ? kLightRounds * (kThreads - kWave) : 4];
    __shared__ LightLine sh_light[2];
    __shared__ int32_t sh_left[4];  // pairs without mass, or merged, of tokens left out; frame after frame
    extern __shared__ __align__(16) unsigned char dyn_lds[];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int b = blockIdx.x;
    const int V = a.V;
    const int beam = a.beam;
    const int64_t trie_stride = a.trie_stride;

    float* dense_lp = reinterpret_cast<float*>(dyn_lds);
    uint16_t* s_tok = reinterpret_cast<uint16_t*>(dyn_lds + (size_t)V * sizeof(float));
    float* s_lp = reinterpret_cast<float*>(dyn_lds + s_lp_lds_offset(V));  // kEntryMajor only
    float* lm_s = reinterpret_cast<float*>(dyn_lds + lm_lds_offset(V, kEntryMajor));
    constexpr bool has_lm = LM != kLmNone;
    // Distances of the candidates beyond the register cache, as the first histogram pass
    // worked them out: the later passes and the selection read them back instead of
    // evaluating the candidate again (row j, this thread's place = its candidate number
    // kRegCand + j).  A thread only ever reads what it wrote itself.
    uint64_t* const dcache = reinterpret_cast<uint64_t*>(dyn_lds + a.dcache_off) + tid;
    // light frames: scores of the candidates, the stays, then the extensions of each round
    // (light_candidates of them; launch_beam makes the distance cache that large)
    double* const light_score = reinterpret_cast<double*>(dyn_lds + a.dcache_off);
    // kReach: the survivors of a light frame, for every second frame each: by token (log-prob; the frame's
    // number in its chunk, and from bit 8 on the token's place in the list, from 1), and listed (one place more
    // of both: for what is not to be written); and per listed token and entry the light frame in which that
    // extension was last merged, at (place << light_lg) + entry
    uint4* const light_tokens = reinterpret_cast<uint4*>(dyn_lds + a.light_off);
    const int light_table_words = V + 1;  // 16 bytes each
    const LightShape light_layout = light_shape(beam, kThreads);
    const int reach_places = reach_list_places(light_layout.blocks, kThreads, V);
    Survivor* const light_list = reinterpret_cast<Survivor*>(light_tokens + light_table_words);
    uint32_t* const light_notes = reinterpret_cast<uint32_t*>(light_list + 2 * (reach_places + 1));
    const int drows = a.dcache_rows;

    StreamState<MB>* const carried =
        a.stream ? static_cast<StreamState<MB>*>(a.stream) + b : nullptr;  // uniform
    // kColdGlobal: this utterance's two generations of trie bookkeeping fields
    ColdSlab<MB>* const cold_gen =
        kColdGlobal ? static_cast<ColdSlab<MB>*>(a.cold) + 2 * (int64_t)b : nullptr;
    const int32_t t_base = carried ? carried->frames_done : 0;
    int32_t len = a.lengths[b];
    len = len < 0 ? 0 : (len > a.T ? a.T : len);
    if (carried && len > a.t_total - t_base) len = max(0, a.t_total - t_base);
    const int64_t g_base = (int64_t)b * a.T;
    const int64_t trace_base = (int64_t)b * a.out_stride + t_base;
    const Survivor* rec_all = a.rec;

    // ---- header chunks: 32 frames x 64 B = 128 threads x 16 B ------------------------
    // Chunk c+1 is loaded into registers while chunk c is decoded and moved into LDS at
    // the chunk boundary, so the only wait for it sits in the outer (per-chunk) loop.
    const uint4* hdr_words = reinterpret_cast<const uint4*>(a.hdr + g_base);
#define FLTOP_LOAD_CHUNK(dst, c)                                                         \
    do {                                                                                 \
        (dst) = make_uint4(0u, 0u, 0u, 0u);                                              \
        if (tid < 4 * kChunk && (c) * kChunk + (tid >> 2) < len)                         \
            (dst) = hdr_words[(int64_t)(c) * (4 * kChunk) + tid];                        \
    } while (0)
#define FLTOP_RING_HEAD(t) (*reinterpret_cast<const HdrHead*>(&ring[(t) % kChunk]))

    uint4 staged;
    FLTOP_LOAD_CHUNK(staged, 0);

    // ---- one-time initialisation ------------------------------------------------
    for (int v = tid; v < V; v += kThreads) dense_lp[v] = -INFINITY;
    for (int i = tid; i < kFine; i += kThreads) hfine[i] = 0u;
    if (tid < kCoarse) hcoarse[tid] = 0u;
    if (LM == kLmLds)
        for (int i = tid; i < V * V; i += kThreads) lm_s[i] = a.lm_table[i];
    for (int g2 = 0; g2 < 2; ++g2) {
        if (tid < kMaxBeam) {
            links_of(g2).par[tid] = -1;
            if (!kColdGlobal) {
                links_of(g2).first_kid[tid] = -1;
                links_of(g2).next_kid[tid] = -1;
            }
            links_of(g2).kidmask[tid] = 0u;
        }
        for (int i = tid; i < kHashSlots; i += kThreads) links_of(g2).ht[i] = -1;
    }
    if (kEntryMajor)
        for (int i = tid; i < 2 * kKidSlots; i += kThreads) (&kidset2[0][0])[i] = kNoKid;
    if (tid == 0) {
        sh_nnew = 0;
        sh_blcount = 0;
        sh_minD = kAllOnes;
        if (FLOOR) {
            sh_floor = kAllOnes;
            sh_toptok = INT32_MAX;
            sh_below = 0;
            sh_nlist = 0;
            sh_nout = 0;
        }
    }
    if (tid < 8) sh_stat[tid] = 0ull;
    if constexpr (kLight) {
        if constexpr (!kReach) {
            for (int i = tid; i < kLightRounds * (kThreads - kWave); i += kThreads) light_kill[i] = 0u;
        } else if (a.light_off != 0) {
            for (int i = tid; i < reach_places << light_layout.lg; i += kThreads) light_notes[i] = 0u;
        }
    }
    if (carried) {  // the beam as the previous chunk left it
        __syncthreads();  // the link arrays were just preset by other threads
        const uint32_t* src = reinterpret_cast<const uint32_t*>(&carried->slab);
        uint32_t* dst = reinterpret_cast<uint32_t*>(&slab_of(0));
        for (int i = tid; i < (int)(sizeof(BeamSlab<MB>) / 4); i += kThreads) dst[i] = src[i];
        const uint32_t* lsrc = reinterpret_cast<const uint32_t*>(carried->par);
        uint32_t* ldst = reinterpret_cast<uint32_t*>(&links_of(0));
        for (int i = tid; i < 4 * kMaxBeam; i += kThreads) ldst[i] = lsrc[i];
    } else if (tid == 0) {
        BeamSlab<MB>& s0 = slab_of(0);
        s0.h[0] = kGolden;
        s0.pb[0] = 0.0;
        s0.pnb[0] = -INFINITY;
        s0.ptot[0] = 0.0;
        s0.last[0] = -1;
        ColdRef<MB>{&slab_of(0), cold_gen}.set(0, 0, 0, 0, 0);
    }
    TrieNode* trie = a.trie + (int64_t)b * trie_stride;
    double lm_ub = 0.0;  // upper bound of any LM term (never below 0)
    bool lm_gaps = false;  // (uniform) pairs of the table have no mass
    if (has_lm) {
        static_assert(kLmBoundParts == kWave, "one partial maximum per lane");
        const float signed_part = a.lm_bound[lane];
        if (LISTED || kReach) lm_gaps = __builtin_amdgcn_ballot_w64(__float_as_int(signed_part) < 0) != 0;
        float part = fabsf(signed_part);
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) part = fmaxf(part, __shfl_xor(part, o, kWave));
        lm_ub = (double)part;
    }
    const double lm_reach = lm_ub * (1.0 + 0x1p-22);  // the same, whichever way the bound was rounded
    __syncthreads();
    if (kEntryMajor && carried) {  // the pair table is not carried: rebuild it from the links
        if (tid < carried->n_live && links_of(0).par[tid] >= 0)
            kidset_insert(kidset2[0], kKidSlots, links_of(0).par[tid], slab_of(0).last[tid]);
        __syncthreads();
    }

    // non-blank survivors up to which no thread has kFlooredFrom candidates (full beam)
    const int floored_above = (kFlooredFrom - 1) * (kThreads / beam);
    int mapped_for = -1;  // kEntryMajor: the beam size the thread -> entry mapping was made for
    int ext_i = 0, ext_g = 0, ext_G = 1;
    int gen = 0;         // beam generation: slab_of(gen), links_of(gen)
    int n_live = 1;
    bool collapsed = false;  // blank-only frames since the beam was last written
    double kmax_v = 0.0, kmin_v = 0.0;  // bounds of the best / worst score
    // the latter is a bound, not an estimate (kReach only: kept by all builds it made the general path's frames up to
    // 4% longer, 128 utterances x 300 frames, V = 32, table, beam 64, R = 0: 1571 -> 1604 us)
    bool kmin_sure = false;
    bool failed = false;     // a frame's survivor records did not fit the workspace
    int prev_out_len = 0;       // streaming: length of the transcript the last call wrote ...
    uint64_t prev_tokens_at = 0, prev_frames_at = 0;  // ... and the rows it wrote it to
    if (carried) {
        prev_out_len = carried->out_len;
        prev_tokens_at = carried->out_tokens_at;
        prev_frames_at = carried->out_frames_at;
        n_live = carried->n_live;
        collapsed = (carried->collapsed & 1) != 0;
        if constexpr (kReach) kmin_sure = (carried->collapsed & 2) != 0;
        kmax_v = carried->kmax;
        kmin_v = carried->kmin;
    }

    // Light frames: wavefronts [0, light_stay_waves) take the entries that stay; behind them sit
    // light_blocks blocks of 1 << light_lg extensions, one block per non-blank survivor and round.
    int links_are = kLinksBuilt;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid / kWave);
    const bool windowed = a.beam_window > 0.0;
    // number of the light frame (above what else stands where the notes are)
    uint32_t light_tag = kReach ? 1u << 24 : 0u;
    int light_lg = 0, light_stay_waves = 1, light_blocks = 0;
    const float light_reach = (float)lm_reach + 0.02f;
    float light_spread = 0.0f, light_scale = 0.0f;  // (not kReach, whose last wavefront keeps them)
    int light_from = 0, light_misses = 0;  // frame from which on headers are believed; how many in turn did not hold
    const double light_slack = lm_ub + 1.0986122886681098 + 1e-3;
    // whether tokens that cannot reach the beam may be left out: the statistics ask for the number of their
    // pairs with mass, which follows from the tokens unless pairs of the table have none
    const bool light_leaves_out = LM == kLmNone || a.stats == nullptr || !lm_gaps;
    // what the bins cover beyond the spread of the beam: how far the cut may fall in one frame (a table
    // spreads the scores); grows where that was not enough
    float light_margin = (float)light_slack + (has_lm ? 8.0f : 0.5f);
    if constexpr (kLight) {
        const LightShape shape = light_shape(beam, kThreads);
        light_lg = shape.lg;
        light_stay_waves = shape.stay_waves;
        light_blocks = shape.blocks;
    }
    // place of an entry's parent in the beam (-1: not there)
    auto parent_place = [&](int j, uint64_t want, int32_t depth) -> int {
        const int32_t code = links_of(gen).par[j];
        if (links_are != kLinksCoded) return code;
        if (code >= 0) return newslot[code];
        if (depth == 0 ||
            ((Tables::of(links_of(gen ^ 1))[Tables::fresh_word(want)] >> ((uint32_t)want & 31u)) & 1u) == 0)
            return -1;
        int p = -1;
        for (int v = 0; v < n_live; ++v)
            if (slab_of(gen).h[v] == want) p = v;
        return p;
    };
    // both generations' tables: empty ones for light frames, empty hash tables for the general path
    auto fill_tables = [&](int v) {
        constexpr int kHalf = kHashSlots / 4;  // 16 bytes each
        static_assert(!kLight || 2 * kHalf <= kThreads, "one store of a thread");
        if (2 * kHalf == kThreads || tid < 2 * kHalf)
            reinterpret_cast<int4*>(links_of(tid / kHalf).ht)[tid % kHalf] = make_int4(v, v, v, v);
    };
    // parent places and children lists from what a light frame left
    auto build_links = [&](Links<MB>* lk) {
        if (tid < n_live) {
            const ColdRef<MB> c{&slab_of(gen), nullptr};
            const int p = parent_place(tid, c.hp(tid), c.plen(tid));
            lk->par[tid] = p;
            if (p >= 0) {
                const int32_t tok = slab_of(gen).last[tid];
                if (kEntryMajor) kidset_insert(kidset2[gen], kKidSlots, p, tok);
                else lk->next_kid[tid] = atomicExch(&lk->first_kid[p], tid);
                atomicOr(&lk->kidmask[p], 1u << (tok & 31));
            }
        }
        links_are = kLinksBuilt;
    };

    // Statistics of this utterance live in LDS, not in 64-bit registers that every thread would
    // carry through the whole kernel.  What the frames of one chunk add up to is wave-uniform
    // and collects in 32-bit counters (scalar registers); once per chunk the last thread of the
    // workgroup (its wavefront has the least to do) moves them into LDS.
    enum : int { kStSurv, kStCand, kStPeak, kStBeam, kStPass, kStExact, kStDrop, kStRecords };
    const bool stat_thread = tid == kThreads - 1;
    uint32_t pd_cand = 0, pd_peak = 0, pd_beam = 0, pd_pass = 0, pd_exact = 0, pd_drop = 0;
    auto flush_stats = [&]() {
        if (stat_thread) {
            atomicAdd(&sh_stat[kStCand], (unsigned long long)pd_cand);
            atomicMax(&sh_stat[kStPeak], (unsigned long long)pd_peak);
            atomicAdd(&sh_stat[kStBeam], (unsigned long long)pd_beam);
            atomicAdd(&sh_stat[kStPass], (unsigned long long)pd_pass);
            if (pd_exact) atomicAdd(&sh_stat[kStExact], (unsigned long long)pd_exact);
            if (pd_drop) atomicAdd(&sh_stat[kStDrop], (unsigned long long)pd_drop);
        }
        pd_cand = pd_peak = pd_beam = pd_pass = pd_exact = pd_drop = 0;
    };
#ifdef FLTOP_PHASE_CLOCKS
    constexpr int kWavesPerGroup = kThreads / kWave >= 4 ? kThreads / kWave / 4 : 1;
    const int ph_grp = (tid / kWave) / kWavesPerGroup;
    const bool ph_rec = lane == 0 && (tid / kWave) % kWavesPerGroup == 0;
    uint64_t ph_clk[16] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    uint64_t ph_last = clock64();
#endif

    int32_t touched = 0;
    const int n_chunks = (len + kChunk - 1) / kChunk;
    for (int c = 0; c < n_chunks; ++c) {
    // ---- chunk boundary: headers of frames [32c, 32c+32) into LDS, next chunk requested --
    lds_barrier();  // nobody still reads the previous chunk's headers
    if constexpr (!kReach) {
        // These builds ask for the frames' top emissions only, and find them where the best other than the blank stood
        // (worked out in each frame: 256 utterances of up to 1500 frames, V = 32, beam 100, 1503 us against 1484).  The
        // first survivor is in the next lane.
        const Survivor first{dpp_or_zero<0x55, 0xf>((int)staged.x), __int_as_float(dpp_or_zero<0x55, 0xf>((int)staged.y))};
        if ((tid & 3) == 0) staged.z = (uint32_t)__float_as_int(frame_top(__int_as_float((int)staged.z), first));
    }
    if (tid < 4 * kChunk) reinterpret_cast<uint4*>(&ring[0])[tid] = staged;
    if constexpr (kReach) {  // (their entries are marked with the frame's number in its chunk)
        if (a.light_off != 0)
            for (int i = tid; i < light_table_words; i += kThreads) light_tokens[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    lds_barrier();
    FLTOP_LOAD_CHUNK(staged, c + 1);
    const int t_end = min(len, (c + 1) * kChunk);

    // ---- classify the chunk's frames (lane l looks at frame 32c + l): blank-only frames
    //      change no prefix and no order, and a run of them costs a few additions ----------
    uint32_t blank_only;  // bit l: blank is the only survivor of frame 32c + l
    int lp_bits;          // lane l: that frame's blank log-prob (fp32 bits), -inf if it was pruned
    uint64_t light_mask = 0;  // bit l: frame 32c + l is a light one ...
    uint32_t h_desc = 0;      // ... lane l: its survivors (13 bits), whether tokens may be left out (bit 14),
                              // blank-only frames behind it (from bit 16)
    int h_top = 0;            // lane l (fp32 bits): its largest log-prob,
    int h_run = 0;            // no less than the sum of the blank-only frames' behind it (and 2e-3 more at most),
    int h_alone = 0;          // the spread of the beam below which no token reaches it,
    int h_grow = 0;           // how far the best total then rises at most, and with those frames
    int h_grow_run = 0;
    uint32_t h_rec = 0;       // and where its records start
    {
        const int fl = c * kChunk + (lane & (kChunk - 1));
        const HdrHead hh = FLTOP_RING_HEAD(fl);
        const bool inside = lane < kChunk && fl < len;
        const bool lone_blank =
            inside && hh.count == 1 && hh.s0.tok == 0 && hh.s0.lp > -INFINITY;
        blank_only = (uint32_t)__ballot(lone_blank);
        lp_bits = __float_as_int(hh.s0.tok == 0 ? hh.s0.lp : -INFINITY);
        if constexpr (kLight && !kReach) {
            const int with_blank = hh.s0.tok == 0 ? 1 : 0;
            const int others = hh.count - with_blank;
            const int run_behind =
                lane + 1 < kChunk ? __builtin_ctz(~(blank_only >> (lane + 1)) | 0x80000000u) : 0;
            const int rounds = light_rounds(light_blocks, others);
            // non-blank survivors (3 bits), whether blank survived (bit 3), extensions per thread (3 bits),
            // blank-only frames behind it (from bit 8)
            h_desc = (uint32_t)(others & 7) | (uint32_t)(with_blank << 3) | (uint32_t)(rounds << 4) |
                     (uint32_t)(run_behind << 8);
            const float frame_best = hh.best;
            h_top = __float_as_int(frame_best);
            const float upto = row32_inclusive_sum(lone_blank ? hh.s0.lp : 0.0f);
            h_run = __float_as_int(
                __int_as_float(__builtin_amdgcn_ds_bpermute((lane + run_behind) << 2, __float_as_int(upto))) - upto);
            light_mask = __ballot(inside && hh.count <= kRegK && others >= 1 && rounds <= kLightRounds &&
                                  fabsf(frame_best) < INFINITY);
            // the sums' rounding has to stay below the 1e-3 that `light_slack` adds (and an overflow of
            // masked rows' log-probs must not get into the bounds): 5 additions of less than 2048 each
            if (__ballot(!(fabsf(upto) < 1024.0f)) != 0) light_mask = 0;
        }
        if constexpr (kReach) {
            const int with_blank = hh.s0.tok == 0 ? 1 : 0;
            const int others = hh.count - with_blank;
            const int run_behind =
                lane + 1 < kChunk ? __builtin_ctz(~(blank_only >> (lane + 1)) | 0x80000000u) : 0;
            const float lpb = with_blank ? hh.s0.lp : -INFINITY;
            const float frame_best = fmaxf(hh.best, lpb);
            // Every entry stays with at least its total and the blank's log-prob.  The margin of 0.02 is far
            // above what fp32 loses below 1e4.
            const bool tame = light_leaves_out && fabsf(frame_best) < 1e4f;
            // (a frame that is none has no survivors here: they are asked for before its turn comes, and its records
            // may not be there)
            const bool light = inside && a.light_off != 0 && others >= 1 && hh.count <= kWave &&
                               (hh.count <= kRegK || hh.rec_base != kNoRecords) && fabsf(frame_best) < INFINITY;
            h_desc = (uint32_t)(light ? hh.count : 0) | (uint32_t)(tame ? 1 << 14 : 0) |
                     (uint32_t)(run_behind << 16);
            h_top = __float_as_int(frame_best);
            h_rec = hh.rec_base;
            const float gap = tame && lpb > -INFINITY ? lpb - hh.best - light_reach : -INFINITY;
            h_alone = __float_as_int(windowed ? fminf(gap, (float)a.beam_window * 0.9999f - 2.1f) : gap);
            // (an entry's own repeat, and its parent's extension)
            const float merges = (1.0f + __expf(light_reach)) * __expf(hh.best - lpb) * 1.0001f + 1e-3f;
            h_grow = __float_as_int(merges);
            const float upto = row32_inclusive_sum(lone_blank ? hh.s0.lp : 0.0f);
            const float run_sum =
                __int_as_float(__builtin_amdgcn_ds_bpermute((lane + run_behind) << 2, __float_as_int(upto))) - upto + 1e-3f;
            h_run = __float_as_int(run_sum);
            h_grow_run = __float_as_int(lpb + merges + run_sum);
            light_mask = __ballot(light);
            // the sums' rounding has to stay below the 1e-3 that `light_slack` adds (and an overflow of
            // masked rows' log-probs must not get into the bounds): 5 additions of less than 2048 each
            if (__ballot(!(fabsf(upto) < 1024.0f)) != 0) light_mask = 0;
        }
        const int chunk_survivors = __builtin_amdgcn_readlane(
            wave_inclusive_scan(inside ? hh.count : 0), kWave - 1);
        // records the chunk's frames take beyond the survivors in their headers
        const int chunk_records = __builtin_amdgcn_readlane(
            wave_inclusive_scan(inside ? max(0, hh.count - kRegK) : 0), kWave - 1);
        flush_stats();  // of the previous chunk (at most 32 frames: the counters cannot wrap)
        if (stat_thread) {
            atomicAdd(&sh_stat[kStSurv], (unsigned long long)chunk_survivors);
            if (chunk_records) atomicAdd(&sh_stat[kStRecords], (unsigned long long)chunk_records);
        }
        if constexpr (kReach) {
            // the lines of the frames' records are asked for ahead of time (light frames last less than a read from
            // memory takes; what comes is not used, and waited for in the next chunk)
            const int part = (tid / kChunk) * 16;  // 128 bytes
            asm volatile("" ::"v"(touched));
            if (light_mask != 0 && hh.count <= kWave && hh.count - kRegK > part && hh.rec_base != kNoRecords)
                touched = *reinterpret_cast<const volatile int32_t*>(&rec_all[(int64_t)hh.rec_base + part]);
        }
        // after a frame whose records did not fit the workspace the utterance is not decoded
        // any further, but its survivors are still counted: the caller learns what to ask for
        if (failed) continue;
    }

    for (int t = c * kChunk; t < t_end; ++t) {
        const int l = t & (kChunk - 1);
        if (FLTOP_RARE(n_live == 0)) {  // the beam died: nothing left to decode
            if (a.frame_beam && tid < t_end - t) a.frame_beam[trace_base + t + tid] = 0;
            t = t_end;  // (the loop keeps its single exit: leaving it from several places costs
            continue;   // every frame a dispatch on the way round)
        }
        // ---- run of blank-only frames --------------------------------------------------
        const int run = __builtin_ctz(~(blank_only >> l) | 0x80000000u);
        if (FLTOP_RARE(run > 0)) {
            // every entry's total takes the run's log-probs one by one, in frame order, as a
            // plain implementation adds them (the owner thread keeps the sum in a register)
            BeamSlab<MB>* const cur_run = &slab_of(gen);
            double own = tid < n_live ? cur_run->ptot[tid] : 0.0;
            for (int k = 0; k < run; ++k) {
                const double x = (double)__int_as_float(__builtin_amdgcn_readlane(lp_bits, l + k));
                own += x;
                kmax_v += x;
                kmin_v += x;
            }
            if (tid < n_live) cur_run->ptot[tid] = own;
            collapsed = true;
            lds_barrier();  // the new totals are read by other threads in the next full frame
            pd_cand += (uint32_t)(n_live * run);
            pd_peak = max(pd_peak, (uint32_t)n_live);
            pd_beam += (uint32_t)(n_live * run);
            if (a.frame_beam && tid < run) a.frame_beam[trace_base + t + tid] = n_live;
            t += run - 1;
            PHASE_MARK(7);
            continue;
        }
        if constexpr (kLight) {
            if constexpr (kReach) {
                if (((light_mask >> l) & 1ull) && t >= light_from) {
#include "fltop_beam_reach.inc"
                }
            } else {
                if ((light_mask >> l) & 1ull) {
                    if (links_are == kLinksBuilt) {
                        // the general path came before: its lists go; no parent is among fresh prefixes
                        if (tid < kMaxBeam) {
                            links_of(gen).first_kid[tid] = -1;
                            links_of(gen).kidmask[tid] = 0u;
                            newslot[tid] = tid;
                        }
                        fill_tables(0);
                        links_are = kLinksCoded;
                        light_spread = light_spread_of((float)(kmax_v - kmin_v) + 1.0f);
                        light_scale = (float)kLightBins * __builtin_amdgcn_rcpf(light_spread + light_margin);
                        lds_barrier();
                    }
#include "fltop_beam_light.inc"
                }
            }
            if (links_are != kLinksBuilt) {  // the general path looks children up from their parents
                build_links(&links_of(gen));
                lds_barrier();
                fill_tables(-1);  // its hash tables again (a barrier follows before anything enters them)
            }
        }
        // (local to the frame: as long as light frames run, none of it takes up a register)
        FrameCtx<MB> fc;
        fc.dense_lp = dense_lp;
        fc.s_tok = s_tok;
        fc.s_lp = s_lp;
        fc.lm_lds = (LdsFloatPtr)lm_s;
        fc.lm_glb = a.lm_table;
        fc.lm_alpha = a.lm_alpha;
        fc.lm_beta = a.lm_beta;
        fc.V = V;
        const FrameHdr hd = ring[t % kChunk];  // all 64 bytes in one round trip
        const int K = hd.count;
        const float top = kReach ? frame_top(hd.best, hd.first[0]) : hd.best;

        BeamSlab<MB>* const cur = &slab_of(gen);
        BeamSlab<MB>* const nxt = &slab_of(gen ^ 1);
        Links<MB>* const lk = &links_of(gen);
        Links<MB>* const lkn = &links_of(gen ^ 1);
        const ColdRef<MB> ccur{cur, kColdGlobal ? cold_gen + gen : nullptr};
        const ColdRef<MB> cnxt{nxt, kColdGlobal ? cold_gen + (gen ^ 1) : nullptr};

        // ---- survivors: registers for K <= 6, LDS staging beyond ------------------------
        const bool big = K > kRegK;
        fc.cur = cur;
        fc.lk = lk;
        fc.big = big;
        fc.collapsed = collapsed;
        // unused places of the inline list hold (-1, -inf), so they can be taken as they are
        fc.t0 = hd.first[0].tok;
        fc.l0 = hd.first[0].lp;
        fc.t1 = hd.first[1].tok;
        fc.l1 = hd.first[1].lp;
        fc.t2 = hd.first[2].tok;
        fc.l2 = hd.first[2].lp;
        fc.t3 = hd.first[3].tok;
        fc.l3 = hd.first[3].lp;
        fc.t4 = hd.first[4].tok;
        fc.l4 = hd.first[4].lp;
        fc.t5 = hd.first[5].tok;
        fc.l5 = hd.first[5].lp;
        if (tid == 0) {
            sh_nnew = 0;
            sh_blcount = 0;
        }
        if (tid >= kThreads / 2 && tid - kThreads / 2 < kMaxBeam / 4)
            reinterpret_cast<int4*>(newslot)[tid - kThreads / 2] = make_int4(-1, -1, -1, -1);
        if (big && hd.rec_base == kNoRecords) {  // uniform: the record array was too small
            failed = true;
            t = t_end;
            continue;
        }
        // survivors ascend by token: the blank, if kept, is the first
        const int nb0 = hd.first[0].tok == 0 ? 1 : 0;
        // Frames with thousands of candidates: nearly all of them lie far below the beam's cut.
        // With the beam full, every entry i stands for one candidate of its own, the better of
        // "i stays" and "i extended by the frame's top token": that is `beam` different
        // candidates, so whatever scores below the worst of these cannot be kept.  One barrier
        // makes that floor known before the extensions are looked at; those below it are only
        // counted, four at a time, and never reach the histogram or the probe of the pair table
        // (in the distance cache they are marked as gone).  (128 utterances, V = 1024, every token
        // kept, beam 64: 38.1 ms per decode without the floor, 11.3 ms with it.  A floor from a
        // histogram of the same few candidates, whose resolution is a bin: 17.0 ms.)
        const bool floored_frame =  // uniform
            FLOOR && big && n_live == beam && K - nb0 > floored_above;
        if (big) {
            const Survivor* recs = rec_all + ((int64_t)hd.rec_base - kRegK);
            const FrameHdr* full = &ring[t % kChunk];
            for (int k = tid; k < K; k += kThreads) {
                const Survivor s = (k < kRegK) ? full->first[k] : recs[k];
                s_tok[k] = (uint16_t)s.tok;
                if (kEntryMajor) {
                    s_lp[k] = s.lp;
                    if (floored_frame && s.lp == top && s.tok != 0) atomicMin(&sh_toptok, s.tok);
                }
                dense_lp[s.tok] = s.lp;
            }
        }
        if (big) lds_barrier();

        PHASE_MARK(0);
        fc.nb0 = nb0;
        fc.Knb = K - fc.nb0;
        fc.div_magic = hd.div_magic;
        const double lp_blank = fc.nb0 ? (double)hd.first[0].lp : -INFINITY;
        // Extension candidate e = i * Knb + k is entry i extended by non-blank survivor k.
        // Thread numbers are taken from the upper half of the wavefronts first (the lower
        // half has the stays).  Plain builds: a thread takes e = e_first, e_first + kThreads, ...
        // Entry-major builds: entry i is shared by G = kThreads / n_live threads, of which
        // number g takes k = g, g + G, g + 2G, ...
        const int n_ext = n_live * fc.Knb;
        const int e_first = (tid + kThreads / 2) & (kThreads - 1);
        if (kEntryMajor && n_live != mapped_for) {  // uniform; the beam is full most of the time
            ext_g = e_first / n_live;
            ext_i = e_first - ext_g * n_live;
            ext_G = kThreads / n_live;
            mapped_for = n_live;
        }
        const int G = ext_G;
        const bool ext_thread = ext_g < G && ext_g < fc.Knb;  // kEntryMajor only
        const int M = kEntryMajor ? (fc.Knb + G - 1) / G  // most candidates any thread has
                                  : (n_ext + kThreads - 1) / kThreads;
        uint64_t selD = kAllOnes;  // with selH: keep D < selD or (D == selD and hash <= selH)
        uint64_t kbest_key = 0;    // upper bound of the best candidate's key
        // upper bound of every candidate score -> reference key
        const double ref = kmax_v + (double)top + lm_ub + 1.0986122886681098 + 1e-3;
        fc.Rk = order_key(ref);
        const uint64_t Rk = fc.Rk;
        if constexpr (FLOOR) {
            if (floored_frame) {
                constexpr bool floored = true;
#include "fltop_beam_frame.inc"
            } else {
                constexpr bool floored = false;
#include "fltop_beam_frame.inc"
            }
        } else {
            constexpr bool floored = false;
#include "fltop_beam_frame.inc"
        }
        // the links phase reads what other threads have just emitted: LDS always, and in
        // kColdGlobal builds their stores to global memory too
        if (kColdGlobal) __syncthreads();
        else lds_barrier();
        PHASE_MARK(5);

        // ---- adopt the new beam; rebuild parent / children links ---------------------
        int n_new = __builtin_amdgcn_readfirstlane(sh_nnew);  // the same in every lane
        if (FLTOP_RARE(n_new > beam)) {
            pd_drop += (uint32_t)(n_new - beam);
            n_new = beam;
        }
        pd_beam += (uint32_t)n_new;
        // A run of blank-only frames that follows inside this chunk is taken here: the thread
        // that owns a place of the new beam adds the run's log-probs to its total, one by one in
        // frame order, behind the barrier this frame ends on anyway.  (A run at the start of a
        // chunk or of the utterance takes the path at the top of the loop.)
        int run_after = 0;
        if (l + 1 < kChunk && n_new > 0)
            run_after = __builtin_ctz(~(blank_only >> (l + 1)) | 0x80000000u);
        double own_total = 0.0;  // of the entry this thread owns in the new beam (for the run)
        if (tid < n_new) {
            int p = -1;
            if constexpr (!kColdGlobal) {
                // Two LDS round trips: everything the entry's own fields can say, asked for
                // together; then ONE lookup, in the table of moves if the parent was in the old
                // beam (did it stay, and where), else in the hash table of the new prefixes
                // (a parent that was not in the beam can only have entered it just now).
                const int32_t code = lkn->par[tid];
                const int32_t depth = cnxt.plen(tid);
                const uint64_t want = cnxt.hp(tid);
                const int32_t tok_me = nxt->last[tid];
                own_total = nxt->ptot[tid];
                uint32_t hs = (uint32_t)want & (kHashSlots - 1);
                const int32_t* where = code >= 0 ? &newslot[code] : &lkn->ht[hs];
                int v = *where;
                if (code >= 0) {
                    p = v;
                } else if (depth > 0 && v >= 0) {  // rare: walk on until found or free
                    for (int probe = 0; probe < kHashSlots; ++probe) {
                        if (nxt->h[v] == want) {
                            p = v;
                            break;
                        }
                        hs = (hs + 1) & (kHashSlots - 1);
                        v = lkn->ht[hs];
                        if (v < 0) break;
                    }
                }
                lkn->par[tid] = p;
                if (p >= 0) {
                    if (kEntryMajor)
                        kidset_insert(kidset2[gen ^ 1], kKidSlots, p, tok_me);
                    else
                        lkn->next_kid[tid] = atomicExch(&lkn->first_kid[p], tid);
                    atomicOr(&lkn->kidmask[p], 1u << (tok_me & 31));
                }
            } else {
                const int32_t code = lkn->par[tid];
                if (code >= 0) {
                    p = newslot[code];  // the parent was in the old beam: did it stay, and where
                } else if (cnxt.plen(tid) > 0) {
                    const uint64_t want = cnxt.hp(tid);
                    uint32_t hs = (uint32_t)want & (kHashSlots - 1);
                    int v = lkn->ht[hs];
                    if (v >= 0) {  // rare: something hashes to this place; walk on until found or free
                        for (int probe = 0; probe < kHashSlots; ++probe) {
                            if (nxt->h[v] == want) {
                                p = v;
                                break;
                            }
                            hs = (hs + 1) & (kHashSlots - 1);
                            v = lkn->ht[hs];
                            if (v < 0) break;
                        }
                    }
                }
                lkn->par[tid] = p;
                if (p >= 0) {
                    if (kEntryMajor)
                        kidset_insert(kidset2[gen ^ 1], kKidSlots, p, nxt->last[tid]);
                    else
                        lkn->next_kid[tid] = atomicExch(&lkn->first_kid[p], tid);
                    atomicOr(&lkn->kidmask[p], 1u << (nxt->last[tid] & 31));
                }
            }
        }
        PHASE_MARK(10);
        // housekeeping behind this frame's last readers: the old generation's links
        // (next used as the new generation of the following frame) and the histogram.
        // The upper half of the threads does it: the lower half has just done the links.
        if (tid >= kThreads / 2) {
            // 16 bytes per store
            const int u = tid - kThreads / 2;
            const int4 ones = make_int4(-1, -1, -1, -1), zeros = make_int4(0, 0, 0, 0);
            // (trip counts known at compile time: straight-line stores, no loops)
            constexpr int kHalf = kThreads / 2;
            auto fill = [&](int4* dst, auto n_tag, const int4& v) {
                constexpr int n = decltype(n_tag)::value;  // 16-byte words to fill
#pragma unroll
                for (int j = 0; j < n / kHalf; ++j) dst[u + j * kHalf] = v;
                if (n % kHalf != 0 && u < n % kHalf) dst[u + (n / kHalf) * kHalf] = v;
            };
            fill(reinterpret_cast<int4*>(lk->ht), std::integral_constant<int, kHashSlots / 4>{}, ones);
            if (kEntryMajor)
                fill(reinterpret_cast<int4*>(kidset2[gen]), std::integral_constant<int, kKidSlots / 4>{},
                     ones);
            if (!kColdGlobal)
                fill(reinterpret_cast<int4*>(lk->first_kid), std::integral_constant<int, kMaxBeam / 4>{},
                     ones);
            fill(reinterpret_cast<int4*>(lk->kidmask), std::integral_constant<int, kMaxBeam / 4>{}, zeros);
            fill(reinterpret_cast<int4*>(hfine), std::integral_constant<int, kFine / 4>{}, zeros);
            if (u < kCoarse / 4) reinterpret_cast<int4*>(hcoarse)[u] = zeros;
        }
        if (tid == 0) {
            sh_minD = kAllOnes;
            if (floored_frame) {
                sh_floor = kAllOnes;
                sh_toptok = INT32_MAX;
                sh_below = 0;
                sh_nlist = 0;
                sh_nout = 0;
            }
            if (a.frame_beam) a.frame_beam[trace_base + t] = n_new;
        }
        if (big)
            for (int k = tid; k < K; k += kThreads) dense_lp[s_tok[k]] = -INFINITY;
        if (n_new > 0) {
            kmax_v = key_value(kbest_key);
            // worst kept score: the selection threshold when there was one
            const bool cut = selD != kAllOnes && selD <= Rk;
            if constexpr (kReach) kmin_sure = cut;
            kmin_v = cut ? key_value(Rk - selD) : kmin_v + (double)top - 4.0;
            if (!(kmin_v <= kmax_v)) kmin_v = kmax_v;
        }
        n_live = n_new;
        gen ^= 1;
        collapsed = run_after > 0;  // otherwise every entry carries its own p_b / p_nb
        if (run_after > 0) {
            double own = own_total;
            if (kColdGlobal && tid < n_new) own = nxt->ptot[tid];
            for (int k = 0; k < run_after; ++k) {
                const double x = (double)__int_as_float(__builtin_amdgcn_readlane(lp_bits, l + 1 + k));
                own += x;
                kmax_v += x;
                kmin_v += x;
            }
            if (tid < n_new) nxt->ptot[tid] = own;
            pd_cand += (uint32_t)(n_new * run_after);
            pd_peak = max(pd_peak, (uint32_t)n_new);
            pd_beam += (uint32_t)(n_new * run_after);
            if (a.frame_beam && tid < run_after) a.frame_beam[trace_base + t + 1 + tid] = n_new;
            t += run_after;
        }
        lds_barrier();
        PHASE_MARK(6);
    }  // frames of the chunk
    }  // chunks
#undef FLTOP_RARE
#undef FLTOP_USUAL
#undef FLTOP_LOAD_CHUNK
#undef FLTOP_RING_HEAD

    flush_stats();
    if (failed) n_live = 0;  // nothing to report, and a stream that carries on finds no beam
    // every trie store must have landed before the back-walk reads the nodes
    __threadfence_block();
    __syncthreads();

    // ---- best prefix (paper: GetHighestScorePrefix) ----------------------------------
    BeamSlab<MB>& fin = slab_of(gen);
    const ColdRef<MB> cfin{&slab_of(gen), kColdGlobal ? cold_gen + gen : nullptr};
    int32_t* wp_node = reinterpret_cast<int32_t*>(hfine);  // the histogram is idle now
    int32_t* wp_depth = wp_node + kWaypoints;
    static_assert(2 * kWaypoints <= kFine, "way-points alias the histogram");
    if (tid == 0) {
        sh_kbest = 0;
        sh_selH = kAllOnes;
        sh_best = -1;
    }
    __syncthreads();
    if (tid < n_live)
        atomicMax((unsigned long long*)&sh_kbest, (unsigned long long)order_key(fin.ptot[tid]));
    __syncthreads();
    if (tid < n_live && order_key(fin.ptot[tid]) == sh_kbest)
        atomicMin((unsigned long long*)&sh_selH, (unsigned long long)fin.h[tid]);
    __syncthreads();
    if (tid < n_live && order_key(fin.ptot[tid]) == sh_kbest && fin.h[tid] == sh_selH)
        sh_best = tid;
    __syncthreads();

    const int best = sh_best;
    if (tid == 0) {
        if (failed) {  // said loudly: no transcript, not an empty one
            a.out_lengths[b] = -1;
            a.out_scores[b] = __int_as_float(0x7fc00000);  // NaN
        } else if (best < 0) {
            a.out_lengths[b] = 0;
            a.out_scores[b] = -INFINITY;
        } else {
            a.out_lengths[b] = cfin.plen(best);
            a.out_scores[b] = (float)fin.ptot[best];
        }
        if (a.stats) {
            atomicAdd((unsigned long long*)&a.stats->frames, (unsigned long long)len);
            atomicAdd((unsigned long long*)&a.stats->sum_survivors, sh_stat[kStSurv]);
            atomicAdd((unsigned long long*)&a.stats->sum_candidates, sh_stat[kStCand]);
            atomicMax((unsigned long long*)&a.stats->peak_candidates, sh_stat[kStPeak]);
            atomicAdd((unsigned long long*)&a.stats->sum_beam, sh_stat[kStBeam]);
            atomicAdd((unsigned long long*)&a.stats->select_passes, sh_stat[kStPass]);
            atomicAdd((unsigned long long*)&a.stats->exact_rankings, sh_stat[kStExact]);
            atomicAdd((unsigned long long*)&a.stats->overflow_drops, sh_stat[kStDrop]);
            if (failed) atomicAdd((unsigned long long*)&a.stats->record_overflows, 1ull);
            atomicAdd((unsigned long long*)&a.stats->survivor_records, sh_stat[kStRecords]);
        }
    }
#ifdef FLTOP_PHASE_CLOCKS
    if (ph_rec && a.stats)
        for (int i = 0; i < 16; ++i)
            atomicAdd((unsigned long long*)&a.stats->phase_clocks[ph_grp * 16 + i],
                      (unsigned long long)ph_clk[i]);
#endif
    // Back-walk: thread 0 follows the every-8th-level links and records way-points; then
    // one thread per way-point walks the (at most 8) parents down to the next way-point.
    // A streaming decode remembers the trie node behind every token it wrote: where the walk
    // meets the node that is already written at that position, everything before it is in
    // place (a node's ancestors never change), so a call rewrites only what has changed.
    int32_t* const out_row = a.out_tokens + (int64_t)b * a.out_stride;
    int32_t* const born_row =
        a.out_token_frames ? a.out_token_frames + (int64_t)b * a.out_stride : nullptr;
    int32_t* const wrote = a.out_nodes ? a.out_nodes + (int64_t)b * a.out_stride : nullptr;
    const bool same_rows = wrote && prev_tokens_at == (uint64_t)(uintptr_t)out_row &&
                           prev_frames_at == (uint64_t)(uintptr_t)born_row;
    const int new_out_len = best >= 0 ? cfin.plen(best) : 0;
    if (best >= 0) {
        int node = cfin.node(best);
        int depth = new_out_len;
        while (depth > 0) {  // uniform: node/depth are re-read from LDS after each batch
            if (tid == 0) {
                int n = 0;
                int nd = node, dp = depth;
                bool met = false;
                while (dp > 0 && n < kWalkers - 1 && nd > 0 && (int64_t)nd < a.trie_stride) {
                    if (same_rows && wrote[dp - 1] == nd) {
                        met = true;
                        break;
                    }
                    wp_node[n] = nd;
                    wp_depth[n] = dp;
                    ++n;
                    const TrieNode tn = trie[nd];
                    nd = tn.xup;
                    dp = (dp - 1) & ~7;
                }
                const bool ok = !met && nd > 0 && (int64_t)nd < a.trie_stride;
                wp_node[n] = nd;             // where the next batch starts ...
                wp_depth[n] = met ? dp : (ok ? dp : 0);  // ... and the last walker stops
                sh_blcount = ok ? dp : 0;    // depth left for the next batch
                sh_nnew = n;
            }
            __syncthreads();
            const int n = sh_nnew;
            if (tid < n) {
                int nd = wp_node[tid];
                int dp = wp_depth[tid];
                const int stop = wp_depth[tid + 1];
                while (dp > stop && nd > 0 && (int64_t)nd < a.trie_stride) {
                    if (same_rows && wrote[dp - 1] == nd) break;
                    const TrieNode tn = trie[nd];
                    out_row[dp - 1] = tn.tok;
                    if (born_row) born_row[dp - 1] = (nd - 1) / beam;  // node id = 1 + frame * beam + slot
                    if (wrote) wrote[dp - 1] = nd;
                    nd = tn.parent;
                    --dp;
                }
            }
            node = wp_node[n];
            depth = sh_blcount;
            __syncthreads();
        }
    }
    if (wrote)  // positions the shorter transcript no longer covers
        for (int q = new_out_len + tid; q < prev_out_len; q += kThreads) wrote[q] = -1;

    // ---- optional: the whole final beam in rank order ---------------------------------
    if (a.nbest_count) {
        if (tid == 0) a.nbest_count[b] = n_live;
        if (tid < n_live) {
            const uint64_t myK = order_key(fin.ptot[tid]);
            const uint64_t myH = fin.h[tid];
            int rank = 0;
            for (int e = 0; e < n_live; ++e) {
                const uint64_t oK = order_key(fin.ptot[e]);
                const uint64_t oH = fin.h[e];
                rank += (oK > myK || (oK == myK && oH < myH)) ? 1 : 0;
            }
            const int64_t row = (int64_t)b * beam + rank;
            const int n = cfin.plen(tid);
            a.nbest_lengths[row] = n;
            a.nbest_pb[row] = collapsed ? fin.ptot[tid] : fin.pb[tid];
            a.nbest_pnb[row] = collapsed ? -INFINITY : fin.pnb[tid];
            int node = cfin.node(tid);
            int32_t* dst = a.nbest_tokens + row * a.out_stride;
            for (int p = n - 1; p >= 0 && node > 0 && (int64_t)node < a.trie_stride; --p) {
                const TrieNode tn = trie[node];
                dst[p] = tn.tok;
                node = tn.parent;
            }
        }
    }

    // ---- streaming: leave the beam for the next chunk -----------------------------------
    if (carried) {
        if constexpr (kLight) {
            if (links_are != kLinksBuilt) {
                __syncthreads();
                build_links(&links_of(gen));
                __syncthreads();
            }
        }
        const uint32_t* src = reinterpret_cast<const uint32_t*>(&slab_of(gen));
        uint32_t* dst = reinterpret_cast<uint32_t*>(&carried->slab);
        for (int i = tid; i < (int)(sizeof(BeamSlab<MB>) / 4); i += kThreads) dst[i] = src[i];
        const uint32_t* lsrc = reinterpret_cast<const uint32_t*>(&links_of(gen));
        uint32_t* ldst = reinterpret_cast<uint32_t*>(carried->par);
        for (int i = tid; i < 4 * kMaxBeam; i += kThreads) ldst[i] = lsrc[i];
        if (tid == 0) {
            carried->frames_done = t_base + len;
            carried->out_len = new_out_len;
            carried->out_tokens_at = (uint64_t)(uintptr_t)out_row;
            carried->out_frames_at = (uint64_t)(uintptr_t)born_row;
            carried->n_live = n_live;
            carried->collapsed = (collapsed ? 1 : 0) | (kmin_sure ? 2 : 0);
            carried->kmax = kmax_v;
            carried->kmin = kmin_v;
        }
    }
}

// A fresh stream: the empty prefix with score 0, no links, no frames seen.
template <int MB>
__global__ __launch_bounds__(kThreadsSmall) void stream_begin_kernel(StreamState<MB>* st, int32_t B,
                                                                     int32_t* out_nodes,
                                                                     int64_t n_out_nodes) {
    constexpr int kThreads = kThreadsSmall;
    constexpr int kMaxBeam = MB;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n_out_nodes;
         i += (int64_t)gridDim.x * kThreads)
        out_nodes[i] = -1;
    for (int32_t b = blockIdx.x; b < B; b += gridDim.x) {
        StreamState<MB>* s = st + b;
        uint32_t* words = reinterpret_cast<uint32_t*>(s);
        for (int i = threadIdx.x; i < (int)(sizeof(StreamState<MB>) / 4); i += kThreads) words[i] = 0u;
        __syncthreads();
        for (int i = threadIdx.x; i < kMaxBeam; i += kThreads) {
            s->par[i] = -1;
            s->first_kid[i] = -1;
            s->next_kid[i] = -1;
        }
        if (threadIdx.x == 0) {
            s->n_live = 1;
            s->slab.h[0] = kGolden;
            s->slab.pb[0] = 0.0;
            s->slab.pnb[0] = -INFINITY;
            s->slab.ptot[0] = 0.0;
            s->slab.last[0] = -1;
        }
        __syncthreads();
    }
}

// The search stage's log-sum-exp, element-wise over two arrays (for checking its rounding): NaN where
// the forms that its builds use would not agree in every bit.
__global__ __launch_bounds__(256) void log_add_kernel(const double* __restrict__ a,
                                                      const double* __restrict__ b,
                                                      double* __restrict__ out, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double x = a[i], y = b[i], r = lse2<false>(x, y);
        out[i] = lse2_any<false>(x, y) == r && lse2<true>(x, y) == r && lse2_any<true>(x, y) == r ? r : NAN;
    }
}

}  // namespace

hipError_t launch_log_add(const double* a, const double* b, double* out, int64_t n,
                          hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(log_add_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256),
                       0, stream, a, b, out, n);
    return hipGetLastError();
}

size_t stream_record_bytes(int32_t beam) {
    return beam <= kBeamSmall ? sizeof(StreamState<kBeamSmall>) : sizeof(StreamState<kBeamLarge>);
}

hipError_t launch_stream_begin(const StreamSpace& sp, int32_t B, int32_t beam, hipStream_t stream) {
    const dim3 grid((unsigned)(B < 1024 ? B : 1024));
    const int64_t n_out_nodes = (int64_t)B * sp.t_total;
    if (beam <= kBeamSmall)
        hipLaunchKernelGGL(stream_begin_kernel<kBeamSmall>, grid, dim3(kThreadsSmall), 0, stream,
                           static_cast<StreamState<kBeamSmall>*>(sp.records), B, sp.out_nodes,
                           n_out_nodes);
    else
        hipLaunchKernelGGL(stream_begin_kernel<kBeamLarge>, grid, dim3(kThreadsSmall), 0, stream,
                           static_cast<StreamState<kBeamLarge>*>(sp.records), B, sp.out_nodes,
                           n_out_nodes);
    return hipGetLastError();
}

// Compute units of the current device (asked once per device).
static hipError_t compute_units(int* n_cu) {
    constexpr int kMaxDevices = 64;
    static int cached[kMaxDevices] = {0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < kMaxDevices && cached[dev] > 0) {
        *n_cu = cached[dev];
        return hipSuccess;
    }
    int n = 0;
    e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (n <= 0) n = 1;
    if (dev >= 0 && dev < kMaxDevices) cached[dev] = n;  // racing callers write the same value
    *n_cu = n;
    return hipSuccess;
}

// Tokens that a frame of a small vocabulary is expected to keep, above which it goes through those that can reach the
// beam only: more than fit its header.
constexpr int kNarrowReachAbove = 8;

hipError_t launch_beam(const int32_t* lengths, int32_t B, int32_t T, int32_t V,
                       const fltop_params& p, const Workspace& ws, const StreamSpace* carried,
                       int32_t* out_tokens, int32_t* out_lengths, float* out_scores,
                       fltop_stats* stats, hipStream_t stream) {
    BeamArgs a;
    a.lengths = lengths;
    a.hdr = ws.hdr;
    a.rec = ws.rec;
    a.trie = carried ? carried->trie : ws.trie;
    a.trie_stride = carried ? carried->trie_stride : ws.trie_stride;
    a.cold = ws.cold;
    a.stream = carried ? carried->records : nullptr;
    a.out_nodes = carried ? carried->out_nodes : nullptr;
    a.t_total = carried ? carried->t_total : T;
    a.out_stride = carried ? carried->t_total : T;
    a.lm_table = p.lm_table;
    a.lm_bound = ws.lm_bound;
    a.lm_alpha = (double)p.lm_weight;
    a.lm_beta = (double)p.insertion_bonus;
    a.beam_window = p.beam_threshold;
    a.frame_beam = p.frame_beam;
    a.out_token_frames = p.out_token_frames;
    a.B = B;
    a.T = T;
    a.V = V;
    a.beam = p.beam;
    a.lm_in_lds = (p.lm_table != nullptr && (size_t)V * V * sizeof(float) <= 16384) ? 1 : 0;
    a.out_tokens = out_tokens;
    a.out_lengths = out_lengths;
    a.out_scores = out_scores;
    a.stats = stats;
    a.nbest_count = p.nbest_count;
    a.nbest_tokens = p.nbest_tokens;
    a.nbest_lengths = p.nbest_lengths;
    a.nbest_pb = p.nbest_pb;
    a.nbest_pnb = p.nbest_pnb;
    // "wide" = frames are expected to hold hundreds of candidates or more: a large vocabulary,
    // or a search that is known to keep every token (R = 0) of a small one with a beam to
    // match (measured on V = 32: from 512 candidates per frame on, the 512-thread build is
    // 9-41% faster; how many tokens a threshold R > 0 keeps is not known here).  Where frames go through the
    // tokens that can reach the beam only (see below) and there are more utterances than CUs, two per CU with
    // 256 threads are faster for fewer candidates, whose blocks of extensions fit those (400 utterances x 60 frames,
    // R = 0, 512 and 256 threads: V = 16, beam 32 265 and 185 us; V = 32, beam 16 232 and 165; V = 64, beam 32 355
    // and 343; V = 32, beam 64 394 and 487; V = 64, beam 60 503 and 703; flat emissions, V = 16, beam 64 424 and
    // 277, V = 64, beam 64 835 and 936).
    const int kept_at_most = p.top_n > 0 && p.top_n < V ? p.top_n : V;
    int n_cu = 0;
    hipError_t qe = compute_units(&n_cu);
    if (qe != hipSuccess) return qe;
    const bool very_dense = (int64_t)B > (int64_t)n_cu * 2;
    const bool short_calls = carried != nullptr && T <= (V <= 64 ? 2 : (p.beam > kBeamTiny ? 8 : 3));
    const bool every_token = V <= 64 && p.rel_threshold == 0.0f;
    const bool every_reach = every_token && p.lm_table == nullptr && p.beam <= kBeamTiny && !very_dense && !short_calls;
    const bool two_per_cu = every_reach && B > n_cu && kept_at_most > kNarrowReachAbove;
    const bool wide = V > 64 || (every_token && (int64_t)p.beam * kept_at_most >= (two_per_cu ? 2048 : 512) &&
                                 (!two_per_cu || p.beam > 32));
    const bool large_beam = p.beam > kBeamSmall;
    const bool huge_beam = p.beam > kBeamLarge;  // 1024-entry build, 1024 threads, one per CU
    if (huge_beam && (carried != nullptr || V > FLTOP_MAX_VOCAB_WIDE_BEAM))
        return hipErrorInvalidValue;  // the entry points refuse these before they get here
    const bool dense = (int64_t)B > (int64_t)n_cu * (wide ? 1 : 2);
    const bool threads_512 = large_beam || (wide && !very_dense);  // as dispatched below
    size_t dyn = lm_lds_offset(V, threads_512);
    if (a.lm_in_lds) dyn += (size_t)V * V * sizeof(float);
    dyn = (dyn + 15) / 16 * 16;
    a.dcache_off = (int32_t)dyn;
    a.dcache_rows = 0;
    a.light_off = 0;
    // Workgroup size: frames of a small vocabulary have a few dozen candidates, and the cost of
    // a frame is its barriers and its longest wavefront, so four wavefronts are best; a large
    // vocabulary leaves hundreds to thousands of candidates per frame, which eight wavefronts
    // (two per SIMD) evaluate twice as fast (measured: V = 1024 27% faster per decode with 512
    // threads, V = 32 at r = 0.01 6% slower).
    // Beam capacity: up to 128 entries the beam state takes 31 to 35 KB of LDS; beyond, the
    // 512-entry build (116 KB, one thread per entry, one workgroup per CU) is used, and beyond
    // that the 1024-entry build (1024 threads, 134 KB, part of the state in global memory).
    // Residency: at two wavefronts per SIMD a CU holds two 256-thread workgroups (one of 512
    // threads).  A batch with more utterances than that over the whole chip is bound by
    // instruction issue, not by one frame's latency, and small frames then run best as two
    // wavefronts per utterance (one for the stays, one for the extensions: the other two of
    // the four mostly repeat wave-uniform bookkeeping), with registers cut for three
    // wavefronts per SIMD and, where a one-shot decode's beam allows, the 64-entry state
    // (20 KB of LDS) so that more workgroups fit a CU.  Measured on B = 4096, V = 32,
    // beam 32, before light frames: 287 M frames/s with the four-wavefront build alone, 470 M with its registers
    // cut for four wavefronts per SIMD, 564 M with two wavefronts per utterance, 679 M with
    // the small state as well.  A streaming decode keeps the 128-entry state throughout (its
    // carried records are laid out for it).
    // (large vocabulary: eight wavefronts per utterance while the whole batch is resident that
    // way, two workgroups per CU, four beyond: B = 1024, V = 1024: 143 M frames/s against
    // 120 M; B = 512: 93 M against 111 M)
    // Which survivor lists to expect.  A threshold R > 0 keeps a share of the vocabulary that falls
    // with R: `likely` is what a frame with competing tokens keeps of it, fitted to where the builds
    // for long lists begin to pay on this repository's emissions (tokens per threads of an entry;
    // time with short lists assumed / with long ones, 160 random calls: R = 0.1: 447 0.96, 1670
    // 1.08; R = 0.01: 16 0.97, 32 1.00, 64 1.02, 113 1.05, 900 1.42; R = 0.003: 16 1.09; R = 0.001:
    // 10 1.03, 16 1.10, 32 1.21).  Results do not depend on it.
    const double share =
        p.rel_threshold > 0.0f ? 0.1 * std::pow(0.01 / (double)p.rel_threshold, 1.25) : 1.0;
    const double likely = fmin((double)kept_at_most, (double)V * fmin(1.0, share));
    const int per_entry = (huge_beam ? kThreadsHuge : kThreadsLarge) / p.beam;  // of a full beam
    const int entry_threads = per_entry > 0 ? per_entry : 1;
    // Long: some thread has kFlooredFrom candidates.
    const bool long_lists =
        kept_at_most > kRegK && likely > (double)((kFlooredFrom - 1) * entry_threads);
    // A beam of hundreds of entries, one thread each, is spread so far that most tokens of the smallest
    // vocabularies can reach its floor, and the pass that lists those costs more than it saves.  The line
    // is drawn for short utterances (32 x 60 frames, time with the list of the time without, beams 257 /
    // 512 / 1000: V = 32, R = 0.01 1.02 / 1.02 / 1.04, V = 128 1.03 / 1.05 / 1.04, V = 256 1.02 / 1.04 / 1.01, V = 500
    // 0.92 / 0.94 / 0.95; R = 0.001: V = 64 1.03 / 1.03 / 1.02, V = 256 0.87 / 0.94 / 0.95).  Longer ones, whose
    // beam is full for most of their frames, would gain from the list from V = 128 on (300 frames: V = 32,
    // R = 0.01 1.01 / 1.02 / 1.03, V = 128 0.96 / 1.00 / 1.02, V = 256 0.85 / 0.90 / 0.91; R = 0.001: V = 128 0.71 /
    // 0.80 / 0.88, V = 256 0.54 / 0.63 / 0.65).  Beams of 129 to 256 have it throughout (V = 29 to 256: 60
    // frames 0.92 to 1.04, 400 frames 0.84 to 1.00).
    const bool few_tokens = p.beam > kBeamLarge / 2 && V < 512;
    // Whole: every token is kept, of a vocabulary that gives no thread that many, or a static
    // top-N is filled: up to three candidates per thread, of which most lie beyond the histogram's
    // window (see kCountAll; the 1024-thread build, which gets there with at most six tokens per
    // frame, gains nothing).
    const bool whole_lists = !long_lists && (p.rel_threshold == 0.0f ||
                                             (!large_beam && likely > (double)entry_threads));
    const bool tiny_state = p.beam <= kBeamTiny && carried == nullptr;
    const bool kept_few = p.rel_threshold > 0.0f || kept_at_most <= kWave;
    // Builds with 256 and 128 threads: frames whose survivors fit their header, and whose extensions fit
    // the threads, run as light ones.  Where no frame can (R = 0: every frame keeps as many), a build
    // without that path is 4-10% faster (64 utterances x 100 frames, beam 64, Top-7: 560 against 594 us; Top-5,
    // beam 65, for which three non-blank tokens fit: 492 against 526).  Nor does it pay for a stream that
    // is fed a frame or two per call: what the first and the last frame of a call set up for it costs more
    // than they gain (64 streams, beam 100, four calls of one frame: 69.1 against 73.5 us, of two 72.0
    // against 75.2; of five 122.5 against 122.7, and beam 8 103.6 against 95.7).
    // Frames that go through the tokens that can reach the beam only (fltop_beam_reach.inc).  Small vocabularies:
    // where frames with competing tokens keep more than the six that fit their header, so that most would
    // take the general path (64 utterances x 500 frames, V = 32, beam 32, R = 0: 2200 -> 705 us; R = 0.01,
    // where plain light frames do: 384 us against 390 when both came, with a table 481 against 535, two utterances fed
    // 25 frames a call, beam 97, table, window 10: 452 against 557).  They have the threads that the general path wants, which
    // frames that turn out to be none take: with 256 where every token is kept, those of flat emissions took up to
    // twice as long (64 x 100 frames, V = 64, beam 64, R = 0: 931 us without these frames, 2126 with 256 threads, 1093
    // with 512; V = 32, beam 16: 407, 584, 309) and the peaked ones no less (batch above: 843).
    // Vocabularies above 64 tokens: where frames keep up to 64 (a
    // lane each), which those that keep every token do not (128 x 400, V = 1024, beam 64, R = 0.01: 757 -> 463 us,
    // with a table in memory 883 -> 803; R = 0 2721 us without, 2853 with it); the largest
    // ones leave no LDS for the survivors by token.  A table spreads the scores, and with 256 threads most lists would
    // be too long (128 x 500, V = 32, beam 64, R = 0: 2567 us without, 4016 with it), with 512 those of small thresholds
    // (64 x 150, V = 512, beam 100, R = 0.003: 542 and 610; V = 1024, beam 64, R = 0.001: 617 and 649; V = 128: 847 and
    // 832).  Small vocabularies that keep every token at beams above 64 have 512 threads without these frames (with 256
    // they leave one block of extensions: 32 x 200, V = 32, beam 128: 1344 and 1533 us; R = 0.0005, V = 32, beam 100,
    // which has 256 threads either way: 1256 -> 795).  Not for streams of a few frames per call,
    // which set up for them in vain (64 streams, V = 64, beam 64, R = 0, six calls of one frame: 200 us, with 256 threads
    // 334; five calls of V = 1024, R = 0.01 without and with them: beam 64, three frames 167 and 178, five 219 and 218;
    // beam 100, five 284 and 289, eight 320 and 333; V = 73, R = 0.003, beam 98, eight 360 and 356).
    const bool narrow_reach = !wide && !dense && !short_calls && likely > (double)kNarrowReachAbove && p.lm_table == nullptr;
    const bool never_light =
        short_calls ||
        (p.rel_threshold == 0.0f && !narrow_reach &&
         !light_possible(kept_at_most, p.beam, dense && tiny_state ? kThreadsDense : kThreadsSmall, kRegK));
    // With a table, one block of extensions (beams above 64) is too little for what large vocabularies list (64 x 200,
    // V = 972, R = 0.01: beam 64 472 us without, 441 with, beam 79 514 and 562; V = 128, beam 79 457 and 391, but 16
    // streams of ten frames a call, beam 100 485 and 524), and what a score window asks of every candidate too
    // much for lists of several rounds (64 x 150, V = 512, R = 0.01, window 10: beam 32 300 and 273, beam 48 326 and
    // 370; R = 0.1 232 and 205).
    const bool table_reach =
        p.lm_table == nullptr ||
        (likely <= 128.0 && p.beam <= (p.beam_threshold > 0.0 ? (likely > 8.0 ? 32 : kBeamTiny) : (V <= 256 && carried == nullptr ? kBeamSmall : kBeamTiny)));
    const bool wide_reach = V <= 64 ? wide && every_reach
                                    : !dense && !large_beam && V <= 2048 && kept_few && !short_calls && table_reach;
    const bool any_reach = narrow_reach || wide_reach;
    // Distance cache: rows for the candidates beyond the one a thread keeps in registers.  A
    // batch that leaves LDS to spare (at most two workgroups per CU) gets 48 KB with 512
    // threads (frames of up to 6656 candidates are evaluated once) or 16 KB with 256; the
    // builds for large batches get one row (1-4 KB: up to two candidates per thread), or as many as light
    // frames need.
    if (!large_beam) {
        const int threads = threads_512 ? kThreadsLarge
                                        : (wide || !dense ? kThreadsSmall : kThreadsDense);
        a.dcache_rows = dense && !wide_reach ? 1 : (wide ? 12 : 8);
        const LightShape shape = light_shape(p.beam, threads);
        // the builds with light frames, whose scores lie there
        const bool plain_light = !wide && !narrow_reach && (tiny_state || !dense);
        const int scores = plain_light ? light_candidates(p.beam, threads)
                                       : (any_reach ? reach_candidates(p.beam, threads, V) : 0);
        const int light_rows = (scores + threads - 1) / threads;
        if (a.dcache_rows < light_rows) a.dcache_rows = light_rows;
        dyn += (size_t)a.dcache_rows * threads * sizeof(uint64_t);
        if (any_reach) {
            a.light_off = (int32_t)dyn;
            const int places = reach_list_places(shape.blocks, threads, V);
            dyn += ((size_t)V + 1) * 16 + 2 * sizeof(Survivor) * (size_t)(places + 1) +
                   ((size_t)places << shape.lg) * sizeof(uint32_t);
        }
    }
    // (A table that does not fit the LDS has more than 64 tokens, which makes a search wide: the builds
    // for others are not made for it.)
    auto launch = [&](auto lm_tag) -> hipError_t {
        constexpr int LM = decltype(lm_tag)::value;
#define FLTOP_LAUNCH_BUILD(THREADS_, MB_, WAVES_, LISTS_)                                   \
    hipLaunchKernelGGL((beam_kernel<LM, THREADS_, MB_, WAVES_, LISTS_>), dim3((unsigned)B), \
                       dim3(THREADS_), dyn, stream, a)
#define FLTOP_LAUNCH_SHORT_OR_LONG(THREADS_, MB_, WAVES_)                         \
    do {                                                                          \
        if (long_lists) FLTOP_LAUNCH_BUILD(THREADS_, MB_, WAVES_, kListsLongest); \
        else FLTOP_LAUNCH_BUILD(THREADS_, MB_, WAVES_, kListsShort);              \
    } while (0)
#define FLTOP_LAUNCH_ANY_LISTS(THREADS_, MB_, WAVES_)                            \
    do {                                                                         \
        if (whole_lists) FLTOP_LAUNCH_BUILD(THREADS_, MB_, WAVES_, kListsWhole); \
        else FLTOP_LAUNCH_SHORT_OR_LONG(THREADS_, MB_, WAVES_);                  \
    } while (0)
        if (huge_beam && long_lists && few_tokens) {
            FLTOP_LAUNCH_BUILD(kThreadsHuge, kBeamHuge, 4, kListsLong);
        } else if (huge_beam) {
            FLTOP_LAUNCH_SHORT_OR_LONG(kThreadsHuge, kBeamHuge, 4);
        } else if (large_beam && long_lists && few_tokens) {
            FLTOP_LAUNCH_BUILD(kThreadsLarge, kBeamLarge, 2, kListsLong);
        } else if (large_beam) {
            FLTOP_LAUNCH_ANY_LISTS(kThreadsLarge, kBeamLarge, 2);
        } else if (wide && very_dense) {
            FLTOP_LAUNCH_BUILD(kThreadsSmall, kBeamSmall, 4, kListsShort);
        } else if (wide_reach) {
            if constexpr (LM == kLmLds) return hipErrorInvalidValue;  // (a table that small has at most 64 tokens)
            else if (whole_lists) FLTOP_LAUNCH_BUILD(kThreadsLarge, kBeamSmall, 2, kListsWhole | kReachFlag);
            else if (long_lists) FLTOP_LAUNCH_BUILD(kThreadsLarge, kBeamSmall, 2, kListsLongest | kReachFlag);
            else FLTOP_LAUNCH_BUILD(kThreadsLarge, kBeamSmall, 2, kListsShort | kReachFlag);
        } else if (wide && dense) {
            FLTOP_LAUNCH_ANY_LISTS(kThreadsLarge, kBeamSmall, 4);
        } else if (wide) {
            FLTOP_LAUNCH_ANY_LISTS(kThreadsLarge, kBeamSmall, 2);
        } else if constexpr (LM == kLmGlobal) {
            return hipErrorInvalidValue;
        } else if (dense && tiny_state && never_light) {
            FLTOP_LAUNCH_BUILD(kThreadsDense, kBeamTiny, 3, kListsWhole);
        } else if (dense && tiny_state) {
            FLTOP_LAUNCH_BUILD(kThreadsDense, kBeamTiny, 3, kListsShort);
        } else if (dense) {
            FLTOP_LAUNCH_BUILD(kThreadsDense, kBeamSmall, 3, kListsShort);
        } else if (never_light) {
            FLTOP_LAUNCH_BUILD(kThreadsSmall, kBeamSmall, 2, kListsWhole);
        } else if (narrow_reach) {
            if constexpr (LM != kLmNone) return hipErrorInvalidValue;  // (calls with a table are none)
            else FLTOP_LAUNCH_BUILD(kThreadsSmall, kBeamSmall, 2, kListsShort | kReachFlag);
        } else {
            FLTOP_LAUNCH_BUILD(kThreadsSmall, kBeamSmall, 2, kListsShort);
        }
        return hipGetLastError();
#undef FLTOP_LAUNCH_ANY_LISTS
#undef FLTOP_LAUNCH_SHORT_OR_LONG
#undef FLTOP_LAUNCH_BUILD
    };
    if (p.lm_table == nullptr) return launch(std::integral_constant<int, kLmNone>{});
    if (a.lm_in_lds) return launch(std::integral_constant<int, kLmLds>{});
    return launch(std::integral_constant<int, kLmGlobal>{});
}

}  // namespace fltop
