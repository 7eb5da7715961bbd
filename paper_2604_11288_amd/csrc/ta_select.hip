// Step 4 of the eviction pass: utility (Eq. 1 / Eq. 3) and protected top-K
// (Alg. 1, utility and top-K steps; Sec. 3.3; Thm. 2-4).
//
// One workgroup per unit.  The total order is (class desc, u desc, position
// desc) and the class sizes are known before any ranking: class 2 (sinks and
// recent window) is a pair of position ranges, class 1 (sponsored) is counted
// from the sponsor mask.  Hence exactly one class straddles the budget - the
// "boundary class" - and only inside it a rank threshold is needed:
//   c2 + c1 <= K : classes 2 and 1 are kept whole, R = K - c2 - c1 slots go to class 0
//   otherwise    : class 2 is kept whole, R = K - c2 slots go to class 1 (pool overflow)
// Three kernels find the R-th largest (u, position) key of that class and write the retained positions in
// ascending order, all over order-preserving 32-bit images of u:
//   select_reg_kernel     rows whose keys fit the registers of a workgroup: one pass over the inputs, the
//                         cut found by binning over the range of the keys and ranking one bin's members
//   select_stream         long rows and many units: one pass with a list of candidates in LDS
//   select_kernel         what neither takes: keys recomputed for every pass of an MSD radix select
//
// Options around the same selection (baselines and Sec. 3.3 as settings):
//   pool_r       the scores are max-pooled over 2 pool_r + 1 positions before the utility
//                (the clustering step of SnapKV)
//   layer_K      per-layer budgets (PyramidKV); idx rows keep the common capacity K
//   k_protected  fixed partition K = K_main + K_protected (template CAPPED): the protected pool
//                takes the k_protected best sponsored tokens, everything else that is not
//                mandatory competes for the main pool by (u, position) alone - two threshold
//                searches instead of one
#include <type_traits>

#include "ta_gather.h"
#include "ta_order.h"
#include "ta_wave.h"

namespace ta {

namespace {

constexpr int SEL_THREADS = 1024;
constexpr int SEL_WAVES = SEL_THREADS / 64;
constexpr int HIST_COPIES = 16;               // privatised histograms, one per lane % 16
constexpr int HIST_STRIDE = 257;              // odd stride: the same bin of different copies sits in different LDS banks

struct SelectArgs {
    const float* A;
    const uint8_t* anchor;
    const uint8_t* spons;
    const float* vouch;
    const int32_t* seq_len;
    const int32_t* layer_K;
    int32_t* idx;
    int32_t* cnt;
    float* margin;                  // [units][2] or null: smallest retained / largest evicted u of the class the cut falls in
    int32_t batch, hkv, n, K;
    int32_t pool_r, k_protected;
    int32_t units;
    int32_t vec_ok;
    Divider by_hkv, by_batch;
    int32_t n_sink, n_recent;
    float alpha, beta, gamma;
};

// Order-preserving map fp32 -> uint32 (larger float <=> larger integer).
__device__ __forceinline__ uint32_t ordered_bits(float u)
{
    uint32_t b = __float_as_uint(u);
    return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

// The inverse map; the ends of the key range stand for "no such position".
__device__ __forceinline__ float margin_value(uint32_t k)
{
    if (k == 0xFFFFFFFFu) return INFINITY;                  // no retained member
    if (k == 0u) return -INFINITY;                          // no evicted member
    return __uint_as_float((k >> 31) ? (k ^ 0x80000000u) : ~k);
}

__device__ __forceinline__ int block_sum(int v, int* s_red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
    if (lane == 0) s_red[wave] = v;
    __syncthreads();
    int t = 0;
    for (int w = 0; w < SEL_WAVES; ++w) t += s_red[w];
    return t;
}

struct RadixState {
    uint32_t digit;      // chosen digit
    uint32_t need;       // keys still needed inside the chosen bin
    uint32_t bin_count;  // population of the chosen bin
    uint32_t all_of_bin; // 1: the chosen bin and everything above it is exactly what is needed
};

// After a histogram pass: s_hist[copy][bin] hold the counts.  Finds the largest
// digit d with sum_{d' >= d} h[d'] >= need.  All threads get the result.
__device__ __forceinline__ RadixState radix_pick(uint32_t (*s_hist)[HIST_STRIDE], uint32_t* s_h,
                                                 RadixState* s_state, uint32_t need)
{
    const int tid = threadIdx.x;
    if (tid < 256) {
        uint32_t t = 0;
#pragma unroll
        for (int c = 0; c < HIST_COPIES; ++c) {
            t += s_hist[c][tid];
            s_hist[c][tid] = 0;
        }
        s_h[tid] = t;
    }
    __syncthreads();
    if (tid < 64) {
        // lane l owns bins 255-4l .. 252-4l (descending), scan over lanes
        uint32_t h0 = s_h[255 - 4 * tid], h1 = s_h[254 - 4 * tid];
        uint32_t h2 = s_h[253 - 4 * tid], h3 = s_h[252 - 4 * tid];
        uint32_t mine = h0 + h1 + h2 + h3;
        uint32_t incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            uint32_t up = __shfl_up(incl, o);
            if (tid >= o) incl += up;
        }
        unsigned long long m = __ballot(incl >= need);
        int first = __ffsll((long long)m) - 1;           // first lane reaching `need`
        if (tid == first) {
            uint32_t above = incl - mine;                  // keys in strictly higher bins
            uint32_t hs[4] = {h0, h1, h2, h3};
            RadixState r;
            r.digit = 0; r.need = 0; r.bin_count = 0; r.all_of_bin = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (above + hs[j] >= need) {
                    r.digit = (uint32_t)(255 - 4 * tid - j);
                    r.need = need - above;
                    r.bin_count = hs[j];
                    r.all_of_bin = (above + hs[j] == need) ? 1u : 0u;
                    break;
                }
                above += hs[j];
            }
            *s_state = r;
        }
    }
    __syncthreads();
    return *s_state;
}

// Four consecutive positions ("a quad") are one thread's unit of work: their operands arrive
// as one 16-byte load each for A and the vouchers and one 4-byte load each for the two flag
// arrays, their keys sit in one 16-byte LDS slot, and their retained members leave in order.
struct Quad {
    float A[4];
    float v[4];
    uint8_t sp[4];
    uint8_t an[4];
};

// ---- form for what the others do not take (rows longer than SR_MAX_N with an option, or with a list that does not
// fit): the keys are recomputed from the inputs in every pass -----------------------------------------------------
template <bool CAPPED>
__global__ void __launch_bounds__(SEL_THREADS)
select_kernel(SelectArgs a)
{
    __shared__ uint32_t s_hist[HIST_COPIES][HIST_STRIDE];
    __shared__ uint32_t s_h[256];
    __shared__ int s_red[SEL_WAVES];
    __shared__ RadixState s_state;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    // Same block -> unit order as the score step: A is read from the L2 that wrote it (unless the second sweep went backwards).
    const int32_t place = (int32_t)blockIdx.x;
    if (place >= a.units) return;
    const int32_t unit = __builtin_amdgcn_readfirstlane(unit_at(place, a.seq_len, a.batch, a.hkv, a.units));
    const int32_t b = (unit / a.hkv) % a.batch;
    const int32_t n = a.n;
    int32_t K = a.K;                                         // capacity of an idx row; the budget unless a layer has its own
    if (a.layer_K) {
        int32_t lo = a.n_sink + a.n_recent;                  // the mandatory tokens must fit (validated: <= a.K)
        lo = lo < 1 ? 1 : lo;
        const int32_t kl = a.layer_K[unit / (a.batch * a.hkv)];
        K = kl < lo ? lo : (kl > K ? K : kl);
    }
    int32_t nb = a.seq_len ? a.seq_len[b] : n;
    nb = nb < 0 ? 0 : (nb > n ? n : nb);
    int32_t* idx = a.idx + (size_t)unit * (size_t)a.K;

    if (nb <= K) {                                           // nothing to evict
        for (int32_t p = tid; p < nb; p += SEL_THREADS) idx[p] = p;
        if (tid == 0) {
            a.cnt[unit] = nb;
            if (a.margin) {
                a.margin[2 * (size_t)unit] = INFINITY;
                a.margin[2 * (size_t)unit + 1] = -INFINITY;
            }
        }
        return;
    }

    const float* A = a.A ? a.A + (size_t)unit * (size_t)n : nullptr;
    const size_t row = (size_t)b * (size_t)n;
    const uint8_t* anchor = a.anchor + row;
    const uint8_t* spons = a.spons + row;
    const float* vouch = a.vouch + row;

    const int32_t ns = a.n_sink < nb ? a.n_sink : nb;
    int32_t rs = nb - a.n_recent;                            // recent window = [rs, nb)
    rs = rs < ns ? ns : rs;
    const int32_t c2 = ns + (nb - rs);
    const int32_t nquads = (nb + 3) >> 2;
    const bool use_A = (a.alpha != 0.0f);
    const bool vec = a.vec_ok != 0;                          // n % 4 == 0 and aligned rows

    for (int i = tid; i < HIST_COPIES * HIST_STRIDE; i += SEL_THREADS) (&s_hist[0][0])[i] = 0;

    auto load_flags = [&](const uint8_t* src, int32_t q, uint8_t (&out)[4]) {
        if (vec) {
            const uchar4 f = *reinterpret_cast<const uchar4*>(src + 4 * q);   // 4q + 3 < n: inside the row
            out[0] = f.x; out[1] = f.y; out[2] = f.z; out[3] = f.w;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) out[c] = (4 * q + c < nb) ? src[4 * q + c] : (uint8_t)0;
        }
    };
    auto load_floats = [&](const float* src, int32_t q, float (&out)[4]) {
        if (vec) {
            const float4 f = *reinterpret_cast<const float4*>(src + 4 * q);
            out[0] = f.x; out[1] = f.y; out[2] = f.z; out[3] = f.w;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) out[c] = (4 * q + c < nb) ? src[4 * q + c] : 0.0f;
        }
    };
    // scores of a quad, max-pooled over [p - r, p + r] clipped to the sequence (r <= 4: the quad and its neighbours)
    auto load_pooled = [&](int32_t q, float (&out)[4]) {
        float w[12];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int32_t qq = q - 1 + j;
            if (vec && qq >= 0 && 4 * qq + 3 < n) {
                const float4 f = *reinterpret_cast<const float4*>(A + 4 * qq);
                w[4 * j + 0] = f.x; w[4 * j + 1] = f.y; w[4 * j + 2] = f.z; w[4 * j + 3] = f.w;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (4 * qq + c >= nb) w[4 * j + c] = -INFINITY;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int32_t p = 4 * qq + c;
                    w[4 * j + c] = (p >= 0 && p < nb) ? A[p] : -INFINITY;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float m = w[4 + c];
#pragma unroll
            for (int d = 1; d <= 4; ++d)
                if (d <= a.pool_r) m = fmaxf(m, fmaxf(w[4 + c - d], w[4 + c + d]));
            out[c] = (4 * q + c < nb) ? m : 0.0f;
        }
    };
    auto load_rest = [&](int32_t q, Quad& x) {               // everything but the sponsor flags
        load_flags(anchor, q, x.an);
        load_floats(vouch, q, x.v);
        if (use_A && a.pool_r > 0) load_pooled(q, x.A);
        else if (use_A) load_floats(A, q, x.A);
        else {
#pragma unroll
            for (int c = 0; c < 4; ++c) x.A[c] = 0.0f;
        }
    };

    // ---- class-1 population
    int local = 0;
    for (int32_t q = tid; q < nquads; q += SEL_THREADS) {
        uint8_t sp[4];
        load_flags(spons, q, sp);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int32_t p = 4 * q + c;
            local += (p >= ns && p < rs && sp[c]) ? 1 : 0;
        }
    }
    const int32_t c1 = block_sum(local, s_red);

    const int bclass = (c2 + c1 <= K) ? 0 : 1;
    const int32_t R = bclass == 0 ? K - c2 - c1 : K - c2;    // slots for the boundary class
    const float nf = (float)nb;
    // fixed partition: P sponsored tokens are protected, M more slots go to the best of everything else
    int32_t P = 0;
    if (CAPPED) {
        P = a.k_protected < c1 ? a.k_protected : c1;
        P = P < K - c2 ? P : K - c2;
    }
    const int32_t M = K - c2 - P;

    // order-preserving key of position p if it belongs to the boundary class (fixed partition:
    // if it is not mandatory), else 0
    auto key_of = [&](int32_t p, float Ap, uint8_t an, uint8_t sp, float v) -> uint32_t {
        if (p < ns || p >= rs) return 0u;
        if (!CAPPED && (sp != 0) != (bclass == 1)) return 0u;
        float r = __fdiv_rn((float)(p + 1), nf);
        float t = use_A ? __fmul_rn(a.alpha, Ap) : 0.0f;
        t = __fadd_rn(t, __fmul_rn(a.beta, r));
        t = __fadd_rn(t, __fmul_rn(a.gamma, (float)an));
        t = __fadd_rn(t, v);
        uint32_t k = ordered_bits(t);
        return k == 0u ? 1u : k;
    };
    auto quad_keys = [&](int32_t q, const Quad& x, uint32_t (&k)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) k[c] = key_of(4 * q + c, x.A[c], x.an[c], x.sp[c], x.v[c]);
    };
    auto keys_at = [&](int32_t q, uint32_t (&k)[4]) {
        Quad x;
        load_flags(spons, q, x.sp);
        load_rest(q, x);
        quad_keys(q, x, k);
    };
    __syncthreads();

    // ---- threshold search ------------------------------------------------
    // Among the positions `member` admits (it gets a quad, its keys, and clears the keys of the
    // others), finds the `want`-th largest (key, position): a member is in the top `want` iff
    // key > T, or key == T and position >= Pt.
    auto find_threshold = [&](auto&& member, uint32_t want, uint32_t& T, int32_t& Pt) {
        uint32_t prefix = 0, need = want;
        bool done = false;
        for (int pass = 0; pass < 4 && !done; ++pass) {
            const int shift = 24 - 8 * pass;
            for (int32_t q = tid; q < nquads; q += SEL_THREADS) {
                uint32_t k4[4];
                keys_at(q, k4);
                member(q, k4);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t k = k4[c];
                    bool in = k != 0u && (pass == 0 || (k >> (shift + 8)) == (prefix >> (shift + 8)));
                    if (in) atomicAdd(&s_hist[lane & (HIST_COPIES - 1)][(k >> shift) & 255u], 1u);
                }
            }
            __syncthreads();
            RadixState r = radix_pick(s_hist, s_h, &s_state, need);
            prefix |= r.digit << shift;
            need = r.need;
            if (r.all_of_bin) {                              // keep every key >= prefix
                T = prefix - 1u;
                Pt = 0x7FFFFFFF;
                done = true;
            } else if (pass == 3) {
                T = prefix;                                  // several positions share u == T
                // the `need` highest positions among them are kept
                int bits = 32 - __clz(nb - 1);
                int ppasses = (bits + 7) / 8;
                uint32_t pprefix = 0, pneed = need;
                for (int pp = 0; pp < ppasses; ++pp) {
                    const int ps = 8 * (ppasses - 1 - pp);
                    for (int32_t q = tid; q < nquads; q += SEL_THREADS) {
                        uint32_t k4[4];
                        keys_at(q, k4);
                        member(q, k4);
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const uint32_t p = (uint32_t)(4 * q + c);
                            bool in = k4[c] == T && (pp == 0 || (p >> (ps + 8)) == (pprefix >> (ps + 8)));
                            if (in) atomicAdd(&s_hist[lane & (HIST_COPIES - 1)][(p >> ps) & 255u], 1u);
                        }
                    }
                    __syncthreads();
                    RadixState qs = radix_pick(s_hist, s_h, &s_state, pneed);
                    pprefix |= qs.digit << ps;
                    pneed = qs.need;
                }
                Pt = (int32_t)pprefix;                       // positions are unique: pneed == 1 here
                done = true;
            }
        }
    };

    uint32_t T = 0xFFFFFFFFu;     // boundary-class position p is kept iff key > T, or key == T and p >= Pt
    int32_t Pt = 0x7FFFFFFF;
    uint32_t T1 = 0xFFFFFFFFu;    // fixed partition: a sponsored position is protected iff key > T1, or key == T1 and p >= Pt1
    int32_t Pt1 = 0x7FFFFFFF;
    if (!CAPPED) {
        if (R > 0) find_threshold([](int32_t, uint32_t (&)[4]) {}, (uint32_t)R, T, Pt);
    } else {
        if (P == c1) {                                       // every sponsored token is protected
            T1 = 0u;
            Pt1 = 0;
        } else if (P > 0) {
            find_threshold([&](int32_t q, uint32_t (&k4)[4]) {
                uint8_t sp[4];
                load_flags(spons, q, sp);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (!sp[c]) k4[c] = 0u;
            }, (uint32_t)P, T1, Pt1);
        }
        if (M > 0) {                                         // more candidates than M remain: nb > K
            find_threshold([&](int32_t q, uint32_t (&k4)[4]) {
                uint8_t sp[4];
                load_flags(spons, q, sp);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int32_t p = 4 * q + c;
                    if (sp[c] && (k4[c] > T1 || (k4[c] == T1 && p >= Pt1))) k4[c] = 0u;   // protected: not a candidate
                }
            }, (uint32_t)M, T, Pt);
        }
    }

    // ---- which positions of a quad are retained (bit c: position 4q + c) --------------------------
    uint32_t kept_min = 0xFFFFFFFFu, gone_max = 0u;          // keys at the cut, over this thread's candidates
    const auto keep_of = [&](int32_t q) -> uint32_t {
        uint32_t keep = 0;
        uint8_t sp[4] = {0, 0, 0, 0};
        uint32_t k4[4] = {0u, 0u, 0u, 0u};
        load_flags(spons, q, sp);
        bool need_keys = false;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int32_t p = 4 * q + c;
            need_keys = need_keys || (p >= ns && p < rs && (CAPPED || (sp[c] != 0) == (bclass == 1)));
        }
        if (need_keys) keys_at(q, k4);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int32_t p = 4 * q + c;
            bool kp = false;
            bool ranked = false;                             // competes for the slots the cut divides
            if (p < nb) {
                if (p < ns || p >= rs) kp = true;
                else if (CAPPED) {
                    const bool prot = sp[c] && (k4[c] > T1 || (k4[c] == T1 && p >= Pt1));   // protected pool
                    kp = prot || (k4[c] > T) || (k4[c] == T && p >= Pt);                  // main pool
                    ranked = !prot;
                } else if ((sp[c] != 0) != (bclass == 1)) kp = sp[c] != 0;   // class 1 above the boundary class, class 0 below it
                else {
                    kp = (k4[c] > T) || (k4[c] == T && p >= Pt);
                    ranked = true;
                }
            }
            if (ranked && kp) kept_min = k4[c] < kept_min ? k4[c] : kept_min;
            if (ranked && !kp) gone_max = k4[c] > gone_max ? k4[c] : gone_max;
            keep |= kp ? (1u << c) : 0u;
        }
        return keep;
    };

    // ---- ascending write-out -------------------------------------------------------------------
    int32_t base = 0;
    // one scan over per-quad counts per round of 4096 positions
    for (int32_t q0 = 0; q0 < nquads; q0 += SEL_THREADS) {
        const int32_t q = q0 + tid;
        const uint32_t keep = q < nquads ? keep_of(q) : 0u;
        const int mine = __popc(keep);
        int incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            int up = __shfl_up(incl, o);
            if (lane >= o) incl += up;
        }
        __syncthreads();
        if (lane == 63) s_red[wave] = incl;
        __syncthreads();
        int woff = 0, total = 0;
        for (int w = 0; w < SEL_WAVES; ++w) {
            int c = s_red[w];
            woff += (w < wave) ? c : 0;
            total += c;
        }
        int32_t slot = base + woff + incl - mine;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (keep & (1u << c)) {
                if (slot < K) idx[slot] = 4 * q + c;
                ++slot;
            }
        }
        base += total;
    }
    if (tid == 0) a.cnt[unit] = base < K ? base : K;
    if (a.margin) {                                          // uniform
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t lo = __shfl_xor(kept_min, o), hi = __shfl_xor(gone_max, o);
            kept_min = lo < kept_min ? lo : kept_min;
            gone_max = hi > gone_max ? hi : gone_max;
        }
        __syncthreads();
        if (lane == 0) {
            s_h[wave] = kept_min;
            s_h[SEL_WAVES + wave] = gone_max;
        }
        __syncthreads();
        if (tid == 0) {
            for (int w = 0; w < SEL_WAVES; ++w) {
                kept_min = s_h[w] < kept_min ? s_h[w] : kept_min;
                gone_max = s_h[SEL_WAVES + w] > gone_max ? s_h[SEL_WAVES + w] : gone_max;
            }
            a.margin[2 * (size_t)unit] = margin_value(kept_min);
            a.margin[2 * (size_t)unit + 1] = margin_value(gone_max);
        }
    }
}


// ---- register form: rows of up to SR_MAX_N positions, one workgroup per unit ---------------------------------
// A thread keeps the keys of its quads in registers (quad r * SR_THREADS + tid in round r), so every input is read
// once, whatever class the cut falls in: the sponsored positions, the ranges of both classes' keys and the keys
// themselves come out of one pass.  The cut is found by binning the boundary class's keys over the range they
// really take (SR_BINS bins between the smallest and the largest: integers that order as the floats do, so an
// outlier costs a few octaves of bins and not the resolution) and ranking the few members of the bin it falls
// in against each other.
constexpr int SR_THREADS = 1024;
constexpr int SR_WAVES = SR_THREADS / 64;
constexpr int SR_MAX_ROUNDS = 8;
constexpr int SR_MAX_N = SR_MAX_ROUNDS * SR_THREADS * 4;
constexpr int SR_BINS = 2048;
constexpr int SR_CAND = 256;                                 // members of a bin that are ranked one against the other

// Rows moved by the workgroup that selects them: one launch fewer, some 2 us, but a workgroup moves no more than one compute
// unit can, and each has one to itself.  Whole pass in us, launch of its own / here, 256 compute units:
//   more units than compute units: never.  The last of them select and move in a second round (4096 positions, 64 rows: 256
//     units 107.9 / 106.4, 264 132.0 / 133.1; 1024 rows: 256 141.6 / 139.0, 264 164.5 / 174.1; ragged 1500..3001, 64 rows: 256
//     69.4 / 67.6, 288 89.4 / 91.4).
//   at least three quarters of them: any budget.  1024 rows, 4096 positions: 128 units 80.6 / 87.1, 160 95.9 / 98.7, 176 110.1 /
//     111.9, 192 114.9 / 113.6, 224 128.2 / 126.4; 8192 positions: 144 144.7 / 146.0, 176 174.3 / 173.9, 192 184.4 / 182.5;
//     2048 positions, half of them kept: 176 82.2 / 83.1, 192 86.2 / 86.5, 240 97.8 / 95.1.  (Fewer rows break even
//     earlier, ragged lengths later: 512 rows 160 83.2 / 83.8, 176 97.3 / 96.6; 1500..3001 positions, 1024 rows 192 89.3 / 91.1,
//     224 94.5 / 94.5, 256 103.9 / 102.3.)
//   fewer: up to 256 rows.  64 rows, 4096 positions: 64 units 40.5 / 38.9, 128 61.9 / 60.4; 256 rows: 8 units 23.9 / 23.9, 32 31.4 /
//     32.2, 128 65.0 / 65.3, 160 80.9 / 79.8; 320 rows: 8 units 23.6 / 24.5, 32 31.6 / 34.2; 512 rows: 16 units 26.5 / 29.5.
constexpr int SR_GATHER_MAX_K = 2048;                      // the list passes through the histogram's memory
constexpr int SR_GATHER_FEW_K = 256;
bool gathers_here(int64_t units, int32_t K)
{
    const int64_t cus = compute_units();
    return units <= cus && K <= (4 * units >= 3 * cus ? SR_GATHER_MAX_K : SR_GATHER_FEW_K);
}

struct SelectRegLds {
    uint32_t hist[32 * 65];                                  // bin b at (b % 32) * 65 + b / 32: 64 lanes read a row of it at once; then the list to gather
    uint32_t part[4 * SR_WAVES], sponsored[SR_WAVES];        // per wavefront: key ranges of both classes (the smallest as complements); sponsored count
    uint32_t bound[SR_WAVES], groups[SR_WAVES];              // per wavefront: a lower bound of the cut (complement); the groups it is over
    uint32_t edge[2][SR_WAVES];                              // per wavefront: smallest retained, largest evicted key
    uint32_t totals[SR_MAX_ROUNDS * SR_WAVES];               // retained positions per round and wavefront
    uint32_t cand[2 * SR_CAND + 4];                          // (position, key) pairs
    uint32_t count;
    struct { uint32_t bin, need, count, all, key, pos; } st;
};

// ---- quads of a row of n positions at any alignment (n % 4 != 0 puts the rows of a batch at odd places): one wide load
// each, which the hardware takes at any byte address.  A quad that would reach past the row's end (the last one, n >= 4)
// is loaded from the row's last four positions and moved down; what lies past the end is 0.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_any __attribute__((aligned(1)));
__device__ __forceinline__ int32_t quad_start(int32_t p, int32_t n) { return p <= n - 4 ? p : n - 4; }
__device__ __forceinline__ float4 load_quad_f(const float* row, int32_t start)
{
    const f32x4_any v = *reinterpret_cast<const f32x4_any*>(row + start);
    return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ uint32_t load_quad_b(const uint8_t* row, int32_t start)
{
    return *reinterpret_cast<const u32_any*>(row + start);
}
__device__ __forceinline__ float4 move_down(float4 v, int32_t by)         // by 0 .. 3 positions
{
    if (by & 1) v = make_float4(v.y, v.z, v.w, 0.0f);
    if (by & 2) v = make_float4(v.z, v.w, 0.0f, 0.0f);
    return v;
}

static_assert(sizeof(SelectRegLds::hist) >= sizeof(uint32_t) * SR_GATHER_MAX_K, "the list to gather");

// SEGS > 0: no attention term, and vouchers of the match or the expansion (0 wherever the sponsor flag is).  The plain positions'
// utilities (no anchor, no voucher) then rise with the position, so the last K - c2 positions before the recent window outrank
// or tie-break every plain one before them.  What can be retained at all is those, the mandatory positions and the flagged
// ones: their positions are collected into a list in LDS, in order, from the flags alone (two bytes per position, 16 positions
// to a load, SEGS times 32 positions per thread), and the list is selected from as a row of one round is.  More of them than the
// list holds (a table that hits nearly everywhere): false, and the caller takes the whole row.  (Not with the margin output, which
// wants the best of the evicted ones, nor with the fixed partition, which ranks both classes.)
// ASK: the vouchers may be anything.  A position whose voucher is not zero joins the list as a flagged one does, and if one of the last
// K - c2 has a voucher below zero, or none (NaN), the whole row is taken.  The flags are counted first: where they alone fill the list no
// voucher is looked at.
// What it measured: where launch_select chooses.
constexpr int SR_LIST = 4 * SR_THREADS;
constexpr int SR_SEG = 32 * SR_THREADS;                    // a thread's flags of a segment are the bits of one word
constexpr int SR_LONG_SEGS = 4;
static_assert(SR_SEG == SR_MAX_N, "a row of one segment is taken by the register form");
static_assert(SR_LONG_SEGS * SR_THREADS <= SR_LIST, "a bit per position has room in the list");
struct SparseList {
    uint32_t entry[SR_LIST];                                 // position; bit 31: sponsored, bit 30: an anchor
    uint32_t totals[SR_LONG_SEGS * SR_WAVES];
    uint32_t below_zero;                                     // ASK: a voucher at the end of the row is
};

// bit i: byte i of four is not zero
__device__ __forceinline__ uint32_t byte_flags(uint32_t x)
{
    const uint32_t high = (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u;
    return ((high >> 7) * 0x01020408u) >> 24 & 15u;
}
// flags of the 16 positions from p on as bits (0 past the row's end; n >= 16)
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
__device__ __forceinline__ u32x4_any load_flags16(const uint8_t* row, int32_t p, int32_t n)
{
    return *reinterpret_cast<const u32x4_any*>(row + (p <= n - 16 ? p : n - 16));
}
__device__ __forceinline__ uint32_t flags16(u32x4_any x, int32_t p, int32_t n)
{
    const uint32_t m = byte_flags(x[0]) | byte_flags(x[1]) << 4 | byte_flags(x[2]) << 8 | byte_flags(x[3]) << 12;
    return p <= n - 16 ? m : p < n ? m >> (p - (n - 16)) : 0u;
}

template <int ROUNDS, bool CAPPED, int GATHER, int SEGS = 0, bool ASK = false>
__device__ __forceinline__ bool select_reg(const SelectArgs& a, const std::conditional_t<GATHER != GATHER_NONE, CompactArgs, int>& g,
                                           SelectRegLds& L, SparseList* list)
{
    constexpr bool SPARSE = SEGS > 0;
    static_assert(!SPARSE || (ROUNDS == 1 && !CAPPED && GATHER == GATHER_NONE), "the list is one round");
    constexpr bool PRUNE = ROUNDS >= 4 && !CAPPED;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    // Same block -> unit order as the score step: A is read from the L2 that wrote it (unless the second sweep went backwards).
    const int32_t place = (int32_t)blockIdx.x;
    if (place >= a.units) return true;
    const int32_t unit = __builtin_amdgcn_readfirstlane(unit_at(place, a.seq_len, a.batch, a.hkv, a.units));
    const int32_t pair = (int32_t)divide((uint32_t)unit, a.by_hkv), l = (int32_t)divide((uint32_t)pair, a.by_batch);
    const int32_t b = pair - l * a.batch;
    const int32_t n = a.n;
    int32_t K = a.K;                                         // capacity of an idx row; the budget unless a layer has its own
    if (a.layer_K) {
        int32_t lo = a.n_sink + a.n_recent;                  // the mandatory tokens must fit (validated: <= a.K)
        lo = lo < 1 ? 1 : lo;
        const int32_t kl = a.layer_K[l];
        K = kl < lo ? lo : (kl > K ? K : kl);
    }
    int32_t nb = a.seq_len ? a.seq_len[b] : n;
    nb = nb < 0 ? 0 : (nb > n ? n : nb);
    int32_t* idx = a.idx + (size_t)unit * (size_t)a.K;

    if (nb <= K) {                                           // nothing to evict
        for (int32_t p = tid; p < nb; p += SR_THREADS) {
            idx[p] = p;
            if constexpr (GATHER != GATHER_NONE) L.hist[p] = (uint32_t)p;
        }
        if (tid == 0) {
            a.cnt[unit] = nb;
            if (a.margin) {
                a.margin[2 * (size_t)unit] = INFINITY;
                a.margin[2 * (size_t)unit + 1] = -INFINITY;
            }
        }
        if constexpr (GATHER != GATHER_NONE) {
            __syncthreads();
            gather_rows<SR_THREADS, GATHER>(g, unit, nb, L.hist, tid);
        }
        return true;
    }

    const float* A = a.A ? a.A + (size_t)unit * (size_t)n : nullptr;
    const size_t row = (size_t)b * (size_t)n;
    const uint8_t* anchor = a.anchor + row;
    const uint8_t* spons = a.spons + row;
    const float* vouch = a.vouch + row;
    const int32_t ns = a.n_sink < nb ? a.n_sink : nb;
    int32_t rs = nb - a.n_recent;                            // recent window = [rs, nb)
    rs = rs < ns ? ns : rs;
    const int32_t c2 = ns + (nb - rs);
    int32_t nquads = (nb + 3) >> 2;
    const bool use_A = (a.alpha != 0.0f);

    if (tid < 32 * 65 / 4) reinterpret_cast<uint4*>(L.hist)[tid] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) L.count = 0u;

    // ---- one pass over the inputs ------------------------------------------------------------------
    uint32_t key[ROUNDS][4];                                 // order-preserving images of u
    uint32_t mid = 0u, spm = 0u;                             // bits 4 r + c: between the mandatory ranges; and sponsored
    uint32_t lo0 = 0xFFFFFFFFu, hi0 = 0u, lo1 = 0xFFFFFFFFu, hi1 = 0u;   // key ranges of the plain and of the sponsored positions
    const float nf = (float)nb, inv = __fdiv_rn(1.0f, nf);
    const float g0 = __fmul_rn(a.gamma, 0.0f);
    int32_t own[4] = {0, 0, 0, 0};                           // SPARSE: positions of this thread's entries; past the last one n
    if constexpr (SPARSE) {
        const int32_t plain_end = rs - (K - c2);             // plain positions before it cannot be retained
        const int32_t tail = plain_end > 0 ? plain_end : 0;  // every position from it on is in the list
        if (nb - tail > SR_LIST) return false;               // uniform
        const auto first = [&](int s) { return SR_SEG * s + 32 * tid; };
        uint32_t in[SEGS], sp[SEGS] = {}, an[SEGS] = {}, upto[SEGS];         // bit i: position first(s) + i; in: is in the list
        u32x4_any f[SEGS][4];
        if (SEGS > 1 || first(0) < tail) {                   // (a short row's wavefronts that have none of it do not work on it)
#pragma unroll
            for (int s = 0; s < SEGS; ++s) {                 // all requested together; past the row its last 16 positions
                f[s][0] = load_flags16(spons, first(s), n);
                f[s][1] = load_flags16(spons, first(s) + 16, n);
                f[s][2] = load_flags16(anchor, first(s), n);
                f[s][3] = load_flags16(anchor, first(s) + 16, n);
            }
        }
        constexpr int ASK_QUADS = 8;                         // of vouchers, per thread in flight, behind the flags
        const int32_t quads = (tail + 3) >> 2;
        float4 v[ASK ? ASK_QUADS : 1];
        const auto load_vouchers = [&](int32_t q0) {
#pragma unroll
            for (int j = 0; ASK && j < ASK_QUADS; ++j) {
                const int32_t q = q0 + j * SR_THREADS + tid;
                v[j] = load_quad_f(vouch, quad_start(4 * (q < quads ? q : quads > 0 ? quads - 1 : 0), n));
            }
        };
        load_vouchers(0);
        if (SEGS > 1 || first(0) < tail) {
#pragma unroll
            for (int s = 0; s < SEGS; ++s) {
                const int32_t p0 = first(s);
                if (SR_SEG * s >= tail) continue;            // uniform
                sp[s] = flags16(f[s][0], p0, n) | flags16(f[s][1], p0 + 16, n) << 16;
                an[s] = flags16(f[s][2], p0, n) | flags16(f[s][3], p0 + 16, n) << 16;
            }
        }
        const auto in_front = [&](int s) {                   // the positions of the word before the tail
            const int32_t left = tail - first(s);
            return left >= 32 ? 0xFFFFFFFFu : left > 0 ? (1u << left) - 1u : 0u;
        };
#pragma unroll
        for (int s = 0; s < SEGS; ++s) {
            const int32_t p0 = first(s);
            in[s] = sp[s] | an[s];
            if (p0 < ns) in[s] |= ns - p0 < 32 ? (1u << (ns - p0)) - 1u : 0xFFFFFFFFu;
            in[s] &= in_front(s);
        }
        if constexpr (ASK) {
            uint32_t* bits = list->entry;
            uint32_t flagged = 0u;
#pragma unroll
            for (int s = 0; s < SEGS; ++s) {
                bits[s * SR_THREADS + tid] = 0u;
                flagged += (uint32_t)__popc(in[s]);
            }
            flagged = wave_sum_dpp(flagged);
            if (lane == 0) list->totals[wave] = flagged;
            if (tid == 0) list->below_zero = 0u;
            __syncthreads();
            if (__builtin_amdgcn_readlane((int)row_sum_dpp(list->totals[lane & (SR_WAVES - 1)]), 0) + nb - tail > SR_LIST) return false;     // uniform
            for (int32_t q0 = 0; q0 < quads;) {
#pragma unroll
                for (int j = 0; j < ASK_QUADS; ++j) {
                    const int32_t q = q0 + j * SR_THREADS + tid;
                    if (q >= quads) continue;
                    const float4 x = move_down(v[j], 4 * q - quad_start(4 * q, n));
                    const uint32_t set = (x.x != 0.0f ? 1u : 0u) | (x.y != 0.0f ? 2u : 0u) | (x.z != 0.0f ? 4u : 0u) | (x.w != 0.0f ? 8u : 0u);
                    if (set) atomicOr(&bits[q >> 3], set << (4 * (q & 7)));
                }
                q0 += ASK_QUADS * SR_THREADS;
                if (q0 < quads) load_vouchers(q0);           // uniform
            }
            bool below = false;
            for (int32_t p = tail + tid; p < nb; p += SR_THREADS) below = below || !(vouch[p] >= 0.0f);
            if (below) list->below_zero = 1u;
            __syncthreads();
            if (list->below_zero != 0u) return false;        // uniform in the workgroup
#pragma unroll
            for (int s = 0; s < SEGS; ++s) in[s] |= bits[s * SR_THREADS + tid] & in_front(s);
        }
#pragma unroll
        for (int s = 0; s < SEGS; ++s) upto[s] = wave_scan_dpp((uint32_t)__popc(in[s]));
        if (lane == 63) {
#pragma unroll
            for (int s = 0; s < SEGS; ++s) list->totals[s * SR_WAVES + wave] = upto[s];
        }
        __syncthreads();                                     // (and every thread has read its bits)
        const uint32_t sums = wave_scan_dpp(lane < SEGS * SR_WAVES ? list->totals[lane] : 0u);
        const int32_t found = __builtin_amdgcn_readlane((int)sums, SEGS * SR_WAVES - 1), m = found + nb - tail;
        if (m > SR_LIST) return false;                       // uniform in the workgroup
#pragma unroll
        for (int s = 0; s < SEGS; ++s) {
            const int e = s * SR_WAVES + wave;               // uniform in the wavefront
            const uint32_t before = e > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)sums, __builtin_amdgcn_readfirstlane(e > 0 ? e - 1 : 0)) : 0u;
            uint32_t at = before + upto[s] - (uint32_t)__popc(in[s]);
            for (uint32_t left = in[s]; left; left &= left - 1u) {
                const int bit = __ffs((int)left) - 1;
                list->entry[at++] = (uint32_t)(first(s) + bit) | ((sp[s] >> bit) & 1u) << 31 | ((an[s] >> bit) & 1u) << 30;
            }
        }
        for (int32_t p = tail + tid; p < nb; p += SR_THREADS)
            list->entry[found + p - tail] = (uint32_t)p | (spons[p] ? 0x80000000u : 0u) | (anchor[p] ? 0x40000000u : 0u);
        __syncthreads();
        nquads = (m + 3) >> 2;
        const uint4 mine = reinterpret_cast<const uint4*>(list->entry)[tid];
        const uint32_t e4[4] = {mine.x, mine.y, mine.z, mine.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool live = 4 * tid + c < m, sps = live && (e4[c] >> 31) != 0u;
            const int32_t p = live ? (int32_t)(e4[c] & 0x3FFFFFFFu) : n;
            own[c] = p;
            float t = __fmul_rn(a.beta, div_by((float)(p + 1), nf, inv));
            t = __fadd_rn(0.0f, t);
            // (a caller's flag other than 0 and 1 counts as in the form that would have the row otherwise)
            const float an1 = ASK && SEGS == 1 ? (live ? (float)anchor[p] : 0.0f) : live && (e4[c] & 0x40000000u) ? 1.0f : 0.0f;
            t = __fadd_rn(t, __fmul_rn(a.gamma, an1));
            t = __fadd_rn(t, (ASK ? live : sps) ? vouch[p] : 0.0f);
            const uint32_t k = ordered_bits(t);
            key[0][c] = k;
            const bool in2 = p >= ns && p < rs;
            mid |= in2 ? 1u << c : 0u;
            spm |= in2 && sps ? 1u << c : 0u;
            lo0 = in2 && !sps && k < lo0 ? k : lo0;
            hi0 = in2 && !sps && k > hi0 ? k : hi0;
            lo1 = in2 && sps && k < lo1 ? k : lo1;
            hi1 = in2 && sps && k > hi1 ? k : hi1;
        }
    } else {
        // The loads of BATCH rounds are issued together, unconditionally (a quad index past the end is clamped and its data
        // masked): with few units nothing else hides a round trip.  Which loads there are is asked once per batch and not per
        // round: behind a branch of its own every round waited for all that was outstanding, 2.2 us per 4096 positions.
        constexpr int BATCH = ROUNDS < 4 ? ROUNDS : 4;
#pragma unroll
        for (int r0 = 0; r0 < ROUNDS; r0 += BATCH) {
            if (r0 * SR_THREADS >= nquads) {                     // uniform: nothing of the row lies this far
#pragma unroll
                for (int r = r0; r < r0 + BATCH; ++r)
#pragma unroll
                    for (int c = 0; c < 4; ++c) key[r][c] = 0u;
                continue;
            }
            uint32_t sp[BATCH], an[BATCH];
            float4 v[BATCH], s[BATCH];
            const auto quad_of = [&](int j) {
                const int32_t q = (r0 + j) * SR_THREADS + tid;
                return q < nquads ? q : nquads - 1;
            };
            const auto load_shared = [&](int j) {                // what the units of a sequence share
                const int32_t start = quad_start(4 * quad_of(j), n);
                sp[j] = load_quad_b(spons, start);
                an[j] = load_quad_b(anchor, start);
                v[j] = load_quad_f(vouch, start);
                s[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                return start;
            };
            if (ROUNDS == 1 && n < 4) {                   // a row of one to three positions
                float vv[4], ss[4];
                sp[0] = an[0] = 0u;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float m = -INFINITY;
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (e < nb && e >= c - a.pool_r && e <= c + a.pool_r && use_A) m = fmaxf(m, A[e]);
                    const bool in = c < nb;
                    sp[0] |= in && spons[c] ? 1u << (8 * c) : 0u;
                    an[0] |= in ? (uint32_t)anchor[c] << (8 * c) : 0u;
                    vv[c] = in ? vouch[c] : 0.0f;
                    ss[c] = in && use_A ? m : 0.0f;
                }
                v[0] = make_float4(vv[0], vv[1], vv[2], vv[3]);
                s[0] = make_float4(ss[0], ss[1], ss[2], ss[3]);
            } else if (!use_A) {
#pragma unroll
                for (int j = 0; j < BATCH; ++j) load_shared(j);
            } else if (a.pool_r == 0) {
#pragma unroll
                for (int j = 0; j < BATCH; ++j) {
                    const int32_t start = load_shared(j);
                    s[j] = load_quad_f(A, start);
                }
            } else {
                // scores max-pooled over [p - r, p + r] clipped to the sequence: r <= 4, so the quad and its neighbours
                float4 w[BATCH][3];
#pragma unroll
                for (int j = 0; j < BATCH; ++j) {
                    load_shared(j);
#pragma unroll
                    for (int e = 0; e < 3; ++e) {
                        const int32_t p = 4 * (quad_of(j) - 1 + e);
                        w[j][e] = load_quad_f(A, quad_start(p < 0 ? 0 : p, n));
                    }
                }
#pragma unroll
                for (int j = 0; j < BATCH; ++j) {
                    const int32_t q = quad_of(j);
                    float x[12], ss[4];
#pragma unroll
                    for (int e = 0; e < 3; ++e) {
                        const int32_t p = 4 * (q - 1 + e);
                        if (n & 3) w[j][e] = move_down(w[j][e], p > n - 4 ? p - (n - 4) : 0);
                        const float y[4] = {w[j][e].x, w[j][e].y, w[j][e].z, w[j][e].w};
#pragma unroll
                        for (int c = 0; c < 4; ++c) x[4 * e + c] = p + c >= 0 && p + c < nb ? y[c] : -INFINITY;
                    }
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float m = x[4 + c];
#pragma unroll
                        for (int d = 1; d <= 4; ++d)
                            if (d <= a.pool_r) m = fmaxf(m, fmaxf(x[4 + c - d], x[4 + c + d]));
                        ss[c] = 4 * q + c < nb ? m : 0.0f;
                    }
                    s[j] = make_float4(ss[0], ss[1], ss[2], ss[3]);
                }
            }
#pragma unroll
            for (int j = 0; j < BATCH; ++j) {
                const int r = r0 + j;
                const int32_t q = r * SR_THREADS + tid;
                if (n >= 4 && (n & 3)) {                         // uniform
                    const int32_t by = q < nquads ? 4 * q - quad_start(4 * q, n) : 0;
                    sp[j] >>= 8 * by;
                    an[j] >>= 8 * by;
                    v[j] = move_down(v[j], by);
                    if (a.pool_r == 0) s[j] = move_down(s[j], by);
                }
                const float Aq[4] = {s[j].x, s[j].y, s[j].z, s[j].w}, vq[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
                const bool no_flags = (sp[j] | an[j]) == 0u;
                if (__ballot(!(no_flags && 4 * q >= ns && 4 * q + 3 < rs)) == 0ull) {   // nothing but class 0
                    mid |= 15u << (4 * r);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float t = use_A ? __fmul_rn(a.alpha, Aq[c]) : 0.0f;
                        t = __fadd_rn(t, __fmul_rn(a.beta, div_by((float)(4 * q + c + 1), nf, inv)));
                        t = __fadd_rn(t, g0);
                        t = __fadd_rn(t, vq[c]);
                        const uint32_t k = ordered_bits(t);
                        key[r][c] = k;
                        lo0 = k < lo0 ? k : lo0;
                        hi0 = k > hi0 ? k : hi0;
                    }
                    continue;
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int32_t p = 4 * q + c;
                    float t = use_A ? __fmul_rn(a.alpha, Aq[c]) : 0.0f;
                    t = __fadd_rn(t, __fmul_rn(a.beta, div_by((float)(p + 1), nf, inv)));
                    t = __fadd_rn(t, __fmul_rn(a.gamma, (float)((an[j] >> (8 * c)) & 0xFFu)));
                    t = __fadd_rn(t, vq[c]);
                    const uint32_t k = ordered_bits(t);
                    key[r][c] = k;
                    const bool sps = ((sp[j] >> (8 * c)) & 0xFFu) != 0u;
                    const bool m = p >= ns && p < rs;
                    mid |= m ? 1u << (4 * r + c) : 0u;
                    spm |= m && sps ? 1u << (4 * r + c) : 0u;
                    lo0 = m && !sps && k < lo0 ? k : lo0;
                    hi0 = m && !sps && k > hi0 ? k : hi0;
                    lo1 = m && sps && k < lo1 ? k : lo1;
                    hi1 = m && sps && k > hi1 ? k : hi1;
                }
            }
        }
    }
    // position of (round, quad element): in a row the quad's, in the list the entry's
    const auto position = [&](int r, int c) { return SPARSE ? own[c] : 4 * (r * SR_THREADS + tid) + c; };
    // over the wavefronts: one value of each in LDS, which every wavefront reduces for itself, a row of 16 lanes per range.
    // (All five by full reductions in both halves: 3500 cycles of the 15 000 of 4096 positions.)
    {
        uint32_t c = 0u;
        if (__ballot(spm)) {                                 // uniform; few wavefronts have a sponsored position
            c = wave_sum_dpp((uint32_t)__popc(spm));
            lo1 = wave_min_dpp(lo1);
            hi1 = wave_max_dpp(hi1);
        }
        // A lower bound of the cut: with at least as many groups of lanes as there are slots, the smallest of the groups' largest
        // keys.  What lies below it is not binned, and the bins are the finer for it.  (With two rounds or
        // fewer the bound costs what it saves; four: 16 384 positions, 512 of them kept, 16.2 -> 14.7 us; eight: 32 767 pooled, 35.4 -> 28.2.)
        if (PRUNE) {
            uint32_t g = hi0;
            if (K - c2 <= 4 * SR_WAVES) g = row_max_dpp(g);                  // uniform
            else if (K - c2 <= 16 * SR_WAVES) g = quad_max_dpp(g);
            const int step = K - c2 <= 4 * SR_WAVES ? 16 : K - c2 <= 16 * SR_WAVES ? 4 : 1;
            const unsigned long long live = __ballot(g != 0u && (lane & (step - 1)) == 0);
            g = wave_min_dpp(g == 0u ? 0xFFFFFFFFu : g);
            if (lane == 0) {
                L.bound[wave] = ~g;
                L.groups[wave] = (uint32_t)__popcll(live);
            }
        }
        lo0 = wave_min_dpp(lo0);
        hi0 = wave_max_dpp(hi0);
        if (lane == 0) {
            L.part[wave] = ~lo0;
            L.part[SR_WAVES + wave] = hi0;
            L.part[2 * SR_WAVES + wave] = ~lo1;
            L.part[3 * SR_WAVES + wave] = hi1;
            L.sponsored[wave] = c;
        }
    }
    __syncthreads();
    int32_t c1;
    {
        static_assert(SR_WAVES == 16, "a row of lanes per value");
        const uint32_t x = row_max_dpp(L.part[lane]);
        c1 = __builtin_amdgcn_readlane((int)row_sum_dpp(L.sponsored[lane & 15]), 0);
        lo0 = ~(uint32_t)__builtin_amdgcn_readlane((int)x, 0);
        hi0 = (uint32_t)__builtin_amdgcn_readlane((int)x, 16);
        lo1 = ~(uint32_t)__builtin_amdgcn_readlane((int)x, 32);
        hi1 = (uint32_t)__builtin_amdgcn_readlane((int)x, 48);
    }
    uint32_t near_cut = 0xFFFFFFFFu;                         // bits as in `mid`: not below the bound
    if (PRUNE) {
        const uint32_t bound = ~(uint32_t)__builtin_amdgcn_readlane((int)row_max_dpp(L.bound[lane & 15]), 0);
        const int32_t groups = __builtin_amdgcn_readlane((int)row_sum_dpp(L.groups[lane & 15]), 0);
        if (groups >= K - c2 && bound > lo0) {               // uniform
            lo0 = bound;
            near_cut = 0u;
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) near_cut |= key[r][c] >= bound ? 1u << (4 * r + c) : 0u;
        }
    }
    const int bclass = (c2 + c1 <= K) ? 0 : 1;
    const int32_t R = bclass == 0 ? K - c2 - c1 : K - c2;    // slots for the boundary class
    // fixed partition: P sponsored tokens are protected, M more slots go to the best of everything else
    int32_t P = 0;
    if (CAPPED) {
        P = a.k_protected < c1 ? a.k_protected : c1;
        P = P < K - c2 ? P : K - c2;
    }
    const int32_t M = K - c2 - P;

    // ---- the cut: among the positions of `members` (bits as above; values val(r, c) in [lo, hi]), a position is in the
    // top `need` iff value > T, or value == T and position >= Pt.  False: the cut falls among more than SR_CAND
    // members that all have the value T, and `need` of these are wanted.  The histogram is clear on entry.
    const auto search = [&](auto&& val, const uint32_t members, uint32_t lo, uint32_t hi, uint32_t& need, uint32_t& T,
                            int32_t& Pt) -> bool {
        for (bool first_level = true;; first_level = false) {
            const uint32_t d = hi - lo;
            const int shift = d < (uint32_t)SR_BINS ? 0 : 21 - __clz((int)d);    // d >> shift < SR_BINS
            int prev = -1;                                   // equal bins in a row go into the histogram as one add
            uint32_t run = 0;
            const auto put = [&]() {
                if (prev >= 0) atomicAdd(&L.hist[(prev & 31) * 65 + (prev >> 5)], run);
            };
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                if (r * SR_THREADS >= nquads) break;         // uniform
                if (__ballot((members >> (4 * r)) & 15u) == 0ull) continue;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t v = val(r, c);
                    if (first_level) {                       // uniform; every member lies in [lo, hi]
                        const int bin = ((members >> (4 * r + c)) & 1u) ? (int)((v - lo) >> shift) : -1;
                        if (bin != prev) {
                            put();
                            prev = bin;
                            run = 0;
                        }
                        ++run;
                        continue;
                    }
                    const int bin = ((members >> (4 * r + c)) & 1u) && v >= lo && v <= hi ? (int)((v - lo) >> shift) : -1;
                    if (bin != prev) {
                        put();
                        prev = bin;
                        run = 0;
                    }
                    ++run;
                }
            }
            put();
            __syncthreads();
            if (wave == 0) {
                // lane l owns the bins 32 (63 - l) .. + 31: the scan over lanes runs downwards through the values
                uint32_t mine = 0;
#pragma unroll
                for (int j = 0; j < 32; ++j) mine += L.hist[j * 65 + 63 - lane];
                const uint32_t incl = wave_scan_dpp(mine);
                const int first = __ffsll((long long)__ballot(incl >= need)) - 1;   // the lane whose bins hold the cut
                const uint32_t above = (uint32_t)__builtin_amdgcn_readlane((int)(incl - mine), first);
                // its 32 bins, one per lane, again from the largest down
                const uint32_t h = lane < 32 ? L.hist[(31 - lane) * 65 + 63 - first] : 0u;
                const uint32_t in2 = above + wave_scan_dpp(h);
                const int at = __ffsll((long long)__ballot(in2 >= need)) - 1;
                if (lane == at) {
                    L.st.bin = (uint32_t)(32 * (63 - first) + 31 - at);
                    L.st.need = need - (in2 - h);
                    L.st.count = h;
                    L.st.all = in2 == need ? 1u : 0u;
                }
            }
            __syncthreads();
            const uint32_t bin = L.st.bin, count = L.st.count, all = L.st.all;
            need = L.st.need;
            lo += bin << shift;
            hi = hi - lo < (1u << shift) - 1u ? hi : lo + ((1u << shift) - 1u);
            if (all) {                                       // everything from the bin's lower end up
                T = lo - 1u;
                Pt = 0x7FFFFFFF;
                return true;
            }
            if (count <= (uint32_t)SR_CAND) {
#pragma unroll
                for (int r = 0; r < ROUNDS; ++r) {
                    if (r * SR_THREADS >= nquads) break;
                    if (__ballot((members >> (4 * r)) & 15u) == 0ull) continue;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const uint32_t v = val(r, c);
                        if (((members >> (4 * r + c)) & 1u) && v >= lo && v <= hi) {
                            const uint32_t e = atomicAdd(&L.count, 1u);
                            L.cand[2 * e] = (uint32_t)position(r, c);
                            L.cand[2 * e + 1] = v;
                        }
                    }
                }
                __syncthreads();
                // a wavefront per candidate, the others in its lanes: a candidate's rank is the number of lanes that hold a larger one.
                // (A thread per candidate that walks through all of them: some 60 cycles for every one.)
                {
                    const unsigned long long* pairs = reinterpret_cast<const unsigned long long*>(L.cand);
                    unsigned long long held[SR_CAND / 64];
#pragma unroll
                    for (int k = 0; k < SR_CAND / 64; ++k) held[k] = 64 * k + lane < (int)count ? pairs[64 * k + lane] : 0ull;
                    for (uint32_t e = (uint32_t)wave; e < count; e += SR_WAVES) {
                        const unsigned long long one = pairs[e];
                        uint32_t rank = 0;
#pragma unroll
                        for (int k = 0; k < SR_CAND / 64; ++k)
                            if (64u * k < count) rank += (uint32_t)__popcll(__ballot(held[k] > one));    // uniform
                        if (lane == 0 && rank == need - 1u) {
                            L.st.key = (uint32_t)(one >> 32);
                            L.st.pos = (uint32_t)one;
                        }
                    }
                }
                if (tid == 0) L.count = 0u;
                __syncthreads();
                T = L.st.key;
                Pt = (int32_t)L.st.pos;
                return true;
            }
            __syncthreads();                                 // the state has been read
            for (int i = tid; i < 32 * 65; i += SR_THREADS) L.hist[i] = 0u;
            __syncthreads();
            if (shift == 0) {
                T = lo;
                return false;
            }
        }
    };
    const auto find_threshold = [&](const uint32_t members, uint32_t lo, uint32_t hi, uint32_t want, uint32_t& T, int32_t& Pt) {
        uint32_t need = want;
        const auto keys = [&](int r, int c) { return key[r][c]; };
        if (search(keys, members, lo, hi, need, T, Pt)) return;
        // many positions share the key T: the `need` highest of them are kept
        uint32_t same = 0u;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) same |= key[r][c] == T ? 1u << (4 * r + c) : 0u;
        uint32_t Tp = 0;
        int32_t unused = 0;
        const auto positions = [&](int r, int c) { return (uint32_t)position(r, c); };
        search(positions, members & same, 0u, (uint32_t)(nb - 1), need, Tp, unused);   // positions are unique: always found
        Pt = unused == 0x7FFFFFFF ? (int32_t)Tp + 1 : (int32_t)Tp;
    };

    uint32_t T = 0xFFFFFFFFu;     // a position that competes is kept iff key > T, or key == T and p >= Pt
    int32_t Pt = 0x7FFFFFFF;
    uint32_t always = 0u, compete;                           // retained whatever the ranking says; ranked
    if (!CAPPED) {
        compete = bclass ? spm : (mid & ~spm);
        always = bclass ? 0u : spm;
        if (R > 0) find_threshold(bclass ? compete : compete & near_cut, bclass ? lo1 : lo0, bclass ? hi1 : hi0, (uint32_t)R, T, Pt);
    } else {
        if (P == c1) always = spm;                           // every sponsored token is protected
        else if (P > 0) {
            uint32_t T1 = 0xFFFFFFFFu;
            int32_t Pt1 = 0x7FFFFFFF;
            find_threshold(spm, lo1, hi1, (uint32_t)P, T1, Pt1);
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int32_t p = 4 * (r * SR_THREADS + tid) + c;
                    const bool prot = key[r][c] > T1 || (key[r][c] == T1 && p >= Pt1);
                    always |= prot ? spm & (1u << (4 * r + c)) : 0u;
                }
            __syncthreads();
            for (int i = tid; i < 32 * 65; i += SR_THREADS) L.hist[i] = 0u;
            __syncthreads();
        }
        compete = mid & ~always;
        if (M > 0) find_threshold(compete, lo0 < lo1 ? lo0 : lo1, hi0 > hi1 ? hi0 : hi1, (uint32_t)M, T, Pt);   // more candidates than M remain: nb > K
    }

    // ---- what is retained, in ascending order: the counts of all rounds are scanned at once, two rounds to a register
    uint32_t keep = always;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        if (r * SR_THREADS >= nquads) break;                 // uniform
        const int32_t q = r * SR_THREADS + tid;
        if (__ballot((compete >> (4 * r)) & 15u)) {          // uniform
            uint32_t above = 0u, level = 0u;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                above |= key[r][c] > T ? 1u << c : 0u;
                level |= key[r][c] == T ? 1u << c : 0u;
            }
            if (level) {                                     // at the cut the position decides
#pragma unroll
                for (int c = 0; c < 4; ++c) above |= position(r, c) >= Pt ? level & (1u << c) : 0u;
            }
            keep |= (above << (4 * r)) & compete;
        }
        if (SPARSE || 4 * q < ns || 4 * q + 3 >= rs) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int32_t p = position(r, c);
                keep |= p < nb && (p < ns || p >= rs) ? 1u << (4 * r + c) : 0u;
            }
        }
    }
    uint32_t kept_min = 0xFFFFFFFFu, gone_max = 0u;          // keys at the cut, over this thread's candidates
    if (a.margin) {                                          // uniform
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t bit = 1u << (4 * r + c), k = key[r][c];
                kept_min = (compete & keep & bit) && k < kept_min ? k : kept_min;
                gone_max = (compete & ~keep & bit) && k > gone_max ? k : gone_max;
            }
    }
    constexpr int PAIRS = (ROUNDS + 1) / 2;
    uint32_t incl2[PAIRS];                                   // inclusive counts within the wavefront, rounds 2j and 2j + 1
#pragma unroll
    for (int j = 0; j < PAIRS; ++j) {
        uint32_t v = (uint32_t)__popc((keep >> (8 * j)) & 15u);
        if (2 * j + 1 < ROUNDS) v |= (uint32_t)__popc((keep >> (8 * j + 4)) & 15u) << 16;
        incl2[j] = wave_scan_dpp(v);                         // at most 256 per field: no carry between the halves
    }
    if (lane == 63) {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) L.totals[r * SR_WAVES + wave] = (incl2[r >> 1] >> (16 * (r & 1))) & 0xFFFFu;
    }
    if (a.margin) {                                          // uniform
        kept_min = wave_min_dpp(kept_min);
        gone_max = wave_max_dpp(gone_max);
        if (lane == 0) {
            L.edge[0][wave] = kept_min;
            L.edge[1][wave] = gone_max;
        }
    }
    __syncthreads();
    // every wavefront scans the ROUNDS * SR_WAVES totals for itself, two per lane
    const uint32_t t0 = 2 * lane < ROUNDS * SR_WAVES ? L.totals[2 * lane] : 0u;
    const uint32_t t1 = 2 * lane < ROUNDS * SR_WAVES ? L.totals[2 * lane + 1] : 0u;
    const uint32_t after = wave_scan_dpp(t0 + t1);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        if (r * SR_THREADS >= nquads) break;                 // uniform
        const int e = r * SR_WAVES + wave;                   // uniform in the wavefront
        const uint32_t upto = (uint32_t)__builtin_amdgcn_readlane((int)after, __builtin_amdgcn_readfirstlane(e >> 1));
        const uint32_t odd = (uint32_t)__builtin_amdgcn_readlane((int)t1, __builtin_amdgcn_readfirstlane(e >> 1));
        const uint32_t even = (uint32_t)__builtin_amdgcn_readlane((int)t0, __builtin_amdgcn_readfirstlane(e >> 1));
        const uint32_t before = upto - odd - ((e & 1) ? 0u : even);
        const uint32_t bits = (keep >> (4 * r)) & 15u;
        if (__ballot(bits) == 0ull) continue;
        const uint32_t incl = (incl2[r >> 1] >> (16 * (r & 1))) & 0xFFFFu;
        int32_t slot = (int32_t)(before + incl) - __popc(bits);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (bits & (1u << c)) {
                if (slot < K) {
                    idx[slot] = position(r, c);
                    if constexpr (GATHER != GATHER_NONE) L.hist[slot] = (uint32_t)position(r, c);
                }
                ++slot;
            }
        }
    }
    if (tid == 0) {
        const int32_t total = (int32_t)__builtin_amdgcn_readlane((int)after, 63);
        a.cnt[unit] = total < K ? total : K;
        if (a.margin) {
            for (int w = 0; w < SR_WAVES; ++w) {
                kept_min = L.edge[0][w] < kept_min ? L.edge[0][w] : kept_min;
                gone_max = L.edge[1][w] > gone_max ? L.edge[1][w] : gone_max;
            }
            a.margin[2 * (size_t)unit] = margin_value(kept_min);
            a.margin[2 * (size_t)unit + 1] = margin_value(gone_max);
        }
    }
    if constexpr (GATHER != GATHER_NONE) {
        // the positions lie in the histogram's memory, which the search has left behind
        const int32_t total = (int32_t)__builtin_amdgcn_readlane((int)after, 63);
        __syncthreads();
        gather_rows<SR_THREADS, GATHER>(g, unit, total < K ? total : K, L.hist, tid);
    }
    return true;
}

template <int ROUNDS, bool CAPPED, int GATHER>
__global__ void __launch_bounds__(SR_THREADS)
select_reg_kernel(SelectArgs a, std::conditional_t<GATHER != GATHER_NONE, CompactArgs, int> g)
{
    __shared__ __align__(16) SelectRegLds L;
    select_reg<ROUNDS, CAPPED, GATHER>(a, g, L, nullptr);
}

template <int ROUNDS, bool ASK>
__global__ void __launch_bounds__(SR_THREADS)
select_sparse_kernel(SelectArgs a)
{
    __shared__ __align__(16) SelectRegLds L;
    __shared__ __align__(16) SparseList list;
    if (!select_reg<1, false, GATHER_NONE, 1, ASK>(a, 0, L, &list)) {
        __syncthreads();
        select_reg<ROUNDS, false, GATHER_NONE>(a, 0, L, nullptr);
    }
}

// ---- streaming form: every input is read once, whatever the length ----------------------------
// One workgroup of four wavefronts per unit walks the sequence from its end in segments and keeps
// the best candidates of the boundary class seen so far in LDS as (key, position) pairs.  A
// position joins the list if it beats the current threshold - the R-th largest (key, position) at
// the last shrink, nothing before the first - and the list is cut back to its R best whenever the
// next segment might not fit (an MSD radix select over the LDS list, the same search as above).
// Walking from the end meets the recent positions first, whose recency term is largest: with a
// non-negative beta the threshold is high after the first shrink and few later positions pass it.
// The order of the walk and of the list only affect the time, never the result: the retained set
// is defined by the total order, and the output is written in ascending position order from a
// bitmap of the sequence (bits of the mandatory positions, of the sponsored ones when they are
// all kept, and of the final R candidates).
// What bounds it: instructions.  (Four segments in flight instead of two: 72.1 -> 75.9 us for 8 units of 131 072 positions; one barrier
// less per segment: 74.0.)  Hence straight-line code per position, one question per wavefront, one LDS addition for all that a
// wavefront adds, addresses of 32 bits: 8 units of 131 072 positions, budget 1024, 72.1 -> 65.3, 256 of them with budget 64 67.5 -> 54.0, 2048 of
// 16 384 78.1 -> 64.1, 2048 of 32 768 142.8 -> 129.0, 1024 of 60 000 130.1 -> 111.4, 2048 of 900 24.6 -> 24.0; scores max-pooled over 7: 8 of
// 131 072 102.3 -> 85.7, over 5: 16 of 85 059 62.4 -> 56.1, over 9: 1024 of 60 000 219.7 -> 186.3.
constexpr int SS_THREADS = 256;
constexpr int SS_BIG_THREADS = 1024;                       // few units with long rows: a workgroup has a compute unit to itself
constexpr int SS_SLACK = 256;                              // list entries beyond R + one segment: new entries between two cuts
constexpr int SS_DEPTH = 2;                                // segments whose operands are in flight
constexpr int SS_HIST_COPIES = 4;
constexpr int SS_MAX_PER_THREAD = 24;                      // list entries a thread holds while the list is compacted
constexpr int SS_FEW_PER_THREAD = 10;                      // ... in the instance for short lists (budgets up to about 1300)
constexpr int SS_BIG_PER_THREAD = 6;                       // ... in a workgroup of SS_BIG_THREADS
constexpr int SS_MAX_CAP = SS_THREADS * SS_MAX_PER_THREAD;
constexpr int SS_MAX_LDS = 144 * 1024;                     // dynamic LDS of a workgroup (list + bitmap)
// Which form runs: this one when a row does not fit the registers of the form above, and for many units, where its small
// workgroups fill the chip and end early on short rows; its cuts cost more with the budget.  us, register / streaming form (units x
// positions, budget):
//   below 1024 units the registers: 320 x 4096, 256 9.0 / 20.2; 512 x 32 768, 1024 41.7 / 55.5; 768 x 1000, 64 10.6 / 12.4, x 8192, 512 19.9 / 27.6,
//     x 16 384, 256 35.6 / 34.7, x 32 768, 1024 64.6 / 66.9.
//   more than 8192 positions, from 1024 units on this one: 1024 x 10 000, 256 44.5 / 28.7, x 32 768, 1024 89.3 / 73.3.
//   up to 8192 positions of one length, up to 1280 units: the registers.  1024 x 1000, 64 13.0 / 13.4, x 2000, 128 13.9 / 18.1, x 8192, 64
//     22.5 / 25.4; 1280 x 1500, 64 15.6 / 16.4, x 8192, 256 26.9 / 27.3; 1536 x 1000, 64 17.4 / 15.2, x 4000, 256 21.2 / 21.1; 2048 x 2048, 256 23.8 /
//     22.8; ragged from a quarter, 1024 x 4096, 256 16.5 / 15.0, x 8192 22.0 / 19.0.
//   budgets from 384 on: up to 2048 units of one length, 1024 of any (two workgroups to a compute unit: twice what runs at once).  2048 x 1000, 400 24.4 / 24.8, x 4096, 384 29.3 / 38.2, x 8192, 1024 43.6 / 59.2;
//     16 384 x 1000, 400 165 / 130, x 4000, 1024 218 / 268; ragged 1024 x 1000, 384 10.9 / 12.7, x 8192, 384 23.2 / 24.5, x 8192, 1024 23.8 / 28.4;
//     3072 x 4096, 512 50.4 / 46.2.
//   budgets from 640 on and rows of more than 2048 positions: up to 2048 units, ragged or not.  With the fills of the outputs, ragged from an
//     eighth: 1056 x 4096, 640 21.1 / 27.9, x 4096, 2048 20.1 / 34.2; 1536 x 8192, 640 36.5 / 37.4; 2048 x 3000, 1024 31.4 / 31.2, x 4096, 640
//     33.8 / 38.6, x 8192, 768 47.2 / 51.7; from a half: 1056 x 8192, 1024 33.6 / 47.0; 1536 x 8192, 640 39.3 / 40.7; 2048 x 4096, 1024 38.9 / 55.3; not
//     1536 x 2048, 768 28.1 / 25.1; 2048 x 2000, 512 35.2 / 34.4; 3072 x 4096, 640 56.3 / 57.4 and from an eighth 50.8 / 49.6.
//   (Ragged: lengths are given.  What they are the host does not know.)
// Long rows: sixteen wavefronts per unit up to 512 units (512 of 65 537: 97 us against 118 with four; 1024 of 40 001: 129 against 92,
// both before the walk lost its branches).
constexpr int64_t SS_MIN_UNITS = 1024;
bool registers_for_many(int64_t units, int32_t n, int32_t K, bool ragged)
{
    if (n > 8 * SR_THREADS) return false;
    if (K < 384) return units <= 1280 && !ragged;
    return units <= (!ragged || (K >= 640 && n > 2 * SR_THREADS) ? 2048 : 1024);
}
constexpr int64_t SS_BIG_MAX_UNITS = 512;

struct StreamLds {
    uint32_t hist[SS_HIST_COPIES][HIST_STRIDE];
    uint32_t h[256];
    int red[SS_BIG_THREADS / 64];
    RadixState state;
    uint32_t count;                                        // entries in the candidate list
};

// The same search as radix_pick, for SS_HIST_COPIES histograms.
__device__ __forceinline__ RadixState stream_pick(StreamLds& L, uint32_t need)
{
    const int tid = threadIdx.x;
    if (tid < 256) {
        uint32_t t = 0;
#pragma unroll
        for (int c = 0; c < SS_HIST_COPIES; ++c) {
            t += L.hist[c][tid];
            L.hist[c][tid] = 0;
        }
        L.h[tid] = t;
    }
    __syncthreads();
    if (tid < 64) {
        const uint32_t h0 = L.h[255 - 4 * tid], h1 = L.h[254 - 4 * tid];
        const uint32_t h2 = L.h[253 - 4 * tid], h3 = L.h[252 - 4 * tid];
        const uint32_t mine = h0 + h1 + h2 + h3;
        uint32_t incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t up = __shfl_up(incl, o);
            if (tid >= o) incl += up;
        }
        const unsigned long long m = __ballot(incl >= need);
        const int first = __ffsll((long long)m) - 1;
        if (tid == first) {
            uint32_t above = incl - mine;
            const uint32_t hs[4] = {h0, h1, h2, h3};
            RadixState r;
            r.digit = 0; r.need = 0; r.bin_count = 0; r.all_of_bin = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (above + hs[j] >= need) {
                    r.digit = (uint32_t)(255 - 4 * tid - j);
                    r.need = need - above;
                    r.bin_count = hs[j];
                    r.all_of_bin = (above + hs[j] == need) ? 1u : 0u;
                    break;
                }
                above += hs[j];
            }
            L.state = r;
        }
    }
    __syncthreads();
    return L.state;
}

// MARGIN: the keys turned away are tracked for the margin output; OPTS: max-pooled scores and the fixed partition, which walks
// the sequence a second time when it has to find the protected tokens first (instances of their own: the default
// ones keep their registers)
template <int THREADS, int PER_THREAD, bool MARGIN, bool OPTS>        // cap <= THREADS * PER_THREAD
__device__ __forceinline__ void select_stream(const SelectArgs& a, const int32_t cap)
{
    constexpr int WAVES = THREADS / 64;
    constexpr int SEG = THREADS * 4;                       // positions per segment
    extern __shared__ uint32_t s_dyn[];                    // [cap] keys, [cap] positions, [ceil(n / 32)] bitmap
    __shared__ StreamLds L;
    uint32_t* ckey = s_dyn;
    uint32_t* cpos = s_dyn + cap;
    uint32_t* bitmap = s_dyn + 2 * cap;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int32_t place = (int32_t)blockIdx.x;
    if (place >= a.units) return;
    const int32_t unit = __builtin_amdgcn_readfirstlane(unit_at(place, a.seq_len, a.batch, a.hkv, a.units));
    const int32_t b = (unit / a.hkv) % a.batch;
    const int32_t n = a.n;
    int32_t K = a.K;
    if (a.layer_K) {
        int32_t lo = a.n_sink + a.n_recent;
        lo = lo < 1 ? 1 : lo;
        const int32_t kl = a.layer_K[unit / (a.batch * a.hkv)];
        K = kl < lo ? lo : (kl > K ? K : kl);
    }
    int32_t nb = a.seq_len ? a.seq_len[b] : n;
    nb = nb < 0 ? 0 : (nb > n ? n : nb);
    int32_t* idx = a.idx + (size_t)unit * (size_t)a.K;
    if (nb <= K) {                                         // nothing to evict
        for (int32_t p = tid; p < nb; p += THREADS) idx[p] = p;
        if (tid == 0) {
            a.cnt[unit] = nb;
            if (a.margin) {
                a.margin[2 * (size_t)unit] = INFINITY;
                a.margin[2 * (size_t)unit + 1] = -INFINITY;
            }
        }
        return;
    }

    const float* A = a.A ? a.A + (size_t)unit * (size_t)n : nullptr;
    const size_t row = (size_t)b * (size_t)n;
    const uint8_t* anchor = a.anchor + row;
    const uint8_t* spons = a.spons + row;
    const float* vouch = a.vouch + row;
    const int32_t ns = a.n_sink < nb ? a.n_sink : nb;
    int32_t rs = nb - a.n_recent;
    rs = rs < ns ? ns : rs;
    const int32_t c2 = ns + (nb - rs);
    const int32_t nquads = (nb + 3) >> 2;    
    const bool use_A = (a.alpha != 0.0f);
    const int32_t words = (nb + 31) >> 5;

    struct Loaded {
        float4 A, v;
        uint32_t sp, an;
        float4 before[OPTS ? 1 : 0], after[OPTS ? 1 : 0];  // the neighbouring quads of A, for the max-pool
    };
    // unconditional loads (the quad index is clamped into the row, the caller masks what lies outside):
    // straight-line loads let the compiler wait for exactly the segment it needs
    const float* A_src = use_A ? A : vouch;                // no attention term: any readable row, the values are not used
    const auto load_quad = [&](int32_t q, Loaded& x) {
        q = q < 0 ? 0 : (q >= nquads ? nquads - 1 : q);
        const int32_t start = quad_start(4 * q, n);        // n >= 4 (the launcher)
        // (offsets of 32 bits from uniform addresses: rows of this form have a bitmap in LDS and are not that long)
        const uint32_t at = (uint32_t)start;
        x.sp = load_quad_b(spons + at, 0);
        x.an = load_quad_b(anchor + at, 0);
        x.v = load_quad_f(reinterpret_cast<const float*>(reinterpret_cast<const char*>(vouch) + 4u * at), 0);
        x.A = load_quad_f(reinterpret_cast<const float*>(reinterpret_cast<const char*>(A_src) + 4u * at), 0);
        if constexpr (OPTS) {
            if (a.pool_r > 0) {                            // uniform
                x.before[0] = load_quad_f(A_src, 4 * (q > 0 ? q - 1 : 0));
                x.after[0] = load_quad_f(A_src, quad_start(4 * q + 4, n));
            }
        }
    };

    // the first segments' operands are requested before anything else: they travel while the sponsored
    // positions are counted
    const int32_t nseg = (nquads + THREADS - 1) / THREADS;
    Loaded ring[SS_DEPTH];
#pragma unroll
    for (int d = 0; d < SS_DEPTH; ++d) load_quad((nseg - 1 - d) * THREADS + tid, ring[d]);


    for (int i = tid; i < SS_HIST_COPIES * HIST_STRIDE; i += THREADS) (&L.hist[0][0])[i] = 0;
    for (int32_t i = tid; i < words; i += THREADS) bitmap[i] = 0u;
    if (tid == 0) L.count = 0u;

    // ---- sponsored positions outside the mandatory ranges (16 flags per load) -------------------
    int local = 0;
    {
        const int32_t n16 = nb >> 4;
        typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
        const u32x4_any* sp16 = reinterpret_cast<const u32x4_any*>(spons);
        for (int32_t i = tid; i < n16; i += THREADS) {
            const u32x4_any f = sp16[i];
            const uint32_t w4[4] = {f[0], f[1], f[2], f[3]};
            const int32_t p0 = 16 * i;
            if (p0 >= ns && p0 + 15 < rs) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // a flag byte is 0 or not: count the non-zero bytes of the word
                    const uint32_t x = w4[j];
                    const uint32_t nz = ((x | (x >> 1) | (x >> 2) | (x >> 3) | (x >> 4) | (x >> 5) | (x >> 6) | (x >> 7)) & 0x01010101u);
                    local += __popc(nz);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int32_t p = p0 + j;
                    const uint32_t byte = (w4[j >> 2] >> (8 * (j & 3))) & 0xFFu;
                    local += (p >= ns && p < rs && byte) ? 1 : 0;
                }
            }
        }
        for (int32_t p = 16 * n16 + tid; p < nb; p += THREADS) local += (p >= ns && p < rs && spons[p]) ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) local += __shfl_xor(local, o);
    if (lane == 0) L.red[wave] = local;
    __syncthreads();                                       // also: histograms, bitmap and count are cleared
    int32_t c1 = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) c1 += L.red[w];

    const int bclass = (c2 + c1 <= K) ? 0 : 1;
    int32_t R = bclass == 0 ? K - c2 - c1 : K - c2;        // slots of the boundary class (more members than that exist)
    // fixed partition: P sponsored tokens are protected, K - c2 - P more slots go to the best of everything else
    const bool capped = OPTS && a.k_protected >= 0;
    int32_t P = 0;
    if (capped) {
        P = a.k_protected < c1 ? a.k_protected : c1;
        P = P < K - c2 ? P : K - c2;
    }
    uint32_t T1 = 0xFFFFFFFFu;                             // a sponsored position is protected iff key > T1, or key == T1 and p >= Pt1
    int32_t Pt1 = 0x7FFFFFFF;
    const float nf = (float)nb, inv = __fdiv_rn(1.0f, nf);

    auto key_of = [&](int32_t p, float Ap, uint32_t an, float v) -> uint32_t {
        const float r = div_by((float)(p + 1), nf, inv);
        float t = use_A ? __fmul_rn(a.alpha, Ap) : 0.0f;
        t = __fadd_rn(t, __fmul_rn(a.beta, r));
        t = __fadd_rn(t, __fmul_rn(a.gamma, an ? 1.0f : 0.0f));
        t = __fadd_rn(t, v);
        const uint32_t k = ordered_bits(t);
        return k == 0u ? 1u : k;
    };

    // ---- the list is cut back to its R best entries; returns their threshold -----------------------
    uint32_t T = 0u;              // a position joins the list iff key > T, or key == T and p >= Pt
    int32_t Pt = 0x7FFFFFFF;
    uint32_t gone_max = 0u;       // largest key this thread has turned away from the list or cut out of it
    const auto shrink = [&](const uint32_t m) {            // m: entries in the list (the same value in every thread)
        uint32_t prefix = 0, need = (uint32_t)R;
        uint32_t Tn = 0u;
        int32_t Pn = 0x7FFFFFFF;
        bool done = false;
        for (int pass = 0; pass < 4 && !done; ++pass) {
            const int shift = 24 - 8 * pass;
            for (uint32_t e = tid; e < m; e += THREADS) {
                const uint32_t k = ckey[e];
                const bool in = pass == 0 || (k >> (shift + 8)) == (prefix >> (shift + 8));
                if (in) atomicAdd(&L.hist[lane & (SS_HIST_COPIES - 1)][(k >> shift) & 255u], 1u);
            }
            __syncthreads();
            const RadixState r = stream_pick(L, need);
            prefix |= r.digit << shift;
            need = r.need;
            if (r.all_of_bin) {
                Tn = prefix - 1u;
                Pn = 0x7FFFFFFF;
                done = true;
            } else if (pass == 3) {
                Tn = prefix;
                const int bits = 32 - __clz(nb - 1);
                const int ppasses = (bits + 7) / 8;
                uint32_t pprefix = 0, pneed = need;
                for (int pp = 0; pp < ppasses; ++pp) {
                    const int ps = 8 * (ppasses - 1 - pp);
                    for (uint32_t e = tid; e < m; e += THREADS) {
                        const uint32_t p = cpos[e];
                        const bool in = ckey[e] == Tn && (pp == 0 || (p >> (ps + 8)) == (pprefix >> (ps + 8)));
                        if (in) atomicAdd(&L.hist[lane & (SS_HIST_COPIES - 1)][(p >> ps) & 255u], 1u);
                    }
                    __syncthreads();
                    const RadixState qs = stream_pick(L, pneed);
                    pprefix |= qs.digit << ps;
                    pneed = qs.need;
                }
                Pn = (int32_t)pprefix;
                done = true;
            }
        }
        // compaction in place: every thread takes its entries into registers, then the kept ones
        // are appended from slot 0 (exactly R of them; their order in the list does not matter)
        uint32_t mk[PER_THREAD], mp[PER_THREAD];
#pragma unroll
        for (int j = 0; j < PER_THREAD; ++j) {
            const uint32_t e = (uint32_t)tid + (uint32_t)j * THREADS;
            mk[j] = e < m ? ckey[e] : 0u;
            mp[j] = e < m ? cpos[e] : 0u;
        }
        if (tid == 0) L.count = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER_THREAD; ++j) {
            if ((uint32_t)j * THREADS >= m) continue;   // uniform: nothing of the list lies this far
            const bool keep = mk[j] > Tn || (mk[j] == Tn && mk[j] != 0u && (int32_t)mp[j] >= Pn);
            if (MARGIN && !keep) gone_max = mk[j] > gone_max ? mk[j] : gone_max;   // (0 beyond the list's end)
            const unsigned long long bal = __ballot(keep);
            uint32_t base = 0;
            if (lane == 0 && bal) base = atomicAdd(&L.count, (uint32_t)__popcll(bal));
            base = __shfl(base, 0);
            if (keep) {
                const uint32_t slot = base + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
                if (slot < (uint32_t)cap) {
                    ckey[slot] = mk[j];
                    cpos[slot] = mp[j];
                }
            }
        }
        __syncthreads();
        T = Tn;
        Pt = Pn;
    };

    // ---- the walk, from the last segment to the first; the operands of SS_DEPTH segments are in flight
    // (a segment is worked on in about a microsecond, a round trip under load takes several)
    for (int pool = OPTS ? 0 : 1; pool < 2; ++pool) {
        const bool protect = pool == 0;
        if constexpr (OPTS) {
            if (protect && !(capped && P > 0 && P < c1)) continue;         // uniform: nothing to find
            if (capped) R = protect ? P : K - c2 - P;
            if (!protect && capped && P > 0 && P < c1) {                   // the first walk's list is the protected pool
                T1 = T;
                Pt1 = Pt;
                const uint32_t m = L.count;
                for (uint32_t e = tid; e < m; e += THREADS) {
                    const uint32_t p = cpos[e];
                    atomicOr(&bitmap[p >> 5], 1u << (p & 31u));
                }
                __syncthreads();
                if (tid == 0) L.count = 0u;
                T = 0u;
                Pt = 0x7FFFFFFF;
                gone_max = 0u;
                __syncthreads();
#pragma unroll
                for (int d = 0; d < SS_DEPTH; ++d) load_quad((nseg - 1 - d) * THREADS + tid, ring[d]);
            }
        }
        for (int32_t top = nseg - 1; top >= 0; top -= SS_DEPTH) {
#pragma unroll
            for (int d = 0; d < SS_DEPTH; ++d) {
                const int32_t sg = top - d;
                const int32_t q = sg * THREADS + tid;
                uint32_t keys[4];
                bool join[4];
                uint32_t always = 0u;                          // bits of the quad that are retained whatever the ranking says
                {
                    Loaded x = ring[d];
                    if (n & 3) {                               // uniform
                        const int32_t by = q == nquads - 1 ? 4 * q - quad_start(4 * q, n) : 0;
                        x.sp >>= 8 * by;
                        x.an >>= 8 * by;
                        x.v = move_down(x.v, by);
                        x.A = move_down(x.A, by);
                    }
                    float Aq[4] = {x.A.x, x.A.y, x.A.z, x.A.w};
                    if constexpr (OPTS) {
                        if (a.pool_r > 0) {                    // uniform; window clipped to [0, nb)
                            const int32_t p4 = 4 * q + 4, by4 = p4 < n ? p4 - quad_start(p4, n) : 0;
                            const float4 after = move_down(x.after[0], by4);
                            float w12[12] = {x.before[0].x, x.before[0].y, x.before[0].z, x.before[0].w, Aq[0], Aq[1], Aq[2], Aq[3],
                                             after.x, after.y, after.z, after.w};
#pragma unroll
                            for (int j = 0; j < 12; ++j) {
                                if (j >= 4 && j < 8 && sg * SEG + SEG <= nb) continue;             // uniform: the segment's own lie in the row
                                if (4 * q - 4 + j < 0 || 4 * q - 4 + j >= nb) w12[j] = -INFINITY;
                            }
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                float m = w12[4 + c];
#pragma unroll
                                for (int e = 1; e <= 4; ++e)
                                    if (e <= a.pool_r) m = fmaxf(m, fmaxf(w12[4 + c - e], w12[4 + c + e]));
                                Aq[c] = m;
                            }
                        }
                    }
                    const float vq[4] = {x.v.x, x.v.y, x.v.z, x.v.w};
                    // Without the fixed partition no lane branches on its flags, which send the lanes of a wavefront every way; a segment between the
                    // mandatory ranges asks once per wavefront whether anything of it can join.
                    if (!capped && sg >= 0 && sg * SEG >= ns && (sg + 1) * SEG <= rs) {     // uniform
                        uint32_t best = 0u;
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const bool member = ((x.sp >> (8 * c)) & 0xFFu) != 0u ? bclass == 1 : bclass == 0;
                            keys[c] = member ? key_of(4 * q + c, Aq[c], (x.an >> (8 * c)) & 0xFFu, vq[c]) : 0u;
                            best = keys[c] > best ? keys[c] : best;
                            join[c] = false;
                        }
                        if (bclass == 0) always = byte_flags(x.sp);        // uniform: class 1 above the boundary class
                        if (__ballot(best != 0u && best >= T)) {           // uniform
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                join[c] = R > 0 && keys[c] != 0u && (keys[c] > T || (keys[c] == T && 4 * q + c >= Pt));
                                if (MARGIN) gone_max = !join[c] && keys[c] > gone_max ? keys[c] : gone_max;
                            }
                        } else if (MARGIN) {
                            gone_max = best > gone_max ? best : gone_max;
                        }
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const int32_t p = 4 * q + c;
                            const uint32_t sp = (x.sp >> (8 * c)) & 0xFFu, an = (x.an >> (8 * c)) & 0xFFu;
                            keys[c] = 0u;
                            join[c] = false;
                            if constexpr (!OPTS) {
                                const bool live = sg >= 0 && p < nb, fixed = p < ns || p >= rs, member = (sp != 0u) == (bclass == 1);
                                keys[c] = key_of(p, Aq[c], an, vq[c]);
                                join[c] = live && !fixed && member && R > 0 && (keys[c] > T || (keys[c] == T && p >= Pt));
                                always |= live && (fixed || (!member && sp != 0u)) ? 1u << c : 0u;     // class 1 above the boundary class
                                if (MARGIN) gone_max = live && !fixed && member && !join[c] && keys[c] > gone_max ? keys[c] : gone_max;
                            } else if (sg >= 0 && p < nb && q < nquads) {
                                if (p < ns || p >= rs) always |= 1u << c;
                                else if (capped) {
                                    keys[c] = key_of(p, Aq[c], an, vq[c]);
                                    bool member = sp != 0u;        // first walk: the protected pool
                                    if (!protect) {
                                        const bool prot = sp != 0u && (P == c1 || keys[c] > T1 || (keys[c] == T1 && p >= Pt1));
                                        member = !prot;
                                        always |= prot && P == c1 ? 1u << c : 0u;
                                    }
                                    join[c] = member && R > 0 && (keys[c] > T || (keys[c] == T && p >= Pt));
                                    if (MARGIN && member && !join[c]) gone_max = keys[c] > gone_max ? keys[c] : gone_max;
                                } else if ((sp != 0u) != (bclass == 1)) always |= (sp != 0u) ? (1u << c) : 0u;   // class 1 above the boundary class, class 0 below it
                                else if (MARGIN || R > 0) {
                                    keys[c] = key_of(p, Aq[c], an, vq[c]);
                                    join[c] = R > 0 && (keys[c] > T || (keys[c] == T && p >= Pt));
                                    if (MARGIN && !join[c]) gone_max = keys[c] > gone_max ? keys[c] : gone_max;
                                }
                            }
                        }
                    }
                }
                // the segment SS_DEPTH further on takes over the registers (past the first segment: a clamped
                // address whose data nobody uses)
                load_quad((sg - SS_DEPTH) * THREADS + tid, ring[d]);
                if (sg >= 0) {                                 // uniform
                    if (always) atomicOr(&bitmap[(4 * q) >> 5], always << ((4 * q) & 31));
                    unsigned long long bal[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) bal[c] = __ballot(join[c]);
                    if (bal[0] | bal[1] | bal[2] | bal[3]) {   // uniform
                        const uint32_t more = (uint32_t)(__popcll(bal[0]) + __popcll(bal[1]) + __popcll(bal[2]) + __popcll(bal[3]));
                        uint32_t base = 0;
                        if (lane == 0) base = atomicAdd(&L.count, more);
                        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            if (join[c]) {
                                const uint32_t slot = base + (uint32_t)__popcll(bal[c] & ((1ull << lane) - 1ull));
                                if (slot < (uint32_t)cap) {    // holds by construction: the list is cut back before it could overflow
                                    ckey[slot] = keys[c];
                                    cpos[slot] = (uint32_t)(4 * q + c);
                                }
                            }
                            base += (uint32_t)__popcll(bal[c]);
                        }
                    }
                    __syncthreads();                           // the segment's entries are in the list
                    const uint32_t m = L.count;
                    __syncthreads();                           // every thread has read the count before anyone adds to it again
                    // Cut back when the next segment might not fit, at the end (to exactly R), and once early: the
                    // first cut gives the threshold that keeps most later positions out of the list.
                    const bool early = T == 0u && m >= 2u * (uint32_t)R && m >= 512u;
                    if (R > 0 && ((sg > 0 && (m + (uint32_t)SEG > (uint32_t)cap || early)) || (sg == 0 && m > (uint32_t)R))) shrink(m);
                }
            }
        }
    }

    // ---- the final candidates join the bitmap; ascending write-out from it --------------------------
    {
        const uint32_t m = L.count;                        // == R (or 0)
        for (uint32_t e = tid; e < m; e += THREADS) {
            const uint32_t p = cpos[e];
            atomicOr(&bitmap[p >> 5], 1u << (p & 31u));
        }
    }
    __syncthreads();
    const int32_t wpt = (words + THREADS - 1) / THREADS;            // consecutive words per thread
    const int32_t w0 = tid * wpt;
    int mine = 0;
    for (int32_t w = w0; w < w0 + wpt && w < words; ++w) mine += __popc(bitmap[w]);
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
    }
    if (lane == 63) L.red[wave] = incl;
    __syncthreads();
    int woff = 0, total = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const int c = L.red[w];
        woff += (w < wave) ? c : 0;
        total += c;
    }
    int32_t slot = woff + incl - mine;
    for (int32_t w = w0; w < w0 + wpt && w < words; ++w) {
        uint32_t bits = bitmap[w];
        while (bits) {
            const int bit = __ffs((int)bits) - 1;
            bits &= bits - 1u;
            if (slot < K) idx[slot] = 32 * w + bit;
            ++slot;
        }
    }
    if (tid == 0) a.cnt[unit] = total < K ? total : K;
    if (MARGIN && a.margin) {                              // uniform
        uint32_t kept_min = 0xFFFFFFFFu;
        const uint32_t m = L.count;
        for (uint32_t e = tid; e < m; e += THREADS) kept_min = ckey[e] < kept_min ? ckey[e] : kept_min;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t lo = __shfl_xor(kept_min, o), hi = __shfl_xor(gone_max, o);
            kept_min = lo < kept_min ? lo : kept_min;
            gone_max = hi > gone_max ? hi : gone_max;
        }
        __syncthreads();                                   // the scan's partial sums have been read
        if (lane == 0) {
            L.h[wave] = kept_min;
            L.h[WAVES + wave] = gone_max;
        }
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                kept_min = L.h[w] < kept_min ? L.h[w] : kept_min;
                gone_max = L.h[WAVES + w] > gone_max ? L.h[WAVES + w] : gone_max;
            }
            a.margin[2 * (size_t)unit] = margin_value(kept_min);
            a.margin[2 * (size_t)unit + 1] = margin_value(gone_max);
        }
    }
}

// WPE: wavefronts per SIMD.  Short candidate lists (budgets up to about 1300): six, which the many short units of a ragged
// batch need to hide their round trips (up to six registers of the instance with the margin output go to scratch for it); long lists keep the registers.
template <int PER_THREAD, int WPE, bool MARGIN, bool OPTS>
__global__ void __launch_bounds__(SS_THREADS) __attribute__((amdgpu_waves_per_eu(WPE)))
select_stream_kernel(SelectArgs a, int32_t cap)
{
    select_stream<SS_THREADS, PER_THREAD, MARGIN, OPTS>(a, cap);
}

// Few units with long rows: 256 of them have a compute unit each, where four wavefronts walk 1024 positions at a time
// (256 rows of 131 072 positions: 203 us); sixteen walk 4096 (89 us).
template <bool MARGIN, bool OPTS>
__global__ void __launch_bounds__(SS_BIG_THREADS)
select_stream_big_kernel(SelectArgs a, int32_t cap)
{
    select_stream<SS_BIG_THREADS, SS_BIG_PER_THREAD, MARGIN, OPTS>(a, cap);
}

// Without an attention term: from a list as above; a row whose list does not hold what is flagged is walked.
template <bool ASK>
__global__ void __launch_bounds__(SS_BIG_THREADS)
select_sparse_long_kernel(SelectArgs a, int32_t cap)
{
    static_assert(SS_BIG_THREADS == SR_THREADS, "one workgroup for both");
    __shared__ __align__(16) SelectRegLds L;
    __shared__ __align__(16) SparseList list;
    if (!select_reg<1, false, GATHER_NONE, SR_LONG_SEGS, ASK>(a, 0, L, &list)) {
        __syncthreads();
        select_stream<SS_BIG_THREADS, SS_BIG_PER_THREAD, false, false>(a, cap);
    }
}

typedef void (*StreamKernel)(SelectArgs, int32_t);
// [margin]; the instances with options track the margin too
constexpr StreamKernel STREAM_FEW[2] = {select_stream_kernel<SS_FEW_PER_THREAD, 6, false, false>, select_stream_kernel<SS_FEW_PER_THREAD, 6, true, false>};
constexpr StreamKernel STREAM_LONG[2] = {select_stream_kernel<SS_MAX_PER_THREAD, 4, false, false>, select_stream_kernel<SS_MAX_PER_THREAD, 4, true, false>};
constexpr StreamKernel STREAM_BIG[2] = {select_stream_big_kernel<false, false>, select_stream_big_kernel<true, false>};
constexpr StreamKernel STREAM_SPARSE[2] = {select_sparse_long_kernel<false>, select_sparse_long_kernel<true>};   // [vouchers that may be anything]
constexpr int SS_SPARSE_LDS = SS_MAX_LDS - (int)(sizeof(SelectRegLds) + sizeof(SparseList));
constexpr StreamKernel STREAM_OPTS = select_stream_kernel<SS_MAX_PER_THREAD, 3, true, true>;
constexpr StreamKernel STREAM_BIG_OPTS = select_stream_big_kernel<true, true>;

DeviceOnce g_setup;

}  // namespace

hipError_t select_setup()
{
    return g_setup.run([](int) {
        hipError_t e = hipSuccess;
        for (StreamKernel k : {STREAM_FEW[0], STREAM_FEW[1], STREAM_LONG[0], STREAM_LONG[1], STREAM_BIG[0], STREAM_BIG[1], STREAM_OPTS, STREAM_BIG_OPTS})
            if (e == hipSuccess)
                e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, SS_MAX_LDS);
        for (StreamKernel k : {STREAM_SPARSE[0], STREAM_SPARSE[1]})
            if (e == hipSuccess)
                e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, SS_SPARSE_LDS);
        return e;
    });
}

hipError_t launch_select(const float* A, const uint8_t* anchor, const uint8_t* spons,
                         const float* vouch, const int32_t* seq_len,
                         int32_t layers, int32_t batch, int32_t hkv, int32_t n, int32_t K,
                         const ta_params& prm, int32_t* idx, int32_t* cnt, hipStream_t st, bool own_vouchers, const CompactArgs* job,
                         bool* gathered)
{
    if (gathered) *gathered = false;
    SelectArgs a;
    a.by_hkv = divider((uint32_t)hkv);
    a.by_batch = divider((uint32_t)batch);
    a.A = (prm.alpha != 0.0f) ? A : nullptr;
    a.anchor = anchor;
    a.spons = spons;
    a.vouch = vouch;
    a.seq_len = seq_len;
    a.layer_K = prm.layer_K;
    a.pool_r = (prm.alpha != 0.0f && prm.pool_k > 1) ? (prm.pool_k - 1) / 2 : 0;
    a.k_protected = prm.k_protected;
    a.idx = idx;
    a.cnt = cnt;
    a.margin = prm.margin;
    a.batch = batch;
    a.hkv = hkv;
    a.n = n;
    a.K = K;
    a.n_sink = prm.n_sink;
    a.n_recent = prm.n_recent;
    a.alpha = prm.alpha;
    a.beta = prm.beta;
    a.gamma = prm.gamma;
    const int64_t units = (int64_t)layers * batch * hkv;
    a.units = (int32_t)units;
    a.vec_ok = (n % 4 == 0) && ((uintptr_t)anchor % 4 == 0) && ((uintptr_t)spons % 4 == 0) &&
               ((uintptr_t)vouch % 16 == 0) && (a.A == nullptr || (uintptr_t)a.A % 16 == 0);
    const unsigned blocks = (unsigned)units;
    const bool capped = prm.k_protected >= 0;
    // The streaming form serves the selection when its candidate list and the bitmap of the sequence fit the LDS of a
    // workgroup (with options only rows that the register form cannot hold).
    const bool opts = capped || a.pool_r > 0;
    const bool list = a.alpha == 0.0f && !capped && !a.margin && a.beta >= 0.0f && a.gamma >= 0.0f;
    if (n >= 4 && (n > SR_MAX_N || (units >= SS_MIN_UNITS && !opts && !registers_for_many(units, n, K, seq_len != nullptr)))) {
        const int64_t rmax = (int64_t)K - prm.n_sink - prm.n_recent;      // most slots the boundary class can have
        const auto list_cap = [&](int threads) { return (rmax + 4 * threads + SS_SLACK + threads - 1) / threads * threads; };
        const auto lds_of = [&](int64_t cap) { return cap * 8 + ((int64_t)n + 31) / 32 * 4; };
        const int64_t big_cap = list_cap(SS_BIG_THREADS), cap = list_cap(SS_THREADS);
        const bool big = units <= SS_BIG_MAX_UNITS && big_cap <= SS_BIG_THREADS * SS_BIG_PER_THREAD && lds_of(big_cap) <= SS_MAX_LDS;
        if (big || (cap <= SS_MAX_CAP && lds_of(cap) <= SS_MAX_LDS)) {
            const hipError_t attr_err = select_setup();
            if (attr_err != hipSuccess) return attr_err;
            const bool few = cap <= SS_THREADS * SS_FEW_PER_THREAD;
            const int m = a.margin ? 1 : 0;
            const bool from_list = list && big && n > SR_MAX_N && n <= SR_LONG_SEGS * SR_SEG && lds_of(big_cap) <= SS_SPARSE_LDS;
            const StreamKernel kernel = from_list ? STREAM_SPARSE[own_vouchers ? 0 : 1] : opts ? (big ? STREAM_BIG_OPTS : STREAM_OPTS) : big ? STREAM_BIG[m] : few ? STREAM_FEW[m] : STREAM_LONG[m];
            const int64_t c = big ? big_cap : cap;
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(big ? SS_BIG_THREADS : SS_THREADS), (size_t)lds_of(c), st, a, (int32_t)c);
            return hipGetLastError();
        }
    }
    if (n <= SR_MAX_N) {
        const auto run = [&](auto capped_tag, auto kind_tag, auto g) {
            constexpr bool CAPPED = decltype(capped_tag)::value;
            constexpr int KIND = decltype(kind_tag)::value;
            auto kernel = n <= 4 * SR_THREADS ? select_reg_kernel<1, CAPPED, KIND> : n <= 8 * SR_THREADS ? select_reg_kernel<2, CAPPED, KIND>
                          : n <= 16 * SR_THREADS ? select_reg_kernel<4, CAPPED, KIND> : select_reg_kernel<8, CAPPED, KIND>;
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(SR_THREADS), 0, st, a, g);
        };
        const std::false_type plain{};
        // From a list: see SparseList.  Not a row of one round, which is as quick as its list; vouchers that have to be asked cost a pass over
        // them, which pays from more than 8192 positions on.  The kernel in us, every position / list: 4096 5.4 / 5.9, 4 x 6000 7.3 / 6.5,
        // 16 384 12.2 / 7.1, 4 x 32 768 18.9 / 8.6; with vouchers asked: 4096 5.5 / 8.6, 8192 8.8 / 9.3, 9000 10.4 / 8.4, 16 384 12.2 / 8.9,
        // 4 x 32 768 18.9 / 10.8.  Rows beyond the registers (above), the walk / list: 4 x 131 072 71.6 / 14.3; with vouchers asked 40 000
        // 31.3 / 15.3, 4 x 131 072 71.6 / 21.7.  Whole pass, one sequence of 131 072 positions in 32 layers, budget 256: 89.5 / 32.2.
        // A row with more flagged positions than the list holds is taken as a whole after all, and pays for finding that out: of 8192 positions
        // 0.4 us, 16 384 1.0, 32 768 2.0; with vouchers asked 9000 and 16 384 1.5, 32 768 3.1 (3.4 and 5.0 with the vouchers read in front of
        // the count; 4 x 131 072, whole call, 87.0 -> 78.8).  (Of more than 16 384 positions four to eight registers are then in scratch.)
        if (list && n > (own_vouchers ? 4 : 8) * SR_THREADS) {
            const auto sparse = own_vouchers ? (n <= 8 * SR_THREADS    ? select_sparse_kernel<2, false>
                                                : n <= 16 * SR_THREADS ? select_sparse_kernel<4, false>
                                                                       : select_sparse_kernel<8, false>)
                                             : (n <= 16 * SR_THREADS ? select_sparse_kernel<4, true> : select_sparse_kernel<8, true>);
            hipLaunchKernelGGL(sparse, dim3(blocks), dim3(SR_THREADS), 0, st, a);
            return hipGetLastError();
        }
        const bool fits = job && !capped && !(job->table && job->Kin_l) && gathers_here(units, K);
        if (fits) {
            *gathered = true;
            if (job->table) run(plain, std::integral_constant<int, GATHER_PAGED>{}, *job);
            else if (job->Kin_l) run(plain, std::integral_constant<int, GATHER_LAYERED>{}, *job);
            else run(plain, std::integral_constant<int, GATHER_DENSE>{}, *job);
        } else if (capped) run(std::true_type{}, std::integral_constant<int, GATHER_NONE>{}, 0);
        else run(plain, std::integral_constant<int, GATHER_NONE>{}, 0);
    } else {
        if (capped) hipLaunchKernelGGL(select_kernel<true>, dim3(blocks), dim3(SEL_THREADS), 0, st, a);
        else hipLaunchKernelGGL(select_kernel<false>, dim3(blocks), dim3(SEL_THREADS), 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace ta
