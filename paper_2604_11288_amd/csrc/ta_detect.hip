// Learned anchor detection (Sec. 5.1 "Learned Anchor Detection"): per position the confidence
//   f(h) = sigmoid(W2 . GELU(W1 . h))
// of a small two-layer perceptron on the hidden state, the anchor flag f(h) > thr and the
// per-anchor sponsor budget of TA-Learned (fixed B) or TA-LearnRank (scale * f(h)).
//
// The first layer is a [positions x d_model] x [d_model x m] contraction on the matrix cores (bf16 MFMA,
// fp32 accumulation).  It is computed as W1 . h^T, so that an accumulator tile has hidden units as rows and
// positions as columns: GELU, the product with W2 and the sum over the hidden units then stay with one
// position.  h and W1 stream through LDS, 64 input features (one 128-byte line per row) at a time, by direct
// global->LDS loads ahead of their use, 16-byte chunks XOR-swizzled by row for conflict-free fragment reads.
// Two forms (below), by the number of positions: one wavefront per share of the features for few positions,
// shared slices for many.  W1 is re-read by every workgroup (from the L2: it is at most 16 MB, 1 MB for the
// usual d_model = 4096, m = 128).
//
// The same kernels, in their second mode, are the embedding-based detector (Sec. 3.2 "Anchor detection",
// third instantiation; TA-Fast-Embedding): W1 holds the anchor-concept embeddings, the contraction
// gives every dot product x . c_e, the squared norms of both operands are summed from the very
// fragments the MFMA consumes (v_dot2_f32_bf16), and the epilogue takes the largest cosine and
// compares it with the threshold.
#include <math.h>

#include "ta_internal.h"
#include "ta_score_common.h"

namespace ta {

namespace {

constexpr int DT_KS = 64;                        // input features per slice

struct DetectArgs {
    const uint4* h;
    const uint4* W1;
    const uint16_t* W2;
    const int32_t* seq_len;
    float* conf;
    uint8_t* anchor;
    float* anchor_B;
    int64_t total;                               // batch * n positions
    int32_t n, dm, m;
    int32_t wrows;                               // rows W1 really has (<= m; the tile repeats the last one)
    int32_t h_row_bytes;                         // bytes between consecutive positions
    float thr, B, scale;
    int32_t rank;
};

// Direct global->LDS load, 16 bytes per lane, lane i lands at lds_base + 16 i (inline assembly so that the compiler does not wait
// for all of them before every LDS read).  STREAM: with the non-temporal hint.
template <bool STREAM = false>
__device__ __forceinline__ void dma16(const void* base, uint32_t off, uint32_t lds_base)
{
    if constexpr (STREAM)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :
                     : "s"(lds_base), "v"(off), "s"(base)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(lds_base), "v"(off), "s"(base)
                     : "memory", "m0");
}

constexpr int vm_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// erf(x) by the rational-exponential formula 7.1.26 of Abramowitz and Stegun,
//   erf(x) = sign(x) (1 - (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) exp(-x^2)),  t = 1 / (1 + p |x|),
// whose absolute error stays below 1.5e-7: the size of an fp32 rounding of the 1 + erf it feeds, at a
// third of the instructions of the library routine and without branches (the epilogue evaluates it
// 128 times per lane while the workgroup streams nothing).
__device__ __forceinline__ float erf_poly(float x)
{
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
    float poly = fmaf(1.061405429f, t, -1.453152027f);
    poly = fmaf(poly, t, 1.421413741f);
    poly = fmaf(poly, t, -0.284496736f);
    poly = fmaf(poly, t, 0.254829592f);
    poly *= t;
    const float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * ax * ax);
    return copysignf(fmaf(-poly, e, 1.0f), x);
}

// acc + sum of the squares of the eight bf16 values of a fragment (fp32)
__device__ __forceinline__ float add_squares(uint4 v, float acc)
{
    union { uint32_t u; bf16x2 b; } c;
    c.u = v.x; acc = __builtin_amdgcn_fdot2_f32_bf16(c.b, c.b, acc, false);
    c.u = v.y; acc = __builtin_amdgcn_fdot2_f32_bf16(c.b, c.b, acc, false);
    c.u = v.z; acc = __builtin_amdgcn_fdot2_f32_bf16(c.b, c.b, acc, false);
    c.u = v.w; acc = __builtin_amdgcn_fdot2_f32_bf16(c.b, c.b, acc, false);
    return acc;
}

enum { MODE_MLP = 0, MODE_COSINE = 1 };

// The order in which a wavefront visits its `steps` steps over the features.  Rows lie a power of two apart more often than not, so workgroups that
// all begin at feature 0 read the same offset within their rows at the same time and crowd a few memory channels.  So the steps lie in 2^log
// parts, and neighbouring workgroups begin with different ones.  The sums of a part start from zero, and the parts' sums are added
// up as a balanced tree (close_part).  A workgroup visits part (start ^ i) as the i-th: whatever its start, the same pairs of the tree meet, with at most
// their operands exchanged, so a row's result does not depend, to the last bit, on where the row stands in the call.  (A start that wraps
// round, each workgroup's another, spreads the reads further but adds up in as many orders.)
// us, all at feature 0 / parts / wrapping starts, d_model 4096: 128 256 rows, 16 concepts, four parts 187 / 150 = 7.0 TB/s / 148; 131 072 positions,
// 128 units, four parts 236 / 192 / 190, 32 768 62 / 57 / 52; 32 units, eight parts 187 / 174 / 171; d_model 2048, 131 072 positions, four parts, 128 units
// 130 / 121 / 99, 64 units 108 / 104 / 101, 32 units 101 / 91 / 92.  Where the wavefronts' parts begin 2 or 4 KB apart and W1 counts as much as h, they crowd the channels
// of the L2 in turn: 64 units with four wavefronts, four parts 235 for 213 at feature 0 (steps dealt out one by one 200, but d_model 2048 22 for 18), so in
// order; 128 units, two parts 402.  Rows that are no multiple of 4 KB apart gain nothing (d_model 3072, 131 072 positions of 32 units 139 / 144).
struct Visit {
    int steps, chunk, parts, base, start, part, at, left;  // at: this step; left: steps of its part, with this one
    // The parts [base, base + parts) of 2^log.  (Workgroup b runs on XCD b mod 8: neighbours of an XCD start at different parts.)
    __device__ __forceinline__ Visit(int n, int log, int of = 1, int share = 0)
        : steps(n), chunk((n + (1 << log) - 1) >> log), parts((1 << log) / of), base(share * parts), start((int)(blockIdx.x >> 3) & (parts - 1)), part(0)
    {
        open();
    }
    __device__ __forceinline__ int steps_in(int first, int count) const    // of that many parts that follow each other
    {
        const int rest = steps - first * chunk, most = count * chunk;
        return rest < 0 ? 0 : (rest > most ? most : rest);
    }
    __device__ __forceinline__ int total() const { return steps_in(base, parts); }
    __device__ __forceinline__ void open()
    {
        at = (base + (start ^ part)) * chunk;
        left = steps_in(base + (start ^ part), 1);
    }
    __device__ __forceinline__ void step()
    {
        ++at;
        --left;
    }
    __device__ __forceinline__ bool last() const { return part + 1 == parts; }
    __device__ __forceinline__ void to_full()              // on to a part that has steps left, if there is one
    {
        while (left == 0 && !last()) {
            ++part;
            open();
        }
    }
};

// The end of a part: level l of the tree holds the sums of 2^(l + 1) parts, and behind the last part the accumulators get its top.
template <int LOG, int N, typename T>
__device__ __forceinline__ void close_part(const Visit& v, T (&acc)[N], T (&tree)[LOG ? LOG : 1][N])
{
    if constexpr (LOG > 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            tree[0][j] += acc[j];
            acc[j] = T{};
        }
#pragma unroll
        for (int l = 1; l < LOG; ++l) {
            if ((v.part + 1) & ((1 << l) - 1)) break;      // uniform
#pragma unroll
            for (int j = 0; j < N; ++j) {
                tree[l][j] += tree[l - 1][j];
                tree[l - 1][j] = T{};
            }
        }
        if (v.last())
#pragma unroll
            for (int j = 0; j < N; ++j) acc[j] = tree[LOG - 1][j];
    }
}

// ---- shared form: the wavefronts of a workgroup share every slice ---------------------------------------
// TW: wavefront rows over the positions (64 TW positions per workgroup); HT: 32-unit hidden tiles
// per wavefront; MH: wavefront columns over the hidden units (m = 32 HT MH); MODE: which epilogue; DT_RING: slice
// buffers, loads run DT_RING - 1 slices ahead; STREAM: see launch_hint; LOG: see Visit
template <int TW, int HT, int MH, int MODE, int DT_RING, bool STREAM, int LOG>
__global__ void __launch_bounds__(64 * TW * MH, 2)
detect_kernel(DetectArgs a)
{
    constexpr int DT_TOKENS = 64 * TW;
    constexpr int THREADS = 64 * TW * MH;
    constexpr int M = 32 * HT * MH;
    constexpr int WAVES = TW * MH;
    constexpr int NI_H = DT_TOKENS / 8;                    // 1 KB loads per slice: h (8 rows each)
    constexpr int NI_W = M / 8;                            //                      W1
    constexpr int LH = NI_H / WAVES;                       // per wavefront
    constexpr int LW = (NI_W + WAVES - 1) / WAVES;         // (wraps: a few duplicate loads when M is small)
    constexpr int LPS = LH + LW;
    constexpr int H_BYTES = DT_TOKENS * 128;               // bytes of the h part of a buffer
    constexpr int BUF_BYTES = H_BYTES + M * 128;

    extern __shared__ uint4 s_buf[];                       // DT_RING buffers, then W2 as floats
    float* s_w2 = reinterpret_cast<float*>(reinterpret_cast<char*>(s_buf) + DT_RING * BUF_BYTES);
    float* s_part = s_w2 + M;                              // [MH][DT_TOKENS] partial sums over hidden units
    float* s_xx = s_part + MH * DT_TOKENS;                 // [DT_TOKENS] squared norms of the positions' rows

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c32 = lane & 31, hf = lane >> 5;
    const int tw = wave % TW, mh = wave / TW;              // position block of 64, hidden column
    const int64_t tile0 = (int64_t)blockIdx.x * DT_TOKENS;
    const int nstages = (a.dm + DT_KS - 1) / DT_KS;        // (the last slice may be half)

    if constexpr (MODE == MODE_MLP)
        for (int j = tid; j < M; j += THREADS) s_w2[j] = bf16_bits_to_float(a.W2[j]);

    // per-lane byte offsets of this wavefront's loads inside a slice (loop invariant)
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4*)s_buf;
    uint32_t off_h[LH], off_w[LW];
    int ins_h[LH], ins_w[LW];
#pragma unroll
    for (int j = 0; j < LH; ++j) {
        const int ins = wave + WAVES * j;
        const int row = ins * 8 + (lane >> 3);
        int64_t t = tile0 + row;
        t = t < a.total ? t : a.total - 1;                 // stay inside the tensor; never stored
        const int chunk = (lane & 7) ^ (row & 7);
        off_h[j] = (uint32_t)((t - tile0) * a.h_row_bytes + chunk * 16);
        ins_h[j] = ins;
    }
#pragma unroll
    for (int j = 0; j < LW; ++j) {
        const int ins = (wave + WAVES * j) % NI_W;
        const int row = ins * 8 + (lane >> 3);
        const int chunk = (lane & 7) ^ (row & 7);
        const int src_row = row < a.wrows ? row : a.wrows - 1;   // missing rows repeat the last one
        off_w[j] = (uint32_t)(src_row * a.dm * 2 + chunk * 16);
        ins_w[j] = ins;
    }
    const uint32_t half_back = ((lane & 7) ^ (lane >> 3)) >= 4 ? 64u : 0u;   // half a slice: the second half repeats the first
    const char* hbase = reinterpret_cast<const char*>(a.h) + tile0 * a.h_row_bytes;
    const char* wbase = reinterpret_cast<const char*>(a.W1);
    Visit ahead(nstages, LOG), now = ahead;                // the slice to request, the slice to work on
    ahead.to_full();
    const auto issue = [&](int i) {
        const uint32_t dst = lds0 + (uint32_t)(i % DT_RING) * BUF_BYTES;
        const int s = ahead.at;
        ahead.step();
        ahead.to_full();
        const char* hs = hbase + (size_t)s * (DT_KS * 2);
        const char* ws = wbase + (size_t)s * (DT_KS * 2);
        const uint32_t back = s * DT_KS + 32 >= a.dm ? half_back : 0u;
#pragma unroll
        for (int j = 0; j < LH; ++j) dma16<STREAM>(hs, off_h[j] - back, __builtin_amdgcn_readfirstlane(dst + ins_h[j] * 1024));
#pragma unroll
        for (int j = 0; j < LW; ++j)
            dma16(ws, off_w[j] - back, __builtin_amdgcn_readfirstlane(dst + H_BYTES + ins_w[j] * 1024));
    };
    const auto wait_but = [](int k) {                      // at most k later slices outstanding
        switch (k) {
            case 0: __builtin_amdgcn_s_waitcnt(vm_imm(0)); break;
            case 1: __builtin_amdgcn_s_waitcnt(vm_imm(LPS)); break;
            default: __builtin_amdgcn_s_waitcnt(vm_imm(2 * LPS)); break;
        }
    };
    static_assert(2 * LPS <= 63, "vmcnt range");

#pragma unroll
    for (int s = 0; s < DT_RING - 1; ++s)
        if (s < nstages) issue(s);

    // fragment slots of this lane inside a buffer (16-byte units), for the four MFMA steps of a slice
    int slot_h[2][4], slot_w[HT][4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const int row = 64 * tw + 32 * tt + c32;
            slot_h[tt][ks] = row * 8 + ((2 * ks + hf) ^ (row & 7));
        }
#pragma unroll
        for (int ht = 0; ht < HT; ++ht) {
            const int row = 32 * (mh * HT + ht) + c32;
            slot_w[ht][ks] = H_BYTES / 16 + row * 8 + ((2 * ks + hf) ^ (row & 7));
        }
    }

    f32x16 acc[2][HT];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int ht = 0; ht < HT; ++ht)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[tt][ht][i] = 0.0f;
    float xx[2] = {0.0f, 0.0f}, cc[HT];                    // cosine mode: squared norms, this lane's half of each row
#pragma unroll
    for (int ht = 0; ht < HT; ++ht) cc[ht] = 0.0f;
    f32x16 acc_tree[2][LOG ? LOG : 1][HT] = {};
    float xx_tree[LOG ? LOG : 1][2] = {}, cc_tree[LOG ? LOG : 1][HT] = {};

    int s = 0;
    for (;;) {
        for (; now.left > 0; now.step(), ++s) {
            const int later = nstages - 1 - s;
            wait_but(later < DT_RING - 2 ? later : DT_RING - 2);
            __syncthreads();                                   // slice s landed everywhere, slice s-1 consumed
            if (s + DT_RING - 1 < nstages) issue(s + DT_RING - 1);
            const uint4* buf = s_buf + (size_t)(s % DT_RING) * (BUF_BYTES / 16);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if (ks == 2 && now.at * DT_KS + 32 >= a.dm) break;   // uniform
                uint4 hraw[2], wraw[HT];
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) hraw[tt] = buf[slot_h[tt][ks]];
#pragma unroll
                for (int ht = 0; ht < HT; ++ht) wraw[ht] = buf[slot_w[ht][ks]];
                if constexpr (MODE == MODE_COSINE) {
#pragma unroll
                    for (int tt = 0; tt < 2; ++tt) xx[tt] = add_squares(hraw[tt], xx[tt]);
#pragma unroll
                    for (int ht = 0; ht < HT; ++ht) cc[ht] = add_squares(wraw[ht], cc[ht]);
                }
                bf16x8 hfrag[2], wfrag[HT];
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) hfrag[tt] = as_frag(hraw[tt]);
#pragma unroll
                for (int ht = 0; ht < HT; ++ht) wfrag[ht] = as_frag(wraw[ht]);
#pragma unroll
                for (int ht = 0; ht < HT; ++ht)
#pragma unroll
                    for (int tt = 0; tt < 2; ++tt)   // rows: hidden units of the tile, columns: positions
                        acc[tt][ht] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfrag[ht], hfrag[tt], acc[tt][ht], 0, 0, 0);
            }
        }
        if constexpr (LOG == 0) break;
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) close_part<LOG>(now, acc[tt], acc_tree[tt]);
        if constexpr (MODE == MODE_COSINE) {
            close_part<LOG>(now, xx, xx_tree);
            close_part<LOG>(now, cc, cc_tree);
        }
        if (now.last()) break;
        ++now.part;
        now.open();
    }

    if constexpr (MODE == MODE_MLP) {
        // ---- epilogue: GELU, weights of the output unit, sum over the hidden units -----------
        // acc[tt][ht][i] is hidden unit 32 (mh HT + ht) + 8 (i / 4) + 4 hf + i % 4 of position 64 tw + 32 tt + c32
        float part[2];
    #pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            float sum = 0.0f;
    #pragma unroll
            for (int ht = 0; ht < HT; ++ht) {
    #pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    asm volatile("" ::: "memory");             // the weights are read where they are used, not all up front
                    const float4 w = *reinterpret_cast<const float4*>(&s_w2[32 * (mh * HT + ht) + 8 * i4 + 4 * hf]);
                    const float wv[4] = {w.x, w.y, w.z, w.w};
    #pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float z = acc[tt][ht][4 * i4 + c];
                        const float gelu = 0.5f * z * (1.0f + erf_poly(z * 0.70710678118654752f));
                        sum = fmaf(wv[c], gelu, sum);
                        asm volatile("" : "+v"(sum));          // consume each value now: no pile-up of live erf results
                    }
                }
            }
            sum += __shfl_xor(sum, 32);                        // the two half-waves hold disjoint hidden units
            part[tt] = sum;
        }
        if (hf == 0) {
    #pragma unroll
            for (int tt = 0; tt < 2; ++tt) s_part[mh * DT_TOKENS + 64 * tw + 32 * tt + c32] = part[tt];
        }
        __syncthreads();
        if (tid < DT_TOKENS) {                                 // THREADS >= DT_TOKENS
            const int64_t t = tile0 + tid;
            if (t < a.total) {
                float out = s_part[tid];
    #pragma unroll
                for (int c = 1; c < MH; ++c) out += s_part[c * DT_TOKENS + tid];
                float conf = 1.0f / (1.0f + expf(-out));
                if (a.seq_len) {
                    const int64_t b = t / a.n;
                    if ((int32_t)(t - b * a.n) >= a.seq_len[b]) conf = 0.0f;   // past the end of its sequence
                }
                const bool is_anchor = conf > a.thr;
                a.conf[t] = conf;
                a.anchor[t] = is_anchor ? 1 : 0;
                a.anchor_B[t] = is_anchor ? (a.rank ? a.scale * conf : a.B) : 0.0f;
            }
        }
    } else {
        // ---- epilogue: largest cosine --------------------------------------------------------
        // reciprocal norms of this wavefront column's concept rows, through LDS (s_w2 is free in this mode)
#pragma unroll
        for (int ht = 0; ht < HT; ++ht) {
            const float c2 = cc[ht] + __shfl_xor(cc[ht], 32);
            if (hf == 0 && tw == 0) s_w2[32 * (mh * HT + ht) + c32] = c2 > 0.0f ? 1.0f / sqrtf(c2) : 0.0f;
        }
        __syncthreads();
        float best[2];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            float b = -INFINITY;
#pragma unroll
            for (int ht = 0; ht < HT; ++ht)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const float4 w = *reinterpret_cast<const float4*>(&s_w2[32 * (mh * HT + ht) + 8 * i4 + 4 * hf]);
                    b = fmaxf(b, acc[tt][ht][4 * i4 + 0] * w.x);
                    b = fmaxf(b, acc[tt][ht][4 * i4 + 1] * w.y);
                    b = fmaxf(b, acc[tt][ht][4 * i4 + 2] * w.z);
                    b = fmaxf(b, acc[tt][ht][4 * i4 + 3] * w.w);
                }
            best[tt] = fmaxf(b, __shfl_xor(b, 32));
            xx[tt] += __shfl_xor(xx[tt], 32);
        }
        if (hf == 0) {
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                s_part[mh * DT_TOKENS + 64 * tw + 32 * tt + c32] = best[tt];
                if (mh == 0) s_xx[64 * tw + 32 * tt + c32] = xx[tt];
            }
        }
        __syncthreads();
        if (tid < DT_TOKENS) {
            const int64_t t = tile0 + tid;
            if (t < a.total) {
                float b = s_part[tid];
#pragma unroll
                for (int c = 1; c < MH; ++c) b = fmaxf(b, s_part[c * DT_TOKENS + tid]);
                const float x2 = s_xx[tid];
                float sim = x2 > 0.0f ? b / sqrtf(x2) : 0.0f;
                if (a.seq_len) {
                    const int64_t sq = t / a.n;
                    if ((int32_t)(t - sq * a.n) >= a.seq_len[sq]) sim = 0.0f;
                }
                a.conf[t] = sim;
                a.anchor[t] = sim > a.thr ? 1 : 0;
            }
        }
    }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---- split form: every wavefront contracts its own share of the features ------------------------------------
// For few positions, and for few hidden units: no workgroup barrier and no shared slice in the loop.  A wavefront has
// a ring of R steps of its own in LDS (64 features of the tile's positions and of all hidden rows, filled by direct
// loads of whole 128-byte lines: with 64-byte pieces the same kernel took 24 instead of 19 us at 4096 positions and 128
// units, and loading the operand fragments straight into registers, where neighbouring lanes lie in different rows,
// 40 us), and the partial sums of the WV wavefronts meet once, in LDS, after the last step.
// PT: 16-position tiles of a workgroup; NT: 16-unit tiles of the hidden layer (concepts); WV wavefronts, each of which
// contracts every SHARES-th step of 64 features; R: steps in flight per wavefront; PW: wavefronts that have such a share of the steps together, each
// half of its parts (2: twice as many requests in flight where the workgroups are few; the sums are those of 1, bit for bit); LOG: see Visit
template <int PT, int NT, int WV, int R, int PW>
struct SplitShape {
    static constexpr int POS = 16 * PT, M = 16 * NT, THREADS = 64 * WV;
    static constexpr int STEP_UNITS = (PT + NT) * 128;     // 16-byte units of a step
    static constexpr int RING_UNITS = WV * R * STEP_UNITS;
    static constexpr int TILE_UNITS = WV * 4 * POS;        // partial sums of one tile of hidden units, every wavefront's
    // tiles exchanged per round: as many as the ring's memory holds
    static constexpr int CH = RING_UNITS >= NT * TILE_UNITS ? NT : (RING_UNITS >= NT / 2 * TILE_UNITS ? (NT + 1) / 2 : (NT + 3) / 4);
    static constexpr int UNITS = RING_UNITS > CH * TILE_UNITS ? RING_UNITS : CH * TILE_UNITS;
    static constexpr int NORMS = PW == 2 ? 4 * WV : WV;    // sums of squares per row: the wavefronts', or those of each one's four groups of lanes
    static constexpr int LDS_BYTES = UNITS * 16 + (M + THREADS + NORMS * M + NORMS * POS) * 4;
};

template <int PT, int NT, int WV, int R, int MODE, bool STREAM, int LOG, int PW>
__global__ void __launch_bounds__(64 * WV)
detect_split_kernel(DetectArgs a)
{
    using S = SplitShape<PT, NT, WV, R, PW>;
    constexpr int POS = S::POS, M = S::M, THREADS = S::THREADS, LPS = 2 * (PT + NT);
    static_assert((R - 1) * LPS <= 63, "vmcnt range");
    extern __shared__ uint4 s_buf[];                       // step rings, then the partial sums
    float* s_w = reinterpret_cast<float*>(s_buf + S::UNITS);   // output weights, or reciprocal norms of the concepts
    float* s_part = s_w + M;
    float* s_cc = s_part + THREADS;                        // cosine mode: squared norms per wavefront
    float* s_xx = s_cc + S::NORMS * M;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, grp = lane >> 4;
    const int64_t tile0 = (int64_t)blockIdx.x * POS;
    const int nsteps = (a.dm + 63) >> 6;                   // (the last one may be half a step)
    constexpr int SHARES = WV / PW;                        // wavefront w: every SHARES-th step from step w % SHARES on, parts by w / SHARES
    constexpr int LOGW = PW == 2 ? LOG - 1 : LOG;
    const int share = wave % SHARES;
    Visit ahead(nsteps > share ? (nsteps - share + SHARES - 1) / SHARES : 0, LOG, PW, wave / SHARES);
    const int mine = ahead.total();
    Visit now = ahead;                                     // the step to work on; ahead: the step to request
    ahead.to_full();

    // A load instruction brings 8 rows x 128 bytes (one line), eight neighbouring lanes per row, chunks XOR-swizzled by row
    uint32_t off[LPS];
    const int lrow = lane >> 3, lchunk = (lane & 7) ^ lrow;
    const uint32_t half_back = lchunk >= 4 ? 64u : 0u;     // half a step: the second half repeats the first
#pragma unroll
    for (int p = 0; p < 2 * PT; ++p) {
        int64_t t = tile0 + 8 * p + lrow;
        t = t < a.total ? t : a.total - 1;                 // stay inside the tensor; never stored
        off[p] = (uint32_t)((t - tile0) * a.h_row_bytes + lchunk * 16);
    }
#pragma unroll
    for (int j = 0; j < 2 * NT; ++j) {
        const int row = 8 * j + lrow;
        off[2 * PT + j] = (uint32_t)((row < a.wrows ? row : a.wrows - 1) * a.dm * 2 + lchunk * 16);   // missing rows repeat the last one
    }
    const char* hbase = reinterpret_cast<const char*>(a.h) + tile0 * a.h_row_bytes;
    const char* wbase = reinterpret_cast<const char*>(a.W1);
    uint4* ring = s_buf + wave * (R * S::STEP_UNITS);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4*)ring;
    const auto half = [&](const Visit& v) { return 64 * (share + SHARES * v.at) + 32 >= a.dm; };
    const auto issue = [&](int i) {
        const uint32_t dst = lds0 + (uint32_t)(i % R) * (S::STEP_UNITS * 16);
        const size_t at = (size_t)(share + SHARES * ahead.at) * 128;
        const uint32_t back = half(ahead) ? half_back : 0u;
        ahead.step();
        ahead.to_full();
#pragma unroll
        for (int j = 0; j < 2 * PT; ++j) dma16<STREAM>(hbase + at, off[j] - back, __builtin_amdgcn_readfirstlane(dst + j * 1024));
#pragma unroll
        for (int j = 2 * PT; j < LPS; ++j) dma16(wbase + at, off[j] - back, __builtin_amdgcn_readfirstlane(dst + j * 1024));
    };
    // this lane's fragments inside a 2 KB tile of 16 rows
    const int slot0 = r16 * 8 + (grp ^ (r16 & 7)), slot1 = r16 * 8 + ((4 + grp) ^ (r16 & 7));

    f32x4 acc[PT][NT];
#pragma unroll
    for (int p = 0; p < PT; ++p)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[p][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float xx[PT], cc[NT];                                  // cosine mode: squared norms, this lane's share
#pragma unroll
    for (int p = 0; p < PT; ++p) xx[p] = 0.0f;
#pragma unroll
    for (int j = 0; j < NT; ++j) cc[j] = 0.0f;
    f32x4 acc_tree[PT][LOGW ? LOGW : 1][NT] = {};
    float xx_tree[LOGW ? LOGW : 1][PT] = {}, cc_tree[LOGW ? LOGW : 1][NT] = {};

#pragma unroll
    for (int i = 0; i < R; ++i)
        if (i < mine) issue(i);
    const auto step = [&](int i, bool more) {
        const uint4* buf = ring + (i % R) * S::STEP_UNITS;
        uint4 f[2][PT + NT];
#pragma unroll
        for (int j = 0; j < PT + NT; ++j) {
            f[0][j] = buf[j * 128 + slot0];
            f[1][j] = buf[j * 128 + slot1];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the fragments are in registers: the buffer is free
        const bool whole = !half(now);
        if (more) issue(i + R);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (s == 1 && !whole) break;                   // uniform
#pragma unroll
            for (int j = 0; j < PT + NT; ++j) asm volatile("" : "+v"(f[s][j].x), "+v"(f[s][j].y), "+v"(f[s][j].z), "+v"(f[s][j].w));
            if constexpr (MODE == MODE_COSINE) {
#pragma unroll
                for (int p = 0; p < PT; ++p) xx[p] = add_squares(f[s][p], xx[p]);
#pragma unroll
                for (int j = 0; j < NT; ++j) cc[j] = add_squares(f[s][PT + j], cc[j]);
            }
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int p = 0; p < PT; ++p)               // rows: hidden units of the tile, columns: positions
                    acc[p][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_frag(f[s][PT + j]), as_frag(f[s][p]), acc[p][j], 0, 0, 0);
        }
    };
    int i = 0;
    for (;;) {
        for (; now.left > 0; now.step(), ++i) {
            const bool more = i + R < mine;
            if (more) __builtin_amdgcn_s_waitcnt(vm_imm((R - 1) * LPS));   // step i is in; R - 1 later ones are on their way
            else __builtin_amdgcn_s_waitcnt(vm_imm(0));
            asm volatile("" ::: "memory");
            step(i, more);
        }
        if constexpr (LOGW == 0) break;
#pragma unroll
        for (int p = 0; p < PT; ++p) close_part<LOGW>(now, acc[p], acc_tree[p]);
        if constexpr (MODE == MODE_COSINE) {
            close_part<LOGW>(now, xx, xx_tree);
            close_part<LOGW>(now, cc, cc_tree);
        }
        if (now.last()) break;
        ++now.part;
        now.open();
    }

    __syncthreads();                                       // every wavefront is done with its ring
    if constexpr (MODE == MODE_MLP)
        for (int j = tid; j < M; j += THREADS) s_w[j] = bf16_bits_to_float(a.W2[j]);
    // ---- the wavefronts' partial sums meet in LDS, CH tiles at a time; a thread owns one position and every
    // (THREADS / POS)-th quad of hidden units of each round
    const auto of_share = [](auto sum, int w) {            // the top of a share's tree is over its wavefronts
        if constexpr (PW == 2) return sum(w) + sum(w + SHARES);
        else return sum(w);
    };
    const auto squares_of_share = [&](auto sum, int w) {   // (the groups of lanes are added up behind the tree, as the shuffles do)
        if constexpr (PW == 2) {
            const auto of = [&](int g) { return sum(g * WV + w) + sum(g * WV + w + SHARES); };
            return (of(0) + of(1)) + (of(2) + of(3));
        } else {
            return sum(w);
        }
    };
    if constexpr (MODE == MODE_COSINE) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            float c = cc[j];
            if constexpr (PW == 1) {
                c += __shfl_xor(c, 16);
                c += __shfl_xor(c, 32);
            }
            if (PW == 2 || grp == 0) s_cc[(PW == 2 ? grp * WV + wave : wave) * M + 16 * j + r16] = c;
        }
#pragma unroll
        for (int p = 0; p < PT; ++p) {
            float x = xx[p];
            if constexpr (PW == 1) {
                x += __shfl_xor(x, 16);
                x += __shfl_xor(x, 32);
            }
            if (PW == 2 || grp == 0) s_xx[(PW == 2 ? grp * WV + wave : wave) * POS + 16 * p + r16] = x;
        }
        __syncthreads();
        for (int j = tid; j < M; j += THREADS) {
            float c = 0.0f;
#pragma unroll
            for (int w = 0; w < SHARES; ++w) c += squares_of_share([&](int v) { return s_cc[v * M + j]; }, w);
            s_w[j] = c > 0.0f ? 1.0f / sqrtf(c) : 0.0f;
        }
    }
    const int pos = tid % POS, q0 = tid / POS;
    float part = MODE == MODE_COSINE ? -INFINITY : 0.0f;
    float4* s_red = reinterpret_cast<float4*>(s_buf);      // [wave][quad of units][position]
    constexpr int CH = S::CH;
    static_assert(NT % CH == 0, "whole rounds");
#pragma unroll
    for (int j0 = 0; j0 < NT; j0 += CH) {
        if (j0) __syncthreads();                           // the previous round has been read
#pragma unroll
        for (int j = 0; j < CH; ++j)
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const f32x4 v = acc[p][j0 + j];
                s_red[(wave * CH * 4 + 4 * j + grp) * POS + 16 * p + r16] = make_float4(v[0], v[1], v[2], v[3]);
            }
        __syncthreads();
        for (int q = q0; q < 4 * CH; q += THREADS / POS) {
            const auto sum = [&](int w) { return *reinterpret_cast<const f32x4*>(&s_red[(w * CH * 4 + q) * POS + pos]); };
            f32x4 z = of_share(sum, 0);
#pragma unroll
            for (int w = 1; w < SHARES; ++w) z += of_share(sum, w);
            const float4 wt = *reinterpret_cast<const float4*>(&s_w[16 * j0 + 4 * q]);
            const float zs[4] = {z[0], z[1], z[2], z[3]}, ws[4] = {wt.x, wt.y, wt.z, wt.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if constexpr (MODE == MODE_MLP)
                    part = fmaf(ws[c], 0.5f * zs[c] * (1.0f + erf_poly(zs[c] * 0.70710678118654752f)), part);
                else
                    part = fmaxf(part, zs[c] * ws[c]);
            }
        }
    }
    s_part[tid] = part;
    __syncthreads();
    if (tid >= POS) return;
    const int64_t t = tile0 + tid;
    if (t >= a.total) return;
    float out = s_part[tid];
#pragma unroll
    for (int k = 1; k < THREADS / POS; ++k) out = MODE == MODE_COSINE ? fmaxf(out, s_part[k * POS + tid]) : out + s_part[k * POS + tid];
    bool past = false;                                     // past the end of its sequence
    if (a.seq_len) {
        const int64_t b = t / a.n;
        past = (int32_t)(t - b * a.n) >= a.seq_len[b];
    }
    if constexpr (MODE == MODE_MLP) {
        const float conf = past ? 0.0f : 1.0f / (1.0f + expf(-out));
        const bool is_anchor = conf > a.thr;
        a.conf[t] = conf;
        a.anchor[t] = is_anchor ? 1 : 0;
        a.anchor_B[t] = is_anchor ? (a.rank ? a.scale * conf : a.B) : 0.0f;
    } else {
        float x2 = 0.0f;
#pragma unroll
        for (int w = 0; w < SHARES; ++w) x2 += squares_of_share([&](int v) { return s_xx[v * POS + tid]; }, w);
        const float sim = past ? 0.0f : (x2 > 0.0f ? out / sqrtf(x2) : 0.0f);
        a.conf[t] = sim;
        a.anchor[t] = sim > a.thr ? 1 : 0;
    }
}

template <int TW, int HT, int MH, int MODE, int RING, bool STREAM, int LOG = 0>
hipError_t launch_one(const DetectArgs& a, hipStream_t st)
{
    constexpr int M = 32 * HT * MH;
    constexpr int DT_TOKENS = 64 * TW;
    const size_t lds = (size_t)RING * (DT_TOKENS + M) * 128 + (size_t)M * 4 + (size_t)(MH + 1) * DT_TOKENS * 4;
    static DeviceOnce setup;                               // dynamic LDS above 64 KB needs the attribute (per instantiation)
    const hipError_t attr_err = setup.run([&](int) {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&detect_kernel<TW, HT, MH, MODE, RING, STREAM, LOG>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    });
    if (attr_err != hipSuccess) return attr_err;
    const unsigned blocks = (unsigned)((a.total + DT_TOKENS - 1) / DT_TOKENS);
    hipLaunchKernelGGL((detect_kernel<TW, HT, MH, MODE, RING, STREAM, LOG>), dim3(blocks), dim3(64 * TW * MH), lds, st, a);
    return hipGetLastError();
}

template <int PT, int NT, int WV, int R, int MODE, bool STREAM, int LOG = 0, int PW = 1>
hipError_t launch_split(const DetectArgs& a, hipStream_t st)
{
    using S = SplitShape<PT, NT, WV, R, PW>;
    static DeviceOnce setup;
    const hipError_t attr_err = setup.run([&](int) {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&detect_split_kernel<PT, NT, WV, R, MODE, STREAM, LOG, PW>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES);
    });
    if (attr_err != hipSuccess) return attr_err;
    const unsigned blocks = (unsigned)((a.total + S::POS - 1) / S::POS);
    hipLaunchKernelGGL((detect_split_kernel<PT, NT, WV, R, MODE, STREAM, LOG, PW>), dim3(blocks), dim3(S::THREADS), S::LDS_BYTES, st, a);
    return hipGetLastError();
}

// Which form runs.  A workgroup of the split form streams all of W1 (1 MB at d_model 4096, 128 units) for its 16, 32 or
// 64 positions, and the sum of these streams is what bounds it (about 12 TB/s over all L2s); a workgroup of the
// shared form does so for 128 or 256 positions but needs many positions to fill the chip.  So: the smallest tile
// that gives every compute unit at most one workgroup (16 positions up to 4096, 32 up to 8192, 64 up to 16384), then
// the shared form where W1's traffic counts.  Measured at d_model 4096 where no other is given, launches of a graph over inputs in turn, in us, split /
// shared form with three buffers / with two:
//   128 units:  16384: 37 / - / 61;  24000: 64.6 / 50.6 / 65.8;  32768: 70.4 / 56 / 69.3;  40000: 98 / 102 / 84;  131072: 254 / 205 / 192;
//               d_model 2048, 16500: 36.0 / 28.9 / 35.2;  24000: 38.5 / 29.8 / 36.3;  32768: 41.8 / 33.6 / 38.4;
//               d_model 1024, 16500: 21.3 / 17.5 / 19.6;  24000: 25.0 / 19.3 / 21.4;  32768: 25.9 / 18.0 / 21.3
//   256 units:  8192: 42 / 64 / -;  16384: 75 / 66 / -;  32768: 147 / 82 / -;  131072: - / 320 (128 positions) / 284 (256)
//   64 units, 64 positions with four wavefronts / 32:  16384: 29.8 / 36.8;  65536: 108 / 133;  131072: 210 / 256
//   32 units, 64 positions with eight wavefronts / 32 with four:  16384: 25.9 / 28.5;  65536: 90.7 / 93.4;  262144: 336 = 6.4 TB/s / 346
//   up to 16 concepts (cosine), 32 positions with four wavefronts / 16 with eight (two per share of the features):  512 rows 10.5 / 6.7;  4096:
//               10.8 / 8.8;  6000: 13.7 / 15.3;  8000: 15.1 / 16.5;  32000: 42 / 47.6;  128256: 150 / 171;  d_model 2048, 4096: 7.8 / 6.7;  100000: 65 / 86
// Parts (Visit) for the streamed rows that crowd, and for up to 16 concepts at any number of rows from d_model 2048 on: with few rows they are in the
// caches, and parts cost their additions (12 000 positions of 2048, 32 units 13.0 / 14.3).
template <int MODE, bool STREAM, bool PARTS>
hipError_t launch_width(const DetectArgs& a, hipStream_t st)
{
    const int64_t P = a.total;
    const int64_t cus = compute_units();
    constexpr int FOUR = PARTS ? 2 : 0, EIGHT = PARTS ? 3 : 0, FOUR_MLP = MODE == MODE_MLP ? FOUR : 0;
    // Rows of few steps: fewer wavefronts, so that each has several steps of its own to keep in flight (d_model 1024, 131072
    // positions: 32 units 52 us with four wavefronts, 56 with eight, 64 units 58 with two, 68 with four; d_model 2048: 100 / 108, 108 / 124).
    const bool narrow = a.dm <= 2048;
    if (MODE == MODE_COSINE && a.wrows <= 16) {            // (both forms of a d_model add up alike: a table's rows and a prompt's get the same results)
        if (a.dm < 2048) return launch_split<2, 1, 4, 2, MODE, STREAM>(a, st);
        if (P <= 4096) return launch_split<1, 1, 8, 2, MODE, STREAM, 2, 2>(a, st);
        return launch_split<2, 1, 4, 2, MODE, STREAM, 2>(a, st);
    }
    switch (a.m) {
        case 32:
            if (P <= 4096) return launch_split<1, 2, 8, 2, MODE, STREAM>(a, st);
            if (P <= 8192) return launch_split<2, 2, 4, 2, MODE, STREAM, FOUR>(a, st);
            if (narrow && P > 24576) return launch_split<2, 2, 4, 2, MODE, STREAM, FOUR>(a, st);
            return launch_split<4, 2, 8, 1, MODE, STREAM, EIGHT>(a, st);
        case 64:
            if (P <= 4096) return launch_split<1, 4, 4, 3, MODE, STREAM>(a, st);
            if (P <= 8192) return launch_split<2, 4, 4, 2, MODE, STREAM>(a, st);
            if (narrow && P > 24576) return launch_split<4, 4, 2, 2, MODE, STREAM, FOUR>(a, st);
            return launch_split<4, 4, 4, 2, MODE, STREAM>(a, st);
        case 128:
            if (P <= 4096) return launch_split<1, 8, 4, 2, MODE, STREAM>(a, st);
            if (P <= 8192) return launch_split<2, 8, 4, 1, MODE, STREAM>(a, st);
            if (P <= 64 * cus) return launch_split<4, 8, 4, 1, MODE, STREAM>(a, st);
            // 128 positions per workgroup; three buffers (one workgroup per compute unit) while that is one round of workgroups
            if (P <= 128 * cus) return launch_one<2, 2, 2, MODE, 3, STREAM, FOUR_MLP>(a, st);
            return launch_one<2, 2, 2, MODE, 2, STREAM, FOUR_MLP>(a, st);
        default:
            if (P <= 4096) return launch_split<1, 16, 4, 1, MODE, STREAM>(a, st);
            if (P <= 8192) return launch_split<2, 16, 4, 1, MODE, STREAM>(a, st);
            if (P <= 32768) return launch_one<2, 2, 4, MODE, 3, STREAM>(a, st);
            return launch_one<4, 2, 4, MODE, 2, STREAM>(a, st);
    }
}

// The rows of h (or x) are read once.  Where they are many the streaming hint leaves the rest of a workgroup's operands in the
// caches (us, without / with it, eight sets of inputs in turn: 128 256 rows of 4096 and 16 concepts 173 / 166; 131 072 positions of 4096
// and 64 units 216 / 204; 8192 of 4096 and 128 units, 64 MiB, 27.5 / 26.8); fewer may lie in the caches from whoever wrote them, and the hint gives
// up what stays there (4096 of 4096 and 128 units 17.3 / 19.1).
template <int MODE>
hipError_t launch_hint(const DetectArgs& a, hipStream_t st)
{
    constexpr int64_t STREAM_BYTES = int64_t(64) << 20;
    if (a.total * a.dm * 2 < STREAM_BYTES) return launch_width<MODE, false, false>(a, st);
    return a.dm >= 2048 && a.h_row_bytes % 4096 == 0 ? launch_width<MODE, true, true>(a, st) : launch_width<MODE, true, false>(a, st);
}

}  // namespace

hipError_t launch_detect(const void* h, int64_t h_row_stride, const void* W1, const void* W2,
                         const int32_t* seq_len, int32_t batch, int32_t n, int32_t dm, int32_t m,
                         float thr, int32_t rank, float B, float scale,
                         float* conf, uint8_t* anchor, float* anchor_B, hipStream_t st)
{
    DetectArgs a;
    a.h = (const uint4*)h;
    a.W1 = (const uint4*)W1;
    a.W2 = (const uint16_t*)W2;
    a.seq_len = seq_len;
    a.conf = conf;
    a.anchor = anchor;
    a.anchor_B = anchor_B;
    a.total = (int64_t)batch * n;
    a.n = n;
    a.dm = dm;
    a.m = m;
    a.h_row_bytes = (int32_t)(h_row_stride * 2);
    a.thr = thr;
    a.B = B;
    a.scale = scale;
    a.rank = rank;
    a.wrows = m;
    return launch_hint<MODE_MLP>(a, st);
}

hipError_t launch_cosine(const void* x, int64_t x_row_stride, const void* C, int32_t E, int64_t rows, int32_t dm,
                         const int32_t* seq_len, int32_t n, float tau, float* sim, uint8_t* anchor, hipStream_t st)
{
    DetectArgs a;
    a.h = (const uint4*)x;
    a.W1 = (const uint4*)C;
    a.W2 = nullptr;
    a.seq_len = seq_len;
    a.conf = sim;
    a.anchor = anchor;
    a.anchor_B = nullptr;
    a.total = rows;
    a.n = n;
    a.dm = dm;
    a.m = E <= 32 ? 32 : (E <= 64 ? 64 : (E <= 128 ? 128 : 256));
    a.wrows = E;
    a.h_row_bytes = (int32_t)(x_row_stride * 2);
    a.thr = tau;
    a.B = 0.0f;
    a.scale = 0.0f;
    a.rank = 0;
    return launch_hint<MODE_COSINE>(a, st);
}

}  // namespace ta
