// Step 3 of the eviction pass: the attention term A_i of Eq. 1 as column sums
// of the observation window's softmax (cumulative attention over heads and
// steps, App. A dormant-token definition; SnapKV/H2O-style scoring, Sec. 2).
//
// Per unit (layer, sequence, KV head): S = Q K^T with M = G*W query rows
// (G query heads of the group x W window rows), d = 128, n keys; row softmax
// over the visible keys; A[i] = sum over rows of the softmax column i.
//
// Column sums need every row's (max, normaliser) over ALL keys before any row
// can be added into a column, so the keys are swept twice:
//   sweep 1 (stats)  : per row, (m, Z) over a chunk of keys -> workspace; m is a logit
//                      the row has had, close enough to its largest (see reduce below),
//                      and Z the sum of 2^(s - m)
//   sweep 2 (colsum) : merge the chunk statistics of a row into one constant
//                      c_r = m_r + log2 Z_r, recompute S, p = 2^(s - c_r),
//                      sum p over the rows -> A
// Both sweeps are one kernel template, a launch each; a unit of one chunk needs no other workgroup's statistics, and
// its workgroup does both in one launch, its rows' constants in LDS (score_once).  A workgroup owns one chunk of keys of
// one unit and streams it through LDS in 64-key stages: a ring of four 16 KB
// buffers (three for units of at most 64 rows) filled by direct global->LDS loads
// issued as many stages ahead but one (no staging registers), 16-byte chunks XOR-swizzled by row so that the
// ds_read_b128 fragment loads are conflict free.  Blocks are numbered so that
// all chunks of a unit run on one XCD (block b lands on XCD b mod 8): the
// unit's Q rows and chunk statistics are then fetched into one L2 only.  The M rows are split
// into RG groups of 64; the workgroup has 2*RG wavefronts, wavefront (rg, kt)
// owns row group rg (its Q fragments stay in 64 registers for the whole chunk)
// and the kt-th 32-key tile of every stage, so one K fragment read from LDS
// feeds two MFMA row tiles.
// The contraction runs on v_mfma_f32_32x32x16_bf16:
//   sweep 1 computes K Q^T (keys x rows): a lane then holds 16 keys of ONE
//           query row, so (m, Z) are two registers per row tile and need no
//           cross-lane traffic until the end of the chunk;
//   sweep 2 computes Q K^T (rows x keys): a lane holds 16 rows of ONE key, so
//           the column sum is a register accumulation plus one half-wave swap.
#include <math.h>

#include <atomic>
#include <type_traits>

#include "ta_match_device.h"
#include "ta_order.h"
#include "ta_score_common.h"

namespace ta {

int compute_units()
{
    static std::atomic<int> cached{0};                     // callers on several threads may race to fill it
    int cu = cached.load(std::memory_order_relaxed);
    if (cu == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu < 1)
            cu = 256;                                      // MI355X
        cached.store(cu, std::memory_order_relaxed);
    }
    return cu;
}

namespace {

constexpr int STAGE_KEYS = 64;
constexpr int MAX_CHUNKS = 32;                   // of a unit
constexpr int STAGE_UNITS = STAGE_KEYS * 16;     // 16-byte units per stage (256 B per key)
// Stage buffers per workgroup; loads run that many minus one stages ahead.  (Eight buffers for
// the wider workgroups, which have a compute unit to themselves, were measured: no gain.)
// Three for units of at most 64 rows: 48 KB, so that three such workgroups share a compute unit.
constexpr int ring_of(int rg) { return rg == 1 ? 3 : 4; }
// Where the query rows of a workgroup pass through on their way to the registers: the last buffers of the ring, or, where
// they would fill the whole of it, buffers of their own behind the stages that are requested with them.
constexpr int q_stage(int rg) { return rg == 4 ? ring_of(rg) - 1 : ring_of(rg) - rg; }
constexpr int lds_stages(int rg) { return q_stage(rg) + rg > ring_of(rg) ? q_stage(rg) + rg : ring_of(rg); }

// Direct global->LDS load of 16 bytes per lane: lane i reads 16 bytes at base + off (base
// wave-uniform, off per lane) and its data lands at lds_base + 16*i (lds_base wave-uniform,
// passed in M0).  Written as inline assembly on purpose: the compiler would otherwise make
// every later LDS read wait for ALL outstanding direct loads, which would serialise the stage
// pipeline; the waits for these loads are explicit below.  Extra outstanding loads only make
// the compiler's own vmcnt waits more conservative.
// STREAM: with the non-temporal hint, for what will not be read again soon.
template <bool STREAM>
__device__ __forceinline__ void load_to_lds_16(const void* base, uint32_t off, uint32_t lds_base)
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

// the same from an address of each lane's own
__device__ __forceinline__ void load_to_lds_16(const uint4* from, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(lds_base), "v"(from)
                 : "memory", "m0");
}

// the value of the lane 32 further on or back
__device__ __forceinline__ float other_half(float v)
{
    const uint32_t u = __float_as_uint(v);
    const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);  // the lower half twice, the upper half twice
    return __uint_as_float((threadIdx.x & 32u) ? sw[0] : sw[1]);
}

// s_waitcnt vmcnt(n) with the other counters left alone (gfx9 encoding)
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// A sweep that also carries the match tiles: workgroups past the score grid each run one tile
// of the anchor match (they start as the first score workgroups retire).  The statistics sweep
// carries them in the two-sweep step, the column-sum sweep when the normalisers are given.
struct RiderArgs {
    MatchArgs m;
    MatchTable tab;
    uint32_t score_blocks;
};

// a workgroup past the score grid: its tile, in the stages' memory
template <int STAGES>
__device__ __forceinline__ void match_tile_of_block(const RiderArgs& r, uint4 (*s_k)[STAGE_UNITS])
{
    static_assert(sizeof(MatchLds) <= sizeof(uint4) * STAGES * STAGE_UNITS, "match tile must fit the stage ring");
    if (threadIdx.x >= MATCH_THREADS) return;              // a tile is the work of four wavefronts
    const uint32_t t = blockIdx.x - r.score_blocks;
    match_expand_tile(r.m, r.tab, (int32_t)(t % (uint32_t)r.m.tiles), (int32_t)(t / (uint32_t)r.m.tiles),
                      (int)threadIdx.x, *reinterpret_cast<MatchLds*>(&s_k[0][0]));
}

// RG row groups of RT 32-row MFMA tiles each per workgroup; 2 * RG wavefronts.
// row_base: first of the 64 * RG rows this call works on (units with more rows than the widest workgroup's 256 take several
// calls; more row groups would leave too few registers per lane)
// ONE: both sweeps over a unit of one chunk are this workgroup's, one after the other: the first leaves the rows' constants in s_one and
// the second finds them there.
template <int RG, int RT, bool COLSUM, bool PAGED, bool STREAM, bool TURNS, bool ONE = false>
__device__ __forceinline__ void score_body(const ScoreArgs& a, uint4 (*s_k)[STAGE_UNITS], int32_t row_base, float* s_one = nullptr);

// one tile per wavefront: four wavefronts per SIMD (at most 128 registers each)
template <int RG, int RT, bool COLSUM, bool PAGED, bool STREAM, bool PASSES, bool TURNS>
__global__ void __launch_bounds__(128 * RG, RT == 1 ? 4 : 2)
score_kernel(ScoreArgs a)
{
    __shared__ uint4 s_k[lds_stages(RG)][STAGE_UNITS];        // 16 KB per stage
    // a workgroup holds 64 * RG rows at a time; a unit with more rows is done in passes over its chunk
    // (the keys of the later passes come from the L2; their column sums are added to the first pass's)
    if constexpr (!PASSES) {
        score_body<RG, RT, COLSUM, PAGED, STREAM, TURNS>(a, s_k, 0);
    } else {
        for (int32_t row_base = 0; row_base < a.rows_pad; row_base += 64 * RG) {
            if (row_base > 0) __syncthreads();             // the previous pass is done with the LDS
            score_body<RG, RT, COLSUM, PAGED, STREAM, TURNS>(a, s_k, row_base);
        }
    }
}

template <int RG, int RT, bool COLSUM, bool PAGED, bool STREAM, bool PASSES, bool TURNS>
__global__ void __launch_bounds__(128 * RG, RT == 1 ? 4 : 2)
score_match_kernel(ScoreArgs a, RiderArgs r)
{
    __shared__ uint4 s_k[lds_stages(RG)][STAGE_UNITS];
    if (blockIdx.x >= r.score_blocks) {
        match_tile_of_block<lds_stages(RG)>(r, s_k);
        return;
    }
    if constexpr (!PASSES) {
        score_body<RG, RT, COLSUM, PAGED, STREAM, TURNS>(a, s_k, 0);
    } else {
        for (int32_t row_base = 0; row_base < a.rows_pad; row_base += 64 * RG) {
            if (row_base > 0) __syncthreads();
            score_body<RG, RT, COLSUM, PAGED, STREAM, TURNS>(a, s_k, row_base);
        }
    }
}

// Both sweeps over units of one chunk each, in one launch: a workgroup sweeps its unit twice.  The second sweep begins with what the
// first has read last, the statistics stay in LDS, and there is no end of a launch in the middle: the second sweeps of some
// workgroups run beside the first ones of others (on the same compute unit with up to 128 rows; with 256 a workgroup fills one).
template <int RG, int RT, bool PAGED, bool STREAM, bool TURNS>
__device__ __forceinline__ void score_once(const ScoreArgs& a, uint4 (*s_k)[STAGE_UNITS])
{
    __shared__ float s_one[32 * RT * RG];
    // (the first sweep with the streaming hint where a unit may have more stages than a.keep_last: see the rule at the launch)
    score_body<RG, RT, false, PAGED, STREAM && (RG == 1 || (RG == 2 && TURNS)), TURNS, true>(a, s_k, 0, s_one);
    __syncthreads();                                       // the constants are in LDS, and nobody uses the stages' memory
    score_body<RG, RT, true, PAGED, STREAM, TURNS, true>(a, s_k, 0, s_one);
}

template <int RG, int RT, bool PAGED, bool STREAM, bool TURNS>
__global__ void __launch_bounds__(128 * RG, RT == 1 ? 4 : 2)
score_once_kernel(ScoreArgs a)
{
    __shared__ uint4 s_k[lds_stages(RG)][STAGE_UNITS];
    score_once<RG, RT, PAGED, STREAM, TURNS>(a, s_k);
}

template <int RG, int RT, bool PAGED, bool STREAM, bool TURNS>
__global__ void __launch_bounds__(128 * RG, RT == 1 ? 4 : 2)
score_once_match_kernel(ScoreArgs a, RiderArgs r)
{
    __shared__ uint4 s_k[lds_stages(RG)][STAGE_UNITS];
    if (blockIdx.x >= r.score_blocks) {
        match_tile_of_block<lds_stages(RG)>(r, s_k);
        return;
    }
    score_once<RG, RT, PAGED, STREAM, TURNS>(a, s_k);
}

template <int RG, int RT, bool COLSUM, bool PAGED, bool STREAM, bool TURNS, bool ONE>
__device__ __forceinline__ void score_body(const ScoreArgs& a, uint4 (*s_k)[STAGE_UNITS], const int32_t row_base, float* s_one)
{
    constexpr int ROW_TILES = RT;
    constexpr int GROUP_ROWS = 32 * RT;                    // rows of one wavefront
    constexpr int THREADS = 128 * RG;
    constexpr int WAVES = 2 * RG;
    constexpr int LPS = 16 / WAVES;                        // 1 KB direct loads per wavefront per stage
    static_assert(LPS >= 1, "unsupported row-group count");
    constexpr int RING = ring_of(RG);
    // waits until the loads of at most k later stages are outstanding (loads complete in issue order)
    const auto wait_but = [](int k) {
        static_assert(RING - 2 <= 6, "cases below");
        switch (k) {
            case 0: __builtin_amdgcn_s_waitcnt(vmcnt_imm(0)); break;
            case 1: __builtin_amdgcn_s_waitcnt(vmcnt_imm(LPS)); break;
            case 2: __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * LPS)); break;
            case 3: __builtin_amdgcn_s_waitcnt(vmcnt_imm(3 * LPS)); break;
            case 4: __builtin_amdgcn_s_waitcnt(vmcnt_imm(4 * LPS)); break;
            case 5: __builtin_amdgcn_s_waitcnt(vmcnt_imm(5 * LPS)); break;
            default: __builtin_amdgcn_s_waitcnt(vmcnt_imm(6 * LPS)); break;
        }
    };

    __shared__ float s_c[COLSUM ? GROUP_ROWS * RG : 1];            // per-row constant m + log2 Z
    __shared__ int32_t s_lim[COLSUM ? GROUP_ROWS * RG : 1];        // per-row last visible key
    // Partial column sums of the row groups, by stage: two halves, one of which is written out while the other fills.
    constexpr int TURN = RING % 2 ? 2 * RING : RING;       // stages of a turn of the main loop: ring buffers and accumulators have their numbers
    constexpr int FLUSH = TURN;                            // stages of a half
    __shared__ float s_part[COLSUM ? 2 * FLUSH : 1][RG][STAGE_KEYS];

    int tid = threadIdx.x;
    if constexpr (ONE) asm volatile("" : "+v"(tid));       // (nothing that follows from it is kept in registers from one sweep for the other)
    const int lane = tid & 63, wave = tid >> 6;
    const int c32 = lane & 31, hf = lane >> 5;
    const int rg = wave % RG, kt = wave / RG;              // row group, key tile of the stage

    int32_t chunk;
    int32_t place = place_of(blockIdx.x, a.nchunks, a.by_chunks, chunk);
    if (place >= a.units) return;
    if (COLSUM && a.backwards) {
        place = a.units - 1 - place;
        chunk = a.nchunks - 1 - chunk;
    }
    const int32_t unit = __builtin_amdgcn_readfirstlane(unit_at(place, a.seq_len, a.batch, a.hkv, a.units));
    const int32_t pair = (int32_t)divide((uint32_t)unit, a.by_hkv);
    const int32_t g = unit - pair * a.hkv;
    const int32_t l = (int32_t)divide((uint32_t)pair, a.by_batch);
    const int32_t b = pair - l * a.batch;
    const int32_t n = a.n, W = a.W;
    int32_t nb = a.seq_len ? __builtin_amdgcn_readfirstlane(a.seq_len[b]) : n;   // (in a scalar register: it is part of every stage's address)
    nb = nb < 0 ? 0 : (nb > n ? n : nb);

    // The chunks divide the sequence's own length, so that a short one is spread over as many workgroups as a long one (cut
    // where the longest is, the last chunks of the others were empty and the rest no shorter.  Whole pass, us: 80 units of
    // 5000..20000 keys 95 -> 64; 192 of them, 256 rows 506 -> 404; 176 units of 1090..8720 keys 146 -> 124).
    const int32_t seq_stages = (nb + STAGE_KEYS - 1) / STAGE_KEYS;
    const int32_t chunk_keys = (int32_t)divide((uint32_t)(seq_stages + a.nchunks - 1), a.by_chunks) * STAGE_KEYS;
    const int32_t key_lo = chunk * chunk_keys;
    int32_t key_hi = key_lo + chunk_keys;
    key_hi = key_hi > n ? n : key_hi;
    // Keys past the end of a ragged sequence are visible to no row: the stages behind it are not streamed at all; their
    // column sums are zeros, an equal share of which every chunk writes.
    const auto zero_share = [&]() {
        const int32_t from = seq_stages * STAGE_KEYS;
        if (from >= n) return;
        const int32_t share = (int32_t)divide((uint32_t)(n - from + a.nchunks - 1), a.by_chunks);
        const int32_t first = from + chunk * share, last = n - first < share ? n : first + share;
        for (int32_t key = first + (int32_t)threadIdx.x; key < last; key += THREADS) a.A[(size_t)unit * n + key] = 0.0f;
    };
    const int32_t key_end = key_hi < nb ? key_hi : nb;
    const int nstages = key_end > key_lo ? (key_end - key_lo + STAGE_KEYS - 1) / STAGE_KEYS : 0;
    // keys <= min_lim are visible to every live row of a full window
    const int32_t min_lim = a.causal ? nb - W : nb - 1;

    if (key_lo >= nb) {
        // the whole chunk lies past the end of this sequence: nothing is visible
        if constexpr (COLSUM) {
            zero_share();
        } else if constexpr (!ONE) {
            float* st = a.ws + (((size_t)unit * a.nchunks + chunk) * a.rows_pad) * 2;
            for (int r = tid; r < a.rows_pad; r += THREADS) {
                st[r * 2] = -INFINITY;
                st[r * 2 + 1] = 0.0f;
            }
        }
        return;
    }

    // Stages whose keys are all visible to every row: [0, nfast).  The column-sum sweep visits them in the reverse order of the
    // statistics sweep: what that sweep read last is the likeliest to still sit in the last-level cache.
    // (Starting at a stage that differs from block to block, as an earlier form did, costs its arithmetic and is faster only where chunks of 1 MB lie 1 MB
    // apart and all run at once.  Whole pass, us, with that / without: 8 units of 4096 keys 21.7 / 20.5, 256 of 16 384 with 64 rows 376 / 365, 2048 of
    // 4096 794 / 785, 24 layers of 8192 keys, 256 rows, 267.5 / 266.1, one sequence of 131 072 4565 / 4540; one sweep, 512 units of 8192 keys 191 / 185, 128 of
    // 32 768 194 / 185, 64 of 32 768 95 / 103, with 64 rows 32 of 65 536 89 / 95.  Every other chunk in the opposite order mends those, 102 and 91, and costs
    // as much elsewhere: 256 rows, 64 of 32 768 keys 135 / 148, two sweeps, 128 rows, 256 of 16 384 350 / 363.)
    int nfast = min_lim >= key_lo + STAGE_KEYS - 1 ? (min_lim - key_lo + 1) / STAGE_KEYS : 0;
    nfast = nfast > nstages ? nstages : nfast;
    const auto stage_pos = [&](int s) { return COLSUM && s < nfast ? nfast - 1 - s : s; };

    // ---- K staging: direct global->LDS loads, 1 KB (4 key rows) per wavefront instruction.
    // Lane i of a load lands at (buffer + block*1 KB + 16*i): LDS slot row*16 + c' receives the
    // 16-byte chunk c' ^ (row & 15) of key row `row`.
    // The byte offset of a lane's 16 bytes inside a stage does not depend on the stage, so a
    // stage costs one scalar base address and no vector arithmetic (except the ragged last one).
    // Paged K: the keys of a stage (64 positions, page_size is a multiple of 64) lie in one page; lane j
    // keeps the page of the j-th page slot of this chunk, so a stage costs a lane read, not a load.
    const uint4* kbase = (a.Kl ? uniform_global_ptr(a.Kl[l]) : a.K + l * a.k_sl) + (PAGED ? 0 : b * a.k_sb) + g * a.k_sh;
    const auto slot_of = [&](int32_t key) { return a.page_shift >= 0 ? key >> a.page_shift : key / a.page_size; };
    const int32_t slot_lo = PAGED ? slot_of(key_lo) : 0;
    int32_t my_page = 0;
    if constexpr (PAGED) {
        const int32_t slot = slot_lo + lane;
        if (slot < a.max_pages) my_page = a.table[(size_t)b * a.max_pages + slot];
        my_page = my_page < 0 ? 0 : (my_page >= a.num_pages ? a.num_pages - 1 : my_page);
    }
    const auto stage_base = [&](int32_t key0) -> const uint4* {
        if constexpr (!PAGED) return kbase + (int64_t)key0 * a.k_sp;
        const int32_t slot = slot_of(key0);
        const int32_t rel = __builtin_amdgcn_readfirstlane(slot - slot_lo);
        int32_t page;
        if (rel < 64) page = __builtin_amdgcn_readlane(my_page, rel);
        else {                                             // chunks longer than 64 pages: read the table
            page = a.table[(size_t)b * a.max_pages + slot];
            page = page < 0 ? 0 : (page >= a.num_pages ? a.num_pages - 1 : page);
        }
        return kbase + (int64_t)page * a.k_spage + (int64_t)(key0 - slot * a.page_size) * a.k_sp;
    };
    const uint32_t lds_ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4*)&s_k[0][0];
    const uint32_t lds_wave = lds_ring + 1024u * (uint32_t)__builtin_amdgcn_readfirstlane(wave);
    uint32_t lane_off[LPS];
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        const int row = (wave + WAVES * j) * 4 + (lane >> 4);
        lane_off[j] = (uint32_t)(row * a.k_sp + ((lane & 15) ^ (row & 15))) * 16u;
    }
    // STREAM: with the streaming hint; in the first sweep up to this stage only, those from it on are for the last-level cache
    int keep_from = 0;
    if constexpr (STREAM && !COLSUM && ONE) keep_from = nstages > a.keep_last ? nstages - a.keep_last : 0;
    else if constexpr (STREAM && !COLSUM) keep_from = place < a.keep_place ? (int)(((uint64_t)nstages * (uint64_t)a.keep_stage) >> 10) : 0;
    auto stage_issue = [&](int s) {
        const int32_t key0 = key_lo + stage_pos(s) * STAGE_KEYS;
        const uint4* sbase = stage_base(key0);
        const uint32_t dst = lds_wave + (uint32_t)(s % RING) * (STAGE_UNITS * 16u);
        const bool whole = key0 + STAGE_KEYS <= n;
        if (whole && (!STREAM || (!COLSUM && s >= keep_from))) {
#pragma unroll
            for (int j = 0; j < LPS; ++j) load_to_lds_16<false>(sbase, lane_off[j], dst + WAVES * j * 1024u);
        } else if (whole) {
#pragma unroll
            for (int j = 0; j < LPS; ++j) load_to_lds_16<true>(sbase, lane_off[j], dst + WAVES * j * 1024u);
        } else {
#pragma unroll
            for (int j = 0; j < LPS; ++j) {
                const int row = (wave + WAVES * j) * 4 + (lane >> 4);
                const int32_t last = n - 1 - key0;         // stay inside the tensor; masked later
                const int32_t rclamp = row > last ? last : row;
                const uint32_t off = (uint32_t)(rclamp * a.k_sp + ((lane & 15) ^ (row & 15))) * 16u;
                load_to_lds_16<false>(sbase, off, dst + WAVES * j * 1024u);
            }
        }
    };
    // ---- Q and the first stages of K are requested together: one round trip to memory brings both.  Q passes through LDS in
    // the layout of a K stage per 64 rows (whole rows of 256 bytes per 16 lanes; loaded straight into the registers, 32 rows
    // of 32 bytes per instruction and the same rows by both key tiles' wavefronts, they took 2 us of the 7 of a launch of
    // two-stage chunks).  Rows past the last one repeat it: their column sums' constant is inf, their statistics are not read.
    // (Both sweeps, with the statistics of all chunks in one round trip and the scalar divisions, us: 8 units of 4096 keys
    // 15.4 -> 11.9; 32 units of 333 keys, 256 rows 20.2 -> 13.5; 192 units of 8192 keys, 256 rows 270 -> 257.)
    constexpr int QS = q_stage(RG), FIRST = QS < RING - 1 ? QS : RING - 1;     // stages of K that are requested with Q
    constexpr int QPW = 64 * RG / 4 / WAVES;                                    // direct loads of Q per wavefront
    const uint4* qunit = (a.Ql ? uniform_global_ptr(a.Ql[l]) : a.Q + l * a.q_sl) + b * a.q_sb + (int64_t)(g * a.G) * a.q_sh;
    const auto head_of = [&](int32_t r) { return (int32_t)(((uint32_t)r * a.inv_W) >> 20); };
#pragma unroll
    for (int j = 0; j < QPW; ++j) {
        const int row = (wave + WAVES * j) * 4 + (lane >> 4);
        int32_t r = row_base + row;
        r = r < a.rows ? r : a.rows - 1;
        const int32_t h = head_of(r);
        load_to_lds_16(qunit + h * a.q_sh + (r - h * W) * 16 + ((lane & 15) ^ (row & 15)), lds_wave + QS * (STAGE_UNITS * 16u) + WAVES * j * 1024u);
    }
    if constexpr (PAGED) asm volatile("" ::"v"(my_page) : "memory");
#pragma unroll
    for (int s = 0; s < FIRST; ++s)
        if (s < nstages) stage_issue(s);
    int32_t my_lim[ROW_TILES];                             // sweep 1: last visible key of this lane's row
#pragma unroll
    for (int t = 0; t < ROW_TILES; ++t) {
        const int32_t r = row_base + GROUP_ROWS * rg + 32 * t + c32;
        my_lim[t] = r >= a.rows ? -1 : (a.causal ? nb - W + (r - head_of(r) * W) : nb - 1);
    }
    // ---- sweep 2: merge the chunk statistics of a row into its constant.  These are ordinary loads behind the direct loads of
    // Q and the first FIRST stages: waiting for them waits for those as well, which the first stage does in any case.  Each half
    // of the chunks is added in index order, then the two halves.
    if constexpr (COLSUM) {
        constexpr int ROWS = GROUP_ROWS * RG, PARTS = THREADS / ROWS;
        static_assert(PARTS == 2, "two threads per row");
        const int lr = tid % ROWS, part = tid / ROWS;
        const int32_t r = row_base + lr;
        float c = INFINITY;
        int32_t lim = -1;
        if (r < a.rows) {
            const int32_t h = head_of(r), w = r - h * W;
            lim = a.causal ? nb - W + w : nb - 1;
            if (a.lse) {
                // the row's normaliser comes from the prefill attention kernel: c = lse * log2(e)
                const float v = a.lse[(((size_t)l * a.batch + b) * ((size_t)a.hkv * a.G) + (size_t)(g * a.G + h)) * W + w];
                if (v > -INFINITY) c = v * 1.4426950408889634f;
            }
        }
        if constexpr (ONE) {
            if (r < a.rows) c = s_one[lr];
        } else if (!a.lse) {                               // uniform
            // Two threads per row, each with half of the chunks, all loads in flight: one round trip however many chunks
            // there are, so that few units can be cut into many.
            static_assert(sizeof(s_part) >= sizeof(float2) * ROWS, "the second halves pass through the partial sums' memory");
            float2* s_mz = reinterpret_cast<float2*>(&s_part[0][0][0]);
            const int32_t half = (a.nchunks + 1) >> 1, ch0 = part * half;
            const float2* st = reinterpret_cast<const float2*>(a.ws) + ((size_t)unit * a.nchunks * a.rows_pad + (r < a.rows_pad ? r : 0));
            float m = -INFINITY, Z = 0.0f;
            const auto merge = [&](auto count_tag) {
                constexpr int COUNT = decltype(count_tag)::value;
                float2 v[COUNT];
#pragma unroll
                for (int j = 0; j < COUNT; ++j) {
                    const int32_t ch = ch0 + j;
                    v[j] = st[(uint32_t)((ch < a.nchunks ? ch : a.nchunks - 1) * a.rows_pad)];
                }
#pragma unroll
                for (int j = 0; j < COUNT; ++j) {
                    const bool in = j < half && ch0 + j < a.nchunks;
                    v[j].x = in ? v[j].x : -INFINITY;
                    v[j].y = in ? v[j].y : 0.0f;
                    m = fmaxf(m, v[j].x);
                }
                const float ref = m > -INFINITY ? m : 0.0f;
#pragma unroll
                for (int j = 0; j < COUNT; ++j) {
                    const float term = v[j].y * fast_exp2(v[j].x - ref);
                    Z += v[j].y > 0.0f ? term : 0.0f;
                }
            };
            static_assert(MAX_CHUNKS <= 32, "cases below");
            if (half <= 2) merge(std::integral_constant<int, 2>{});
            else if (half <= 8) merge(std::integral_constant<int, 8>{});
            else merge(std::integral_constant<int, 16>{});
            if (part == 1) s_mz[lr] = make_float2(m, Z);
            __syncthreads();
            if (part == 0) {
                const float2 o = s_mz[lr];
                const float mm = fmaxf(m, o.x);
                if (mm > -INFINITY) {
                    const float z = Z * fast_exp2(m - mm) + o.y * fast_exp2(o.x - mm);
                    if (z > 0.0f) c = mm + log2f(z);
                }
            }
            if (r >= a.rows) c = INFINITY;
        }
        if (part == 0) {
            s_c[lr] = c;
            s_lim[lr] = lim;
        }
    }

    // ---- Q and stage 0 are in (loads complete in issue order; with sweep 2, waiting for the statistics has waited for both)
    {
        const int later = nstages - 1;
        wait_but(later < FIRST - 1 ? (later < 0 ? 0 : later) : FIRST - 1);
    }
    __syncthreads();
    bf16x8 qf[ROW_TILES][8];
#pragma unroll
    for (int t = 0; t < ROW_TILES; ++t)
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            qf[t][ks] = as_frag(s_k[QS + rg][(32 * t + c32) * 16 + ((2 * ks + hf) ^ (c32 & 15))]);

    float cst[ROW_TILES][16];
    if constexpr (COLSUM) {
#pragma unroll
        for (int t = 0; t < ROW_TILES; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                cst[t][i] = s_c[GROUP_ROWS * rg + 32 * t + 8 * (i >> 2) + 4 * hf + (i & 3)];
    }

    float m_run[ROW_TILES], z_run[ROW_TILES];
#pragma unroll
    for (int t = 0; t < ROW_TILES; ++t) { m_run[t] = -INFINITY; z_run[t] = 0.0f; }
    const float sc = a.scale_log2;

    // LDS slots of this lane's eight K fragments inside a stage buffer
    const int krow = 32 * kt + c32;
    int kslot[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) kslot[ks] = krow * 16 + ((2 * ks + hf) ^ (krow & 15));

    // every wavefront has its rows: their buffers take the stages that are still missing of the first RING - 1
#pragma unroll
    for (int t = 0; t < ROW_TILES; ++t)
        asm volatile("" ::"v"(qf[t][0]), "v"(qf[t][1]), "v"(qf[t][2]), "v"(qf[t][3]), "v"(qf[t][4]), "v"(qf[t][5]),
                     "v"(qf[t][6]), "v"(qf[t][7])
                     : "memory");
    __syncthreads();
#pragma unroll
    for (int s = FIRST; s < RING - 1; ++s)
        if (s < nstages) stage_issue(s);

    // ---- main loop, software pipelined over stages -------------------------------------
    // Iteration s issues the MFMAs of stage s while the vector ALUs reduce the
    // accumulators of stage s-1 (softmax statistics or column sums), so the matrix pipe
    // and the VALU of a wavefront overlap instead of alternating.
    int ahead = -1;                                        // the stage that the main loop has left off at, its own request made
    const auto stage_sync = [&](int s) {
        if (s > 0) {
            // stage s has landed once at most the loads of the later stages issued so far
            // (up to RING - 2 of them) are outstanding
            const int later = nstages - 1 - s;
            wait_but(later < RING - 2 ? later : RING - 2);
            // The partial column sums that this wavefront has written to LDS are there before it reaches the barrier.  The barrier asks
            // the compiler for this wait, but where it is reached over a loop's back edge (clang of ROCm 7.2) there was none, and now
            // and then a stage's sums were flushed before a wavefront's part of them had arrived: one pass in 500 of 1024
            // units of 2000 keys, 32 columns in front of the last partial stage.
            if constexpr (COLSUM) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __syncthreads();                               // every wavefront: stage s landed, stage s-1 consumed
        }
        if (s != ahead && s + RING - 1 < nstages) stage_issue(s + RING - 1);   // overwrites the buffer of stage s-1
    };
    // eight steps of 16 features, in two halves: the fragments of a half, and its products
    const auto fragments = [&](int ring, int half, bf16x8 (&kf)[8]) {
        const uint4* buf = &s_k[ring][0];
#pragma unroll
        for (int ks = 4 * half; ks < 4 * half + 4; ++ks) kf[ks] = as_frag(buf[kslot[ks]]);
    };
    const auto products = [&](int half, const bf16x8 (&kf)[8], f32x16 (&acc)[ROW_TILES]) {
        if (half == 0) {
#pragma unroll
            for (int t = 0; t < ROW_TILES; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
        }
#pragma unroll
        for (int ks = 4 * half; ks < 4 * half + 4; ++ks)
#pragma unroll
            for (int t = 0; t < ROW_TILES; ++t) {
                if constexpr (!COLSUM)   // keys x rows: acc[t][i] = key tile + 8*(i/4) + 4*hf + i%4, this lane's row
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[t][ks], acc[t], 0, 0, 0);
                else                     // rows x keys: acc[t][i] = row 64*rg + 32*t + 8*(i/4) + 4*hf + i%4, key tile + c32
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[t][ks], kf[ks], acc[t], 0, 0, 0);
            }
    };
    const auto mma = [&](int s, f32x16 (&acc)[ROW_TILES]) {
        bf16x8 kf[8];
        fragments(s % RING, 0, kf);
        fragments(s % RING, 1, kf);
        products(0, kf, acc);
        products(1, kf, acc);
    };
    // online update of a row tile's statistics from its accumulators (the exact running maximum)
    const auto online = [&](f32x16& acc, int t, auto masked_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        float tmax = acc[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, acc[i]);
        const float mnew = fmaxf(m_run[t], tmax * sc);
        const float mref = (MASKED && mnew == -INFINITY) ? 0.0f : mnew;   // every key hidden so far
        float sum = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += fast_exp2(fmaf(acc[i], sc, -mref));
        z_run[t] = z_run[t] * fast_exp2(m_run[t] - mref) + sum;
        m_run[t] = mnew;
    };
    // Reduction of the accumulators of a fully visible stage, a row tile after the other, then what is left of it.
    // Statistics: the reference of a row's exponents does not have to be the maximum: any logit the row has had keeps Z at 1 or
    // more, and fp32 holds sums far above it.  So a stage only sums against the reference it finds (no maximum,
    // no rescaling); one whose sum passes 2^64 - the first of the chunk, whose reference is -inf, and any
    // with a logit 64 octaves above the reference - is reduced again with the maximum.
    float sums[COLSUM ? 1 : ROW_TILES];                    // of the stage: a key's over the rows so far; a row's over the keys, by tile
    const auto reduce_tile = [&](int t, const f32x16 (&acc)[ROW_TILES]) {
        if constexpr (COLSUM) {
            if (t == 0) sums[0] = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) sums[0] += fast_exp2(fmaf(acc[t][i], sc, -cst[t][i]));
        } else {
            sums[t] = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) sums[t] += fast_exp2(fmaf(acc[t][i], sc, -m_run[t]));
        }
    };
    const auto write_colsum = [&](float colsum, int slot) {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(colsum), __float_as_uint(colsum), false, false);
        colsum = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        if (hf == 0) s_part[slot][rg][32 * kt + c32] = colsum;
    };
    const auto reduce_rest = [&](int slot, f32x16 (&acc)[ROW_TILES]) {
        if constexpr (COLSUM) {
            write_colsum(sums[0], slot);
        } else {
            bool small = true;
#pragma unroll
            for (int t = 0; t < ROW_TILES; ++t) small = small && sums[t] < 1.8446744e19f;
            if (__ballot(!small) == 0ull) {                // uniform
#pragma unroll
                for (int t = 0; t < ROW_TILES; ++t) z_run[t] += sums[t];
            } else {
#pragma unroll
                for (int t = 0; t < ROW_TILES; ++t) online(acc[t], t, std::integral_constant<bool, false>{});
            }
        }
    };
    const auto reduce = [&](int s, f32x16 (&acc)[ROW_TILES]) {
#pragma unroll
        for (int t = 0; t < ROW_TILES; ++t) reduce_tile(t, acc);
        reduce_rest(s % (2 * FLUSH), acc);
    };
    // of a stage some key of which is hidden from some row
    const auto reduce_masked = [&](int s, f32x16 (&acc)[ROW_TILES]) {
        const int32_t tile_key0 = key_lo + stage_pos(s) * STAGE_KEYS + 32 * kt;
        float colsum = 0.0f;
#pragma unroll
        for (int t = 0; t < ROW_TILES; ++t) {
            if constexpr (!COLSUM) {
                const int32_t lim = my_lim[t];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int32_t key = tile_key0 + 8 * (i >> 2) + 4 * hf + (i & 3);
                    acc[t][i] = key <= lim ? acc[t][i] : -INFINITY;
                }
                online(acc[t], t, std::integral_constant<bool, true>{});
            } else {
                const int32_t key = tile_key0 + c32;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int row = GROUP_ROWS * rg + 32 * t + 8 * (i >> 2) + 4 * hf + (i & 3);
                    const float p = fast_exp2(fmaf(acc[t][i], sc, -cst[t][i]));
                    colsum += key <= s_lim[row] ? p : 0.0f;
                }
            }
        }
        if constexpr (COLSUM) write_colsum(colsum, s % (2 * FLUSH));
    };
    // Column sums of the stages before `to` that have not been written yet: the row groups' partial sums added up (complete after
    // the barrier that follows their reduction), FLUSH stages at a time - a turn's, four, six in the narrow workgroups - and a stage per
    // wavefront.  With a store in every stage, by the first wavefront, that one has more to do than the others, and the wait for its loads waits for the
    // stores among them.  (Measured with bursts of eight stages, before the main loop went by turns: one sweep, us, a store in every stage /
    // bursts, 192 units of 8192 keys, 256 rows 127.6 / 121.9, 512 of 1500..3001 57.2 / 54.8, 2048 of 2048..16 384 871 / 862, 256 of 16 384
    // 194.8 / 193; without any stores 180, whatever the size of the bursts: most of what they cost is the memory's.)
    int flushed = 0;
    const auto flush = [&](int to) {
        if constexpr (COLSUM) {
            for (int s = flushed + __builtin_amdgcn_readfirstlane(wave); s < to; s += WAVES) {
                const int32_t key = key_lo + stage_pos(s) * STAGE_KEYS + lane;
                if (key < key_hi) {
                    float v = s_part[s % (2 * FLUSH)][0][lane];
#pragma unroll
                    for (int w = 1; w < RG; ++w) v += s_part[s % (2 * FLUSH)][w][lane];
                    float* dst = &a.A[(size_t)unit * n + key];
                    *dst = row_base > 0 ? *dst + v : v;    // (this workgroup's, from the pass before: a barrier lies between them)
                }
            }
            flushed = to;
        }
    };
    // The main loop: whole turns of TURN stages, as long as every stage that they request is a fully visible one too.  The barrier stands
    // in the middle of a stage: in front of it the stage's first products and half of the reduction of the one before, with the last reads
    // of its buffer, which is free behind it; behind it the first fragments of the next stage are read, under the stage's
    // other products.  So neither the matrix pipe nor the vector unit waits for LDS behind a barrier, which the two wavefronts of a
    // SIMD reach together.  What a stage needs is known or steps on by itself - the buffer's number, the wait, the address -
    // and costs some 20 scalar instructions, not 60 and ten branches.  (One sweep / two, us, all stages
    // as in (A) / this: 256 units of 16 384 keys, 256 rows 325 / 280, 633 / 570; 192 of 8192, 256 rows 129 / 114, 253 / 238; 256 of 4096,
    // 512 rows 171 / 149, 336 / 303; 128 rows, 256 units of 16 384 198 / 187, 383 / 365, 2048 of 2048..16 384 873 / 857, 1690 / 1600.)
    const auto turns = [&](int& s, f32x16 (&acc_even)[ROW_TILES], f32x16 (&acc_odd)[ROW_TILES]) {
        if (s + TURN + RING - 1 >= nfast) return;
        bf16x8 kf[8];
        stage_sync(s);                                     // requests s + RING - 1
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        fragments(1 % RING, 0, kf);
        int p = stage_pos(s + RING);                       // place of the stage to request
        const char* from = PAGED ? nullptr : reinterpret_cast<const char*>(kbase + (int64_t)(key_lo + p * STAGE_KEYS) * a.k_sp);
        const int64_t step = (COLSUM ? -1 : 1) * (int64_t)STAGE_KEYS * a.k_sp * 16;
        const auto run = [&](int end, auto stream_tag) {
            for (; s + TURN + RING - 1 < end; s += TURN) {
                const int half = s % (2 * TURN) == 1 ? 0 : TURN;
#pragma unroll
                for (int j = 0; j < TURN; ++j) {           // stage s + j: buffer (1 + j) % RING
                    f32x16 (&acc)[ROW_TILES] = (1 + j) & 1 ? acc_odd : acc_even;
                    f32x16 (&before)[ROW_TILES] = j & 1 ? acc_odd : acc_even;
                    fragments((1 + j) % RING, 1, kf);
                    products(0, kf, acc);
                    reduce_tile(0, before);
                    wait_but(RING - 2);                    // the next stage is in
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // this one has been read, and the partial sums are in LDS
                    __syncthreads();
                    const uint4* src = PAGED ? stage_base(key_lo + p * STAGE_KEYS) : reinterpret_cast<const uint4*>(from);
                    const uint32_t dst = lds_wave + (uint32_t)((1 + j) % RING) * (STAGE_UNITS * 16u);
#pragma unroll
                    for (int i = 0; i < LPS; ++i) load_to_lds_16<decltype(stream_tag)::value>(src, lane_off[i], dst + WAVES * i * 1024u);
                    from += step;
                    p += COLSUM ? -1 : 1;
                    fragments((2 + j) % RING, 0, kf);
                    products(1, kf, acc);
#pragma unroll
                    for (int t = 1; t < ROW_TILES; ++t) reduce_tile(t, before);
                    reduce_rest(half + j, before);
                    if (j == 1 && s > TURN) flush(s - 1);
                }
            }
        };
        if constexpr (STREAM && !COLSUM) run(keep_from < nfast ? keep_from : nfast, std::integral_constant<bool, true>{});
        run(nfast, std::integral_constant<bool, STREAM && COLSUM>{});
        ahead = s;
    };
    // (A) fully visible stages: MFMAs of stage s and the reduction of stage s-1 in one block.
    // Two accumulator sets alternate (loops unrolled by two or by a turn) so that no registers are copied.
    if (nfast > 0) {
        f32x16 acc_even[ROW_TILES], acc_odd[ROW_TILES];
        stage_sync(0);
        mma(0, acc_even);
        int s = 1;
        if constexpr (TURNS) turns(s, acc_even, acc_odd);
        for (; s + 1 < nfast; s += 2) {
            stage_sync(s);
            mma(s, acc_odd);
            reduce(s - 1, acc_even);
            if (s - flushed > FLUSH) flush(s - 1);         // these were reduced in front of this stage's barrier
            stage_sync(s + 1);
            mma(s + 1, acc_even);
            reduce(s, acc_odd);
        }
        if (s < nfast) {                                   // one more stage, into the odd set
            stage_sync(s);
            mma(s, acc_odd);
            reduce(s - 1, acc_even);
            reduce(s, acc_odd);
        } else {
            reduce(s - 1, acc_even);
        }
        // at most FLUSH + 2 stages are pending: the next ones go elsewhere
        if constexpr (COLSUM) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if constexpr (COLSUM) __syncthreads();
        flush(nfast);
    }
    // (B) the few stages near the causal diagonal or past the sequence end: masked, not pipelined
    for (int s = nfast; s < nstages; ++s) {
        stage_sync(s);
        if (s - flushed >= FLUSH) flush(s);
        f32x16 acc_cur[ROW_TILES];
        mma(s, acc_cur);
        reduce_masked(s, acc_cur);
    }
    if constexpr (COLSUM) {
        __syncthreads();
        flush(nstages);
        if (row_base == 0) zero_share();
    }

    if constexpr (!COLSUM) {
        // merge the two half-waves (disjoint key subsets of the same row), then the two
        // key-tile wavefronts of the row group through LDS, then store
        __syncthreads();                                       // staging buffers are idle now
        float* s_m = reinterpret_cast<float*>(&s_k[0][0]);
        float* s_z = s_m + GROUP_ROWS * RG;
#pragma unroll
        for (int t = 0; t < ROW_TILES; ++t) {
            const float mo = other_half(m_run[t]), zo = other_half(z_run[t]);
            const float mf = fmaxf(m_run[t], mo);
            float zf = 0.0f;
            if (mf > -INFINITY) zf = z_run[t] * fast_exp2(m_run[t] - mf) + zo * fast_exp2(mo - mf);
            m_run[t] = mf;
            z_run[t] = zf;
        }
        if (kt == 1 && hf == 0) {
#pragma unroll
            for (int t = 0; t < ROW_TILES; ++t) {
                s_m[GROUP_ROWS * rg + 32 * t + c32] = m_run[t];
                s_z[GROUP_ROWS * rg + 32 * t + c32] = z_run[t];
            }
        }
        __syncthreads();
        if (kt == 0 && hf == 0) {
            float* st = a.ws + (((size_t)unit * a.nchunks + chunk) * a.rows_pad) * 2;
#pragma unroll
            for (int t = 0; t < ROW_TILES; ++t) {
                const int32_t r = GROUP_ROWS * rg + 32 * t + c32;
                const float mo = s_m[r], zo = s_z[r];
                const float mf = fmaxf(m_run[t], mo);
                float zf = 0.0f;
                if (mf > -INFINITY) zf = z_run[t] * fast_exp2(m_run[t] - mf) + zo * fast_exp2(mo - mf);
                if constexpr (ONE) {
                    s_one[r] = zf > 0.0f ? mf + log2f(zf) : INFINITY;
                } else {
                    st[(row_base + r) * 2] = mf;
                    st[(row_base + r) * 2 + 1] = zf;
                }
            }
        }
    }
}

// Workgroups narrower than a match tile: the match runs as a launch of its own in front of the sweep.
hipError_t match_in_front(const ScoreArgs& a, const MatchRider& m, hipStream_t st)
{
    return launch_match(m.tok, a.seq_len, a.batch, a.n, *m.tab, m.anchor_B, m.allow, m.anchor, m.spons, m.vouch, st);
}

RiderArgs rider_args(const ScoreArgs& a, const MatchRider& m, unsigned blocks)
{
    RiderArgs r;
    r.m = make_match_args(m.tok, a.seq_len, a.batch, a.n, m.anchor_B, m.allow, m.anchor, m.spons, m.vouch);
    r.tab = *m.tab;
    r.score_blocks = blocks;
    return r;
}

template <int RG, int RT, bool COLSUM, bool STREAM, bool PASSES, bool TURNS>
hipError_t launch_sweep(const ScoreArgs& a, unsigned blocks, const MatchRider* rider, hipStream_t st)
{
    if constexpr (RG == 1) {
        if (rider) {
            const hipError_t e = match_in_front(a, *rider, st);
            if (e != hipSuccess) return e;
        }
    } else if (rider) {
        const RiderArgs r = rider_args(a, *rider, blocks);
        const dim3 grid(blocks + (unsigned)r.m.tiles * (unsigned)r.m.batch);
        if (a.table) hipLaunchKernelGGL((score_match_kernel<RG, RT, COLSUM, true, STREAM, PASSES, TURNS>), grid, dim3(128 * RG), 0, st, a, r);
        else hipLaunchKernelGGL((score_match_kernel<RG, RT, COLSUM, false, STREAM, PASSES, TURNS>), grid, dim3(128 * RG), 0, st, a, r);
        return hipGetLastError();
    }
    if (a.table) hipLaunchKernelGGL((score_kernel<RG, RT, COLSUM, true, STREAM, PASSES, TURNS>), dim3(blocks), dim3(128 * RG), 0, st, a);
    else hipLaunchKernelGGL((score_kernel<RG, RT, COLSUM, false, STREAM, PASSES, TURNS>), dim3(blocks), dim3(128 * RG), 0, st, a);
    return hipGetLastError();
}

template <int RG, int RT, bool STREAM, bool TURNS>
hipError_t launch_once(const ScoreArgs& a, unsigned blocks, const MatchRider* rider, hipStream_t st)
{
    if constexpr (RG == 1) {
        if (rider) {
            const hipError_t e = match_in_front(a, *rider, st);
            if (e != hipSuccess) return e;
        }
    } else if (rider) {
        const RiderArgs r = rider_args(a, *rider, blocks);
        const dim3 grid(blocks + (unsigned)r.m.tiles * (unsigned)r.m.batch);
        if (a.table) hipLaunchKernelGGL((score_once_match_kernel<RG, RT, true, STREAM, TURNS>), grid, dim3(128 * RG), 0, st, a, r);
        else hipLaunchKernelGGL((score_once_match_kernel<RG, RT, false, STREAM, TURNS>), grid, dim3(128 * RG), 0, st, a, r);
        return hipGetLastError();
    }
    if (a.table) hipLaunchKernelGGL((score_once_kernel<RG, RT, true, STREAM, TURNS>), dim3(blocks), dim3(128 * RG), 0, st, a);
    else hipLaunchKernelGGL((score_once_kernel<RG, RT, false, STREAM, TURNS>), dim3(blocks), dim3(128 * RG), 0, st, a);
    return hipGetLastError();
}

template <int RG, int RT, bool PASSES, bool TURNS>
hipError_t launch_rg(ScoreArgs a, int64_t units, const MatchRider* rider, int32_t gathered, hipStream_t st)
{
    // One launch per sweep over all units.  (Splitting the units into cache-sized groups
    // so that sweep 2 re-reads its keys from the last-level cache was measured slower.)
    a.units = (int32_t)units;
    const unsigned blocks = (unsigned)(8ll * ((units + 7) / 8) * a.nchunks);
    // More workgroups than run at once: the second sweep takes them in the opposite order, so that it begins with the keys that
    // the first has read last and that the last-level cache (256 MB) still holds.  (Whole pass, us, units of several chunks, in the same order / the
    // opposite: 320 units of 4096 keys, K = 1024 190 / 184, 384 of 8000 309 / 305, 320 of 16 384 491 / 491, with 64 rows 486 / 493, 256 rows, 192 units of
    // 8192 248 / 249; ragged ones lose by it, 320 of 2048..8192 178 / 182, 336 of 4096..16 384 410 / 422.)  Where all run at once the stages of each do that
    // already.
    constexpr int64_t RESIDENT = RG == 1 ? 3 : (RG == 2 ? 2 : 1);       // workgroups per compute unit, by their stage rings
    const bool rounds = blocks > RESIDENT * compute_units();
    a.backwards = !a.lse && rounds;
    // Keys that will not be read again are loaded with the streaming hint, which leaves less to evict: those of the only or the
    // second sweep, and in the first all but the last LLC_BYTES, which the second will begin with - of the last units or, where all
    // run at once, of the last stages of each.  (Counted as if every sequence had n keys.  The last units of a ragged batch are its shortest, of
    // which less is kept.)  (Whole pass, us, units of several chunks, the first sweep without / with: 320 units of 4096 keys 151 / 150, 384 of 8000 318 / 305,
    // 320 of 16 384 507 / 491, with 64 rows 522 / 493, 256 of 16 384 389 / 383, with 64 rows 385 / 368, ragged 336 of 4096..16 384 438 / 422, but 320 of
    // 2048..8192 180 / 182; the second: 384 of 8000 317 / 305, 256 of 16 384 401 / 383, 320 of 4096 149.8 / 149.9; one sweep: 256 units of 4096 keys 59 / 52,
    // of 16 384 208 / 195.  Streaming both sweeps of 256 units of 4096 keys: 5 % slower.)  Not below SMALL_BYTES, where the keys may
    // be in the caches (64 units of 4096 keys 31 -> 33), and not the first sweep of 256 rows, which is bound by arithmetic
    // and loses more to the test than it gains; passes over a chunk's rows read its keys several times.  Where an eighth of the
    // keys or more is gathered next and the cache holds a good part of them, the second sweep leaves them there (evict pass,
    // 1024 rows gathered, over 256 units of 4096 keys 151 -> 145, over 320 186.2 -> 184.4).  Units of one chunk have rules of their own, below.
    constexpr int64_t LLC_BYTES = int64_t(256) << 20, SMALL_BYTES = int64_t(128) << 20;
    const int64_t bytes = units * a.n * 256;
    const bool stream = !PASSES && bytes > SMALL_BYTES && !(gathered >= a.n / 8 && bytes <= 2 * LLC_BYTES);
    const auto column_sums = [&](const MatchRider* with) {
        if (stream) return launch_sweep<RG, RT, true, !PASSES, PASSES, TURNS>(a, blocks, with, st);
        return launch_sweep<RG, RT, true, false, PASSES, TURNS>(a, blocks, with, st);
    };
    if (a.lse) return column_sums(rider);                  // the row normalisers are given: column sums alone
    if (PASSES || a.nchunks > 1) {
        a.keep_place = 0x7FFFFFFF;
        a.keep_stage = 1024;
        if (rounds) a.keep_place = (int32_t)(units - units * LLC_BYTES / bytes);
        else a.keep_stage = (int32_t)(1024 - 1024 * LLC_BYTES / bytes);
        constexpr bool FIRST = RG < 4;
        const hipError_t e = FIRST && bytes > LLC_BYTES ? launch_sweep<RG, RT, false, FIRST, PASSES, TURNS>(a, blocks, rider, st)
                                                        : launch_sweep<RG, RT, false, false, PASSES, TURNS>(a, blocks, rider, st);
        if (e != hipSuccess) return e;
        return column_sums(nullptr);
    }
    // One chunk per unit: no workgroup needs another one's statistics, and one launch does both sweeps (score_once).  (Whole pass, us, two
    // launches / one.  128 rows: 512 units of 700 keys 62.1 / 56.4, of 3000 162.5 / 156.0, 1024 of 1500 187 / 170, paged 2048 of 1500..3001 534 /
    // 491, 4096 968 / 871, 2048 of 5000 1012 / 949, of 2048..16 384 1772 / 1686; 64 rows, 2048 of 2000 489 / 454, of 2048..16 384 1835 / 1660;
    // 256 rows, 256 of 1000 63.0 / 56.4, 2048 of 2000 756 / 707, of 8000 2404 / 2292.)
    // The second sweep has the streaming hint: the cache is full of the keys of the workgroups that run at once, and what they read for the last time should
    // not displace them.  Neither sweep has it where there are up to SMALL_BYTES of keys and a third of them or more is gathered next: the cache then has
    // room for both.  (Whole pass, us, without / with, K rows gathered.  1024 of 3000 keys 313 / 294, of 1500, K = 1024 317 / 315, of 900, K = 500 187 / 183,
    // 256 rows, 512 of 1500, K = 1024 211 / 207; 512 of 1900 140.6 / 140.2 with K = 500, 178.7 / 180.7 with 1024.  Up to SMALL_BYTES: 512 of 700, K = 600
    // 95.0 / 97.3, of 1000, K = 800 123.0 / 124.9, paged 500..1000, K = 400 90.9 / 92.9, 256 rows, 256 of 1000, K = 500 72.2 / 75.0; but 512 of 1000, K = 250
    // 83.3 / 83.1, of 700, K = 16 50.3 / 50.5, 1024 of 500, K = 128 98.5 / 97.6, and the scores alone, 512 of 180 15.1 / 14.2.)
    // The first sweep, with up to 128 rows, has the hint as well but for the last keep_last stages of a unit: twice what a workgroup's share of
    // the cache holds, 64 stages (1 MB), 42 with 64 rows.  Without it long units of 64 rows lose more to what the workgroups push out of the cache
    // between a unit's sweeps than one launch gives.  (Whole pass, us, two launches / one without / with the hint: 64 rows, 512 units of 32 768 keys
    // 1448 / 1506 / 1424, of 16 384 746 / 762 / 728, paged 1671 / 1688 / 1638 of 32 768, 2048 of 2048..16 384 1800 / 1685 / 1641; 128 rows, 512 of
    // 8000 412 / 399 / 385, of 16 384 781 / 778 / 753, 2048 of 6000 1215 / 1150 / 1122, of 16 384 2991 / 2996 / 2966, of 2048..16 384 1768 / 1706 /
    // 1669.  With the share itself 4096 of 3000 1257 for 1241, with three times the share 512 of 8000 393, 2048 of 6000 1153.)  128 rows with fewer than
    // 48 stages (no TURNS) would stream nothing and go without the test.
    // Several chunks per unit in one launch, the workgroups of a unit waiting for each other's statistics, was measured as well: 256
    // units of 4096 keys 144.7 / 139.9, 8 of 4096 18.1 / 19.4, 256 of 8000 201 / 211.
    // (These instances come last: the compiler emits kernels in the order of use here, and the two launches of a pass run 0.5 % faster with less code
    // between them: 256 units of 4096 keys, K = 1024 146.1 -> 145.3.)
    if constexpr (!PASSES) {
        a.backwards = 0;
        const int64_t at_once = blocks < RESIDENT * compute_units() ? blocks : RESIDENT * compute_units();
        a.keep_last = (int32_t)(2 * LLC_BYTES / (STAGE_KEYS * 256) / at_once);
        // (a pass takes workgroups of two wavefronts, and one chunk of 48 stages per unit, only with more keys than that)
        if constexpr (RG == 4 || (RG == 2 && !TURNS)) {
            if (bytes <= SMALL_BYTES && 3 * (int64_t)gathered >= a.n) return launch_once<RG, RT, false, TURNS>(a, blocks, rider, st);
        }
        return launch_once<RG, RT, true, TURNS>(a, blocks, rider, st);
    }
    return hipErrorInvalidValue;                           // (not reached)
}

}  // namespace

namespace {

int32_t padded_rows(int32_t rows)
{
    if (rows <= 128) return 128;
    if (rows <= 256) return 256;
    return 512;
}

struct ScorePlan {
    int32_t rows, rows_pad;
    int32_t chunk_keys, nchunks;       // chunks per unit, and what one has of a sequence of n keys (a shorter one is divided by as many)
    int64_t units;
};

// The plan whose statistics ta_workspace_bytes makes room for: chunks as long as possible while the grid still offers about
// two workgroups per compute unit, at least 512 keys, never more than 32 per unit.
ScorePlan base_plan(const ta_layout& lay)
{
    ScorePlan p;
    p.rows = (lay.hq / lay.hkv) * lay.window;
    p.rows_pad = padded_rows(p.rows);
    p.units = (int64_t)lay.layers * lay.batch * lay.hkv;
    const int64_t want_blocks = 2 * (int64_t)compute_units();
    int64_t per_unit = (want_blocks + p.units - 1) / p.units;            // chunks per unit we would like
    per_unit = per_unit < 1 ? 1 : (per_unit > MAX_CHUNKS ? MAX_CHUNKS : per_unit);
    int64_t ck = ((lay.n + per_unit - 1) / per_unit + STAGE_KEYS - 1) / STAGE_KEYS * STAGE_KEYS;
    if (ck < 512) ck = 512;
    while (ck * MAX_CHUNKS < lay.n) ck += STAGE_KEYS;
    p.chunk_keys = (int32_t)ck;
    p.nchunks = (lay.n + p.chunk_keys - 1) / p.chunk_keys;
    return p;
}

int64_t stats_bytes(const ScorePlan& p, int64_t nchunks) { return p.units * nchunks * p.rows_pad * 2 * (int64_t)sizeof(float); }

// The room for statistics that a workspace of ws_bytes (at least the base plan's) offers: that of MAX_CHUNKS chunks per unit, at
// most 8 MiB, or if the workspace has less the base plan's.  There is nothing between the two: the chunks group the sums of a
// row's normaliser, and its last bits should not follow the exact size of the caller's buffer.
int64_t stats_room(const ta_layout& lay, int64_t ws_bytes)
{
    const ScorePlan p = base_plan(lay);
    const int64_t need = stats_bytes(p, p.nchunks), most = stats_bytes(p, MAX_CHUNKS);
    const int64_t full = most < (int64_t(8) << 20) ? most : int64_t(8) << 20;
    return full > need && ws_bytes >= full ? full : need;
}

// The plan that runs, given `room` bytes for the statistics (at least the base plan's): the chunk count whose fullest compute
// unit is done first.  A workgroup costs its stages plus the prologue (Q fragments, first stages, statistics merge) and
// epilogue, about SETUP stages' time; a compute unit that gets k of them costs k times that, and one workgroup of four
// wavefronts alone (rows_pad 128) does not quite fill it.  At most 32 chunks per unit, of at least two stages.  (Score step in
// us, base plan / this one: 8 units of 4096 keys, 128 rows 22 / 19, 256 rows 32 / 23; 64 units of 4096 keys 39 / 36; 192
// units of 8192 keys, 256 rows 316 / 281: 576 workgroups on 256 compute units that hold one each become 768.)
ScorePlan make_plan(const ta_layout& lay, int64_t room)
{
    ScorePlan p = base_plan(lay);
    constexpr int64_t SETUP = 6, ALONE = 115;              // stages; per cent
    const int64_t cus = compute_units(), stages = (lay.n + STAGE_KEYS - 1) / STAGE_KEYS;
    int64_t best = -1;
    for (int64_t c = 1; c <= MAX_CHUNKS && (c == 1 || stages >= 2 * c); ++c) {
        const int64_t per_chunk = (stages + c - 1) / c, chunks = (stages + per_chunk - 1) / per_chunk;
        if (chunks > p.nchunks && stats_bytes(p, chunks) > room) break;
        const int64_t k = (p.units * chunks + cus - 1) / cus;
        const int64_t cost = k * (per_chunk + SETUP) * (k == 1 && p.rows_pad == 128 ? ALONE : 100);
        if (best < 0 || cost < best) {
            best = cost;
            p.chunk_keys = (int32_t)(per_chunk * STAGE_KEYS);
        }
    }
    p.nchunks = (lay.n + p.chunk_keys - 1) / p.chunk_keys;
    return p;
}

}  // namespace

size_t score_workspace_bytes(const ta_layout& lay)
{
    const ScorePlan p = base_plan(lay);
    return (size_t)stats_bytes(p, p.nchunks);              // per-chunk row statistics (m, Z)
}

int64_t score_grid_blocks(const ta_layout& lay)
{
    const ScorePlan p = make_plan(lay, INT64_MAX);
    const int64_t base = base_plan(lay).nchunks;
    return 8 * ((p.units + 7) / 8) * (p.nchunks > base ? p.nchunks : base);
}

// Units of at most 64 rows: two wavefronts per workgroup instead of four of which two work on padding (score step, two sweeps,
// us: 256 units of 4096 keys 104 -> 95, of 16384 keys 387 -> 369, of 40000 keys 481 -> 463; 8 units of 4096 keys 13.6 -> 13.2).
// Such a workgroup cannot take a match tile along, so where there is one to take, the keys have to be many enough (256 MB) for
// the gain to pay for a launch of its own, some 5 us.  Paged keys, which cost the wider workgroups more, gain from half as many on
// (whole pass, with the match in the sweep / in front, us: 8 units of 1000 keys 19.9 / 23.6, 64 of 4000 42.4 / 45.4, 256 of 3000
// 91.0 / 87.6, of 4096 115.1 / 113.3).
constexpr int64_t NARROW_KEYS = int64_t(1) << 20, NARROW_KEYS_PAGED = int64_t(1) << 19;

hipError_t launch_score(const void* Q, const void* K, const ta_layout& lay, const int32_t* seq_len,
                        int causal, float* A, float* ws, size_t ws_bytes, const float* lse, const MatchRider* rider,
                        const ta_paged_kv* pg, const LayerPtrs* lp, hipStream_t st, int32_t gathered)
{
    const ScorePlan p = make_plan(lay, lse ? INT64_MAX : stats_room(lay, (int64_t)ws_bytes));
    ScoreArgs a;
    a.Ql = lp ? reinterpret_cast<const uint4* const*>(&lp->Q[0]) : nullptr;
    a.Kl = lp ? reinterpret_cast<const uint4* const*>(&lp->K[0]) : nullptr;
    a.lse = lse;
    a.table = pg ? pg->block_table : nullptr;
    a.k_spage = pg ? pg->stride[1] / 8 : 0;
    a.page_size = pg ? pg->page_size : 0;
    a.max_pages = pg ? pg->max_pages : 0;
    a.num_pages = pg ? pg->num_pages : 0;
    a.page_shift = -1;
    if (pg && (pg->page_size & (pg->page_size - 1)) == 0) {
        a.page_shift = 0;
        while ((1 << a.page_shift) < pg->page_size) ++a.page_shift;
    }
    a.Q = (const uint4*)Q;
    a.K = (const uint4*)K;
    a.seq_len = seq_len;
    a.A = A;
    a.ws = ws;
    a.q_sl = lay.q_stride[0] / 8;
    a.q_sb = lay.q_stride[1] / 8;
    a.q_sh = lay.q_stride[2] / 8;
    if (pg) {
        a.k_sl = pg->stride[0] / 8;
        a.k_sb = 0;
        a.k_sp = (int32_t)(pg->stride[2] / 8);
        a.k_sh = pg->stride[3] / 8;
    } else {
        a.k_sl = lay.kv_stride[0] / 8;
        a.k_sb = lay.kv_stride[1] / 8;
        a.k_sh = lay.kv_stride[2] / 8;
        a.k_sp = (int32_t)(lay.kv_stride[3] / 8);
    }
    a.batch = lay.batch;
    a.hkv = lay.hkv;
    a.G = lay.hq / lay.hkv;
    a.W = lay.window;
    a.inv_W = (1u << 20) / (uint32_t)lay.window + 1;
    a.by_chunks = divider((uint32_t)p.nchunks);
    a.by_hkv = divider((uint32_t)lay.hkv);
    a.by_batch = divider((uint32_t)lay.batch);
    a.n = lay.n;
    a.rows = p.rows;
    a.rows_pad = p.rows_pad;
    a.nchunks = p.nchunks;
    a.causal = causal;
    a.scale_log2 = (float)(1.4426950408889634 / sqrt((double)lay.d));
    // The kernels with the main loop of whole turns: with more than 128 rows from chunks of 12 stages on, for up to 128 rows from chunks of 48.  Two
    // workgroups or more share a compute unit there and cover each other's waits, the longer code has to be fetched, and it pays for itself later.  (Whole
    // pass, us, without / with: 8 units of 4096 keys, chunks of 2 stages, 18.37 / 18.5, 512 paged ones of 1500..3001, of up to 47, 139.2 / 139.8, 256 of 4096,
    // of 32, 144.4 / 144.3; one sweep over 256 of 16 384, of 128, 193 / 188; narrow workgroups 256 of 4096 47.5 / 47.5.  512 rows, two sweeps: 8 units of
    // 4096 keys, chunks of 2, 30.5 / 33.3, of 9000, of 5, 42.9 / 48.2, 256 of 700, of 11, 79.0 / 79.8, of 1000, of 16, 104 / 101, of 4096 333 / 299,
    // although its column sums hold 24 registers of a lane in scratch, 6 without: those of the state between the passes, outside the loop.)
    const int32_t stages = p.chunk_keys / STAGE_KEYS;
    switch (a.rows_pad) {
        // two 32-row tiles per wavefront (one tile per wavefront with twice the wavefronts - four
        // per SIMD instead of two - was measured: same time at 128 rows, 5 % slower at 256)
        case 128:
            if (p.rows <= 64 && (!rider || p.units * lay.n >= (a.table ? NARROW_KEYS_PAGED : NARROW_KEYS))) return launch_rg<1, 2, false, false>(a, p.units, rider, gathered, st);
            if (stages >= 48) return launch_rg<2, 2, false, true>(a, p.units, rider, gathered, st);
            return launch_rg<2, 2, false, false>(a, p.units, rider, gathered, st);
        case 256:
            if (stages >= 12) return launch_rg<4, 2, false, true>(a, p.units, rider, gathered, st);
            return launch_rg<4, 2, false, false>(a, p.units, rider, gathered, st);
        // 512 rows: two passes of 256 (eight row groups at once leave 128 registers per lane: spills, 3x slower), in kernels of
        // their own: the pass loop costs the column sums' main loop the registers that keep its two pipes busy (1.5 %)
        default:
            if (stages >= 12) return launch_rg<4, 2, true, true>(a, p.units, rider, gathered, st);
            return launch_rg<4, 2, true, false>(a, p.units, rider, gathered, st);
    }
}

}  // namespace ta
