// Incremental form of the eviction pass: one generation step for every
// sequence and unit (Sec. 3.1 "after each generation step"; Alg. 1 with its
// budget-decay step; Sec. 3.2 "Token selection").
//
// Two launches per step, or, where units are not too many and the caller has words for them to count in, the second alone
// (FUSED below):
//   decode_seq_vouch_kernel  per sequence: append the token, test the anchor table at the new
//                            position only, set its budget; voucher and sponsor flag of every
//                            position from the current budgets
//   decode_unit_kernel       one to eight wavefronts per unit: write the new k/v row into the
//                            free slot, add the decode queries' softmax weights over
//                            the cached rows to A (H2O-style cumulative attention,
//                            Eq. 1), free the slot that ranks last under the
//                            (class, u, position) order; trailing workgroups of the same
//                            launch do B_i <- decay * B_i for every position
// The unit kernel is the hot one: it reads the unit's K slots once (HBM bound,
// (K+1) * 256 B per unit per step).  The logits of the group's query heads over the
// slots are a thin contraction that runs on the matrix cores (16-row key tiles x 16
// head columns), fed with whole key rows that are turned into operand fragments
// through a small LDS tile.
#include <math.h>
#include <type_traits>

#include "ta_internal.h"
#include "ta_order.h"
#include "ta_wave.h"

namespace ta {

namespace {

constexpr int DU_THREADS = 256;
constexpr int MAX_GROUP = 16;                              // query heads per KV head (the columns of an MFMA tile)

struct DecodeTable {
    int32_t rid[TA_MAX_TABLE][TA_MAX_GRAM];                // n-grams reversed: rid[e][0] = last token
    int32_t len[TA_MAX_TABLE];
    int32_t E;
    float B;
};

// K/V slots kept in a paged pool (ta_decode_state::pages): strides in 16-byte units.
struct SlotPages {
    const int32_t* table;                                  // [batch][max_pages]
    int64_t s_layer, s_page, s_slot, s_head;
    int32_t page_size, max_pages, num_pages;
    int32_t page_shift;                                    // log2(page_size) when it is a power of two, else -1
};

__device__ __forceinline__ int32_t page_index(const SlotPages& pg, int32_t slot)
{
    return pg.page_shift >= 0 ? slot >> pg.page_shift : slot / pg.page_size;
}

__device__ __forceinline__ int32_t clamp_page(const SlotPages& pg, int32_t page)
{
    return page < 0 ? 0 : (page >= pg.num_pages ? pg.num_pages - 1 : page);
}

// ---- state initialisation -----------------------------------------------------
constexpr int INIT_ITERS = 2;
constexpr int INIT_ROWS = DU_THREADS / 16 * INIT_ITERS;    // rows of one of the two tensors per workgroup

struct InitArgs {
    const int32_t* tok;
    const int32_t* seq_len;
    const uint8_t* anchor;
    const float* anchor_B;
    const float* A;
    const int32_t* idx;
    const int32_t* cnt;
    const uint4* Kout;
    const uint4* Vout;
    int64_t rows;                                          // units * slots
    int64_t slot_blocks, row_blocks;                       // workgroups of the slot tables; of the keys, and as many of the values
    int64_t seq_blocks;                                    // of the per-sequence arrays
    Divider by_slots, by_hkv, by_batch;
    int32_t n;
    float B;
};

// Per-sequence arrays of 256 positions.
__device__ __forceinline__ void init_sequence(const ta_decode_state& st, const InitArgs& a, int32_t r)
{
    const int32_t tiles = (st.cap + DU_THREADS - 1) / DU_THREADS;
    const int b = r / tiles;
    const int p = (r - b * tiles) * DU_THREADS + (int)threadIdx.x;
    int32_t nb = a.seq_len ? a.seq_len[b] : a.n;
    nb = nb < 0 ? 0 : (nb > a.n ? a.n : nb);
    if (p == 0) st.len[b] = nb;
    if (p >= st.cap) return;
    const size_t o = (size_t)b * st.cap + p;
    if (p < nb) {
        const size_t i = (size_t)b * a.n + p;
        const uint8_t an = a.anchor[i];
        st.tok[o] = a.tok[i];
        st.anchor[o] = an;
        st.budget[o] = an ? (a.anchor_B ? a.anchor_B[i] : a.B) : 0.0f;
    } else {
        st.tok[o] = 0;
        st.anchor[o] = 0;
        st.budget[o] = 0.0f;
    }
}

// The unit of a row of the flat [units][slots] order.
__device__ __forceinline__ int32_t init_unit(const InitArgs& a, int64_t row, int32_t slots)
{
    return a.rows <= 0x7FFFFFFF ? (int32_t)divide((uint32_t)row, a.by_slots) : (int32_t)(row / slots);
}

// Position and accumulated attention of a slot per thread.
__device__ __forceinline__ void init_slots(const ta_decode_state& st, const InitArgs& a, int64_t row)
{
    if (row >= a.rows) return;
    const int32_t slots = st.K + 1;
    const int32_t unit = init_unit(a, row, slots), s = (int32_t)(row - (int64_t)unit * slots);
    int32_t p = a.idx[(size_t)unit * st.K + (s < st.K ? s : st.K - 1)];
    const bool kept = s < st.K && s < a.cnt[unit];
    p = p < 0 ? 0 : (p >= a.n ? a.n - 1 : p);
    st.pos[row] = kept ? p : -1;
    st.A[row] = kept && a.A ? a.A[(size_t)unit * a.n + p] : 0.0f;
}

// The slot tables, the keys, the values, then the per-sequence arrays.  Rows move as in the compaction: INIT_ROWS consecutive slots of the
// flat [units][slots] order and one tensor per workgroup, 16 lanes per row, all loads of a lane before its first store, bound by HBM; the slot tables, two
// dependent loads each, have threads of their own.  (us, both tensors by 64 rows behind their slots' tables / this: 256 units of 1025 slots
// 53.2 / 45.3, over pages 53.9 / 46.1; 64 of 1025 17.5 / 14.4; 8192 of 65 97.7 / 89.5; 4096 of 257 183 / 175; 16 384 of 257 734 / 702.  Keys stored without the
// streaming hint, for the first step to find in the last-level cache: 44.6, 44.8, 13.2, 85.3, 166.5, 699, but what comes next, in use the model's
// next pass, then writes them back: a read of 1 GiB behind 4096 of 257 takes 302 us instead of 286.)
template <bool PAGED>
__global__ void __launch_bounds__(DU_THREADS)
decode_init_kernel(ta_decode_state st, InitArgs a, SlotPages pg)
{
    int64_t block = (int64_t)blockIdx.y * GRID_LINE + blockIdx.x;
    if (block < a.slot_blocks) {
        init_slots(st, a, block * DU_THREADS + threadIdx.x);
        return;
    }
    block -= a.slot_blocks;
    if (block >= 2 * a.row_blocks) {
        if (block < 2 * a.row_blocks + a.seq_blocks) init_sequence(st, a, (int32_t)(block - 2 * a.row_blocks));
        return;
    }
    const bool values = block >= a.row_blocks;
    if (values) block -= a.row_blocks;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int32_t slots = st.K + 1;
    const int64_t row0 = block * INIT_ROWS;
    const int32_t unit0 = init_unit(a, row0, slots);       // uniform
    const int32_t slot0 = (int32_t)(row0 - (int64_t)unit0 * slots);
    const int lane16 = threadIdx.x & 15, rsub = threadIdx.x >> 4;
    const u32x4* in = reinterpret_cast<const u32x4*>(values ? a.Vout : a.Kout);
    u32x4* out = reinterpret_cast<u32x4*>(values ? st.Vc : st.Kc);
    int64_t to[INIT_ITERS];
    bool live[INIT_ITERS];
    int32_t slot[INIT_ITERS], count[INIT_ITERS];
    u32x4 v[INIT_ITERS];
#pragma unroll
    for (int i = 0; i < INIT_ITERS; ++i) {
        const int32_t off = 16 * i + rsub;
        const int32_t du = (int32_t)divide((uint32_t)(slot0 + off), a.by_slots);
        live[i] = row0 + off < a.rows;
        const int32_t unit = live[i] ? unit0 + du : unit0;
        const int32_t s = live[i] ? slot0 + off - du * slots : slot0;
        const int32_t sr = s < st.K ? s : st.K - 1;        // a readable row; the spare slot is zeroed
        v[i] = __builtin_nontemporal_load(&in[((int64_t)unit * st.K + sr) * 16 + lane16]);
        slot[i] = s;
        count[i] = a.cnt[unit];
        if (PAGED) {
            const int32_t pair = (int32_t)divide((uint32_t)unit, a.by_hkv), g = unit - pair * st.hkv;
            const int32_t l = (int32_t)divide((uint32_t)pair, a.by_batch), b = pair - l * st.batch;
            const int32_t j = page_index(pg, s);
            const int32_t page = clamp_page(pg, pg.table[(size_t)b * pg.max_pages + j]);
            to[i] = l * pg.s_layer + g * pg.s_head + (int64_t)page * pg.s_page + (int64_t)(s - j * pg.page_size) * pg.s_slot + lane16;
        } else {
            to[i] = ((int64_t)unit * slots + s) * 16 + lane16;
        }
    }
    const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < INIT_ITERS; ++i) {
        if (!live[i]) continue;
        const u32x4 row = slot[i] < st.K && slot[i] < count[i] ? v[i] : zero;
        __builtin_nontemporal_store(row, &out[to[i]]);
    }
}

// ---- step, sequence part ---------------------------------------------------------
// Voucher and sponsor flag of every position from the current budgets (Eq. 2): the same for all
// units of a sequence, so it is computed once per sequence and step, not once per cached row.
struct VouchArgs {
    int32_t L;
    float pw[TA_MAX_SPAN + 1];
};

// Sequence part of a step, one launch: every workgroup reads the old length (nobody writes it here),
// a sequence's last workgroup appends the token, tests the table at the new
// position and publishes the new length in `stepped` (0: the sequence is at capacity and is left
// alone); the others compute the vouchers of their positions, which depend on earlier positions
// only and so not on anything the append writes.
__global__ void __launch_bounds__(256)
decode_seq_vouch_kernel(ta_decode_state st, const int32_t* new_tok, DecodeTable tab, VouchArgs a)
{
    const int b = blockIdx.y;
    const size_t row = (size_t)b * st.cap;
    if (blockIdx.x == gridDim.x - 1) {                     // the append: one wavefront
        const int e = (int)threadIdx.x;
        if (e >= 64) return;
        // (the launch's table lies in host memory: requested together with the length, not behind it)
        const int32_t len_old = st.len[b], t0 = new_tok[b];
        int32_t rid[TA_MAX_GRAM];
#pragma unroll
        for (int k = 0; k < TA_MAX_GRAM; ++k) rid[k] = tab.rid[e][k];
        const int32_t gram = e < tab.E ? tab.len[e] : 0;
        if (len_old < 0 || len_old >= st.cap) {
            if (e == 0) st.stepped[b] = 0;
            return;
        }
        const int32_t p = len_old;
        int32_t* tok = st.tok + row;
        bool hit = gram > 0 && t0 == rid[0] && p - gram + 1 >= 0;
        int32_t before[TA_MAX_GRAM];
#pragma unroll
        for (int k = 1; k < TA_MAX_GRAM; ++k) before[k] = tok[p >= k ? p - k : 0];
#pragma unroll
        for (int k = 1; k < TA_MAX_GRAM; ++k) hit = hit && (k >= gram || before[k] == rid[k]);
        const bool any = __ballot(hit) != 0ull;
        if (e == 0) {
            tok[p] = t0;
            st.anchor[row + p] = any ? 1 : 0;
            st.budget[row + p] = any ? tab.B : 0.0f;
            st.stepped[b] = (p + 1) | (any ? (1 << 30) : 0);   // new length; bit 30: the new token is an anchor
        }
        return;
    }
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= st.cap) return;
    const uint8_t* anchor = st.anchor + row;
    const float* budget = st.budget + row;
    // the flags of the L positions before p, eight requested at a time, with the length; bit k - 1: position p - k
    const int32_t len_old = st.len[b];
    const uint8_t own = anchor[p];
    unsigned long long near = 0ull;
    for (int k0 = 1; k0 <= a.L; k0 += 8) {                 // uniform
        uint8_t f[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) f[j] = anchor[p >= k0 + j ? p - k0 - j : 0];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (f[j] && p >= k0 + j && k0 + j <= a.L) near |= 1ull << (k0 + j - 1);
    }
    if (len_old >= st.cap || p > len_old) return;          // at capacity; positions 0 .. len_old exist after the append
    const uint8_t sp = near != 0ull ? 1 : 0;
    float v = 0.0f;
    while (near) {                                         // increasing distance, as in the fixed-order sum
        const int k = __ffsll((long long)near);
        near &= near - 1ull;
        v = __fadd_rn(v, __fmul_rn(budget[p - k], a.pw[k]));
    }
    st.vouch[row + p] = v;
    // bit 0: sponsored; bit 1: the position is an anchor itself (the new position's flag travels in
    // `stepped`: it is being written by another workgroup of this launch)
    st.spons[row + p] = sp | (p < len_old && own ? 2 : 0);
}

// Trailing workgroups of the unit launch: budget decay of 256 positions each, and the new length.
// Units read neither array (they take the length from `stepped`), so the two kinds of workgroup
// touch disjoint memory.
__device__ __forceinline__ void decay_rider(const ta_decode_state& st, int r, float decay)
{
    const int tiles = (st.cap + 255) >> 8;
    const int b = r / tiles, tile = r - b * tiles;
    const int32_t len_new = st.stepped[b] & 0x3FFFFFFF;
    if (len_new == 0) return;
    float* B = st.budget + (size_t)b * st.cap;
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int p = tile * 256 + j * 64 + (int)threadIdx.x;
        v[j] = B[p < len_new ? p : 0];                      // len_new >= 1
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int p = tile * 256 + j * 64 + (int)threadIdx.x;
        if (p < len_new) B[p] = __fmul_rn(decay, v[j]);
    }
    if (tile == 0 && threadIdx.x == 0) st.len[b] = len_new;
}

// ---- step, unit part ----------------------------------------------------------------
struct UnitArgs {
    const uint4* q_new;
    const uint4* k_new;
    const uint4* v_new;
    int32_t* evicted;
    int32_t n_sink, n_recent;
    float alpha, beta, gamma;
    float scale_log2;
    int32_t last_query;                                    // 1: A holds this step's attention, not the running sum
    int32_t pg_off;                                        // paged slots: offset (in floats) of the page list in the wavefront's LDS
    int32_t units;                                         // workgroups beyond this many decay the budgets
    int32_t group;                                         // query heads per KV head
    Divider by_hkv, by_batch;
    float decay;
};

// A step as one launch (FUSED below): what its sequence part works with, and the words in which the workgroups of a sequence count
// themselves once they have read the length, which the last of them moves on.
constexpr int NEAR_SPAN = 7;                               // positions before its own whose flags a slot's one 8-byte load brings
constexpr int SYNC_LINES = 8;                              // lines of 32 words on which a sequence's units count, then one for the lines that are complete and the tiles of positions
constexpr int SYNC_WORDS = (SYNC_LINES + 1) * 32;          // of a sequence: one line took 1 to 5 us per step, the units' additions following one another
constexpr int COUNT_BITS = 8, MAX_TILES = 64 - COUNT_BITS;   // of the last line's number: a count of up to SYNC_LINES + MAX_TILES, and a bit per tile
static_assert(SYNC_LINES + MAX_TILES < (1 << COUNT_BITS), "the count");
constexpr int TILE_PER = 4;                                // positions of a thread in flight
static_assert(SYNC_WORDS == TA_DECODE_SYNC_WORDS, "as the header states it");
struct StepArgs {
    const int32_t* new_tok;
    int32_t* sync;                                         // [batch][SYNC_WORDS], zero between steps
    int32_t per_seq;                                       // units of a sequence
    int32_t tiles, tile_shift;                             // tiles of 1 << tile_shift positions
    int32_t parts;                                         // what the last line counts up to
    int32_t lead;                                          // workgroups of positions in front of the units: all or none
    int32_t L;                                             // at most NEAR_SPAN
    unsigned long long span;                               // the bytes of a slot's eight flags that its L predecessors are
    uint32_t span_bits;                                    // and their bits
    float pw[NEAR_SPAN + 1];
    int4 rid[TA_MAX_TABLE];                                // n-grams reversed
    int32_t len[TA_MAX_TABLE];                             // 0 past the table's end
    float B;
};

// Is the token that is appended at position p an anchor?  Lane e tests entry e: inputs requested, then tested.
struct AnchorTest {
    int32_t t0, gram, before[TA_MAX_GRAM];
    int4 rid;
};
__device__ __forceinline__ AnchorTest request_anchor(const ta_decode_state& st, const StepArgs& f, int b, int32_t p)
{
    static_assert(TA_MAX_GRAM == 4, "an entry is one int4");
    const int e = (int)threadIdx.x & 63;
    const int32_t* tok = st.tok + (size_t)b * st.cap;
    AnchorTest t;
    t.t0 = f.new_tok[b];
    t.rid = f.rid[e];
    t.gram = f.len[e];
#pragma unroll
    for (int k = 1; k < TA_MAX_GRAM; ++k) t.before[k] = tok[p >= k ? p - k : 0];
    return t;
}
__device__ __forceinline__ bool is_anchor(const AnchorTest& t, int32_t p)
{
    const int32_t rid[TA_MAX_GRAM] = {t.rid.x, t.rid.y, t.rid.z, t.rid.w};
    bool hit = t.gram > 0 && t.t0 == rid[0] && p - t.gram + 1 >= 0;
#pragma unroll
    for (int k = 1; k < TA_MAX_GRAM; ++k) hit = hit && (k >= t.gram || t.before[k] == rid[k]);
    return __ballot(hit) != 0ull;
}

// units of a sequence that count on a line
__device__ __forceinline__ int32_t units_on(int32_t per_seq, int32_t line) { return (per_seq - line + SYNC_LINES - 1) / SYNC_LINES; }

// An index that the compiler takes to differ from lane to lane.  Where it sees one address, it adds up what the lanes of a wavefront add itself and
// waits right there for the sum that comes back, and for all that was requested before.
__device__ __forceinline__ uint32_t lane_index(uint32_t i)
{
    asm volatile("" : "+v"(i));
    return i;
}

// The last line's first two words, as one: below, how many lines are complete and how many tiles of positions have read the length; above, a bit
// per tile, set once its vouchers are in memory.
__device__ __forceinline__ unsigned long long* total_of(const StepArgs& f, int b)
{
    return reinterpret_cast<unsigned long long*>(f.sync + (size_t)b * SYNC_WORDS + 32 * SYNC_LINES);
}
__device__ __forceinline__ unsigned long long add_to_total(const StepArgs& f, int b, unsigned long long v)
{
    const uint32_t at = lane_index((uint32_t)(b * (SYNC_WORDS / 2) + 16 * SYNC_LINES));
    return __hip_atomic_fetch_add(reinterpret_cast<unsigned long long*>(f.sync) + at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long vouched(unsigned long long total) { return total >> COUNT_BITS; }
__device__ __forceinline__ bool completes(const StepArgs& f, unsigned long long total) { return (int32_t)((uint32_t)total & ((1u << COUNT_BITS) - 1u)) == f.parts - 1; }

// Append of a sequence in the one-launch form, by the first wavefront of whichever of its workgroups counts in last.  The length is all that it
// overwrites and others read (the new position's token, flag and budget are nothing to them, the flag that they test themselves).  Sets the
// words back to zero.  p_new: the length before the step; t0: the token; an: is it an anchor there.
__device__ __forceinline__ void append(const ta_decode_state& st, const StepArgs& f, int b, int32_t p_new, int32_t t0, bool an, float decay)
{
    const int lane = (int)threadIdx.x;
    if (lane < SYNC_LINES) __hip_atomic_store(&f.sync[(size_t)b * SYNC_WORDS + 32 * lane], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lane != 0) return;
    __hip_atomic_store(total_of(f, b), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool live = p_new >= 0 && p_new < st.cap;        // else: at capacity, left alone
    if (live) {
        const size_t o = (size_t)b * st.cap + p_new;
        st.tok[o] = t0;
        st.anchor[o] = an ? 1 : 0;
        st.budget[o] = __fmul_rn(decay, an ? f.B : 0.0f);
        st.len[b] = p_new + 1;
    }
    st.stepped[b] = live ? (p_new + 1) | (an ? (1 << 30) : 0) : 0;
}

// Workgroups of positions of the one-launch form: vouchers and flags of a tile of positions, then the decay of its budgets.  Units may need those
// budgets, and may run before or after, but nobody waits for anybody, whatever else the chip runs and wherever workgroups are placed (steps
// of other states may overlap: one that waited could hold the place of the one it waits for).  A budget is overwritten only once all vouchers
// that are computed from it are in memory, which their tile's bit says: a unit that needs a voucher adds the budgets up, then looks at the
// bit of the position's tile, and where it is set takes the voucher that is there (vouchers_of_slots).  The last NEAR_SPAN budgets of a tile
// belong to vouchers of the next one too: of the two workgroups the one that sets its bit second overwrites them.
// A chain of five round trips (inputs, vouchers stored, bit set, budgets stored, counted with the bit), some 5 us beside the units' key stream.
template <int THREADS>
__device__ __forceinline__ void vouch_and_decay(const ta_decode_state& st, const StepArgs& f, int r, float decay, int32_t* s_x)
{
    constexpr int PER = TILE_PER, CHUNK = PER * THREADS;
    float* s_B = reinterpret_cast<float*>(s_x) + 4;        // budgets of NEAR_SPAN positions and those of a chunk
    const int b = r / f.tiles, tile = r - b * f.tiles;
    const int tid = (int)threadIdx.x;
    const size_t row = (size_t)b * st.cap;
    const int32_t p_new = st.len[b], t0 = f.new_tok[b];
    const bool live = p_new >= 0 && p_new < st.cap;        // else: at capacity, left alone
    const int32_t first = tile << f.tile_shift, end = tile == f.tiles - 1 ? st.cap : first + (1 << f.tile_shift);
    const uint8_t* anchor = st.anchor + row;
    float* B = st.budget + row;
    const int32_t exist = live ? (end < p_new + 1 ? end : p_new + 1) : first;      // with the appended position
    int32_t q = first;
    do {                                                   // one round unless rows are long (the first does not wait for the length)
        unsigned long long near[PER];
        float own[PER + 1];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int32_t p = q + j * THREADS + tid < st.cap ? q + j * THREADS + tid : st.cap - 1;
            __builtin_memcpy(&near[j], anchor + (p > NEAR_SPAN ? p - NEAR_SPAN : 0), 8);       // (any address; a row has more than NEAR_SPAN)
            own[j] = B[p];
        }
        own[PER] = B[tid < NEAR_SPAN && q >= NEAR_SPAN ? q - NEAR_SPAN + tid : 0];
        if (q != first) __syncthreads();                   // the chunk before has been read
#pragma unroll
        for (int j = 0; j < PER; ++j) s_B[NEAR_SPAN + j * THREADS + tid] = own[j];
        if (tid < NEAR_SPAN) s_B[tid] = own[PER];
        __syncthreads();                                   // the budgets are in LDS
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int32_t p = q + j * THREADS + tid;
            if (p >= exist) continue;
            if (p < NEAR_SPAN) near[j] <<= 8 * (NEAR_SPAN - p);
            float v = 0.0f;
            if ((near[j] & f.span) != 0ull) {
#pragma unroll 1
                for (int k = 1; k <= f.L; ++k)             // increasing distance, as in the fixed-order sum
                    if (((near[j] >> (8 * (NEAR_SPAN - k))) & 0xFFull) != 0ull) v = __fadd_rn(v, __fmul_rn(s_B[NEAR_SPAN + j * THREADS + tid - k], f.pw[k]));
            }
            __hip_atomic_store(&st.vouch[row + p], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            st.spons[row + p] = ((near[j] & f.span) != 0ull ? 1 : 0) | (p < p_new && (near[j] >> 56) != 0ull ? 2 : 0);     // as decode_seq_vouch_kernel
        }
        q += CHUNK;
    } while (q < exist);
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(p_new) : "memory");                    // this wavefront's vouchers are where every workgroup reads them
    __syncthreads();
    unsigned long long total = 0ull;
    if (tid == 0) {
        total = add_to_total(f, b, (1ull << (COUNT_BITS + tile)) + 1ull);
        s_x[0] = (int32_t)(uint32_t)total;
        s_x[1] = (int32_t)(uint32_t)(total >> 32);
    }
    __syncthreads();                                       // which tiles' vouchers are done
    total = (unsigned long long)(uint32_t)s_x[1] << 32 | (uint32_t)s_x[0];
    const unsigned long long done = vouched(total);
    const int32_t from = tile > 0 && (done >> (tile - 1) & 1ull) ? first - NEAR_SPAN : first;
    int32_t to = tile == f.tiles - 1 || (done >> (tile + 1) & 1ull) ? end : end - NEAR_SPAN;
    to = live ? (to < p_new ? to : p_new) : from;          // (the new position's budget comes with the append)
    const bool kept = end - first <= CHUNK;                // one round: the budgets are in LDS still
    for (q = from + tid; q < to; q += CHUNK) {
        float v[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int32_t p = q + j * THREADS < to ? q + j * THREADS : q;
            v[j] = kept ? s_B[NEAR_SPAN + p - first] : B[p];
        }
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (q + j * THREADS < to) B[q + j * THREADS] = __fmul_rn(decay, v[j]);
    }
    if (tid < 64 && completes(f, total)) append(st, f, b, p_new, t0, live && is_anchor(request_anchor(st, f, b, p_new), p_new), decay);
}

__device__ __forceinline__ uint32_t ordered_bits(float u)
{
    uint32_t b = __float_as_uint(u);
    return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// the two 8-byte halves of a 16-byte load as MFMA operand fragments (four bf16 each)
__device__ __forceinline__ s16x4 lo_half(const uint4& v)
{
    union { uint2 u; s16x4 s; } c;
    c.u = make_uint2(v.x, v.y);
    return c.s;
}
__device__ __forceinline__ s16x4 hi_half(const uint4& v)
{
    union { uint2 u; s16x4 s; } c;
    c.u = make_uint2(v.z, v.w);
    return c.s;
}

// A bit per byte of eight flags.
__host__ __device__ __forceinline__ uint32_t flag_bits(unsigned long long flags)
{
    const auto four = [](uint32_t x) {                     // 0x80 in every byte that is not zero, then their four bits together
        const uint32_t high = (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u;
        return ((high >> 7) * 0x01020408u) >> 24 & 15u;
    };
    return four((uint32_t)flags) | four((uint32_t)(flags >> 32)) << 4;
}

// What is asked of a slot's eight flags, as the bytes that they are loaded as or a bit each: is one of its L predecessors an anchor, is the
// one k positions before, is the slot's own position.
__device__ __forceinline__ bool sponsored(unsigned long long near, const StepArgs& f) { return (near & f.span) != 0ull; }
__device__ __forceinline__ bool sponsored(uint32_t near, const StepArgs& f) { return (near & f.span_bits) != 0u; }
__device__ __forceinline__ bool flag_before(unsigned long long near, int k) { return ((near >> (8 * (NEAR_SPAN - k))) & 0xFFull) != 0ull; }
__device__ __forceinline__ bool flag_before(uint32_t near, int k) { return ((near >> (NEAR_SPAN - k)) & 1u) != 0u; }

// One-launch form: the flags of a lane's slots; s_x[8 + wave] tells the other wavefronts whether one of them is plain - ranks below all
// sponsored ones.
template <int SPL, typename Near>
__device__ __forceinline__ void flags_of_slots(const UnitArgs& a, const StepArgs& fs, int wave, int32_t len_new,
                                               const int32_t (&p0)[SPL], const Near (&near)[SPL], uint8_t (&fl0)[SPL], float (&v0)[SPL], int32_t* s_x)
{
    const int lane = (int)threadIdx.x & 63;
    bool plain = false;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
        const int32_t p = p0[j];
        fl0[j] = (uint8_t)((sponsored(near[j], fs) ? 1 : 0) | (flag_before(near[j], 0) ? 2 : 0));
        v0[j] = 0.0f;
        plain = plain || (p >= a.n_sink && p < len_new - a.n_recent && !(fl0[j] & 1));
    }
    const bool some = __ballot(plain) != 0ull;
    if (lane == 0) s_x[8 + wave] = some ? 1 : 0;
}

// Behind the barrier that follows: is the new position an anchor, and the slots' vouchers if they decide.
template <int WAVES, int SPL, typename Near>
__device__ __forceinline__ uint8_t vouchers_of_slots(const ta_decode_state& st, const StepArgs& fs, int b, const int32_t (&p0)[SPL],
                                                     const Near (&near)[SPL], float (&v0)[SPL], const int32_t* s_x)
{
    const uint8_t an_new = (uint8_t)s_x[16];
    int some = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) some |= s_x[8 + w];
    if (some == 0) {                                       // uniform in the workgroup: vouchers decide
        const float* budget = st.budget + (size_t)b * st.cap;
#pragma unroll
        for (int j = 0; j < SPL; ++j)
#pragma unroll 1
            for (int k = 1; k <= fs.L; ++k) {              // increasing distance, as in the fixed-order sum
                if (p0[j] >= k && flag_before(near[j], k))
                    v0[j] = __fadd_rn(v0[j], __fmul_rn(budget[p0[j] - k], fs.pw[k]));
            }
#pragma unroll
        for (int j = 0; j < SPL; ++j) asm volatile("" : "+v"(v0[j])::"memory");    // the budgets have been read
        const unsigned long long done = vouched(__hip_atomic_load(total_of(fs, b), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
#pragma unroll
        for (int j = 0; j < SPL; ++j)                      // (without a sponsor, free slots among them: zero whatever the tile does)
            if (sponsored(near[j], fs) && (done >> (p0[j] >> fs.tile_shift) & 1ull))
                v0[j] = __hip_atomic_load(&st.vouch[(size_t)b * st.cap + p0[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < SPL; ++j) asm volatile("" : "+v"(v0[j])::"memory");
        __syncthreads();                                   // every wavefront's vouchers are in registers
    }
    return an_new;
}

// A unit is the work of one workgroup of WAVES wavefronts.  SMALL: at most WAVES * SPL * 64 slots, so a
// lane's slots (position, voucher, flags, accumulated attention) stay in its registers from the
// first round trip to the ranking and nothing loops over slots; without it (more slots than a lane holds, and no
// attention term) one wavefront loops over them.
// DT_RING: 16-row key tiles in flight per wavefront.
// WAVES == 1: no workgroup barriers.
// WAVES > 1 (one wavefront would stream a unit's keys one tile after the other): each wavefront has SPL * 64 of
// the slots in its registers and streams every WAVES-th key tile; the slot table, the logits and four small exchanges
// (first free slot, softmax statistics, free count, worst key) go through LDS, with four workgroup barriers.  Every logit,
// every softmax statistic (of a head by one wavefront, in the single wavefront's order; the wavefronts take every
// WAVES-th head) and every slot's key is computed by the same instructions as in the single-wavefront form: all forms
// give the same bits.
// FUSED: the step is this one launch.  A unit tests the table at the new position itself and finds its slots' sponsors by one 8-byte
// load of flags each.  Vouchers it needs only where no plain slot is left to evict: any plain slot ranks below every
// sponsored one, and its own voucher is zero.  It counts itself in once it has read what the append overwrites, and the last workgroup
// of a sequence to do so appends.
template <int GH, bool PAGED, bool SCORED, bool SMALL, int DT_RING, int WAVES, int SPL, bool FUSED = false>
__device__ __forceinline__ void decode_unit(const ta_decode_state& st, const UnitArgs& a, const SlotPages& pg, const StepArgs* fs = nullptr)
{
    extern __shared__ float s_dyn[];
    static_assert(!FUSED || (WAVES > 1 && SMALL), "one launch: several wavefronts per unit");
    static_assert(WAVES == 1 || SCORED || FUSED, "several wavefronts: an attention term or one launch");
    static_assert(SMALL || !SCORED, "with an attention term a unit's slots are in registers");

    const int lane = threadIdx.x & 63;
    const int wave = WAVES > 1 ? (int)(threadIdx.x >> 6) : 0;
    const int sub = lane & 15, grp = lane >> 4;            // 16 lanes per key row, 4 rows per instruction
    int unit = (int)blockIdx.x;
    if constexpr (FUSED) unit -= fs->lead;
    if (unit < 0 || unit >= a.units) {                     // in front of the units or behind them: workgroups of positions
        if constexpr (FUSED) vouch_and_decay<64 * WAVES>(st, *fs, unit < 0 ? unit + fs->lead : unit - a.units, a.decay, reinterpret_cast<int32_t*>(s_dyn));
        else if (wave == 0) decay_rider(st, unit - a.units, a.decay);
        return;
    }
    const int slots = st.K + 1;
    const int G = a.group;
    const int pair = (int)divide((uint32_t)unit, a.by_hkv), l = (int)divide((uint32_t)pair, a.by_batch);
    const int g = unit - pair * st.hkv, b = pair - l * st.batch;
    int32_t* pos = st.pos + (size_t)unit * slots;
    float* A = st.A + (size_t)unit * slots;
    uint4* Kc = reinterpret_cast<uint4*>(st.Kc) + (PAGED ? l * pg.s_layer + g * pg.s_head : (int64_t)unit * slots * 16);
    uint4* Vc = reinterpret_cast<uint4*>(st.Vc) + (PAGED ? l * pg.s_layer + g * pg.s_head : (int64_t)unit * slots * 16);
    const int sbase = wave * (SPL * 64);                           // first slot of this wavefront's share

    // Everything that does not depend on loaded data is requested first, in the order it is needed
    // (loads of a wavefront return in order), and unconditionally (clamped addresses, results masked
    // afterwards): straight-line loads let the compiler wait for exactly the load it needs.
    // FUSED: the length before the step; else what the sequence part of the step, which has run, left
    const int32_t stepped = FUSED ? st.len[b] : st.stepped[b];
    int32_t p0[SPL];
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
        const int s = sbase + lane + 64 * j;
        p0[j] = SMALL ? pos[s < slots ? s : slots - 1] : 0;
    }
    const uint4* nsrc = ((lane & 16) ? a.v_new : a.k_new) + ((size_t)(l * st.batch + b) * st.hkv + g) * 16;
    const uint4 nrow = nsrc[lane & 15];                    // lanes 0-15: the new key row, 16-31: the new value row

    int32_t* s_pg = reinterpret_cast<int32_t*>(s_dyn + a.pg_off);
    if (PAGED) {
        const int npg = page_index(pg, slots - 1) + 1;
        for (int j = lane; j < npg; j += 64) s_pg[j] = clamp_page(pg, pg.table[(size_t)b * pg.max_pages + j]);
        __builtin_amdgcn_wave_barrier();
    }
    const auto row_at = [&](int row) -> int64_t {           // 16-byte index of a slot's first chunk
        if (!PAGED) return (int64_t)row * 16;
        const int32_t j = page_index(pg, row);
        return (int64_t)s_pg[j] * pg.s_page + (int64_t)(row - j * pg.page_size) * pg.s_slot;
    };
    int32_t* s_pos = reinterpret_cast<int32_t*>(s_dyn);
    const int wstride = (slots + 3) & ~3;                  // logits of a head: padded to whole 16-byte groups
    // scored only: per wavefront one 16-row key tile (4 KB) and a copy of the new key row; with several
    // wavefronts 64 words for what they exchange; scored only: the logits
    uint4* s_t = reinterpret_cast<uint4*>(s_dyn + wstride) + 256 * wave;
    uint4* s_kn = reinterpret_cast<uint4*>(s_dyn + wstride) + 256 * WAVES + 16 * wave;
    int32_t* s_x = reinterpret_cast<int32_t*>(reinterpret_cast<uint4*>(s_dyn + wstride) + (SCORED ? (256 + 16) * WAVES : 0));
    float* s_w = reinterpret_cast<float*>(s_x) + (WAVES > 1 ? 64 : 0);

    const int i16 = sub, kq = grp;
    // this wavefront's tiles are wave, wave + WAVES, ...; `tile` below counts them, tile_of gives the unit's tile
    const int ntiles = (((slots + 15) >> 4) - wave + WAVES - 1) / WAVES;
    const auto tile_of = [&](int tile) { return wave + WAVES * tile; };
    uint4 qf[4], tiles[DT_RING][4];                        // DT_RING tiles in flight
    // Key rows are read once per step: the non-temporal hint keeps them from displacing the slot tables,
    // the accumulated attention and the per-sequence arrays in the caches (231 -> 210 us on 16 384 units).
    // Also where they would fit the last-level cache: without the hint they stay there from step to step if nothing comes between, but in use
    // the model's forward pass does, and then they cost what they displace (us per step, with the hint / up to 272 MB of keys without, behind a read of
    // 1 GiB: 256 units x 1025 slots 17.4 / 18.1, 1024 x 257 17.6 / 18.9, 8192 x 101 48.4 / 53.0, 4096 x 257 55.8 / 60.0, 2048 x 1025 93.0 / 96.9; back to
    // back: 15.0 / 16.5, 16.6 / 17.3, 48.1 / 43.7, 54.6 / 48.0, 92.6 / 88.7).
    const auto load_tile = [&](int tile, uint4 (&dst)[4]) {
        if (!PAGED) {                                      // dense unit: one uniform base, a 32-bit byte offset per lane
            const char* base = reinterpret_cast<const char*>(Kc);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                int row = tile_of(tile) * 16 + 4 * t + grp;
                row = row < slots ? row : slots - 1;       // past the last slot: a valid row, masked at the store
                {
                    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
                    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + (uint32_t)(row * 256 + sub * 16)));
                    dst[t] = make_uint4(v.x, v.y, v.z, v.w);
                }
            }
            return;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            int row = tile_of(tile) * 16 + 4 * t + grp;
            row = row < slots ? row : slots - 1;
            typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(&Kc[row_at(row) + sub]));
            dst[t] = make_uint4(v.x, v.y, v.z, v.w);
        }
    };
    if (SCORED) {
        const uint4* qrow = a.q_new + ((size_t)(l * st.batch + b) * st.hq + g * G + (i16 < G ? i16 : 0)) * 16;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint4 v = qrow[kq + 4 * t];
            qf[t] = i16 < G ? v : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < DT_RING; ++j) load_tile(j, tiles[j]);     // past the last tile: the last row again, never used
    }

    // ---- the slot table goes to LDS; lowest-numbered free slot ---------------------------------
    int first_free = 0x7FFFFFFF;
    if (SMALL) {
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int s = sbase + lane + 64 * j;
            if (s < slots) {
                s_pos[s] = p0[j];
                if (p0[j] < 0) first_free = first_free < s ? first_free : s;
            }
        }
    }
    for (int s0 = lane; !SMALL && s0 < slots; s0 += SPL * 64) {    // more slots than a lane's registers hold
        int32_t p4[SPL];
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int s = s0 + 64 * j;
            p4[j] = pos[s < slots ? s : slots - 1];
        }
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int s = s0 + 64 * j;
            if (s < slots) {
                s_pos[s] = p4[j];
                if (p4[j] < 0) first_free = first_free < s ? first_free : s;
            }
        }
    }
    int f = wave_min_dpp(first_free);
    if (FUSED) asm volatile("" ::"v"(stepped));            // read in front of the barrier: a unit may count itself in right behind it
    if (WAVES > 1) {
        if (lane == 0) s_x[wave] = f;
        __syncthreads();                                   // every share of the slot table is in LDS
        f = s_x[0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) f = s_x[w] < f ? s_x[w] : f;
    }
    const int32_t len_new = FUSED ? (stepped < 0 || stepped >= st.cap ? 0 : stepped + 1) : stepped & 0x3FFFFFFF;
    uint8_t an_new = FUSED ? 0 : (uint8_t)((stepped >> 30) & 1);
    // A unit counts itself in on its line, and a line's last unit counts the line; the sums before its own additions come back while it goes on.
    bool counted = false;
    int32_t before = -1;
    uint32_t sum = ~0u;                                    // (no count there can be)
    const int32_t line = FUSED ? (l * st.hkv + g) & (SYNC_LINES - 1) : 0;
    const auto count_in = [&]() {
        if (!FUSED || wave != 0 || counted) return;
        counted = true;
        if (lane == 0) before = __hip_atomic_fetch_add(&fs->sync[lane_index((uint32_t)(b * SYNC_WORDS + 32 * line))], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const auto count_line = [&]() {
        if (!FUSED || wave != 0 || lane != 0 || before != units_on(fs->per_seq, line) - 1) return;
        before = -1;
        sum = (uint32_t)add_to_total(*fs, b, 1ull);
    };
    const auto is_last = [&]() { return wave == 0 && completes(*fs, (uint32_t)__builtin_amdgcn_readfirstlane((int)sum)); };
    if (len_new == 0 || f >= slots) {                      // a sequence at capacity, or no room: nothing to do
        if (wave == 0 && lane == 0 && a.evicted) a.evicted[unit] = -1;
        if constexpr (FUSED) {
            count_in();
            count_line();
            if (is_last()) append(st, *fs, b, stepped, fs->new_tok[b], len_new != 0 && is_anchor(request_anchor(st, *fs, b, stepped), stepped), a.decay);
        }
        return;                                            // (every wavefront of the unit: the same test)
    }
    const int32_t p_new = len_new - 1;
    const float lenf = (float)len_new, len_inv = __fdiv_rn(1.0f, lenf);

    // the per-position inputs of the utility and the accumulated attention of the first SPL * 64 slots
    // are requested now and used after the key stream: they travel while the keys do
    const size_t srow = (size_t)b * st.cap;
    const uint8_t* spons = st.spons + srow;               // bit 0: sponsored, bit 1: anchor
    const float* vouch = st.vouch + srow;
    float v0[SPL], a0[SPL];
    uint8_t fl0[SPL];
    unsigned long long bytes[FUSED ? SPL : 1];             // flags of the positions p - NEAR_SPAN .. p of a slot, a byte each
    // the same, zeroes in front of the sequence; behind the key stream a bit each, which takes half the registers (paged slots, four
    // wavefronts of three slots per lane: three registers in scratch cost 1536 units x 513 slots 41.5 -> 47.4 us)
    using Near = std::conditional_t<SCORED, uint32_t, unsigned long long>;
    Near near[FUSED ? SPL : 1];
#pragma unroll
    for (int j = 0; SMALL && j < SPL; ++j) {
        const int s = sbase + lane + 64 * j;
        if (s == f) p0[j] = p_new;
        if (s >= slots) p0[j] = -2;
        const int32_t pc = p0[j] < 0 ? 0 : p0[j];
        if constexpr (FUSED) {
            __builtin_memcpy(&bytes[j], st.anchor + srow + (pc > NEAR_SPAN ? pc - NEAR_SPAN : 0), 8);     // (any address)
        } else {
            v0[j] = vouch[pc];
            fl0[j] = spons[pc];
        }
        if (SCORED) {
            const float av = A[s < slots ? s : slots - 1];
            a0[j] = (!a.last_query && p0[j] >= 0 && s != f) ? av : 0.0f;
        } else {
            a0[j] = 0.0f;
        }
    }
    if (lane < 16) {
        if (wave == 0) Kc[row_at(f) + lane] = nrow;
        if (SCORED) s_kn[lane] = nrow;
    } else if (lane < 32 && wave == 0) Vc[row_at(f) + lane - 16] = nrow;
    __builtin_amdgcn_wave_barrier();                       // the slot table is in LDS for every lane

    // The flags have arrived.  A unit that will not need vouchers has read all that anybody overwrites and counts itself in early: what its
    // sequence's last one then does hides behind the key stream (256 units x 1025 slots 17.1 -> 16.5 us).  That the first wavefront has a plain
    // slot is enough to know.
    const auto take_flags = [&]() {
        AnchorTest test = {};
        if constexpr (FUSED && !SCORED) {
            if (wave == WAVES - 1) test = request_anchor(st, *fs, b, p_new);
        }
        bool plain = false;
#pragma unroll
        for (int j = 0; FUSED && j < SPL; ++j) {
            const int32_t p = p0[j];
            const unsigned long long eight = p < NEAR_SPAN ? bytes[j] << (8 * (NEAR_SPAN - (p < 0 ? 0 : p))) : bytes[j];
            if constexpr (SCORED) near[j] = flag_bits(eight);
            else near[j] = eight;
            plain = plain || (p >= a.n_sink && p < len_new - a.n_recent && !sponsored(near[j], *fs));
        }
        if (wave == 0 && __ballot(plain) != 0ull) count_in();
        // The table, for the unit.  s_x[16]: is the new position an anchor; s_x[17]: its token.  (Looked up here: the inputs kept in registers
        // through the key stream took nine of them.)
        if constexpr (FUSED) {
            if (wave == WAVES - 1) {
                if constexpr (SCORED) test = request_anchor(st, *fs, b, p_new);
                const bool an = is_anchor(test, p_new);
                if (lane == 0) {
                    s_x[16] = an ? 1 : 0;
                    s_x[17] = test.t0;
                }
            }
        }
    };

    float m_h[GH], inv_h[GH];
    if constexpr (!SCORED && FUSED) {
        take_flags();
        flags_of_slots(a, *fs, wave, len_new, p0, near, fl0, v0, s_x);
        __syncthreads();                                   // every wavefront has read its flags
        an_new = vouchers_of_slots<WAVES>(st, *fs, b, p0, near, v0, s_x);
        count_in();
    }
    if (SCORED) {
        // logits of a 16-row key tile from its rows' fragments
        const auto frag_logits = [&](const uint4 (&frag)[4]) -> f32x4 {
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(lo_half(frag[t]), lo_half(qf[t]), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(hi_half(frag[t]), hi_half(qf[t]), acc, 0, 0, 0);
            }
            return acc;                                    // rows 4 kq .. 4 kq + 3 of the tile, head i16
        };
        // The new key's logit goes into the free slot, from the wavefront whose tile holds it (every row of this pseudo-tile is the
        // new key, so every lane of a head gets that head's logit).  Several wavefronts: it is computed while the second pass's
        // tiles are on their way.
        const bool has_free = WAVES == 1 || (f >> 4) % WAVES == wave;
        float new_logit = 0.0f;
        const auto new_key = [&]() {
            if (!has_free) return;                         // uniform
            uint4 knf[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint4 v = s_kn[kq + 4 * t];
                knf[t] = make_uint4(v.x, v.y, v.z, v.w);
            }
            new_logit = frag_logits(knf)[0] * a.scale_log2;
        };
        const auto store_tile = [&](int tile, const f32x4& acc) {
            const int s = tile_of(tile) * 16 + 4 * kq;
            if (i16 < G && s < wstride) {
                const int4 p4 = *reinterpret_cast<const int4*>(&s_pos[s]);   // padded to whole groups of four
                float4 o;
                o.x = (s + 0 < slots && p4.x >= 0) ? acc[0] * a.scale_log2 : -INFINITY;
                o.y = (s + 1 < slots && p4.y >= 0) ? acc[1] * a.scale_log2 : -INFINITY;
                o.z = (s + 2 < slots && p4.z >= 0) ? acc[2] * a.scale_log2 : -INFINITY;
                o.w = (s + 3 < slots && p4.w >= 0) ? acc[3] * a.scale_log2 : -INFINITY;
                *reinterpret_cast<float4*>(&s_w[i16 * wstride + s]) = o;
            }
        };
        // One tile: its rows go to LDS as soon as they are there, which frees its registers for the
        // tile DT_RING further on; the fragments come back out of LDS in the matrix layout.
        const auto one_tile = [&](int tile, uint4 (&regs)[4], bool reload) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int r = 4 * t + grp;
                s_t[r * 16 + (sub ^ r)] = make_uint4(regs[t].x, regs[t].y, regs[t].z, regs[t].w);
            }
            if (reload) load_tile(tile + DT_RING, regs);
            uint4 frag[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const uint4 v = s_t[i16 * 16 + ((kq + 4 * t) ^ i16)];
                frag[t] = make_uint4(v.x, v.y, v.z, v.w);
            }
            store_tile(tile, frag_logits(frag));
        };
        // Passes of DT_RING tiles.  While every tile of a pass has a successor DT_RING further on, the
        // pass is straight-line code (first pass apart from the loop: other loads are still in flight
        // around it); the last one or two passes test every tile.
        int tb = 0;
        if (2 * DT_RING <= ntiles) {
#pragma unroll
            for (int j = 0; j < DT_RING; ++j) one_tile(j, tiles[j], true);
            if (WAVES > 1) new_key();
            if constexpr (FUSED) take_flags();
            for (tb = DT_RING; tb + 2 * DT_RING <= ntiles; tb += DT_RING) {
#pragma unroll
                for (int j = 0; j < DT_RING; ++j) one_tile(tb + j, tiles[j], true);
            }
        } else if (WAVES > 1) {
            new_key();
            if constexpr (FUSED) take_flags();
        }
        for (; tb < ntiles; tb += DT_RING) {
#pragma unroll
            for (int j = 0; j < DT_RING; ++j)
                if (tb + j < ntiles) one_tile(tb + j, tiles[j], tb + j + DT_RING < ntiles);
        }
        if (WAVES == 1) new_key();
        __builtin_amdgcn_wave_barrier();                   // behind the tile's own logit for the slot
        if (has_free && i16 < G && kq == 0) s_w[i16 * wstride + f] = new_logit;
        if constexpr (FUSED) {
            count_line();
            flags_of_slots(a, *fs, wave, len_new, p0, near, fl0, v0, s_x);
        }
        if (WAVES > 1) __syncthreads();                    // the logits of every wavefront's tiles are in LDS
        else __builtin_amdgcn_wave_barrier();
        if constexpr (FUSED) {
            an_new = vouchers_of_slots<WAVES>(st, *fs, b, p0, near, v0, s_x);
            count_in();
        }
        // softmax statistics of all heads at once: one pass for the maxima, one for the sums.  Several
        // wavefronts: each takes every WAVES-th head (a head's reduction runs in one wavefront, in the
        // single wavefront's order) and the results are exchanged through LDS.
        // a head's logits in registers, all requested at once (a loop over the slots, one LDS round trip per 64 of them and
        // pass, took 4.2 of the 18.7 us of a unit of 1025 slots); lanes past the last slot add exp2(-inf) = 0
        constexpr int NV = WAVES * SPL;
        const auto one_head = [&](int h, float& m, float& inv) {
            float lg[NV];
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const int s = lane + 64 * j;
                const float x = s_w[h * wstride + (s < slots ? s : slots - 1)];
                lg[j] = s < slots ? x : -INFINITY;
            }
            m = lg[0];
#pragma unroll
            for (int j = 1; j < NV; ++j) m = fmaxf(m, lg[j]);
            m = wave_max_dpp(m);
            float z = 0.0f;
#pragma unroll
            for (int j = 0; j < NV; ++j) z += __builtin_amdgcn_exp2f(lg[j] - m);
            inv = __builtin_amdgcn_rcpf(wave_sum_dpp(z));
        };
        if constexpr (WAVES == 1) {
#pragma unroll
            for (int h = 0; h < GH; ++h) {
                m_h[h] = -INFINITY;
                inv_h[h] = 0.0f;
                if (h < G) one_head(h, m_h[h], inv_h[h]);
            }
        } else {
            static_assert(GH <= 16, "the exchange area holds 16 heads");
            float* s_stat = reinterpret_cast<float*>(s_x) + 32;            // [0..16): maxima, [16..32): reciprocal sums
            for (int h = wave; h < G; h += WAVES) {
                float m, inv;
                one_head(h, m, inv);
                if (lane == 0) {
                    s_stat[h] = m;
                    s_stat[16 + h] = inv;
                }
            }
            if constexpr (FUSED) count_line();
            __syncthreads();                               // every head's statistics
#pragma unroll
            for (int h = 0; h < GH; ++h) {
                m_h[h] = h < G ? s_stat[h] : -INFINITY;
                inv_h[h] = h < G ? s_stat[16 + h] : 0.0f;
            }
        }
    }

    // ---- new attention mass per slot, then the rank of the slot, in one pass (a lane handles the
    // same slots in both, so the mass stays in a register)
    unsigned long long worst = ~0ull;
    int nfree = 0;
    const auto rank_slot = [&](int s, int32_t p, float v, uint8_t fl, float a_old, const float (&lg)[GH]) {
        const uint8_t sp = fl & 1, an = (s == f) ? an_new : (uint8_t)((fl >> 1) & 1);
        if (p == -2) return;                               // past the last slot
        if (p < 0) { ++nfree; return; }
        float mass = 0.0f;
        if (SCORED) {
            float add = 0.0f;
#pragma unroll
            for (int h = 0; h < GH; ++h) add += h < G ? __builtin_amdgcn_exp2f(lg[h] - m_h[h]) * inv_h[h] : 0.0f;
            // cumulative mass over the steps, or (TOVA's step-wise rule) this step's mass alone
            mass = a_old + add;
            A[s] = mass;
        } else if (s == f) {
            A[s] = 0.0f;
        }
        const float r = div_by((float)(p + 1), lenf, len_inv);
        float t = SCORED ? __fmul_rn(a.alpha, mass) : 0.0f;
        t = __fadd_rn(t, __fmul_rn(a.beta, r));
        t = __fadd_rn(t, __fmul_rn(a.gamma, (float)an));
        t = __fadd_rn(t, v);
        const unsigned cls = (p < a.n_sink || p >= len_new - a.n_recent) ? 2u : (sp ? 1u : 0u);
        // (class, u, position) packed so that the smallest integer ranks last
        const unsigned long long key = ((unsigned long long)cls << 62) |
                                       ((unsigned long long)ordered_bits(t) << 30) | (unsigned long long)(uint32_t)p;
        worst = key < worst ? key : worst;
    };
    // The logits of a lane's slots (of one slot where heads are many) are read in one go, past the last head or slot those of the
    // last: a test per head had every read wait for the one before, 3000 cycles of the 31 700 of a unit of 1025 slots.
    float lg[SMALL ? SPL : 1][GH];
    const auto read_logits = [&](int j) {
        if (!SCORED) return;
        const int s = sbase + lane + 64 * j;
#pragma unroll
        for (int h = 0; h < GH; ++h) lg[j][h] = s_w[(h < G ? h : G - 1) * wstride + (s < slots ? s : slots - 1)];
    };
    if (GH <= 8) {
#pragma unroll
        for (int j = 0; SMALL && j < SPL; ++j) read_logits(j);
    }
#pragma unroll
    for (int j = 0; SMALL && j < SPL; ++j) {
        if (GH > 8) read_logits(j);
        rank_slot(sbase + lane + 64 * j, p0[j], v0[j], fl0[j], a0[j], lg[j]);
    }
    for (int s0 = lane; !SMALL && s0 < slots; s0 += SPL * 64) {    // more slots than a lane's registers hold
        int32_t p4[SPL];
        float v4[SPL];
        uint8_t fl4[SPL];
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int s = s0 + 64 * j;
            p4[j] = s < slots ? ((s == f) ? p_new : s_pos[s]) : -2;
            const int32_t pc = p4[j] < 0 ? 0 : p4[j];
            v4[j] = vouch[pc];
            fl4[j] = spons[pc];
        }
#pragma unroll
        for (int j = 0; j < SPL; ++j) rank_slot(s0 + 64 * j, p4[j], v4[j], fl4[j], 0.0f, lg[0]);
    }
    nfree = __ballot(nfree > 0) != 0ull ? 1 : 0;           // is a slot of this wavefront's still free?
    worst = wave_min_dpp(worst);
    if (WAVES > 1) {
        if constexpr (FUSED && !SCORED) count_line();
        if constexpr (FUSED) {
            if (is_last()) append(st, *fs, b, p_new, s_x[17], an_new != 0, a.decay);
        }
        // without an attention term no barrier lies between the last exchange and this one: other words
        int32_t* s_e = s_x + (SCORED ? 8 : 32);
        if (lane == 0) {
            s_e[wave] = nfree;
            s_e[8 + 2 * wave] = (int32_t)(uint32_t)worst;
            s_e[9 + 2 * wave] = (int32_t)(uint32_t)(worst >> 32);
        }
        __syncthreads();                                   // every wavefront's free count and worst key
        nfree = 0;
        worst = ~0ull;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            nfree += s_e[w];
            const unsigned long long k = ((unsigned long long)(uint32_t)s_e[9 + 2 * w] << 32) | (uint32_t)s_e[8 + 2 * w];
            worst = k < worst ? k : worst;
        }
    }
    const int32_t evict_pos = nfree > 0 ? -1 : (int32_t)(worst & 0x3FFFFFFFull);
    if (SMALL) {                                           // a lane's slots are in its registers, the new position with them
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int s = sbase + lane + 64 * j;
            if (s == f || (p0[j] >= 0 && p0[j] == evict_pos)) pos[s] = p0[j] == evict_pos ? -1 : p0[j];
        }
    } else {
        for (int s = lane; s < slots; s += 64) {
            const int32_t p = (s == f) ? p_new : s_pos[s];
            if (s == f || (p >= 0 && p == evict_pos)) pos[s] = (p == evict_pos) ? -1 : p;
        }
    }
    if (wave == 0 && lane == 0 && a.evicted) a.evicted[unit] = evict_pos;
}

// How a unit's slots are spread: over `waves` wavefronts with `spl` slots per lane in registers; spl 0 (no attention term): one
// wavefront that loops over its slots.
struct UnitForm {
    int waves, spl;
};
constexpr int LOOP_SPL = 5;                                // slots per lane and round trip of that loop

// Which one, with an attention term.  A wavefront waits for its tiles, so what counts is how many wavefronts stream at once;
// where units are many, their barriers and their LDS do: from 257 slots on, and with up to two sequences' units at any
// budget worth ranking, shared is ahead (us per step, one wavefront / this form: 257 slots, 256 units 14.9 / 11.0, 1024 units
// 23.0 / 19.4, 4096 units 63.7 / 55, 16 384 units 225 / 201; 129 slots, 4096 units 36.6 / 34.6; 65 slots, 4096 units 22.1 /
// 24.5; 701 slots, 1024 units 48.1 / 38; 1501 slots, 2048 units 198 / 125).  More wavefronts with fewer slots per lane where
// a budget leaves the choice (1025 slots, 256 units: four wavefronts 20.4, eight 19.3; 601 slots: 14.9, 15.3).
// Paged slots follow the same lines (16 per page: 257 slots, 256 units 20.7 / 12.9, 4096 units 64.8 / 60.8; 193 slots, 16 384 units
// 169.5 / 164.6; 513 slots 427.7 / 416.7); at 16 384 units of 257 slots they lose 1 % to 4 % (219.5 / 222.0, after prompts of up
// to 16 384 positions 227 / 237).
//
// A step as one launch wants several wavefronts per unit, and is ahead of two while there are not so many units that their counting
// shows.  us per step (replayed from a graph), one launch / two: 256 units x 257 slots 8.6 / 10.3, x 1025 15.2 / 17.0 (paged 16.3 / 18.0), x 501 with
// 8 heads per group 10.7 / 12.6; 1024 x 257 15.8 / 16.8, x 1025 46.9 / 48.7 (paged 51.4 / 53.0); 1536 x 513 paged 41.8 / 43.3; 3072 x 129 25.1 / 25.5, x 257
// 41.7 / 42.7; 4096 x 129 31.3 / 31.7, x 257 54.2 / 55.0, x 513 96.3 / 98.1.  So where it can be had, two wavefronts share a unit that one would hold up
// to 1792 units; 2048 of them fill the chip, and the workgroups of positions begin behind them (1024 units x 65 slots 8.6 / 10.2; 1536 x 65
// 10.6 / 11.6, x 101 12.5 / 13.8, paged 13.7 / 15.2; 1792 x 31 9.4 / 9.9, x 65 11.0 / 12.1, paged 12.2 / 13.6; 2048 x 31 11.7 / 10.2, x 65 13.3 / 13.1, x 101
// 14.7 / 15.3).
//
// Without an attention term a unit only reads its slot table and flags, so that one launch takes as many wavefronts as hold all slots, while
// the chip starts them at once (us per step, one launch / two, there with a wavefront per unit: 16 units x 1501 slots 7.5 / 14.6; 256 x 1025
// 6.9 / 12.2, paged 7.3 / 12.8; 1024 x 2001 12.1 / 19.2; 1536 x 1501 13.7 / 16.6; 2048 x 501 8.8 / 10.4; 3072 x 501 10.5 / 11.1; 4096 x 201 8.9 / 9.0, paged
// 9.8 / 9.4, and as the calls are issued 9.9 / 11.9; 256 x 257 up to 57 344 positions 7.5 / 6.9, as issued 9.1 / 12.5; with 16 384 wavefronts, before
// anything was counted: 2048 x 1025 13.1 / 13.9, paged 15.9 / 14.5; 4096 x 257 11.3 / 11.5, paged 12.6 / 11.3).
static_assert(TA_MAX_DECODE_K + 1 <= 8 * 4 * 64, "the widest form");
constexpr int FEW_UNITS = 512, FEW_UNITS_ONE_LAUNCH = 1792, ONE_LAUNCH_UNITS = 4096, ONE_LAUNCH_PLAIN_WAVES = 12288;
// one: a step of one launch can be had, and is taken if several wavefronts share a unit
UnitForm unit_form(bool scored, int slots, int64_t units, bool one)
{
    if (!scored) {
        const UnitForm all = slots <= 256 ? UnitForm{2, 2} : slots <= 512 ? UnitForm{4, 2} : slots <= 768 ? UnitForm{4, 3} : slots <= 1536 ? UnitForm{8, 3} : UnitForm{8, 4};
        if (one && units * all.waves <= ONE_LAUNCH_PLAIN_WAVES) return all;
        return {1, slots <= LOOP_SPL * 64 ? LOOP_SPL : 0};
    }
    if (units > (one ? FEW_UNITS_ONE_LAUNCH : FEW_UNITS) && slots <= 112) return {1, 2};
    if (units > FEW_UNITS && slots <= 256) return {2, 2};
    if (slots <= 512) return {4, 2};
    if (slots <= 768) return {4, 3};
    if (slots <= 1536) return {8, 3};
    return {8, 4};                                         // at most 2048 slots
}

// Can a step be one launch: given words to count in (two of them are one number of eight bytes), a span whose flags one load holds, and not
// too many units.
bool one_launch(const ta_params& prm, const ta_decode_state& st, int64_t units, const int32_t* sync)
{
    return sync && ((uintptr_t)sync & 7) == 0 && units <= ONE_LAUNCH_UNITS && prm.span_L <= NEAR_SPAN && st.cap > NEAR_SPAN;
}
// And in this form: rows not so long that a tile of positions takes its workgroup more rounds than the units hide.  Two launches spread them better
// where sequences are few and units short.  us per step, one launch / two, sequences as long as the rows: 256 units x 257 slots of one sequence, 57 344
// positions in one round 8.7 / 10.5, 65 536 in two 11.9 / 10.7; x 1025, 131 072 in two 16.8 / 20.5; 1024 x 257 of four, 65 536 in two 19.4 / 22.7, 200 000 in
// four 23.9 / 29.2; 1024 x 65, 40 960 in two 11.2 / 11.4, in four 17.4 / 11.4; without an attention term 1024 x 501, 65 536 in two 11.0 / 11.5, 131 072 in four
// 17.5 / 13.7.
int rounds_of(const ta_decode_state& st, UnitForm f) { return (int)((st.cap - 1) / ((int64_t)MAX_TILES * TILE_PER * 64 * f.waves)) + 1; }
bool rows_fit(bool scored, const ta_decode_state& st, UnitForm f)
{
    if (f.waves >= 8) return rounds_of(st, f) <= 2;
    if (st.batch < 4) return rounds_of(st, f) <= 1;
    return rounds_of(st, f) <= (scored ? 2 : 1) * (f.waves >= 4 ? 2 : 1);
}
// The workgroups of positions: behind the units, whose keys they leave the memory to (us per step, in front / behind: 256 units x 1025 slots 15.7 /
// 15.1, 1024 x 257 16.5 / 16.0); in front of them where their chain of round trips is what takes longest, which is without an
// attention term (512 x 1025 7.5 / 9.1, 1024 x 1025 10.0 / 12.1, 3072 x 501 10.8 / 12.1, 4096 x 201 9.0 / 10.7) or with several rounds (1024 x 257, rows
// of 40 960 positions in two 18.8 / 21.0; 256 x 1025, 131 072 in two 17.0 / 19.2).
bool positions_first(bool scored, const ta_decode_state& st, UnitForm f) { return !scored || rounds_of(st, f) > 1; }

// Key tiles in flight: two per wavefront where wavefronts share a unit - enough with all that then share a compute unit, and the
// registers let more of them do so (six, us per step: 1025 slots, 256 units 21.0 -> 19.8, 1024 units 56.6 -> 52.7; 1501
// slots, 1024 units 94.4 -> 75.4).  One wavefront per unit: three at four wavefronts per SIMD; paged slots need
// more registers for their addresses: four at three wavefronts per SIMD instead of spilling.
template <int GH, bool PAGED, bool SCORED, bool SMALL, int WAVES, int SPL>
__global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu((WAVES > 1 ? 2 : PAGED ? 3 : 4))))
decode_unit_kernel(ta_decode_state st, UnitArgs a, SlotPages pg)
{
    decode_unit<GH, PAGED, SCORED, SMALL, (WAVES > 1 ? 2 : PAGED ? 4 : 3), WAVES, SPL>(st, a, pg);
}

// Paged slots: at most 128 registers (none of them in scratch), so that two workgroups of eight wavefronts share a compute unit as
// those of the two-launch form do: with 131 to 135 they did not, and where units are more than compute units the step fell behind two
// launches (us per step, 135 / 128 registers / two launches: 320 units x 1135 slots 29.3 / 25.7 / 28.0, 512 x 1025 33.7 / 30.0 / 31.5, 1024 x 1025
// 63.2 / 55.0 / 55.3, 256 x 1025 17.9 / 17.8 / 20.0; from a graph, with none in scratch, 25.1, 28.0, 51.4, 16.3 / 27.0, 29.5, 53.0, 18.0).
template <int GH, bool PAGED, bool SCORED, int WAVES, int SPL>
__global__ void __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(PAGED && SCORED ? 4 : 2)))
decode_step_kernel(ta_decode_state st, UnitArgs a, SlotPages pg, StepArgs f)
{
    decode_unit<GH, PAGED, SCORED, true, 2, WAVES, SPL, true>(st, a, pg, &f);
}

using UnitKernel = void (*)(ta_decode_state, UnitArgs, SlotPages);
using StepKernel = void (*)(ta_decode_state, UnitArgs, SlotPages, StepArgs);

template <int GH, bool PAGED, bool SCORED>
StepKernel step_kernel(UnitForm f)
{
    switch (f.waves * 8 + f.spl) {
        case 2 * 8 + 2: return decode_step_kernel<GH, PAGED, SCORED, 2, 2>;
        case 4 * 8 + 2: return decode_step_kernel<GH, PAGED, SCORED, 4, 2>;
        case 4 * 8 + 3: return decode_step_kernel<GH, PAGED, SCORED, 4, 3>;
        case 8 * 8 + 3: return decode_step_kernel<GH, PAGED, SCORED, 8, 3>;
        default: return decode_step_kernel<GH, PAGED, SCORED, 8, 4>;
    }
}

template <int GH, bool PAGED>
UnitKernel unit_kernel(bool scored, UnitForm f)
{
    if (!scored) return f.spl ? decode_unit_kernel<GH, PAGED, false, true, 1, LOOP_SPL> : decode_unit_kernel<GH, PAGED, false, false, 1, LOOP_SPL>;
    switch (f.waves * 8 + f.spl) {
        case 1 * 8 + 2: return decode_unit_kernel<GH, PAGED, true, true, 1, 2>;
        case 2 * 8 + 2: return decode_unit_kernel<GH, PAGED, true, true, 2, 2>;
        case 4 * 8 + 2: return decode_unit_kernel<GH, PAGED, true, true, 4, 2>;
        case 4 * 8 + 3: return decode_unit_kernel<GH, PAGED, true, true, 4, 3>;
        case 8 * 8 + 3: return decode_unit_kernel<GH, PAGED, true, true, 8, 3>;
        default: return decode_unit_kernel<GH, PAGED, true, true, 8, 4>;
    }
}

DeviceOnce g_setup;

SlotPages slot_pages(const ta_decode_state& st)
{
    SlotPages pg = {};
    pg.page_size = 1;
    pg.page_shift = -1;
    if (st.pages) {
        const ta_paged_kv& p = *st.pages;
        pg.table = p.block_table;
        pg.s_layer = p.stride[0] / 8;
        pg.s_page = p.stride[1] / 8;
        pg.s_slot = p.stride[2] / 8;
        pg.s_head = p.stride[3] / 8;
        pg.page_size = p.page_size;
        pg.max_pages = p.max_pages;
        pg.num_pages = p.num_pages;
        if ((p.page_size & (p.page_size - 1)) == 0) {
            pg.page_shift = 0;
            while ((1 << pg.page_shift) < p.page_size) ++pg.page_shift;
        }
    }
    return pg;
}

template <int GH>
hipError_t unit_attributes()
{
    // dynamic LDS above 64 KB (large budgets with an attention term) needs the attribute
    hipError_t e = hipSuccess;
    for (const UnitForm f : {UnitForm{1, 2}, UnitForm{2, 2}, UnitForm{4, 2}, UnitForm{4, 3}, UnitForm{8, 3}, UnitForm{8, 4}})
        for (const UnitKernel k : {unit_kernel<GH, false>(true, f), unit_kernel<GH, true>(true, f)})
            if (e == hipSuccess)
                e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    for (const UnitForm f : {UnitForm{2, 2}, UnitForm{4, 2}, UnitForm{4, 3}, UnitForm{8, 3}, UnitForm{8, 4}})
        for (const StepKernel k : {step_kernel<GH, false, true>(f), step_kernel<GH, true, true>(f)})
            if (e == hipSuccess)
                e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    return e;
}

template <int GH>
void launch_unit(const ta_decode_state& st, const UnitArgs& a, const SlotPages& pg, const StepArgs* one, unsigned grid, size_t lds, UnitForm f,
                 hipStream_t s)
{
    if (one) {
        // (how many heads a group has is nothing to a unit without an attention term)
        const StepKernel kernel = a.alpha != 0.0f ? (st.pages ? step_kernel<GH, true, true>(f) : step_kernel<GH, false, true>(f))
                                                  : (st.pages ? step_kernel<4, true, false>(f) : step_kernel<4, false, false>(f));
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * f.waves), lds, s, st, a, pg, *one);
        return;
    }
    const bool scored = a.alpha != 0.0f;
    const UnitKernel kernel = st.pages ? unit_kernel<GH, true>(scored, f) : unit_kernel<GH, false>(scored, f);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * f.waves), lds, s, st, a, pg);
}

}  // namespace

hipError_t decode_setup()
{
    return g_setup.run([](int) {
        hipError_t e = unit_attributes<4>();
        if (e == hipSuccess) e = unit_attributes<8>();
        if (e == hipSuccess) e = unit_attributes<MAX_GROUP>();
        return e;
    });
}

hipError_t launch_decode_init(const ta_decode_state& st, const int32_t* tok, const int32_t* seq_len, int32_t n,
                              const uint8_t* anchor, const float* anchor_B, const float* A,
                              const int32_t* idx, const int32_t* cnt, const void* Kout, const void* Vout,
                              float B, hipStream_t s)
{
    InitArgs a;
    a.tok = tok;
    a.seq_len = seq_len;
    a.anchor = anchor;
    a.anchor_B = anchor_B;
    a.A = A;
    a.idx = idx;
    a.cnt = cnt;
    a.Kout = (const uint4*)Kout;
    a.Vout = (const uint4*)Vout;
    a.rows = (int64_t)st.layers * st.batch * st.hkv * (st.K + 1);
    a.slot_blocks = (a.rows + DU_THREADS - 1) / DU_THREADS;
    a.row_blocks = Kout ? (a.rows + INIT_ROWS - 1) / INIT_ROWS : 0;      // (paged state whose rows are in place already: none)
    a.by_slots = divider((uint32_t)(st.K + 1));
    a.by_hkv = divider((uint32_t)st.hkv);
    a.by_batch = divider((uint32_t)st.batch);
    a.n = n;
    a.B = B;
    a.seq_blocks = (int64_t)((st.cap + DU_THREADS - 1) / DU_THREADS) * st.batch;
    const GridLines grid(a.slot_blocks + 2 * a.row_blocks + a.seq_blocks);
    const SlotPages pg = slot_pages(st);
    if (st.pages) hipLaunchKernelGGL(decode_init_kernel<true>, dim3(grid.x, grid.lines), dim3(DU_THREADS), 0, s, st, a, pg);
    else hipLaunchKernelGGL(decode_init_kernel<false>, dim3(grid.x, grid.lines), dim3(DU_THREADS), 0, s, st, a, pg);
    return hipGetLastError();
}

hipError_t launch_decode_step(const ta_decode_state& st, const int32_t* new_tok, const void* q_new,
                              const void* k_new, const void* v_new, const MatchTable& tab,
                              const ta_params& prm, int32_t* evicted, int32_t* sync, hipStream_t s)
{
    UnitArgs a;
    a.q_new = (const uint4*)q_new;
    a.k_new = (const uint4*)k_new;
    a.v_new = (const uint4*)v_new;
    a.evicted = evicted;
    a.n_sink = prm.n_sink;
    a.n_recent = prm.n_recent;
    a.alpha = prm.alpha;
    a.beta = prm.beta;
    a.gamma = prm.gamma;
    a.scale_log2 = (float)(1.4426950408889634 / sqrt((double)st.d));
    a.last_query = prm.last_query;
    const unsigned units = (unsigned)(st.layers * st.batch * st.hkv);
    const int G = st.hq / st.hkv;
    const int slots = st.K + 1;
    // slot table; with an attention term also one key tile, the new key row and the logits
    const size_t wstride = (size_t)((slots + 3) & ~3);
    const SlotPages pg = slot_pages(st);
    const size_t page_list = st.pages ? (size_t)((slots - 1) / pg.page_size + 1) : 0;      // the pages of the unit's slots
    // per wavefront a key tile and the new key row; several wavefronts: 64 words more
    const auto scored_floats = [&](int waves) { return wstride + (1024 + 64) * (size_t)waves + (waves > 1 ? 64 : 0) + (size_t)G * wstride; };
    const bool scored = prm.alpha != 0.0f;
    const bool can = one_launch(prm, st, units, sync);
    const UnitForm shared = unit_form(scored, slots, units, can);
    const bool one = can && shared.waves > 1 && rows_fit(scored, st, shared);
    const UnitForm form = one ? shared : unit_form(scored, slots, units, false);
    size_t lds_floats = scored ? scored_floats(form.waves) : wstride + (form.waves > 1 ? 64 : 0);
    a.pg_off = (int32_t)lds_floats;
    a.units = (int32_t)units;
    a.group = G;
    a.by_hkv = divider((uint32_t)st.hkv);
    a.by_batch = divider((uint32_t)st.batch);
    a.decay = prm.budget_decay;
    lds_floats += page_list;
    if (one && lds_floats < 4 + NEAR_SPAN + (size_t)TILE_PER * 64 * form.waves) lds_floats = 4 + NEAR_SPAN + (size_t)TILE_PER * 64 * form.waves;
    const size_t lds = lds_floats * sizeof(float);
    if (lds > 160 * 1024) return hipErrorInvalidValue;      // (a unit's logits are at most 15 360: 113 KB in all)
    const hipError_t attr_err = decode_setup();
    if (attr_err != hipSuccess) return attr_err;
    if (one) {
        const int32_t per_seq = (int32_t)(units / (unsigned)st.batch);
        StepArgs sa;
        sa.tile_shift = 0;                                 // TILE_PER positions per thread, more where that would be too many tiles
        while ((1 << sa.tile_shift) < TILE_PER * 64 * form.waves || ((st.cap - 1) >> sa.tile_shift) >= MAX_TILES) ++sa.tile_shift;
        sa.tiles = ((st.cap - 1) >> sa.tile_shift) + 1;
        sa.parts = (per_seq < SYNC_LINES ? per_seq : SYNC_LINES) + sa.tiles;
        const uint64_t grid = (uint64_t)units + (uint64_t)sa.tiles * (uint64_t)st.batch;
        if (grid > 0x7FFFFFFFull) return hipErrorInvalidValue;
        sa.lead = positions_first(scored, st, form) ? (int32_t)(grid - units) : 0;
        sa.new_tok = new_tok;
        sa.sync = sync;
        sa.per_seq = per_seq;
        sa.L = prm.span_L;
        sa.span = prm.span_L > 0 ? ((1ull << (8 * prm.span_L)) - 1ull) << (8 * (NEAR_SPAN - prm.span_L)) : 0ull;
        sa.span_bits = flag_bits(sa.span);
        for (int k = 0; k <= NEAR_SPAN; ++k) sa.pw[k] = tab.pw[k];
        for (int e = 0; e < TA_MAX_TABLE; ++e) {
            sa.rid[e] = make_int4(tab.rid[e][0], tab.rid[e][1], tab.rid[e][2], tab.rid[e][3]);
            sa.len[e] = e < tab.E ? tab.len[e] : 0;
        }
        sa.B = tab.B;
        if (G <= 4) launch_unit<4>(st, a, pg, &sa, (unsigned)grid, lds, form, s);
        else if (G <= 8) launch_unit<8>(st, a, pg, &sa, (unsigned)grid, lds, form, s);
        else launch_unit<MAX_GROUP>(st, a, pg, &sa, (unsigned)grid, lds, form, s);
        return hipGetLastError();
    }
    DecodeTable dt;
    for (int e = 0; e < TA_MAX_TABLE; ++e) {
        for (int k = 0; k < TA_MAX_GRAM; ++k) dt.rid[e][k] = tab.rid[e][k];
        dt.len[e] = tab.len[e];
    }
    dt.E = tab.E;
    dt.B = tab.B;
    VouchArgs va;
    va.L = prm.span_L;
    for (int k = 0; k <= TA_MAX_SPAN; ++k) va.pw[k] = tab.pw[k];
    // the units, then one workgroup per 256 positions for the budget decay
    const unsigned tiles = (unsigned)((st.cap + 255) / 256);
    const uint64_t grid = (uint64_t)units + (uint64_t)tiles * (uint64_t)st.batch;
    if (grid > 0x7FFFFFFFull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(decode_seq_vouch_kernel, dim3(tiles + 1, (unsigned)st.batch), dim3(256), 0, s, st, new_tok, dt, va);
    if (G <= 4) launch_unit<4>(st, a, pg, nullptr, (unsigned)grid, lds, form, s);
    else if (G <= 8) launch_unit<8>(st, a, pg, nullptr, (unsigned)grid, lds, form, s);
    else launch_unit<MAX_GROUP>(st, a, pg, nullptr, (unsigned)grid, lds, form, s);
    return hipGetLastError();
}

}  // namespace ta
