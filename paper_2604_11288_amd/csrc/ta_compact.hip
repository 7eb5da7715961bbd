// Step 5 of the eviction pass: gather of the retained K/V rows (index_select
// along the sequence dimension, Sec. 3.2 "Token selection"; Alg. 1, eviction
// step).  Pure data movement, bound by HBM.
//
// A 256-byte row (d = 128 bf16) is moved by 16 lanes with one 16-byte load and one 16-byte store each, two rows in flight
// per lane.  A workgroup takes 32 consecutive rows of the flat [units][K] order and one of the two tensors: the first half of the launch
// moves the keys, the second the values.  The memory's changes between reading and writing bound it, and these cost
// least where few places are open at a time.  (us, 64 rows of both tensors of one unit per workgroup / this: 256 units x 1000 rows 47.6 / 43.9,
// 1024 x 512 94.6 / 88.3 = 6.1 TB/s read and written, 8192 x 200 306 / 270, over pages 329 / 286; one or four rows in flight per lane 49.8 and 45.8, 101 and
// 91.8, 301 and 278.)
// By flat rows, as units alone left the last workgroup of each with what does not fill it, half of them all but empty
// at 33 rows: 32 rows of one unit per workgroup / this, 16 384 x 33 119 / 90, over pages 153 / 97, x 16 over pages 68 / 50, x 4 27.7 / 14.5, 65 536 x 8 over
// pages 201 / 94, 2048 x 40 19.4 / 17.1; 32 rows of one unit take as long as before, 64 x 1024 13.2 / 13.3, 16 384 x 64 170 / 170, and some 0.3 us more with
// one list for all units.  (Workgroups that lie within a unit in code of their own, with what follows from the unit uniform: 2 to 4 % slower.)
#include "ta_gather.h"

namespace ta {

namespace {

constexpr int COMPACT_THREADS = 256, COMPACT_ITERS = 2;
constexpr int ROWS_PER_ITER = COMPACT_THREADS / 16;      // 16 rows per pass over the block
constexpr int ROWS_PER_BLOCK = ROWS_PER_ITER * COMPACT_ITERS;

template <bool PAGED, bool LAYERED, bool DST_PAGED = false>
__global__ void __launch_bounds__(COMPACT_THREADS)
compact_kernel(CompactArgs a)
{
    const uint32_t block = blockIdx.z * GRID_LINE + blockIdx.x;
    if (block >= a.blocks) return;
    const bool values = blockIdx.y != 0;
    const int64_t row0 = (int64_t)block * ROWS_PER_BLOCK;
    const int32_t unit0 = a.rows <= 0x7FFFFFFF ? (int32_t)divide((uint32_t)row0, a.by_K) : (int32_t)(row0 / a.K);   // uniform
    const int32_t slot0 = (int32_t)(row0 - (int64_t)unit0 * a.K);
    const int lane16 = threadIdx.x & 15;
    int32_t unit[COMPACT_ITERS], r[COMPACT_ITERS], p[COMPACT_ITERS], count[COMPACT_ITERS];
    int32_t h[COMPACT_ITERS], b[COMPACT_ITERS], l[COMPACT_ITERS];
#pragma unroll
    for (int j = 0; j < COMPACT_ITERS; ++j) {
        const int32_t off = (int32_t)(threadIdx.x >> 4) + j * ROWS_PER_ITER, s = slot0 + off;
        const bool in = row0 + off < a.rows;
        const int32_t du = (int32_t)divide((uint32_t)s, a.by_K);
        unit[j] = in ? unit0 + du : unit0;
        r[j] = in ? s - du * a.K : 0;
        const int32_t pair = (int32_t)divide((uint32_t)unit[j], a.by_hkv);
        h[j] = unit[j] - pair * a.hkv;
        l[j] = (int32_t)divide((uint32_t)pair, a.by_batch);
        b[j] = pair - l[j] * a.batch;
        const int32_t sel = a.idx_shared ? b[j] : unit[j];
        p[j] = a.idx[(size_t)sel * (size_t)a.K + r[j]];
        count[j] = in ? a.cnt[sel] : 0;
    }
    bool any = false;
#pragma unroll
    for (int j = 0; j < COMPACT_ITERS; ++j) any = any || r[j] < count[j];
    if (__ballot(any) == 0ull) return;                     // the wavefront's rows are all past the retained ones
    u32x4 v[COMPACT_ITERS];
#pragma unroll
    for (int j = 0; j < COMPACT_ITERS; ++j) {
        const RowSource<PAGED, LAYERED> rows(a, l[j], b[j], h[j], lane16);
        const u32x4* in = reinterpret_cast<const u32x4*>(LAYERED ? global_ptr(values ? a.Vin_l[l[j]] : a.Kin_l[l[j]]) : (values ? a.Vin : a.Kin));
        const int32_t q = r[j] < count[j] ? p[j] : 0;      // (past the retained rows: a row of the tensor, not stored)
        v[j] = __builtin_nontemporal_load(&in[rows(q < 0 ? 0 : (q >= a.n ? a.n - 1 : q))]);
    }
    // The compacted rows are not read again by this pass: streaming stores keep them from
    // lingering in the caches as dirty lines that the next kernel's reads would have to evict.
#pragma unroll
    for (int j = 0; j < COMPACT_ITERS; ++j) {
        if (r[j] >= count[j]) continue;
        u32x4* out = reinterpret_cast<u32x4*>(LAYERED ? global_ptr(values ? a.Vout_l[l[j]] : a.Kout_l[l[j]]) : (values ? a.Vout : a.Kout));
        int64_t off = ((int64_t)(LAYERED ? unit[j] - l[j] * a.hkv * a.batch : unit[j]) * a.K + r[j]) * 16 + lane16;
        if (DST_PAGED) {
            const int32_t slot = r[j] / a.d_page_size;
            int32_t page = a.d_table[(size_t)b[j] * a.d_max_pages + slot];
            page = page < 0 ? 0 : (page >= a.d_num_pages ? a.d_num_pages - 1 : page);
            off = l[j] * a.d_layer + (int64_t)page * a.d_page + (int64_t)(r[j] - slot * a.d_page_size) * a.d_pos + h[j] * a.d_head + lane16;
        }
        __builtin_nontemporal_store(v[j], &out[off]);
    }
}

// Writes a table of per-layer addresses, handed over by value, to device memory: the kernels of the
// pass then read their layer's entries from there.  (Arrays inside those kernels' own argument
// structs were measured first: a run-time choice between a table entry and the base pointer made
// the compiler copy the whole argument block to scratch memory per lane - the compaction took
// 690 us instead of 42 - and the statistics sweep reloaded arguments inside its stage loop.)
// N layers of the five tables, packed: small argument blocks stay on the fast path (the table of
// a 32-layer model is 1.3 KB).
template <int N>
struct PackedLayerPtrs {
    const void* p[5][N];
};

template <int N>
__global__ void layer_table_kernel(PackedLayerPtrs<N> t, LayerPtrs* dst, int32_t layers)
{
    const void** out[5] = {dst->Q, dst->K, dst->V, const_cast<const void**>(reinterpret_cast<void* const*>(dst->Kout)),
                           const_cast<const void**>(reinterpret_cast<void* const*>(dst->Vout))};
    for (int i = (int)threadIdx.x; i < 5 * layers; i += (int)blockDim.x) {
        const int arr = i / layers, l = i - arr * layers;
        out[arr][l] = t.p[arr][l];
    }
}

template <int N>
void launch_layer_table_n(const LayerPtrs& h, LayerPtrs* dev_table, int32_t layers, hipStream_t st)
{
    PackedLayerPtrs<N> t;
    for (int l = 0; l < N; ++l) {
        const bool on = l < layers;
        t.p[0][l] = on ? h.Q[l] : nullptr;
        t.p[1][l] = on ? h.K[l] : nullptr;
        t.p[2][l] = on ? h.V[l] : nullptr;
        t.p[3][l] = on ? h.Kout[l] : nullptr;
        t.p[4][l] = on ? h.Vout[l] : nullptr;
    }
    hipLaunchKernelGGL(layer_table_kernel<N>, dim3(1), dim3(256), 0, st, t, dev_table, layers);
}

}  // namespace

hipError_t launch_layer_table(const LayerPtrs& host_table, LayerPtrs* dev_table, int32_t layers, hipStream_t st)
{
    if (layers <= 32) launch_layer_table_n<32>(host_table, dev_table, layers, st);
    else launch_layer_table_n<TA_MAX_LAYER_PTRS>(host_table, dev_table, layers, st);
    return hipGetLastError();
}

CompactArgs make_compact_args(const void* Kin, const void* Vin, const int32_t* idx, const int32_t* cnt, const ta_layout& lay, int32_t K,
                              int32_t idx_shared, void* Kout, void* Vout, const ta_paged_kv* pg, const LayerPtrs* lp,
                              const ta_paged_kv* dst_pg)
{
    CompactArgs a;
    a.d_table = dst_pg ? dst_pg->block_table : nullptr;
    a.d_layer = dst_pg ? dst_pg->stride[0] / 8 : 0;
    a.d_page = dst_pg ? dst_pg->stride[1] / 8 : 0;
    a.d_pos = dst_pg ? dst_pg->stride[2] / 8 : 0;
    a.d_head = dst_pg ? dst_pg->stride[3] / 8 : 0;
    a.d_page_size = dst_pg ? dst_pg->page_size : 1;
    a.d_max_pages = dst_pg ? dst_pg->max_pages : 0;
    a.d_num_pages = dst_pg ? dst_pg->num_pages : 0;
    a.Kin_l = lp ? reinterpret_cast<const uint4* const*>(&lp->K[0]) : nullptr;
    a.Vin_l = lp ? reinterpret_cast<const uint4* const*>(&lp->V[0]) : nullptr;
    a.Kout_l = lp ? reinterpret_cast<uint4* const*>(&lp->Kout[0]) : nullptr;
    a.Vout_l = lp ? reinterpret_cast<uint4* const*>(&lp->Vout[0]) : nullptr;
    a.Kin = (const uint4*)Kin;
    a.Vin = (const uint4*)Vin;
    a.idx = idx;
    a.cnt = cnt;
    a.Kout = (uint4*)Kout;
    a.Vout = (uint4*)Vout;
    if (pg) {
        a.s_layer = pg->stride[0] / 8;
        a.s_page = pg->stride[1] / 8;
        a.s_pos = pg->stride[2] / 8;
        a.s_head = pg->stride[3] / 8;
        a.s_batch = 0;
        a.table = pg->block_table;
        a.page_size = pg->page_size;
        a.max_pages = pg->max_pages;
        a.num_pages = pg->num_pages;
    } else {
        a.s_layer = lay.kv_stride[0] / 8;
        a.s_batch = lay.kv_stride[1] / 8;
        a.s_head = lay.kv_stride[2] / 8;
        a.s_pos = lay.kv_stride[3] / 8;
        a.table = nullptr;
        a.s_page = 0;
        a.page_size = a.max_pages = a.num_pages = 0;
    }
    a.batch = lay.batch;
    a.hkv = lay.hkv;
    a.n = lay.n;
    a.K = K;
    a.idx_shared = idx_shared;
    a.rows = (int64_t)lay.layers * lay.batch * lay.hkv * K;
    a.blocks = (uint32_t)((a.rows + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK);
    a.by_K = divider((uint32_t)K);
    a.by_hkv = divider((uint32_t)lay.hkv);
    a.by_batch = divider((uint32_t)lay.batch);
    return a;
}

hipError_t launch_compact(const void* Kin, const void* Vin, const int32_t* idx, const int32_t* cnt,
                          const ta_layout& lay, int32_t K, int32_t idx_shared,
                          void* Kout, void* Vout, const ta_paged_kv* pg, const LayerPtrs* lp, hipStream_t st,
                          const ta_paged_kv* dst_pg)
{
    const CompactArgs a = make_compact_args(Kin, Vin, idx, cnt, lay, K, idx_shared, Kout, Vout, pg, lp, dst_pg);
    const int64_t blocks = (a.rows + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK;
    if (blocks > 0x7FFFFFFFll) return hipErrorInvalidValue;              // (Divider)
    const GridLines lines(blocks);
    const dim3 grid(lines.x, 2, lines.lines), block(COMPACT_THREADS);
    if (dst_pg && pg) hipLaunchKernelGGL((compact_kernel<true, false, true>), grid, block, 0, st, a);
    else if (dst_pg) hipLaunchKernelGGL((compact_kernel<false, false, true>), grid, block, 0, st, a);
    else if (pg && lp) hipLaunchKernelGGL((compact_kernel<true, true>), grid, block, 0, st, a);
    else if (pg) hipLaunchKernelGGL((compact_kernel<true, false>), grid, block, 0, st, a);
    else if (lp) hipLaunchKernelGGL((compact_kernel<false, true>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((compact_kernel<false, false>), grid, block, 0, st, a);
    return hipGetLastError();
}

}  // namespace ta
