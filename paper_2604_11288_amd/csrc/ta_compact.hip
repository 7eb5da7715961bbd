// Step 5 of the eviction pass: gather of the retained K/V rows (index_select
// along the sequence dimension, Sec. 3.2 "Token selection"; Alg. 1, eviction
// step).  Pure data movement, bound by HBM.
//
// A 256-byte row (d = 128 bf16) is moved by 16 lanes with one 16-byte load and one 16-byte store each, two rows in flight
// per lane.  A workgroup takes 32 consecutive output rows of one unit and one of the two tensors: the first half of the launch
// moves the keys, the second the values.  The memory's changes between reading and writing bound it, and these cost
// least where few places are open at a time.  (us, 64 rows of both tensors per workgroup / this: 256 units x 1024 rows 46.6 / 44.2,
// 1024 x 512 95 / 90, in one run of rows 96.5 / 83.3 = 6.4 TB/s read and written, 1024 x 777 141.5 / 132, 4096 x 100 80.8 / 73.4; one
// tensor, 64 rows of 256 threads 45.5, 92.7, 88.8, 136.5, 76.5; 16 rows of 128 threads 43.9, 89.4, 85, 132.9, 69.7, but 2048 x 20 11.0 for 9.3.)
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
    const int32_t unit = (int32_t)divide(block, a.by_blocks);
    const int32_t blk = (int32_t)block - unit * a.blocks_per_unit;
    const bool values = blockIdx.y != 0;
    const int32_t pair = (int32_t)divide((uint32_t)unit, a.by_hkv), h = unit - pair * a.hkv;
    const int32_t l = (int32_t)divide((uint32_t)pair, a.by_batch), b = pair - l * a.batch;
    const int32_t sel = a.idx_shared ? b : unit;
    const int lane16 = threadIdx.x & 15;
    const int32_t row0 = blk * ROWS_PER_BLOCK + (int32_t)(threadIdx.x >> 4);
    const int32_t* idx = a.idx + (size_t)sel * (size_t)a.K;
    int32_t p[COMPACT_ITERS];
#pragma unroll
    for (int j = 0; j < COMPACT_ITERS; ++j) {              // requested together with the count
        const int32_t r = row0 + j * ROWS_PER_ITER;
        p[j] = idx[r < a.K ? r : a.K - 1];
    }
    int32_t cnt = a.cnt[sel];
    cnt = cnt > a.K ? a.K : cnt;
    if (blk * ROWS_PER_BLOCK >= cnt) return;              // whole block past the retained rows
    const RowSource<PAGED, LAYERED> rows(a, l, b, h, lane16);
    const u32x4* in = reinterpret_cast<const u32x4*>(LAYERED ? global_ptr(values ? a.Vin_l[l] : a.Kin_l[l]) : (values ? a.Vin : a.Kin));
    u32x4* out = reinterpret_cast<u32x4*>(LAYERED ? global_ptr(values ? a.Vout_l[l] : a.Kout_l[l]) : (values ? a.Vout : a.Kout));
    u32x4 v[COMPACT_ITERS];
#pragma unroll
    for (int j = 0; j < COMPACT_ITERS; ++j) {
        const int32_t r = row0 + j * ROWS_PER_ITER;        // (past the last row: an index within the tensor, not stored)
        const int32_t q = r < cnt ? p[j] : p[0];
        v[j] = __builtin_nontemporal_load(&in[rows(q < 0 ? 0 : (q >= a.n ? a.n - 1 : q))]);
    }
    // The compacted rows are not read again by this pass: streaming stores keep them from
    // lingering in the caches as dirty lines that the next kernel's reads would have to evict.
    const int64_t out_base = (int64_t)(LAYERED ? unit - l * a.hkv * a.batch : unit) * a.K * 16 + lane16;
#pragma unroll
    for (int j = 0; j < COMPACT_ITERS; ++j) {
        const int32_t r = row0 + j * ROWS_PER_ITER;
        if (r >= cnt) continue;
        int64_t off = out_base + (int64_t)r * 16;
        if (DST_PAGED) {
            const int32_t slot = r / a.d_page_size;
            int32_t page = a.d_table[(size_t)b * a.d_max_pages + slot];
            page = page < 0 ? 0 : (page >= a.d_num_pages ? a.d_num_pages - 1 : page);
            off = l * a.d_layer + (int64_t)page * a.d_page + (int64_t)(r - slot * a.d_page_size) * a.d_pos + h * a.d_head + lane16;
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
    a.blocks_per_unit = (K + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK;
    a.blocks = (uint32_t)((int64_t)lay.layers * lay.batch * lay.hkv * a.blocks_per_unit);
    a.by_blocks = divider((uint32_t)a.blocks_per_unit);
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
    const int64_t blocks = (int64_t)lay.layers * lay.batch * lay.hkv * a.blocks_per_unit;
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
