// Step 5's arguments, and the gather of one unit's rows by a workgroup that has just selected them.
#pragma once
#include "ta_internal.h"
#include "ta_order.h"

namespace ta {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct CompactArgs {
    const uint4* Kin;
    const uint4* Vin;
    const int32_t* idx;
    const int32_t* cnt;
    uint4* Kout;
    uint4* Vout;
    int64_t s_layer, s_batch, s_head, s_pos;   // input strides in 16-byte units
    int32_t batch, hkv, n, K;
    int32_t idx_shared;
    int64_t rows;                              // units * K, of either tensor
    uint32_t blocks;
    Divider by_K, by_hkv, by_batch;
    // paged input: rows are addressed through the block table (s_batch unused, s_page per page)
    const int32_t* table;
    int64_t s_page;
    int32_t page_size, max_pages, num_pages;
    // one tensor per layer: DEVICE tables; layer l reads Kin_l[l], Vin_l[l] and writes Kout_l[l], Vout_l[l]
    const uint4* const* Kin_l;
    const uint4* const* Vin_l;
    uint4* const* Kout_l;
    uint4* const* Vout_l;
    // paged output: row r of a unit goes to slot r of its sequence's pages in the destination pools
    const int32_t* d_table;
    int64_t d_layer, d_page, d_pos, d_head;    // destination strides in 16-byte units
    int32_t d_page_size, d_max_pages, d_num_pages;
};

// marks a pointer read from a device table as a global address (else it is accessed with flat instructions)
template <typename T>
__device__ __forceinline__ T* global_ptr(T* p)
{
    typedef __attribute__((address_space(1))) T* gp;
    return (T*)(gp)(uintptr_t)p;
}

CompactArgs make_compact_args(const void* Kin, const void* Vin, const int32_t* idx, const int32_t* cnt, const ta_layout& lay, int32_t K,
                              int32_t idx_shared, void* Kout, void* Vout, const ta_paged_kv* pg, const LayerPtrs* lp,
                              const ta_paged_kv* dst_pg);

// Where the rows of a unit lie (16-byte units; a lane moves the 16 bytes lane16 of a row).
template <bool PAGED, bool LAYERED>
struct RowSource {
    const CompactArgs& a;
    int32_t b;
    int64_t base;
    __device__ RowSource(const CompactArgs& args, int32_t l, int32_t seq, int32_t h, int lane16)
        : a(args), b(seq), base((LAYERED ? 0 : l * args.s_layer) + (PAGED ? 0 : seq * args.s_batch) + h * args.s_head + lane16) {}
    __device__ __forceinline__ int64_t operator()(int32_t p) const
    {
        if (PAGED) {
            const int32_t slot = p / a.page_size;
            int32_t page = a.table[(size_t)b * a.max_pages + slot];
            page = page < 0 ? 0 : (page >= a.num_pages ? a.num_pages - 1 : page);
            return base + (int64_t)page * a.s_page + (int64_t)(p - slot * a.page_size) * a.s_pos;
        }
        return base + (int64_t)p * a.s_pos;
    }
};

// How a selection kernel moves the rows it has selected: not at all (a launch of its own does), or from this kind of cache.
enum Gather { GATHER_NONE, GATHER_DENSE, GATHER_PAGED, GATHER_LAYERED };

// The rows `list[0 .. cnt)` of a unit, by all threads of the workgroup: 16 lanes per row, the loads of GROUP rows of K and V
// per lane before the first store.
template <int THREADS, int KIND>
__device__ __forceinline__ void gather_rows(const CompactArgs& a, const int32_t unit, const int32_t cnt, const uint32_t* list, const int tid)
{
    constexpr bool PAGED = KIND == GATHER_PAGED, LAYERED = KIND == GATHER_LAYERED;
    constexpr int STEP = THREADS / 16, GROUP = 4;
    const int32_t h = unit % a.hkv, b = (unit / a.hkv) % a.batch, l = unit / (a.hkv * a.batch);
    const int lane16 = tid & 15, rsub = tid >> 4;
    const RowSource<PAGED, LAYERED> src(a, l, b, h, lane16);
    const u32x4* Kin = reinterpret_cast<const u32x4*>(LAYERED ? global_ptr(a.Kin_l[l]) : a.Kin);
    const u32x4* Vin = reinterpret_cast<const u32x4*>(LAYERED ? global_ptr(a.Vin_l[l]) : a.Vin);
    const int64_t out = (int64_t)(LAYERED ? unit - l * a.hkv * a.batch : unit) * a.K * 16 + lane16;
    u32x4* Kout = reinterpret_cast<u32x4*>(LAYERED ? global_ptr(a.Kout_l[l]) : a.Kout) + out;
    u32x4* Vout = reinterpret_cast<u32x4*>(LAYERED ? global_ptr(a.Vout_l[l]) : a.Vout) + out;
    for (int32_t r0 = rsub; r0 < cnt; r0 += GROUP * STEP) {
        u32x4 k[GROUP], v[GROUP];
        int64_t from[GROUP];
#pragma unroll
        for (int j = 0; j < GROUP; ++j) {
            const int32_t r = r0 + j * STEP;
            from[j] = src((int32_t)list[r < cnt ? r : cnt - 1]);   // past the end: the last row again, not stored
        }
#pragma unroll
        for (int j = 0; j < GROUP; ++j) {
            k[j] = __builtin_nontemporal_load(&Kin[from[j]]);
            v[j] = __builtin_nontemporal_load(&Vin[from[j]]);
        }
#pragma unroll
        for (int j = 0; j < GROUP; ++j) {
            const int32_t r = r0 + j * STEP;
            if (r < cnt) {
                __builtin_nontemporal_store(k[j], &Kout[(int64_t)r * 16]);
                __builtin_nontemporal_store(v[j], &Vout[(int64_t)r * 16]);
            }
        }
    }
}

}  // namespace ta
