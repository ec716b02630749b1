// Sweep-block copy of the relabelled matrix (Algorithm 1, the SpMV line, on
// large power-law matrices): the setup kernels that cut the rows into sweep
// blocks and store each block's entries in column order.
//
// Why: in row order the 64 gathers of one wavefront instruction fall on up
// to 64 different 128-byte lines of x, and beyond L2 each line costs a
// memory request.  A wavefront that walks a block's entries in column order
// gathers neighbouring columns in one instruction, which share lines, above
// all in the dense head of x where the hub-first relabelling put the most
// gathered columns.  (Measured at R-MAT scale 26, FP32: 1.02e9 -> 6.5e8
// read requests per SpMV at about the same L2 hit rate.)  The row sums are
// then accumulated in LDS (one slot per row of the block) instead of in row
// order.
//
// Build (all on the device, stream-ordered): the block table (first owned
// row and first entry of every block); the relabelling fill then writes each
// entry's row within its block and position within it (one 32-bit word, in
// row order); one segmented radix sort of the relabelled column indices with
// those words as values (rocPRIM, one segment per block, keys sorted on the
// bits above the line offset so that entries of one line keep their row
// order); then the rows and, gathered by the sorted positions, the values.
// Entries of x past its first SW_HEAD_BYTES are not gathered by the sweep: a
// pass before it lays them out in the order of the tables built here (tail
// columns: panels of x that fit LDS; see k_sweep_tail).
#include <cstring>

#include <rocprim/device/device_segmented_radix_sort.hpp>

#include "../../include/lanczos_topk.h"
#include "lz_spmv.h"

namespace lz {

namespace {

// One workgroup per segment through all radix passes, no partitioning of
// the segments by size: rocPRIM's partitioned path reads segment counts back
// to the host, which a stream-ordered solve cannot do.
//
// Digits of 8 bits, or of 10 where that saves a pass: 17 to 20 bits take two
// passes instead of three (R-MAT 25 FP32, 20 bits: 17.4 -> 15.2 ms).  Past 20
// bits both take three, and the wider digits' passes cost more (1024 counters,
// workgroups of 1024).
using SortConfig8 = rocprim::segmented_radix_sort_config<8, rocprim::kernel_config<256, 16>,
                                                         rocprim::DisabledWarpSortConfig, false>;
using SortConfig10 = rocprim::segmented_radix_sort_config<10, rocprim::kernel_config<1024, 8>,
                                                          rocprim::DisabledWarpSortConfig, false>;

hipError_t sort_blocks(void* tmp, size_t& bytes, const uint32_t* keys_in, uint32_t* keys_out, const uint32_t* vin,
                       uint32_t* vout, int64_t nnz, int64_t nb, const int64_t* begin, int bit0, int bit1,
                       hipStream_t s) {
    if (bit1 - bit0 > 16 && bit1 - bit0 <= 20)
        return rocprim::segmented_radix_sort_pairs<SortConfig10>(tmp, bytes, keys_in, keys_out, vin, vout,
                                                                 (unsigned int)nnz, (unsigned int)nb, begin, begin + 1,
                                                                 (unsigned int)bit0, (unsigned int)bit1, s);
    return rocprim::segmented_radix_sort_pairs<SortConfig8>(tmp, bytes, keys_in, keys_out, vin, vout,
                                                            (unsigned int)nnz, (unsigned int)nb, begin, begin + 1,
                                                            (unsigned int)bit0, (unsigned int)bit1, s);
}

// Block table: ob[b] = first row whose end item lies at or after b * items
// (n if none), e[b] = first entry of block b.  When the device did
// not choose the sweep-block copy every block is empty (e = 0), so the sort
// that follows has nothing to do.
__global__ __launch_bounds__(BLOCK) void k_sw_blocks(const State* st, const int64_t* __restrict__ rp, int64_t n,
                                                     int64_t nnz, int64_t nb, int64_t items, int32_t* ob,
                                                     int64_t* e, uint32_t* queue) {
    const bool on = st->status == 0 && st->reordered && st->packed == PACK_SWEEP;
    if (blockIdx.x == 0 && threadIdx.x < 8) queue[threadIdx.x] = 0u;
    for (int64_t b = (int64_t)blockIdx.x * BLOCK + threadIdx.x; b <= nb; b += (int64_t)gridDim.x * BLOCK) {
        if (!on) {
            ob[b] = 0;
            e[b] = 0;
            continue;
        }
        const int64_t target = b * items;
        int64_t lo = 0, hi = n;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (rp[mid + 1] + SW_W * mid >= target)
                hi = mid;
            else
                lo = mid + 1;
        }
        ob[b] = (int32_t)lo;
        e[b] = lo < n ? max(rp[lo], target - SW_W * lo) : nnz;
    }
}

// Panel of a column: -1 in the head of x, 0 .. np - 1, np past the last panel.
template <class VT> __device__ __forceinline__ int sweep_panel(int32_t c, int np) {
    constexpr int64_t HEAD = SW_HEAD_BYTES / (int64_t)sizeof(VT), COLS = SW_PANEL_BYTES / (int64_t)sizeof(VT);
    return c < HEAD ? -1 : (int)min<int64_t>((c - HEAD) / COLS, np);
}

// Offsets of the tail panels in every block: seg[p * nb + b] = entries of block
// b before panel p (p <= np).  Columns ascend by panel within a block, so every
// entry that opens a panel writes the offsets of the panels since the one
// before it; one workgroup per block.
template <class VT>
__global__ __launch_bounds__(BLOCK) void k_sw_panels(const State* st, int64_t nb, const int64_t* __restrict__ e,
                                                     const int32_t* __restrict__ col, int np,
                                                     uint32_t* __restrict__ seg) {
    if (st->status != 0 || !st->reordered || st->packed != PACK_SWEEP) return;
    for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
        const int64_t e0 = e[b];
        const int cnt = (int)(e[b + 1] - e0);
        const int32_t* c = col + e0;
        for (int k = threadIdx.x; k < cnt; k += BLOCK) {
            const int p = sweep_panel<VT>(c[k], np), before = k > 0 ? sweep_panel<VT>(c[k - 1], np) : -1;
            for (int q = before + 1; q <= p; ++q) seg[q * nb + b] = (uint32_t)k;
        }
        const int last = cnt > 0 ? sweep_panel<VT>(c[cnt - 1], np) : -1;
        for (int q = last + 1 + (int)threadIdx.x; q <= np; q += BLOCK) seg[q * nb + b] = (uint32_t)cnt;
    }
}

// Entry counts of the segments (panel p of block b), to be scanned.
__global__ __launch_bounds__(BLOCK) void k_sw_seg_len(const State* st, int64_t nb, int64_t segs,
                                                      const uint32_t* __restrict__ seg, uint64_t* __restrict__ pre) {
    if (st->status != 0 || !st->reordered || st->packed != PACK_SWEEP) return;
    for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < segs; i += (int64_t)gridDim.x * BLOCK)
        pre[i] = seg[i + nb] - seg[i];
}

// The tail entries panel by panel, block by block: their columns within the
// panel; their stored column words become their positions in that order.
template <class VT>
__global__ __launch_bounds__(BLOCK) void k_sw_tail_fill(const State* st, int64_t nb, const int64_t* __restrict__ e,
                                                        const uint32_t* __restrict__ seg, int np, uint64_t* pre,
                                                        int32_t* __restrict__ col, uint16_t* __restrict__ tcol) {
    constexpr int64_t HEAD = SW_HEAD_BYTES / (int64_t)sizeof(VT), COLS = SW_PANEL_BYTES / (int64_t)sizeof(VT);
    if (st->status != 0 || !st->reordered || st->packed != PACK_SWEEP) return;
    for (int64_t b = blockIdx.x; b < nb; b += gridDim.x) {
        const int64_t e0 = e[b];
        const int k1 = (int)seg[np * nb + b];
        for (int k = (int)seg[b] + (int)threadIdx.x; k < k1; k += BLOCK) {
            const int64_t c = col[e0 + k] - HEAD, p = c / COLS;
            const int64_t v = (int64_t)pre[p * nb + b] + (k - (int64_t)seg[p * nb + b]);
            tcol[v] = (uint16_t)(c - p * COLS);
            col[e0 + k] = (int32_t)(uint32_t)v;
        }
        if (b == nb - 1 && threadIdx.x == 0)
            pre[np * nb] = pre[np * nb - 1] + (seg[np * nb + b] - seg[(np - 1) * nb + b]);
    }
}

template <class VT> void launch_sweep_tail_setup(const Plan& p, const Bufs& b, hipStream_t s) {
    const int64_t segs = (int64_t)p.sw_np * p.sw_nb;
    const unsigned gb = (unsigned)std::min<int64_t>(p.sw_nb, 16384);
    hipLaunchKernelGGL(k_sw_panels<VT>, dim3(gb), dim3(BLOCK), 0, s, b.st, p.sw_nb, b.swe, b.swcol, p.sw_np,
                       b.swseg);
    hipLaunchKernelGGL(k_sw_seg_len, dim3((unsigned)std::min<int64_t>((segs + BLOCK - 1) / BLOCK, 8192)),
                       dim3(BLOCK), 0, s, b.st, p.sw_nb, segs, b.swseg, b.swpre);
    launch_scan(&b.st->reordered, b.swpre, segs, b.swbsum, s);
    hipLaunchKernelGGL(k_sw_tail_fill<VT>, dim3(gb), dim3(BLOCK), 0, s, b.st, p.sw_nb, b.swe, b.swseg, p.sw_np,
                       b.swpre, b.swcol, b.swtcol);
}

// Measured on MI355X, R-MAT 26 FP32 (grid / slices per block / entries per
// thread in flight -> fill ms): 1024/32/1 22.6, 1024/8/8 17.2, 512/16/8
// 15.4, 256/16/8 17.2, 512/32/4 22.8, 1024/64/2 36.0, 256/8/16 12.3,
// 256/8/32 12.4, 256/4/16 12.3, 512/8/16 13.1, 128/8/32 20.5.  The first
// form, one wavefront per block with the rows found by binary search in LDS,
// took 27.9 ms.
constexpr int SWF_THREADS = 256;
constexpr int SWF_GRID = 256;
constexpr int SWF_SLICES = 8;         // work items per block
constexpr int SWF_G = 4;              // groups of 256 entries a wavefront has in flight (16 entries per lane)

// Rows within the block and values of the column-sorted entries: the sorted
// payload of entry p of block b holds its row within the block and its
// position in the block's row-ordered entries, from which its value is
// gathered.  Those gathers fall anywhere in the block (up to 512 KB of values
// in FP32, 2 MB in FP64).  So XCD x (workgroup i runs on XCD i mod 8) takes
// the blocks b = x mod 8 in order, and its workgroups draw the slices of
// those blocks from one counter per XCD: at any time an XCD works on one or
// two blocks, whose values stay in its L2 while they are gathered.  The
// payload stream and the outputs bypass L2.  Every entry's outputs depend on
// the entry alone, so the order in which slices are drawn does not matter.
// A workgroup draws its next slice before working on the current one, and
// each lane keeps 16 entries in flight, so the chain of dependent loads
// (payload, then value) is paid once per 16 entries.  Outputs go to
// sweep_place.
template <class VT>
__global__ __launch_bounds__(SWF_THREADS) void k_sw_fill(const State* st, const VT* __restrict__ val2, int64_t nb,
                                                         const int64_t* __restrict__ e,
                                                         const uint32_t* __restrict__ src,
                                                         uint16_t* __restrict__ rl, VT* __restrict__ val,
                                                         uint32_t* queue) {
    __shared__ uint32_t s_item[2];
    if (st->status != 0 || !st->reordered || st->packed != PACK_SWEEP) return;
    constexpr uint32_t POSMASK = (1u << SW_POSBITS) - 1u;
    typedef uint16_t us4 __attribute__((ext_vector_type(4)));
    typedef VT V4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t xcd = blockIdx.x & 7u;
    const int64_t nbx = (nb - xcd + 7) / 8;      // blocks of this XCD
    const int64_t items = nbx * SWF_SLICES;
    if (threadIdx.x == 0)
        s_item[0] = __hip_atomic_fetch_add(queue + xcd, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    for (int it = 0;; it ^= 1) {
        const int64_t item = s_item[it];
        if (item >= items) break;
        if (threadIdx.x == 0)
            s_item[it ^ 1] = __hip_atomic_fetch_add(queue + xcd, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int64_t b = xcd + 8 * (item / SWF_SLICES), slice = item % SWF_SLICES;
        const int64_t e0 = e[b], e1 = e[b + 1];
        if (e0 < e1) {
            // Groups of 256 entries that hold entries of the block.
            const int64_t f = e0 >> 8;
            const int ng = (int)(((e1 + 255) >> 8) - f);
            const int g1 = (int)((int64_t)ng * (slice + 1) / SWF_SLICES);
            for (int g = (int)((int64_t)ng * slice / SWF_SLICES) + wave * SWF_G; g < g1;
                 g += SWF_G * SWF_THREADS / 64) {
                uint32_t w[SWF_G][4];
                VT v[SWF_G][4];
#pragma unroll
                for (int u = 0; u < SWF_G; ++u)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int64_t k = ((f + g + u) << 8) + i * 64 + lane;
                        w[u][i] = __builtin_nontemporal_load(src + min(max(k, e0), e1 - 1));
                    }
#pragma unroll
                for (int u = 0; u < SWF_G; ++u)
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[u][i] = val2[e0 + (w[u][i] & POSMASK)];
#pragma unroll
                for (int u = 0; u < SWF_G; ++u) {
                    const int64_t k = (f + g + u) << 8;
                    if (g + u >= g1) break;
                    if (k >= e0 && k + 256 <= e1) {
                        us4 r4;
                        V4 v4;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            r4[i] = (uint16_t)(w[u][i] >> SW_POSBITS);
                            v4[i] = v[u][i];
                        }
                        __builtin_nontemporal_store(r4, (us4*)(rl + k + lane * 4));
                        __builtin_nontemporal_store(v4, (V4*)(val + k + lane * 4));
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int64_t ki = k + i * 64 + lane;
                            if (ki >= e0 && ki < e1) {
                                rl[ki] = (uint16_t)(w[u][i] >> SW_POSBITS);
                                val[ki] = v[u][i];
                            }
                        }
                    }
                }
            }
        }
        __syncthreads();                         // the next item is visible; this one is no longer read
    }
}

}  // namespace

bool sweep_applies(int64_t n, int64_t nnz, int prec, int request) {
    if (request == LZ_SWEEP_OFF || n < 2 || nnz <= 0) return false;
    // The sort counts entries and blocks in 32 bits.
    if (nnz >= (int64_t(1) << 32) - 1) return false;
    if (request == LZ_SWEEP_ON) return true;
    return n >= SWEEP_AUTO_MIN_N && (uint64_t)n * storage_bytes(prec) >= SWEEP_AUTO_MIN_X_BYTES;
}

size_t sweep_sort_bytes(int64_t nnz, int64_t nb) {
    size_t narrow = 0, wide = 0;
    if (sort_blocks(nullptr, narrow, nullptr, nullptr, nullptr, nullptr, nnz, nb, nullptr, 0, 32, nullptr) ==
            hipSuccess &&
        sort_blocks(nullptr, wide, nullptr, nullptr, nullptr, nullptr, nnz, nb, nullptr, 0, 20, nullptr) ==
            hipSuccess &&
        narrow > 0)
        return std::max(narrow, wide);
    // No device to ask (the sort's size query looks up the GPU): its two
    // double buffers plus slack; a solve checks the real size before use.
    return (size_t)nnz * 8 + ((size_t)1 << 20);
}

void launch_sweep_blocks(const Plan& p, const Bufs& b, hipStream_t s) {
    if (!p.sweep) return;
    const int gb = (int)std::min<int64_t>((p.sw_nb + BLOCK) / BLOCK, 1024);
    hipLaunchKernelGGL(k_sw_blocks, dim3(gb), dim3(BLOCK), 0, s, b.st, b.rp2, p.n, p.nnz, p.sw_nb, p.sw_items,
                       b.swob, b.swe, b.swq);
}

hipError_t launch_sweep_sort(const Plan& p, const Bufs& b, hipStream_t s) {
    if (!p.sweep) return hipSuccess;
    size_t need = 0;
    hipError_t err = sort_blocks(nullptr, need, nullptr, nullptr, nullptr, nullptr, p.nnz, p.sw_nb, nullptr,
                                 p.sw_bit0, p.sw_bit1, s);
    if (err != hipSuccess) return err;
    if (need > p.sw_sort_bytes) return hipErrorInvalidValue;
    size_t bytes = p.sw_sort_bytes;
    err = sort_blocks(b.swtmp, bytes, (const uint32_t*)b.col2, (uint32_t*)b.swcol, b.swvin, b.swsrc, p.nnz,
                      p.sw_nb, b.swe, p.sw_bit0, p.sw_bit1, s);
    if (err != hipSuccess) return err;
    switch (p.prec) {
        case 0:
            hipLaunchKernelGGL(k_sw_fill<double>, dim3(SWF_GRID), dim3(SWF_THREADS), 0, s, b.st,
                               (const double*)b.val2, p.sw_nb, b.swe, b.swsrc, b.swrl, (double*)b.swval, b.swq);
            break;
        case 1:
            hipLaunchKernelGGL(k_sw_fill<float>, dim3(SWF_GRID), dim3(SWF_THREADS), 0, s, b.st,
                               (const float*)b.val2, p.sw_nb, b.swe, b.swsrc, b.swrl, (float*)b.swval, b.swq);
            break;
        default:
            hipLaunchKernelGGL(k_sw_fill<uint16_t>, dim3(SWF_GRID), dim3(SWF_THREADS), 0, s, b.st,
                               (const uint16_t*)b.val2, p.sw_nb, b.swe, b.swsrc, b.swrl, (uint16_t*)b.swval,
                               b.swq);
            break;
    }
    if (p.sw_np > 0) {
        if (p.prec == 0)
            launch_sweep_tail_setup<double>(p, b, s);
        else if (p.prec == 1)
            launch_sweep_tail_setup<float>(p, b, s);
        else
            launch_sweep_tail_setup<uint16_t>(p, b, s);
    }
    return hipGetLastError();
}

}  // namespace lz
