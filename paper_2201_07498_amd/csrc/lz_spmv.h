// CSR SpMV core over merge-path tiles (Algorithm 1, the SpMV line), shared by
// the Lanczos step and the standalone SpMV.
//
// Walk the matrix as one sequence of items: the entries of row 0, an end
// marker for row 0, the entries of row 1, its end marker, and so on
// (nnz + n items; entry p of row r is item p + r, the end of row r is item
// rowptr[r+1] + r).  Tile t is items [t*TILE, (t+1)*TILE), one tile per
// wavefront at a time, so a tile holds at most TILE entries plus row ends
// whatever the row lengths (long rows, empty rows).  Row r is owned by the
// tile holding its end marker; tile t owns rows ob[t] .. ob[t+1]-1 and its
// entries are [t*TILE - ob[t], (t+1)*TILE - ob[t+1]).  A tile
//   * loads its col/val entries, gathers x and keeps the products in its
//     LDS slice;
//   * sums its owned rows: rows of up to LONGR entries by one lane each,
//     longer ones by the whole wavefront;
//   * may hold a head piece (its first owned row began in an earlier tile)
//     and a tail piece (row ob[t+1] continues into later tiles).
// A row whose first entry lies in tile t1 and whose end lies in tile t2 > t1
// has tail pieces in t1..t2-1 and the head piece in t2.  Every piece is
// published device-coherently and counted on the owner's ticket; the last
// piece to arrive adds all of them in tile order, so the row sum does not
// depend on which wavefront finishes last.
//
// The epilogue is four callbacks, all called by one lane:
//   pre(r)       a value the row epilogue needs (e.g. an entry of another
//                vector), loaded for the first 64 owned rows together with
//                the tile's entries;
//   row(r, s, p) owned row r with its whole sum s and p = pre(r);
//   piece(r, s)  one piece of a split row (for sums that are linear in the
//                row sum, such as alpha);
//   fin(r, s)    a split row's whole sum, from the finalising wavefront.
#pragma once

#include <type_traits>

#include "lz_device.h"

namespace lz {

constexpr int WAVES = BLOCK / 64;
constexpr int TP = TILE / 64;          // tile entries per lane
constexpr int LONGR = 64;              // rows longer than this are summed by the whole wavefront

// Orders this wavefront's LDS writes before its later LDS reads (LDS
// operations of one wavefront complete in order; this stops the compiler
// from moving them).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// True in exactly one wavefront: the last of `count` to arrive.  Lane 0
// publishes the wavefront's partial (st_dev) before calling.
__device__ __forceinline__ bool last_wave(uint32_t* ticket, uint32_t count) {
    uint32_t t = 0;
    if ((threadIdx.x & 63) == 0) {
        __builtin_amdgcn_s_waitcnt(0);
        t = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    t = (uint32_t)lane_value((int)t, 0);
    const bool last = t == count - 1u;
    if (last && (threadIdx.x & 63) == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return last;
}

// Tile of item i, clamped so that malformed input cannot index outside the
// tile tables.
__device__ __forceinline__ int64_t item_tile(int64_t i, int64_t n_tiles) {
    const int64_t t = i / TILE;
    return t < 0 ? 0 : (t >= n_tiles ? n_tiles - 1 : t);
}
// Owner tile of row r (the tile of its end marker).
__device__ __forceinline__ int64_t row_owner(const int64_t* rp, int64_t r, int64_t n_tiles) {
    return item_tile(rp[r + 1] + r, n_tiles);
}

// Sum of p[b..e) in four interleaved chains, combined in a fixed order.
template <class AT>
__device__ __forceinline__ AT lds_sum(const AT* p, int b, int e) {
    AT s0 = AT(0), s1 = AT(0), s2 = AT(0), s3 = AT(0);
    int k = b;
    for (; k + 4 <= e; k += 4) {
        s0 += p[k];
        s1 += p[k + 1];
        s2 += p[k + 2];
        s3 += p[k + 3];
    }
    for (; k < e; ++k) s0 += p[k];
    return (s0 + s1) + (s2 + s3);
}

// Whole-wavefront sum of p[b..e): lane-strided partials, then the butterfly.
template <class AT>
__device__ __forceinline__ AT lds_wave_sum(const AT* p, int b, int e, int lane) {
    AT s = AT(0);
    for (int k = b + lane; k < e; k += 64) s += p[k];
    return wave_sum(s);
}

// Tiles handled by this wavefront out of tiles [tb, te) (all tiles, or one
// slab of a host-resident matrix): the range is split evenly over the eight
// XCDs (workgroup i runs on XCD i mod 8), so neighbouring tiles, which gather
// neighbouring parts of x in a banded matrix, share one L2.
struct TileRange {
    int64_t first, end, stride;
};
template <int NW = WAVES>
__device__ __forceinline__ TileRange wave_tiles(int64_t tb, int64_t te) {
    const int64_t xcd = blockIdx.x & 7, nb8 = gridDim.x >> 3;
    const int64_t nt = te - tb;
    const int64_t lo = tb + nt * xcd / 8, hi = tb + nt * (xcd + 1) / 8;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t w = (int64_t)(blockIdx.x >> 3) * NW + wave;
    return {lo + w, hi, nb8 * NW};
}


// Adds the pieces of the split row r (tail pieces in tiles t1..t2-1, head
// piece in t2) in tile order; called by every lane of the finalising
// wavefront, returns the sum in all lanes.
__device__ __forceinline__ double split_total(const double* head, const double* tail, int64_t t1, int64_t t2,
                                              int lane) {
    double s = 0.0;
    for (int64_t i = t1 + lane; i < t2; i += 64) s += ld_dev(&tail[i]);
    s = wave_sum(s);
    return s + ld_dev(&head[t2]);
}

// Loads of the matrix streams (column indices and values), which every SpMV
// reads exactly once.  With NT they are non-temporal (the L2 does not keep
// them).  Measured on MI355X (SpMV per step, plain / non-temporal): FP64
// R-MAT 20 102.0 / 100.9 us, R-MAT 23 2.037 / 2.016 ms, R-MAT 26 24.4 /
// 23.7 ms; FP32 77.6 / 82.8 us, 1.552 / 1.577 ms, 18.8 / 19.0 ms.  So only
// the FP64 storage streams them non-temporally.
template <bool NT, class T> __device__ __forceinline__ T stream_load(const T* p) {
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

// Bytes at the head of x gathered with ordinary loads (the L2 of one XCD);
// the rest non-temporally.  Measured on MI355X, step SpMV with and without:
// R-MAT scale 23 FP32 1542 -> 1375 us, scale 26 FP32 18.67 -> 18.37 ms and
// BF16 13.92 -> 13.63 ms; FP64 and R-MAT scale 20 unchanged.  A boundary at
// 1, 4 or 16 MB measured the same.
constexpr uint32_t GATHER_WARM_BYTES = 4u << 20;

// Stored entries a lane loads side by side: E words of 4 bytes and E values
// with one load each of at most 16 bytes.  A load then covers 64 E consecutive
// entries, so that fewer loads share a line with the next: the L1 returns in
// order and waits for lines in flight half of this kernel's time.  Measured,
// one entry per lane and load -> E, step SpMV: R-MAT 20 FP64 101 -> 93 us, R-MAT
// 23 BF16 1.203 -> 1.159 ms, ER 500k FP32 60.4 -> 59.2 us, R-MAT 20 FP32 75.5 ->
// 75.2 us.
template <class VT> struct TileVec {
    static constexpr int E = sizeof(VT) == 8 ? 2 : 4;
    typedef int32_t C __attribute__((ext_vector_type(E), aligned(4)));
    typedef VT V __attribute__((ext_vector_type(E), aligned(sizeof(VT))));
};
// Place of the k-th stored entry (of cnt) of a column-sorted tile or group: in
// a whole run of 64 E entries, entries k, k + 64, ... that one gather
// instruction should take from neighbouring columns sit E apart, so that lane
// l's i-th loaded entry is the run's (64 i + l)-th; a last, partial run is
// stored in order.
template <class VT> __device__ __forceinline__ int sorted_place(int k, int cnt) {
    constexpr int E = TileVec<VT>::E;
    const int g = k & ~(64 * E - 1), o = k & (64 * E - 1);
    return g + 64 * E <= cnt ? g + (o & 63) * E + (o >> 6) : k;
}

// The products of one wavefront's share of stored entries [base, base+cnt)
// in LDS, in two halves: tile_load issues the col/val loads of a lane together;
// tile_gather issues the 16 gathers of x, runs `between` (loads of later work)
// and writes the products.  Lanes past the end re-read the last entries (same
// cache lines), so every load is unconditional; with fewer entries than a lane
// takes (cnt < E) the load is by element.  Row-ordered storage (slotbits = 0):
// entry base+k lands in pw[k].  Column-sorted storage: each column word is (col
// << slotbits) | slot and the product lands in pw[slot], the entry's position
// in row order, so the row sums add the same values in the same order as for
// row-ordered storage (lanes past the end rewrite the last entries' products).
// With CACHED, xs holds x[0..hn) in LDS and gathers of those entries read it.
// With OFF32 (every byte offset into x below 2^32), each load is a
// wave-uniform base in scalar registers plus a 32-bit per-lane offset; 64-bit
// per-lane addresses would otherwise take about half of the kernel's vector
// registers and limit its occupancy.
template <class VT> struct TileEntries {
    static constexpr int NV = TP / TileVec<VT>::E;
    typename TileVec<VT>::C ci[NV];
    typename TileVec<VT>::V vv[NV];
};
template <class VT>
__device__ __forceinline__ void tile_load(TileEntries<VT>& t, const int32_t* __restrict__ col,
                                          const VT* __restrict__ val, int64_t base, int cnt, int lane) {
    constexpr int E = TileVec<VT>::E, NV = TileEntries<VT>::NV;
    using C = typename TileVec<VT>::C;
    using V = typename TileVec<VT>::V;
    if (cnt <= 0) return;
    if (cnt < E) {
#pragma unroll
        for (int q = 0; q < NV; ++q)
#pragma unroll
            for (int i = 0; i < E; ++i) {
                t.ci[q][i] = col[base + min(i, cnt - 1)];
                t.vv[q][i] = val[base + min(i, cnt - 1)];
            }
        return;
    }
    constexpr bool NT = sizeof(VT) == 8;
    const char* cb = (const char*)(col + base);
    const char* vb = (const char*)(val + base);
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const uint32_t o = (uint32_t)min(q * 64 * E + lane * E, cnt - E);
        t.ci[q] = stream_load<NT>((const C*)(cb + o * 4u));
        t.vv[q] = stream_load<NT>((const V*)(vb + o * (uint32_t)sizeof(VT)));
    }
}
template <class VT, class AT, bool CACHED, bool OFF32, class Between>
__device__ __forceinline__ void tile_gather(const TileEntries<VT>& t, const VT* __restrict__ x, const VT* xs, int hn,
                                            int cnt, int slotbits, AT* pw, int lane, Between&& between) {
    constexpr int E = TileVec<VT>::E, NV = TileEntries<VT>::NV;
    if (cnt <= 0) {
        between();
        return;
    }
    // Entries of x past the first GATHER_WARM_BYTES are gathered
    // non-temporally: after the hub-first relabelling they are the rarely
    // used columns, and keeping their lines out of L2 leaves it to the warm
    // head of x.
    auto gather = [&](uint32_t c) -> VT {
        const bool warm = c < GATHER_WARM_BYTES / (uint32_t)sizeof(VT);
        if (CACHED && (int)c < hn) return xs[c];
        const VT* px = OFF32 ? (const VT*)((const char*)x + c * (uint32_t)sizeof(VT)) : x + c;
        return warm ? *px : __builtin_nontemporal_load(px);
    };
    const uint32_t smask = (1u << slotbits) - 1u;
    VT xv[TP];
#pragma unroll
    for (int q = 0; q < NV; ++q)
#pragma unroll
        for (int i = 0; i < E; ++i) xv[q * E + i] = gather((uint32_t)t.ci[q][i] >> slotbits);
    between();
    if (slotbits) {
#pragma unroll
        for (int q = 0; q < NV; ++q)
#pragma unroll
            for (int i = 0; i < E; ++i)
                pw[(uint32_t)t.ci[q][i] & smask] = to_a(VT(t.vv[q][i]), AT(0)) * to_a(xv[q * E + i], AT(0));
    } else {
        typedef AT P __attribute__((ext_vector_type(E)));
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            P pr;
#pragma unroll
            for (int i = 0; i < E; ++i) pr[i] = to_a(VT(t.vv[q][i]), AT(0)) * to_a(xv[q * E + i], AT(0));
            if ((q + 1) * 64 * E <= cnt) {               // the whole run is live: one aligned store
                *(P*)(pw + q * 64 * E + lane * E) = pr;
            } else {
                const int k = max(min(q * 64 * E + lane * E, cnt - E), 0);
#pragma unroll
                for (int i = 0; i < E; ++i) pw[min(k + i, cnt - 1)] = pr[i];
            }
        }
    }
}

// Row bounds and pre() of a tile's first 128 owned rows (as offsets of the
// tile's entries; -1 for a first row that began in an earlier tile), and the
// bounds of the rows a split concerns: the start of the first owned row and the
// row continuing past the tile.  All loaded with the tile's entries, so a tile
// waits for two rounds of requests (entries, then gathers) before its sums are
// written.
constexpr int TROWS = 2;
struct TileRows {
    int64_t t, t0, r_lo, r_hi, rb_lo, rb_hi, re_hi;
    int b[TROWS], e[TROWS];
    double pv[TROWS];
    int cnt;
};
template <class Pre>
__device__ __forceinline__ TileRows tile_rows(const int64_t* __restrict__ rp, int64_t t, int64_t r_lo, int64_t r_hi,
                                              int64_t n, int64_t items, int lane, Pre&& pre) {
    TileRows q;
    q.t = t;
    q.r_lo = r_lo;
    q.r_hi = r_hi;
    q.t0 = t * TILE - r_lo;
    q.cnt = (int)(min<int64_t>((t + 1) * TILE, items) - r_hi - q.t0);
#pragma unroll
    for (int i = 0; i < TROWS; ++i) {
        const int64_t r = r_lo + i * 64 + lane;
        q.b[i] = 0;
        q.e[i] = 0;
        q.pv[i] = 0.0;
        if (r < r_hi) {
            q.b[i] = (int)max<int64_t>(rp[r] - q.t0, -1);
            q.e[i] = (int)(rp[r + 1] - q.t0);
            q.pv[i] = pre(r);
        }
    }
    q.rb_lo = r_lo < n ? rp[r_lo] : 0;
    q.rb_hi = r_hi < n ? rp[r_hi] : 0;
    q.re_hi = r_hi < n ? rp[r_hi + 1] : 0;
    return q;
}

// Sums of one tile from its products pw[0..cnt) in row order: owned rows
// (one lane each up to LONGR entries, else the whole wavefront), then the
// head and tail pieces of split rows.  The two pieces are published together
// and take their tickets in one round trip (lane 0 the head's, lane 1 the
// tail's).  With that, the row bounds loaded for 128 rows ahead of the gathers
// and the kernel's state in one round of loads, step SpMV measured (whole solve,
// before -> after): R-MAT 150k FP64 2.97 -> 2.76 ms, R-MAT 20 FP32 7.75 -> 7.20
// ms, FP64 10.7 -> 10.3 ms, ER 500k FP32 2.56 -> 2.46 ms.
template <class AT, class Pre, class Row, class Piece, class Fin>
__device__ __forceinline__ void tile_sums(const TileRows& q, const AT* pw, const int64_t* __restrict__ rp, int64_t n,
                                          int64_t n_tiles, uint32_t* tk, double* head, double* tail, int lane,
                                          Pre&& pre, Row&& row, Piece&& piece, Fin&& fin) {
    const int64_t t = q.t, t0 = q.t0, r_lo = q.r_lo, r_hi = q.r_hi;
    const int cnt = q.cnt;
    const bool split_head = r_lo < r_hi && q.rb_lo < t0;
    const bool split_tail = r_hi < n && q.rb_hi < t0 + cnt;
    double head_s = 0.0;
    // 64 owned rows from `base` on.
    auto rows = [&](int64_t base, int b, int e, double pv) {
        const int64_t r = base + lane;
        const bool valid = r < r_hi;
        b = max(b, 0);
        const bool islong = valid && e - b > LONGR;
        AT s = (valid && !islong) ? lds_sum(pw, b, e) : AT(0);
        uint64_t mask = __ballot(islong);
        while (mask) {
            const int L = __builtin_ctzll(mask);
            mask &= mask - 1;
            const AT ss = lds_wave_sum(pw, lane_value(b, L), lane_value(e, L), lane);
            if (lane == L) s = ss;
        }
        if (valid) {
            if (split_head && r == r_lo) {
                head_s = (double)s;
                piece(r, head_s);
            } else {
                row(r, (double)s, pv);
            }
        }
    };
#pragma unroll
    for (int i = 0; i < TROWS; ++i)
        if (r_lo + i * 64 < r_hi) rows(r_lo + i * 64, q.b[i], q.e[i], q.pv[i]);
    for (int64_t base = r_lo + TROWS * 64; base < r_hi; base += 64) {
        const int64_t r = base + lane;
        int b = 0, e = 0;
        double pv = 0.0;
        if (r < r_hi) {
            b = (int)(rp[r] - t0);
            e = (int)(rp[r + 1] - t0);
            pv = pre(r);
        }
        rows(base, b, e, pv);
    }
    if (!split_head && !split_tail) return;
    // Publish the pieces, count them, finish a row whose last piece this was.
    const int64_t h1 = split_head ? item_tile(q.rb_lo + r_lo, n_tiles) : 0;
    const int64_t t1 = split_tail ? item_tile(q.rb_hi + r_hi, n_tiles) : 0;
    const int64_t t2 = split_tail ? item_tile(q.re_hi + r_hi, n_tiles) : 0;
    if (split_head && lane == 0) st_dev(&head[t], head_s);
    if (split_tail) {
        const AT ss = lds_wave_sum(pw, (int)(max(q.rb_hi, t0) - t0), cnt, lane);
        if (lane == 0) {
            piece(r_hi, (double)ss);
            st_dev(&tail[t], (double)ss);
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    uint32_t got = 0;
    if ((lane == 0 && split_head) || (lane == 1 && split_tail))
        got = __hip_atomic_fetch_add(lane == 0 ? &tk[t] : &tk[t2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool head_last = split_head && (uint32_t)lane_value((int)got, 0) == (uint32_t)(t - h1);
    const bool tail_last = split_tail && (uint32_t)lane_value((int)got, 1) == (uint32_t)(t2 - t1);
    if (head_last) {
        if (lane == 0) __hip_atomic_store(&tk[t], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const double tot = split_total(head, tail, h1, t, lane);
        if (lane == 0) fin(r_lo, tot);
    }
    if (tail_last) {
        if (lane == 0) __hip_atomic_store(&tk[t2], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const double tot = split_total(head, tail, t1, t2, lane);
        if (lane == 0) fin(r_hi, tot);
    }
}

// The workgroup's product buffer: one TILE slice per wavefront, contiguous,
// so a group of NW tiles has one row-ordered array of NW * TILE slots.
template <class AT, int NW>
__device__ __forceinline__ AT* prod_lds() {
    __shared__ __align__(16) AT prod[NW * TILE];
    return prod;
}

// Wavefront per tile over tiles [tb, te) (tile indices and the tables stay
// those of the whole matrix); each wavefront walks its own tiles.
// slotbits = PACK_SLOTBITS for tile-sorted storage, 0 for row order.
template <class VT, class AT, int NW, bool CACHED, bool OFF32, class Pre, class Row, class Piece, class Fin>
__device__ __forceinline__ void spmv_tiles(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                           const VT* __restrict__ val, const VT* __restrict__ x, const VT* xs,
                                           int hn, int64_t n, int64_t nnz, int64_t n_tiles, int64_t tb,
                                           int64_t te, int slotbits, const int32_t* __restrict__ ob, uint32_t* tk,
                                           double* head, double* tail, Pre&& pre, Row&& row, Piece&& piece,
                                           Fin&& fin) {
    const int lane = threadIdx.x & 63;
    AT* pw = prod_lds<AT, NW>() + (threadIdx.x >> 6) * TILE;
    const TileRange tr = wave_tiles<NW>(tb, te);
    const int64_t items = nnz + n;
    if constexpr (CACHED && sizeof(VT) == 2) {
        // One workgroup per CU, so 16 wavefronts and, in BF16, registers to
        // spare (FP32 would spill): the entries and row bounds of the next tile
        // are loaded while the gathers of this one are in flight and its rows
        // are summed.  R-MAT 23 step SpMV 1.146 -> 1.129 ms.
        auto owned = [&](int64_t t, int64_t& lo, int64_t& hi) {
            lo = hi = 0;
            if (t < tr.end) {
                lo = ob[t];
                hi = ob[t + 1];
            }
        };
        if (tr.first >= tr.end) return;
        int64_t r_lo, r_hi, n_lo, n_hi;
        owned(tr.first, r_lo, r_hi);
        owned(tr.first + tr.stride, n_lo, n_hi);
        TileRows q = tile_rows(rp, tr.first, r_lo, r_hi, n, items, lane, pre);
        TileEntries<VT> en;
        tile_load(en, col, val, q.t0, q.cnt, lane);
        for (int64_t t = tr.first; t < tr.end; t += tr.stride) {
            const int64_t tn = t + tr.stride;
            TileRows qn{};
            TileEntries<VT> nx;
            const TileRows cur = q;
            tile_gather<VT, AT, CACHED, OFF32>(en, x, xs, hn, cur.cnt, slotbits, pw, lane, [&] {
                if (tn < tr.end) {
                    qn = tile_rows(rp, tn, n_lo, n_hi, n, items, lane, pre);
                    tile_load(nx, col, val, qn.t0, qn.cnt, lane);
                    owned(tn + tr.stride, n_lo, n_hi);
                }
            });
            wave_sync();
            tile_sums(cur, pw, rp, n, n_tiles, tk, head, tail, lane, pre, row, piece, fin);
            wave_sync();
            q = qn;
            en = nx;
        }
        return;
    }
    int64_t r_lo = 0, r_hi = 0;
    if (tr.first < tr.end) {
        r_lo = ob[tr.first];
        r_hi = ob[tr.first + 1];
    }
    for (int64_t t = tr.first; t < tr.end; t += tr.stride) {
        // Row bounds of the next tile, loaded while this one works.
        const int64_t tn = t + tr.stride;
        int64_t n_lo = 0, n_hi = 0;
        if (tn < tr.end) {
            n_lo = ob[tn];
            n_hi = ob[tn + 1];
        }
        const TileRows q = tile_rows(rp, t, r_lo, r_hi, n, items, lane, pre);
        TileEntries<VT> en;
        tile_load(en, col, val, q.t0, q.cnt, lane);
        tile_gather<VT, AT, CACHED, OFF32>(en, x, xs, hn, q.cnt, slotbits, pw, lane, [] {});
        wave_sync();
        tile_sums(q, pw, rp, n, n_tiles, tk, head, tail, lane, pre, row, piece, fin);
        wave_sync();
        r_lo = n_lo;
        r_hi = n_hi;
    }
}

// Group-sorted storage: the entries of each group of GROUP_TILES consecutive
// tiles are stored in column order with GROUP_SLOTBITS-bit slots (positions
// in the group's row order).  A workgroup takes NW / GROUP_TILES groups at a
// time; wavefront w loads the (w % GROUP_TILES)-th TILE of its group's stored
// entries, so one wavefront instruction gathers from a narrow column range.
// The products land in the group's row-ordered slice of the workgroup buffer,
// and after a barrier each wavefront sums its own tile.  Group sets are split
// contiguously over the eight XCDs.  Every wavefront runs the same number of
// iterations (the barriers need it).
template <class VT, class AT, int NW, bool CACHED, bool OFF32, class Pre, class Row, class Piece, class Fin>
__device__ __forceinline__ void spmv_groups(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                            const VT* __restrict__ val, const VT* __restrict__ x, const VT* xs,
                                            int hn, int64_t n, int64_t nnz, int64_t n_tiles,
                                            const int32_t* __restrict__ ob, uint32_t* tk, double* head,
                                            double* tail, Pre&& pre, Row&& row, Piece&& piece, Fin&& fin) {
    static_assert(NW % GROUP_TILES == 0, "whole groups per workgroup");
    constexpr int GPW = NW / GROUP_TILES;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wi = w % GROUP_TILES;
    AT* pg = prod_lds<AT, NW>() + (w / GROUP_TILES) * (GROUP_TILES * TILE);
    const int64_t items = nnz + n;
    const int64_t n_groups = (n_tiles + GROUP_TILES - 1) / GROUP_TILES;
    const int64_t n_sets = (n_groups + GPW - 1) / GPW;
    const int64_t xcd = blockIdx.x & 7, nb8 = gridDim.x >> 3;
    const int64_t lo = n_sets * xcd / 8, hi = n_sets * (xcd + 1) / 8;
    for (int64_t gs = lo + (blockIdx.x >> 3); gs < hi; gs += nb8) {
        const int64_t tg = (gs * GPW + w / GROUP_TILES) * GROUP_TILES;
        const bool live = tg < n_tiles;
        const int64_t te = min<int64_t>(tg + GROUP_TILES, n_tiles);
        const int64_t g0 = live ? tg * TILE - ob[tg] : nnz;
        const int64_t gend = !live || te >= n_tiles ? nnz : te * TILE - ob[te];
        const int64_t t = tg + wi;
        const bool has = t < n_tiles;
        TileRows q{};
        if (has) q = tile_rows(rp, t, ob[t], ob[t + 1], n, items, lane, pre);
        const int cw = (int)max<int64_t>(0, min<int64_t>(TILE, gend - g0 - (int64_t)wi * TILE));
        TileEntries<VT> en;
        tile_load(en, col, val, g0 + (int64_t)wi * TILE, cw, lane);
        tile_gather<VT, AT, CACHED, OFF32>(en, x, xs, hn, cw, GROUP_SLOTBITS, pg, lane, [] {});
        __syncthreads();
        if (has) tile_sums(q, pg + (q.t0 - g0), rp, n, n_tiles, tk, head, tail, lane, pre, row, piece, fin);
        __syncthreads();
    }
}

// ------------------------------------------------------------ sweep blocks
// The sweep-block copy of the relabelled matrix (layout in lz_internal.h).
struct SweepArgs {
    const int32_t* ob;    // first owned row of every block (nb + 1)
    const int64_t* e;     // first entry of every block (nb + 1)
    const int32_t* col;   // columns, column order within each block
    const uint16_t* rl;   // row of each entry relative to ob[b] (at sweep_place)
    const void* val;      // values (at sweep_place)
    int64_t nb;
    // Tail columns (np > 0): entries seg[b] .. seg[np * nb + b] - 1 of block b
    // gather from xg, the tail entries' values of x in the order k_sweep_tail
    // leaves them, and their column words are positions in xg.
    const uint32_t* seg;
    const void* xg;
    int np;
};
// The tail entries panel by panel, block by block: columns within the panel,
// and the start of panel p at pre[p * nb] (the total at pre[np * nb]).
struct TailArgs {
    const uint16_t* col;
    const uint64_t* pre;
    int64_t nb;
    int np;
};
// Entries per lane and round.  Measured with 8 / 12 / 16, step SpMV of R-MAT 25
// FP32: 3.63 / 3.56 / 3.57 ms (the LDS of the row sums limits occupancy to two
// wavefronts per SIMD, so registers cost nothing).
constexpr int SW_U = 12;
// Rows per block and wavefronts per workgroup (their row sums fill the LDS, so
// one workgroup per CU), per storage precision.  Measured on MI355X, step SpMV
// (rows/wavefronts): R-MAT 25 with the tail pass FP64 4096/4 4.46 ms, 2048/8
// 4.75; FP32 2048/8 3.28-3.36 ms, 2048/4 3.34, 4096/4 3.16; BF16 2048/8 2.93 ms,
// 2048/4 2.90, 4096/4 3.08.  R-MAT 26 without it, where the shapes were chosen:
// FP64 14.3 and 16.5 ms; FP32 12.4, 13.2, 12.6; BF16 9.7, 10.3, 11.7.
template <int P> struct SweepShape { static constexpr int ROWS = 2048, WAVES = 8; };
template <> struct SweepShape<0> { static constexpr int ROWS = 4096, WAVES = 4; };
constexpr int SWEEP_GRID_MAX = 16384;
static_assert(SweepShape<0>::ROWS == sweep_rows(0) && SweepShape<1>::ROWS == sweep_rows(1) &&
                  SweepShape<2>::ROWS == sweep_rows(2) && SweepShape<0>::ROWS <= SW_ROWS_MAX,
              "sweep block rows");

// Where rows and values of entry k of the block with entries [e0, e1) are
// stored: a group of 256 entries (k / 256) wholly inside the block holds the
// four entries i, i + 64, i + 128, i + 192 of a lane side by side, so that a
// lane reads them with one load; the block's first and last, partial groups
// are stored in order.
__device__ __forceinline__ int64_t sweep_place(int64_t k, int64_t e0, int64_t e1) {
    const int64_t g = k & ~int64_t(255);
    const int o = (int)(k & 255);
    return g >= e0 && g + 256 <= e1 ? g + (o & 63) * 4 + (o >> 6) : k;
}

// What bounds it: beside the streams (10 bytes an entry in FP32), the L1.  In
// row order every gather of a rarely used column fetched a line of its own
// from beyond L2; with those columns fetched ahead (k_sweep_tail) the rest of
// x fits L2, and the L1 is busy or held up by lines in flight for 70 % of the
// time.  Step SpMV of R-MAT 25 FP32, all gathers in the sweep -> tail columns
// ahead, rounds pipelined and one block per wavefront: 5.07 -> 3.28 ms (0.39
// of it k_sweep_tail); a head of 1, 2, 4, 8 MiB gave 3.63, 3.57, 3.60, 3.90 ms
// on the same grid, a grid of 512, 1024, 2048 workgroups and one per eight
// blocks 3.56, 3.56, 3.34, 3.28 ms.
// Wavefront per sweep block, blocks dealt round-robin over all wavefronts
// of the grid.  A block zeroes its row sums in LDS (owned rows, then the row
// continuing past it), walks its entries in stored (column) order, 64 * SW_U
// at a time, adding each product into its row's sum with an LDS atomic, and
// then hands every owned row to the epilogue, one lane per row.  The sums
// are binary64 in every storage mode: a hub row can put all of a block's
// 2^18 products into one sum, and a binary32 chain that long loses about
// sqrt(2^18) units of its last place (on a matrix with such rows, binary32
// sums put the FP32-storage Ritz values 1.6e-6 from the FP64 ones); the
// products of FP32 and BF16 values are exact in binary64.  Split rows
// work as for tiles: the block that owns a row whose entries began in
// earlier blocks publishes a head piece, every block a row continues past
// publishes a tail piece, and the last piece to arrive on the owner's ticket
// adds them in block order.  Each wavefront has its own sums and adds into
// them in a fixed instruction order, so the result does not depend on timing.
template <class VT, int NW, int ROWS, bool TAIL, bool OFF32, class Pre, class Row, class Piece, class Fin>
__device__ __forceinline__ void spmv_sweep(const SweepArgs& sw, const int64_t* __restrict__ rp,
                                           const VT* __restrict__ x, int64_t n, uint32_t* tk, double* head,
                                           double* tail, Pre&& pre, Row&& row, Piece&& piece, Fin&& fin) {
    constexpr int64_t ITEMS = (int64_t)SW_W * ROWS;
    constexpr int STEP = 64 * SW_U;
    static_assert(SW_U % 4 == 0, "whole groups of 256 entries per round");
    typedef uint16_t us4 __attribute__((ext_vector_type(4)));      // four entries of a lane
    typedef VT V4 __attribute__((ext_vector_type(4)));
    __shared__ double ys_all[NW][ROWS + 1];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double* ys = ys_all[w];
    const int32_t* __restrict__ col = sw.col;
    const uint16_t* __restrict__ rlv = sw.rl;
    const VT* __restrict__ val = (const VT*)sw.val;
    const VT* __restrict__ xg = (const VT*)sw.xg;
    const int64_t nw = (int64_t)gridDim.x * NW;
    for (int64_t b = (int64_t)blockIdx.x * NW + w; b < sw.nb; b += nw) {
        const int64_t r0 = sw.ob[b], r1 = sw.ob[b + 1];
        const int64_t e0 = sw.e[b], e1 = sw.e[b + 1];
        const int nown = (int)(r1 - r0);
        // Entries [et, ft) are tail entries.
        const int64_t et = TAIL ? e0 + sw.seg[b] : e1, ft = TAIL ? e0 + sw.seg[sw.np * sw.nb + b] : e1;
        for (int i = lane; i <= nown; i += 64) ys[i] = 0.0;
        wave_sync();
        // Whole rounds of 64 * SW_U entries, pipelined over three of them:
        // while the products of one are added, the gathers of the next and the
        // streams of the one after that are in flight.  The steady loop has no
        // branch but its exits, and a round takes 18 (FP64 21) stream loads, so
        // that all of it fits the 63 loads a wavefront can wait on by count.
        struct Round {
            int c[SW_U];
            us4 r[SW_U / 4];
            V4 v[SW_U / 4];
            VT g[SW_U];
        };
        auto load = [&](Round& t, int64_t at) {
            const int32_t* cb = col + at;
            const uint16_t* rb = rlv + at;
            const VT* vb = val + at;
#pragma unroll
            for (int q = 0; q < SW_U; ++q) t.c[q] = __builtin_nontemporal_load(cb + (uint32_t)(q * 64 + lane));
#pragma unroll
            for (int q = 0; q < SW_U / 4; ++q) {
                t.r[q] = __builtin_nontemporal_load((const us4*)(rb + (uint32_t)(q * 256 + lane * 4)));
                t.v[q] = __builtin_nontemporal_load((const V4*)(vb + (uint32_t)(q * 256 + lane * 4)));
            }
        };
        auto from = [](const VT* base, int c) {
            return OFF32 ? *(const VT*)((const char*)base + (uint32_t)c * (uint32_t)sizeof(VT)) : base[(uint32_t)c];
        };
        auto gather = [&](Round& t, int64_t at) {
            const int lo = TAIL ? (int)min<int64_t>(et - at, STEP) : 0, hi = TAIL ? (int)min<int64_t>(ft - at, STEP) : 0;
#pragma unroll
            for (int q = 0; q < SW_U; ++q) {
                const int i = q * 64 + lane;
                t.g[q] = from(TAIL && i >= lo && i < hi ? xg : x, t.c[q]);
            }
        };
        auto add = [&](const Round& t) {
#pragma unroll
            for (int q = 0; q < SW_U; ++q)
                __hip_atomic_fetch_add(ys + min((int)t.r[q / 4][q % 4], nown),
                                       to_a(VT(t.v[q / 4][q % 4]), 0.0) * to_a(t.g[q], 0.0), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WAVEFRONT);
        };
        // Entries [k0, k1) outside whole rounds.
        auto sweep_part = [&](int64_t k0, int64_t k1) {
            for (int64_t at = k0; at < k1; at += STEP) {
                const int left = (int)min<int64_t>(k1 - at, STEP);
                int c[SW_U], r[SW_U];
                VT v[SW_U], g[SW_U];
#pragma unroll
                for (int q = 0; q < SW_U; ++q) {
                    const int64_t k = at + min(q * 64 + lane, left - 1), kp = sweep_place(k, e0, e1);
                    c[q] = __builtin_nontemporal_load(col + k);
                    r[q] = (int)__builtin_nontemporal_load(rlv + kp);
                    v[q] = __builtin_nontemporal_load(val + kp);
                }
#pragma unroll
                for (int q = 0; q < SW_U; ++q) {
                    const int64_t k = at + min(q * 64 + lane, left - 1);
                    g[q] = from(TAIL && k >= et && k < ft ? xg : x, c[q]);
                }
#pragma unroll
                for (int q = 0; q < SW_U; ++q)
                    if (q * 64 + lane < left)
                        __hip_atomic_fetch_add(ys + min(r[q], nown), to_a(v[q], 0.0) * to_a(g[q], 0.0),
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
        };
        // Rounds start at multiples of 256 entries, so that no load shares a
        // cache line with the next: a load that hits a line still in flight
        // holds up the L1 until the line has come.
        const int64_t a0 = min((e0 + 255) & ~int64_t(255), e1);
        const int rounds = (int)((e1 - a0) / STEP);
        sweep_part(e0, a0);
        if (rounds > 0) {
            auto at = [&](int i) { return a0 + (int64_t)min(i, rounds - 1) * STEP; };
            Round ra, rb, rc;
            load(ra, at(0));
            gather(ra, at(0));
            load(rb, at(1));
            for (int i = 0;;) {
                gather(rb, at(i + 1));
                load(rc, at(i + 2));
                add(ra);
                if (++i == rounds) break;
                gather(rc, at(i + 1));
                load(ra, at(i + 2));
                add(rb);
                if (++i == rounds) break;
                gather(ra, at(i + 1));
                load(rb, at(i + 2));
                add(rc);
                if (++i == rounds) break;
            }
        }
        sweep_part(a0 + (int64_t)rounds * STEP, e1);
        wave_sync();
        const bool split_head = nown > 0 && rp[r0] < e0;
        double head_s = 0.0;
        for (int i = lane; i < nown; i += 64) {
            const int64_t rr = r0 + i;
            const double s = ys[i];
            if (i == 0 && split_head) {
                head_s = s;
                piece(rr, s);
            } else {
                row(rr, s, pre(rr));
            }
        }
        if (split_head) {
            if (lane == 0) st_dev(&head[b], head_s);
            const int64_t t1 = (rp[r0] + SW_W * r0) / ITEMS;
            if (last_wave(&tk[b], (uint32_t)(b - t1 + 1))) {
                const double tot = split_total(head, tail, t1, b, lane);
                if (lane == 0) fin(r0, tot);
            }
        }
        if (r1 < n) {
            const int64_t rb = rp[r1];
            if (rb < e1) {
                const double s = ys[nown];
                if (lane == 0) {
                    piece(r1, s);
                    st_dev(&tail[b], s);
                }
                const int64_t t1 = (rb + SW_W * r1) / ITEMS, t2 = (rp[r1 + 1] + SW_W * r1) / ITEMS;
                if (last_wave(&tk[t2], (uint32_t)(t2 - t1 + 1))) {
                    const double tot = split_total(head, tail, t1, t2, lane);
                    if (lane == 0) fin(r1, tot);
                }
            }
        }
        wave_sync();
    }
}

}  // namespace lz
