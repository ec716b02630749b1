// Host-resident matrices: slab planning, device buffers and the copy stream
// (the passes themselves are ooc_pass in lz_ooc.h).
#include <algorithm>
#include <vector>

#include "lz_ooc.h"
#include "lz_spmv.h"

namespace lz {

// A slab's column indices and values from pinned host memory to a staging buffer.
// The host link bounds it (57.5 GB/s for one large copy): 16 workgroups keep
// 512 KiB in flight, several times what the link's latency asks for.  The kernels
// beside it run slower while it does, since they share 16 CUs with loads of host
// latency and their grids wait for the last workgroup: R-MAT 20 FP32 in one slab,
// step SpMV 138 -> 232 us, orthogonalisation kernels of 48 columns 41 -> 105 and
// 124 us against copies by the runtime, out of 2.3 ms of copy a step.  Whole solves
// took 0.64 to 0.94 of the time with those copies in every mix measured (1.4M to
// 16M entries, slabs of 2^18 to 2^24, none to 95 % resident).  Loads are aligned to 16 bytes of the source, which
// starts anywhere; the stores take what alignment that leaves.  Copies by the
// runtime cost the host thread 70 to 450 us inside a call about once per slab,
// while the copy stream idled.  16.1M FP32 entries, 16 steps, slabs of 2^18 / 2^20 /
// 2^22 / 2^24 entries: 76.7 / 62.7 / 48.3 / 51.8 -> 62.6 / 47.0 / 43.4 / 42.2 ms a
// solve.  256 / 128 / 64 / 32 workgroups with 4 loads a thread took 25.2 / 23.8 /
// 23.1 / 21.9 ms where 16 with 8 took 21.7, 8 with 4 27.9 (8.4M entries, half
// resident, slabs of 2^20).
constexpr int PULL_GRID = 16, PULL_U = 8;
__global__ __launch_bounds__(BLOCK) void k_pull(const char* __restrict__ src0, char* __restrict__ dst0, int64_t bytes0,
                                                const char* __restrict__ src1, char* __restrict__ dst1,
                                                int64_t bytes1) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u4any __attribute__((ext_vector_type(4), aligned(1)));
    const int64_t T = (int64_t)gridDim.x * BLOCK, first = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const char* src = a == 0 ? src0 : src1;
        char* dst = a == 0 ? dst0 : dst1;
        const int64_t bytes = a == 0 ? bytes0 : bytes1;
        const int64_t head = min<int64_t>(bytes, (int64_t)(-(uintptr_t)src & 15u)), words = (bytes - head) >> 4;
        const u4* s = (const u4*)(src + head);
        char* d = dst + head;
        for (int64_t i = first; i < words; i += PULL_U * T) {
            u4 v[PULL_U];
#pragma unroll
            for (int q = 0; q < PULL_U; ++q) v[q] = __builtin_nontemporal_load(s + min(i + q * T, words - 1));
#pragma unroll
            for (int q = 0; q < PULL_U; ++q)
                if (i + q * T < words) *(u4any*)(d + (i + q * T) * 16) = v[q];
        }
        if (first < head) dst[first] = src[first];
        const int64_t done = head + words * 16;
        if (first < bytes - done) dst[done + first] = src[done + first];
    }
}

hipError_t ooc_pull(const Ooc& o, int i, int64_t e0, int64_t e1) {
    const int64_t cb = (e1 - e0) * 4, vb = (e1 - e0) * (int64_t)o.vb;
    if (o.dcol) {
        const int g = (int)std::max<int64_t>(1, std::min<int64_t>(PULL_GRID, (std::max(cb, vb) + BLOCK * 16 - 1) / (BLOCK * 16)));
        hipLaunchKernelGGL(k_pull, dim3(g), dim3(BLOCK), 0, o.cs, (const char*)(o.dcol + e0), (char*)o.scol[i], cb,
                           o.dval + (size_t)e0 * o.vb, o.sval[i], vb);
        return hipGetLastError();
    }
    // Pinned memory that the device cannot address, or not all of it.
    hipError_t e = hipMemcpyAsync(o.scol[i], o.hcol + e0, (size_t)cb, hipMemcpyHostToDevice, o.cs);
    if (e == hipSuccess)
        e = hipMemcpyAsync(o.sval[i], o.hval + (size_t)e0 * o.vb, (size_t)vb, hipMemcpyHostToDevice, o.cs);
    return e;
}

namespace {
// Streams and events of the host-resident solves, created on first use per
// host thread and device and kept for the process: a freshly created pair of
// streams has been measured to block the host thread for milliseconds during
// its first few dozen copies and cross-stream waits.
struct StreamSet {
    hipStream_t ks = nullptr, cs = nullptr;
    hipEvent_t join = nullptr;
    hipEvent_t ready[2] = {nullptr, nullptr};
    hipEvent_t freed[2] = {nullptr, nullptr};
};
constexpr int MAX_DEVICES = 64;
thread_local StreamSet stream_sets[MAX_DEVICES];

hipError_t stream_set(StreamSet** out) {
    int d = 0;
    hipError_t e = hipGetDevice(&d);
    if (e != hipSuccess) return e;
    if (d < 0 || d >= MAX_DEVICES) return hipErrorInvalidDevice;
    StreamSet& S = stream_sets[d];
    if (!S.join) {
        StreamSet N;
        const unsigned ef = hipEventDisableTiming;
        if ((e = hipStreamCreateWithFlags(&N.ks, hipStreamNonBlocking)) == hipSuccess &&
            (e = hipStreamCreateWithFlags(&N.cs, hipStreamNonBlocking)) == hipSuccess &&
            (e = hipEventCreateWithFlags(&N.ready[0], ef)) == hipSuccess &&
            (e = hipEventCreateWithFlags(&N.ready[1], ef)) == hipSuccess &&
            (e = hipEventCreateWithFlags(&N.freed[0], ef)) == hipSuccess &&
            (e = hipEventCreateWithFlags(&N.freed[1], ef)) == hipSuccess &&
            (e = hipEventCreateWithFlags(&N.join, ef)) == hipSuccess) {
            S = N;
        } else {
            for (hipStream_t x : {N.ks, N.cs})
                if (x) (void)hipStreamDestroy(x);
            for (hipEvent_t x : {N.ready[0], N.ready[1], N.freed[0], N.freed[1], N.join})
                if (x) (void)hipEventDestroy(x);
            return e;
        }
    }
    *out = &S;
    return hipSuccess;
}
}  // namespace

// True if a kernel may read [h, h + bytes) of host memory at its host address:
// the device addresses it there, and one pinned allocation holds all of it.
// (The runtime's copies check their range, a kernel would fault.)
static bool device_reads(const void* h, size_t bytes) {
    void *d = nullptr, *base = nullptr;
    size_t size = 0;
    return hipHostGetDevicePointer(&d, (void*)h, 0) == hipSuccess && d == h &&
           hipMemGetAddressRange((hipDeviceptr_t*)&base, &size, (hipDeviceptr_t)h) == hipSuccess && h >= base &&
           bytes <= size && (size_t)((const char*)h - (const char*)base) <= size - bytes;
}

hipError_t ooc_begin(Ooc& o, hipStream_t* s) {
    StreamSet* S = nullptr;
    hipError_t e = stream_set(&S);
    if (e != hipSuccess) return e;
    o.ks = S->ks;
    o.cs = S->cs;
    o.join = S->join;
    for (int i = 0; i < 2; ++i) {
        o.ready[i] = S->ready[i];
        o.freed[i] = S->freed[i];
    }
    if ((e = hipEventRecord(o.join, *s)) != hipSuccess) return e;
    if ((e = hipStreamWaitEvent(o.ks, o.join, 0)) != hipSuccess) return e;
    *s = o.ks;
    return hipSuccess;
}

hipError_t ooc_end(Ooc& o, hipStream_t user) {
    hipError_t e;
    if ((e = hipEventRecord(o.join, o.ks)) != hipSuccess) return e;
    return hipStreamWaitEvent(user, o.join, 0);
}

hipError_t ooc_prepare(Plan& p, const Bufs& b, Ooc& o, int64_t slab_nnz, int64_t resident_nnz, hipStream_t s) {
    hipError_t e;
    // Status of the row-pointer checks and the tile table built from them.
    std::vector<int32_t> ob((size_t)p.n_tiles + 1);
    int32_t status = 0;
    if ((e = hipMemcpyAsync(&status, &b.st->status, sizeof(int32_t), hipMemcpyDeviceToHost, s)) != hipSuccess) return e;
    if ((e = hipMemcpyAsync(ob.data(), b.ob, ob.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s)) != hipSuccess)
        return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    o.tb.assign(1, 0);
    o.eb.assign(1, 0);
    o.nres = 0;
    o.next = 0;
    o.validated = false;
    o.streamed = 0;
    p.g_slab = 8;
    // Bad row pointers: no slabs; every later kernel sees the status and returns.
    if (status != 0) return hipSuccess;

    // Slabs: greedy runs of whole tiles of at most slab_nnz entries.  Tile t
    // starts at entry t*TILE - ob[t] (the items before it are its entries and
    // the row ends of rows 0 .. ob[t]-1); a tile holds at most TILE entries.
    auto ent = [&](int64_t t) -> int64_t { return t >= p.n_tiles ? p.nnz : t * TILE - ob[t]; };
    for (int64_t t = 0; t < p.n_tiles;) {
        int64_t u = t + 1;
        while (u < p.n_tiles && ent(u + 1) - ent(t) <= slab_nnz) ++u;
        o.tb.push_back(u);
        o.eb.push_back(ent(u));
        t = u;
    }
    const int ns = o.nslab();
    for (int k = 0; k < ns; ++k)
        if (o.eb[k + 1] < o.eb[k] || o.eb[k + 1] - o.eb[k] > slab_nnz) return hipErrorInvalidValue;
    if (o.eb[ns] != p.nnz) return hipErrorInvalidValue;
    while (o.nres < ns && o.eb[o.nres + 1] <= resident_nnz) ++o.nres;

    // One grid for every slab launch: enough wavefronts for the largest slab,
    // and the alpha partials of all slabs (ns * grid) fit the partial buffer.
    int64_t maxt = 0, maxe = 0;
    for (int k = 0; k < ns; ++k) {
        maxt = std::max(maxt, o.tb[k + 1] - o.tb[k]);
        if (k >= o.nres) maxe = std::max(maxe, o.eb[k + 1] - o.eb[k]);
    }
    int64_t g = std::min<int64_t>(p.g_tile, (maxt + WAVES - 1) / WAVES);
    g = (g + 7) / 8 * 8;
    const int64_t cap = (int64_t)std::max(std::max(p.g_tile, p.g_dense), 2048) * 64;
    if ((int64_t)ns * g > cap) g = cap / ns / 8 * 8;
    if (g < 8) return hipErrorInvalidValue;
    p.g_slab = (int32_t)g;

    // Resident slabs: one copy, on the solve's stream.
    const int64_t eres = o.eb[o.nres];
    if (eres > 0) {
        if ((e = device_alloc((void**)&o.rcol, (size_t)eres * 4)) != hipSuccess) return e;
        if ((e = device_alloc((void**)&o.rval, (size_t)eres * o.vb)) != hipSuccess) return e;
        if ((e = hipMemcpyAsync(o.rcol, o.hcol, (size_t)eres * 4, hipMemcpyHostToDevice, s)) != hipSuccess) return e;
        if ((e = hipMemcpyAsync(o.rval, o.hval, (size_t)eres * o.vb, hipMemcpyHostToDevice, s)) != hipSuccess)
            return e;
        o.streamed += eres * (int64_t)(4 + o.vb);
    }
    // Staging buffers and the copy stream for the others.
    o.dcol = nullptr;
    o.dval = nullptr;
    if (o.nres < ns) {
        if (device_reads(o.hcol, (size_t)p.nnz * 4) && device_reads(o.hval, (size_t)p.nnz * o.vb)) {
            o.dcol = o.hcol;
            o.dval = o.hval;
        } else {
            (void)hipGetLastError();
        }
        const size_t me = (size_t)std::max<int64_t>(maxe, 1);
        for (int i = 0; i < 2; ++i) {
            if ((e = device_alloc((void**)&o.scol[i], me * 4)) != hipSuccess) return e;
            if ((e = device_alloc((void**)&o.sval[i], me * o.vb)) != hipSuccess) return e;
        }
        for (int i = 0; i < 2; ++i)
            if ((e = hipEventRecord(o.freed[i], s)) != hipSuccess) return e;
    }
    return hipSuccess;
}

void ooc_release(Ooc& o) {
    // The streams and events stay cached for the next solve on this thread.
    if (o.ks) (void)hipStreamSynchronize(o.ks);
    if (o.cs) (void)hipStreamSynchronize(o.cs);
    o.ks = o.cs = nullptr;
    o.join = nullptr;
    for (int i = 0; i < 2; ++i) {
        o.ready[i] = o.freed[i] = nullptr;
        if (o.scol[i]) (void)hipFree(o.scol[i]);
        if (o.sval[i]) (void)hipFree(o.sval[i]);
        o.scol[i] = nullptr;
        o.sval[i] = nullptr;
    }
    if (o.rcol) (void)hipFree(o.rcol);
    if (o.rval) (void)hipFree(o.rval);
    o.rcol = nullptr;
    o.rval = nullptr;
}

}  // namespace lz
