// Level-1 packing of the lenses (flow chart of Sec. 2.4, "Lenses packed into
// level-1 grids"): every lens gets the index of the level-1 cell holding it,
// the lenses are stably sorted by that index (so a cell's lenses keep their
// input order and every run is bitwise reproducible), and cell_start[c] is
// the first sorted lens of cell c.  The sorted FP64 arrays are what every
// later kernel reads: the direct sum streams them in order, the near/far
// split of the interpolation uses cell_start.
//
// The sort is a least-significant-digit radix sort over 8-bit digits of the
// cell index, as many passes as the largest index needs.  Each pass counts
// the digits per block of 1024 lenses, takes the exclusive prefix sum of
// those counts in digit-major, block-minor order, and scatters every block's
// lenses to their digit's slots in input order (a lens's rank among the
// lenses of its wave with the same digit comes from ballots over the digit's
// bits), so every pass, and with it the whole sort, is stable whatever the
// distribution of lenses over the cells.  cell_start is the exclusive prefix
// sum of the per-cell counts.
//
// Up to 8192 lenses in up to 16384 cells (what one workgroup's LDS and 32-bit keys
// hold) are packed by one workgroup in one launch instead (k_pack_small): the 16
// or more launches of the above take about 7 us each however few lenses they see.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "plan.hpp"

namespace irs {

namespace {

// level-1 cell of a lens
__device__ __forceinline__ int32_t cell_of(const DevGeom &g, double x, double y)
{
    int64_t cx = (int64_t)floor((x - g.a1) / g.w1);
    int64_t cy = (int64_t)floor((y - g.b1) / g.h1);
    cx = cx < 0 ? 0 : (cx > g.n1x - 1 ? g.n1x - 1 : cx);
    cy = cy < 0 ? 0 : (cy > g.n1y - 1 ? g.n1y - 1 : cy);
    return (int32_t)(cy * g.n1x + cx);
}

__global__ void k_cell_keys(DevGeom g, const double *__restrict__ x,
                            const double *__restrict__ y, int32_t n,
                            int32_t *__restrict__ key, int32_t *__restrict__ idx)
{
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    key[i] = cell_of(g, x[i], y[i]);
    idx[i] = i;
}

__global__ void k_gather(const int32_t *__restrict__ perm, const int32_t *__restrict__ skey,
                         const double *__restrict__ x, const double *__restrict__ y,
                         const double *__restrict__ m, int32_t n, int32_t n1x,
                         double *__restrict__ sx, double *__restrict__ sy,
                         double *__restrict__ sm, uint32_t *__restrict__ cxy,
                         double2 *__restrict__ sxy)
{
    const int32_t p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int32_t i = perm[p];
    sx[p] = x[i];
    sy[p] = y[i];
    sxy[p] = make_double2(x[i], y[i]);
    if (m) sm[p] = m[i];
    const int32_t c = skey[p];
    cxy[p] = ((uint32_t)(c / n1x) << 16) | (uint32_t)(c % n1x);
}

constexpr int kScanThreads = 256;
constexpr int kScanPer = 4;                              // elements per thread
constexpr int kScanBlock = kScanThreads * kScanPer;      // elements per block

// Exclusive prefix sum of a block's wave sums in LDS (kScanThreads / 64 of them).
__device__ __forceinline__ int32_t block_exclusive(int32_t v, int32_t *s_wave, int32_t &total)
{
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    // inclusive scan within the wave
    int32_t x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    int32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) {
        if (w < wave) before += s_wave[w];
        total += s_wave[w];
    }
    __syncthreads();
    return before + x - v;
}

// out[i] = sum of in[j] for j < i within block i / kScanBlock; sums[b] = the
// block's total.  out may be in (each thread reads its elements before it
// writes them).
__global__ __launch_bounds__(kScanThreads) void k_scan_local(const int32_t *in,
                                                             int32_t n, int32_t *out,
                                                             int32_t *__restrict__ sums)
{
    __shared__ int32_t s_wave[kScanThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanPer;
    int32_t v[kScanPer], t = 0;
#pragma unroll
    for (int e = 0; e < kScanPer; ++e) {
        v[e] = base + e < n ? in[base + e] : 0;
        t += v[e];
    }
    int32_t total;
    int32_t run = block_exclusive(t, s_wave, total);
#pragma unroll
    for (int e = 0; e < kScanPer; ++e) {
        if (base + e < n) out[base + e] = run;
        run += v[e];
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// exclusive prefix sum of the nb block totals in place (one workgroup)
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(int32_t *__restrict__ sums, int32_t nb)
{
    __shared__ int32_t s_wave[kScanThreads / 64];
    int32_t carry = 0;
    for (int32_t b0 = 0; b0 < nb; b0 += kScanThreads) {
        const int32_t b = b0 + (int32_t)threadIdx.x;
        const int32_t v = b < nb ? sums[b] : 0;
        int32_t total;
        const int32_t ex = block_exclusive(v, s_wave, total);
        if (b < nb) sums[b] = carry + ex;
        carry += total;
    }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_add(int32_t *__restrict__ out, int32_t n,
                                                           const int32_t *__restrict__ sums)
{
    const int64_t i = (int64_t)blockIdx.x * kScanThreads + threadIdx.x;
    if (i < n) out[i] += sums[i / kScanBlock];
}

__global__ void k_cell_count(const int32_t *__restrict__ key, int32_t n, int32_t *__restrict__ cnt)
{
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) atomicAdd(&cnt[key[i]], 1);
}

// The whole packing of n <= kSmallLenses lenses into ncell <= kSmallCells cells
// by one workgroup: keys (cell, lens index) are all different, so sorting them
// orders the lenses as the stable sort by cell does, whatever the sort; this is a
// bitonic one, whose time does not depend on how the lenses lie.  A thread holds
// E keys next to each other: steps over shorter distances stay in its registers,
// those over less than 64 E in its wave, the others go through LDS.  cell_start
// comes from a search in the sorted keys.  The input lies in the output arrays
// (x, y in sxy, m in sx): every thread holds its lenses in registers before the
// first is written.
//
// Bound by latency: 22 us for 2277 lenses, where the launches of the radix sort
// take about 130 with the gaps between them.  A whole field, plan to map: 2277
// lenses and 2048^2 pixels 1113 -> 953 us; 256^2 pixels and 50, 2277, 5787 and
// 7975 lenses 381 / 306, 815 / 698, 985 / 849 and 1084 / 949 us.
constexpr int kSmallThreads = 1024;
constexpr int kSmallLenses = 8 * kSmallThreads, kSmallCells = 16384;
constexpr int kSmallBits = 13;
static_assert(1 << kSmallBits == kSmallLenses && kSmallCells <= 1 << (31 - kSmallBits), "32-bit keys");

// a and b in ascending order, or descending
__device__ __forceinline__ void order2(uint32_t &a, uint32_t &b, bool up)
{
    const uint32_t lo = min(a, b), hi = max(a, b);
    a = up ? lo : hi;
    b = up ? hi : lo;
}

template <int E>
__global__ __launch_bounds__(kSmallThreads) void k_pack_small(
    DevGeom g, int32_t n, int32_t ncell, int32_t *__restrict__ cell_start,
    int32_t *__restrict__ order, uint32_t *__restrict__ cxy, double *sx, double *sy, double *sm,
    double *sxy)
{
    constexpr int T = kSmallThreads;
    __shared__ uint32_t key[E * T];
    const int tid = threadIdx.x;
    uint32_t v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = e * T + tid;
        v[e] = i < n ? (uint32_t)cell_of(g, sxy[i], sxy[n + i]) << kSmallBits | (uint32_t)i
                     : UINT32_MAX;
    }
    // v[e] is key number tid E + e; merges of k keys, distances j
#pragma unroll
    for (int k = 2; k <= E; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1)
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (!(e & j)) order2(v[e], v[e | j], ((tid * E + e) & k) == 0);
    for (int kt = 2; kt <= T; kt <<= 1) {                  // k = kt E
        const bool up = (tid & kt) == 0;
        for (int jt = kt >> 1; jt > 0; jt >>= 1) {         // j = jt E: thread tid ^ jt's keys
            const bool low = ((tid & jt) == 0) == up;
            uint32_t o[E];
            if (jt < 64) {
#pragma unroll
                for (int e = 0; e < E; ++e) o[e] = (uint32_t)__shfl_xor((int)v[e], jt);
            } else {
                __syncthreads();
#pragma unroll
                for (int e = 0; e < E; ++e) key[e * T + tid] = v[e];
                __syncthreads();
#pragma unroll
                for (int e = 0; e < E; ++e) o[e] = key[e * T + (tid ^ jt)];
            }
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = low ? min(v[e], o[e]) : max(v[e], o[e]);
        }
#pragma unroll
        for (int j = E >> 1; j > 0; j >>= 1)
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (!(e & j)) order2(v[e], v[e | j], up);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) key[tid * E + e] = v[e];
    __syncthreads();
    double x[E], y[E], m[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = e * T + tid;
        const int i = p < n ? (int)(key[p] & (kSmallLenses - 1)) : 0;
        x[e] = sxy[i];
        y[e] = sxy[n + i];
        m[e] = sm ? sx[i] : 1.0;
    }
    for (int c = tid; c <= ncell; c += T) {
        // the first sorted lens of a cell >= c
        int lo = 0, hi = n;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if ((key[mid] >> kSmallBits) < (uint32_t)c) lo = mid + 1;
            else hi = mid;
        }
        cell_start[c] = lo;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = e * T + tid;
        if (p >= n) continue;
        const int32_t c = (int32_t)(key[p] >> kSmallBits);
        order[p] = (int32_t)(key[p] & (kSmallLenses - 1));
        cxy[p] = ((uint32_t)(c / g.n1x) << 16) | (uint32_t)(c % g.n1x);
        sx[p] = x[e];
        sy[p] = y[e];
        if (sm) sm[p] = m[e];
        ((double2 *)sxy)[p] = make_double2(x[e], y[e]);
    }
}

constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;
constexpr int kSortThreads = 256;
constexpr int kSortPer = 4;
constexpr int kSortBlock = kSortThreads * kSortPer;  // keys per block and pass
static_assert(kSortThreads == kRadix, "one digit per thread in the block tables");

// hist[d * nblk + b] = number of keys of block b whose digit at `shift` is d
__global__ __launch_bounds__(kSortThreads) void k_digit_hist(const int32_t *__restrict__ key,
                                                             int32_t n, int shift, int32_t nblk,
                                                             int32_t *__restrict__ hist)
{
    __shared__ int32_t s_cnt[kRadix];
    s_cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortBlock;
#pragma unroll
    for (int e = 0; e < kSortPer; ++e) {
        const int64_t i = base + (int64_t)e * kSortThreads + threadIdx.x;
        if (i < n) atomicAdd(&s_cnt[(key[i] >> shift) & (kRadix - 1)], 1);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * nblk + blockIdx.x] = s_cnt[threadIdx.x];
}

// Stable scatter of block b's keys (and their values) to the slots that the
// scanned table `offs` gives its digits.  The block's keys are taken in input
// order: four rounds of 256, each round wave by wave.
__global__ __launch_bounds__(kSortThreads) void k_digit_scatter(
    const int32_t *__restrict__ key_in, const int32_t *__restrict__ val_in, int32_t n, int shift,
    int32_t nblk, const int32_t *__restrict__ offs, int32_t *__restrict__ key_out,
    int32_t *__restrict__ val_out)
{
    __shared__ int32_t s_off[kRadix];
    s_off[threadIdx.x] = offs[(int64_t)threadIdx.x * nblk + blockIdx.x];
    __syncthreads();
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const uint64_t below = (1ull << lane) - 1ull;
    const int64_t base = (int64_t)blockIdx.x * kSortBlock;
    for (int e = 0; e < kSortPer; ++e) {
        const int64_t i = base + (int64_t)e * kSortThreads + threadIdx.x;
        const bool valid = i < n;
        const int32_t kv = valid ? key_in[i] : 0;
        const int32_t vv = valid ? val_in[i] : 0;
        const int d = (kv >> shift) & (kRadix - 1);
        // lanes of this wave holding a valid key with the same digit
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRadixBits; ++b) {
            const bool bit = (d >> b) & 1;
            const uint64_t set = __ballot(bit);
            same &= bit ? set : ~set;
        }
        const int32_t rank = (int32_t)__popcll(same & below);
        const bool last = (same >> lane) == 1ull;  // highest lane of its digit
        for (int w = 0; w < kSortThreads / 64; ++w) {
            if (wave == w && valid) {
                const int32_t pos = s_off[d] + rank;
                key_out[pos] = kv;
                val_out[pos] = vv;
                if (last) s_off[d] = pos + 1;
            }
            __syncthreads();
        }
    }
}

}  // namespace

irs_status pack_level1(irs_plan_s *p, const double *hx, const double *hy, const double *hm)
{
    const int32_t n = (int32_t)p->n_lens;
    const int64_t ncell64 = (int64_t)p->dg.n1x * p->dg.n1y;
    if (ncell64 >= INT32_MAX || p->dg.n1x > 65535 || p->dg.n1y > 65535) {
        set_error("level-1 grid too large (at most 65535 cells per side)");
        return IRS_E_INVALID;
    }
    const int32_t ncell = (int32_t)ncell64;
    hipStream_t s = p->stream;

    int bits = 0;
    while (bits < 31 && ((ncell - 1) >> bits) != 0) ++bits;
    // the index buffer that the sort's last pass writes is the plan's (the
    // input index of every packed lens)
    double *ux = nullptr, *uy = nullptr, *um = nullptr;
    int32_t *key = nullptr, *val = nullptr, *key2 = nullptr, *val2 = nullptr;
    int32_t *cnt = nullptr, *hist = nullptr, *sums = nullptr;
    const bool odd = (bits + kRadixBits - 1) / kRadixBits % 2 != 0;
    {
        DevArena a;
        a.add(p->d_landed, kLandedSlots);
        a.add(p->d_cell_start, (size_t)ncell + 1);
        IRS_HIP(a.alloc(&p->d_cells));
    }
    if (n > 0) {
        DevArena a;
        a.add(p->d_x, n);
        a.add(p->d_y, n);
        if (hm) a.add(p->d_m, n);
        a.add(p->d_cxy, n);
        a.add(p->d_xy, 2 * (size_t)n);
        IRS_HIP(a.alloc(&p->d_lenses));
        IRS_HIP(dev_alloc(&p->d_order, sizeof(int32_t) * (size_t)n));
        (odd ? val2 : val) = p->d_order;
    }
    p->h_cell_start.assign((size_t)ncell + 1, 0);
    if (n == 0) {
        IRS_HIP(hipMemsetAsync(p->d_cell_start, 0, sizeof(int32_t) * (size_t)(ncell + 1), s));
        IRS_HIP(hipStreamSynchronize(s));
        return IRS_OK;
    }
    const size_t nb = sizeof(double) * (size_t)n;
    if (n <= kSmallLenses && ncell <= kSmallCells) {
        double *in = (double *)p->d_xy;
        IRS_HIP(hipMemcpyAsync(in, hx, nb, hipMemcpyHostToDevice, s));
        IRS_HIP(hipMemcpyAsync(in + n, hy, nb, hipMemcpyHostToDevice, s));
        if (hm) IRS_HIP(hipMemcpyAsync(p->d_x, hm, nb, hipMemcpyHostToDevice, s));
#define IRS_PACK(E)                                                                            \
    hipLaunchKernelGGL(k_pack_small<E>, dim3(1), dim3(kSmallThreads), 0, s, p->dg, n, ncell,   \
                       p->d_cell_start, p->d_order, p->d_cxy, p->d_x, p->d_y, p->d_m, in)
        if (n <= kSmallThreads) IRS_PACK(1);
        else if (n <= 2 * kSmallThreads) IRS_PACK(2);
        else if (n <= 4 * kSmallThreads) IRS_PACK(4);
        else IRS_PACK(8);
#undef IRS_PACK
        IRS_HIP(hipGetLastError());
        IRS_HIP(hipMemcpyAsync(p->h_cell_start.data(), p->d_cell_start,
                               sizeof(int32_t) * (size_t)(ncell + 1), hipMemcpyDeviceToHost, s));
        IRS_HIP(hipStreamSynchronize(s));
        return IRS_OK;
    }
    void *temp = nullptr, *sort = nullptr;
    irs_status st = IRS_OK;
    const int32_t nscan = ncell + 1;  // per-cell counts then a zero: cell_start[ncell] = n
    const int32_t nblk = (n + kSortBlock - 1) / kSortBlock;
    const int32_t nhist = kRadix * nblk;
    const int32_t nsums = (std::max(nscan, nhist) + kScanBlock - 1) / kScanBlock;

    auto fail = [&](hipError_t e, const char *what) {
        st = hip_fail(e, what);
    };
#define IRS_TRY(call)                                 \
    do {                                              \
        hipError_t e_ = (call);                       \
        if (e_ != hipSuccess) {                       \
            fail(e_, #call);                          \
            goto done;                                \
        }                                             \
    } while (0)
    // exclusive prefix sum of in[0, len) into out (three launches)
    auto scan = [&](const int32_t *in, int32_t len, int32_t *out) {
        const int32_t nb = (len + kScanBlock - 1) / kScanBlock;
        hipLaunchKernelGGL(k_scan_local, dim3(nb), dim3(kScanThreads), 0, s, in, len, out, sums);
        hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kScanThreads), 0, s, sums, nb);
        hipLaunchKernelGGL(k_scan_add, dim3((len + kScanThreads - 1) / kScanThreads),
                           dim3(kScanThreads), 0, s, out, len, (const int32_t *)sums);
        return hipGetLastError();
    };

    {
        DevArena a, b;
        a.add(ux, n);
        a.add(uy, n);
        if (hm) a.add(um, n);
        IRS_TRY(a.alloc(&temp));
        b.add(key, n);
        b.add(key2, n);
        b.add(odd ? val : val2, n);
        b.add(cnt, nscan);
        b.add(hist, nhist);
        b.add(sums, nsums);
        IRS_TRY(b.alloc(&sort));
    }
    IRS_TRY(hipMemcpyAsync(ux, hx, nb, hipMemcpyHostToDevice, s));
    IRS_TRY(hipMemcpyAsync(uy, hy, nb, hipMemcpyHostToDevice, s));
    if (hm) IRS_TRY(hipMemcpyAsync(um, hm, nb, hipMemcpyHostToDevice, s));

    {
        const int tb = 256;
        const int nbk = (n + tb - 1) / tb;
        hipLaunchKernelGGL(k_cell_keys, dim3(nbk), dim3(tb), 0, s, p->dg, ux, uy, n, key, val);
        IRS_TRY(hipGetLastError());
        // cell_start: exclusive prefix sum of the per-cell counts
        IRS_TRY(hipMemsetAsync(cnt, 0, sizeof(int32_t) * (size_t)nscan, s));
        hipLaunchKernelGGL(k_cell_count, dim3(nbk), dim3(tb), 0, s, key, n, cnt);
        IRS_TRY(hipGetLastError());
        IRS_TRY(scan(cnt, nscan, p->d_cell_start));
        // stable sort of (cell, lens index) pairs by cell
        for (int shift = 0; shift < bits; shift += kRadixBits) {
            hipLaunchKernelGGL(k_digit_hist, dim3(nblk), dim3(kSortThreads), 0, s, key, n, shift,
                               nblk, hist);
            IRS_TRY(hipGetLastError());
            IRS_TRY(scan(hist, nhist, hist));
            hipLaunchKernelGGL(k_digit_scatter, dim3(nblk), dim3(kSortThreads), 0, s,
                               (const int32_t *)key, (const int32_t *)val, n, shift, nblk,
                               (const int32_t *)hist, key2, val2);
            IRS_TRY(hipGetLastError());
            std::swap(key, key2);
            std::swap(val, val2);
        }
        hipLaunchKernelGGL(k_gather, dim3(nbk), dim3(tb), 0, s, val, key, ux, uy, um, n,
                           p->dg.n1x, p->d_x, p->d_y, p->d_m, p->d_cxy, (double2 *)p->d_xy);
        IRS_TRY(hipGetLastError());
        IRS_TRY(hipMemcpyAsync(p->h_cell_start.data(), p->d_cell_start,
                               sizeof(int32_t) * (size_t)(ncell + 1), hipMemcpyDeviceToHost, s));
        IRS_TRY(hipStreamSynchronize(s));
    }
done:
#undef IRS_TRY
    dev_free(temp);
    dev_free(sort);
    return st;
}

}  // namespace irs
