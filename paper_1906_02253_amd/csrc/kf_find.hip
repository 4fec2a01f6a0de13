// Combinatorial track finding on gfx950.
//
//   a1  bin hits per (event, layer, phi bin, z|r bin): counting sorts
//       into 32-byte records (paper Sec. 3.2: hits handed in by the caller;
//       binning makes the per-layer hit search a contiguous range scan);
//   a2  order seeds by (event, eta bin, phi bin), events optionally largest
//       first, so that a wave's seeds share hit
//       bins (paper Sec. 3.2: seeds grouped close in eta and phi for cache
//       reuse of hit data);
//   a3-a7 one persistent kernel walks tiles of seeds through the detector
//       layer by layer (paper Sec. 2: KF-based finding; Sec. 3.1: layer-to-
//       layer propagation; Sec. 4: hit-search windows, candidate scoring):
//       each lane owns one candidate slot (max_cands slots per seed), keeps
//       its state in registers, propagates to its next surface, scans the
//       window's bins for hits passing the chi2 cut, then the seed's lanes
//       rank the children of all its candidates side by side and materialise
//       the survivors with the Kalman update.  Hit lists are recovered from per-step
//       back-pointers at the end.
#include "kf_find.hpp"
#include "kf_math.hpp"
#include "kf_mlp.hpp"

namespace kfmi {

static_assert(sizeof(BinnedHit) == 32, "BinnedHit is two 16-byte loads");

// ------------------------------------------------------------------ binning
__device__ inline int phi_bin_of(float phi, int nb)
{
    int b = (int)floorf((phi + float(kPi)) * float(nb) / float(2.0 * kPi));
    return b < 0 ? 0 : (b > nb - 1 ? nb - 1 : b);
}

__device__ inline int coord_bin_of(float v, float lo, float hi, int nb)
{
    float t = floorf((v - lo) * float(nb) / (hi - lo));
    if (!(t >= 0.0f)) t = 0.0f;
    if (t > float(nb - 1)) t = float(nb - 1);
    return (int)t;
}

__device__ inline int event_of(const int32_t* off, int n_events, int64_t i)
{
    int lo = 0, hi = n_events;            // off[lo] <= i < off[hi]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= i) lo = mid;
        else hi = mid;
    }
    return lo;
}

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// exclusive scan over the workgroup of one value per lane; lds holds one int
// per wave
__device__ inline int block_scan_excl(int v, int* total, int* lds)
{
    const int ln = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (ln >= o) incl += u;
    }
    if (ln == 63) lds[w] = incl;
    __syncthreads();
    int woff = 0, tot = 0;
    for (int q = 0; q < nw; ++q) {
        const int s = lds[q];
        woff += q < w ? s : 0;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return woff + incl - v;
}

// Hits are binned in one of two ways.  A few (bin_direct) in one launch of
// one workgroup, or a few, per (event, layer): it streams the layer numbers of
// its event, lists its layer's hits, counts them per (phi, z|r) bin in LDS,
// scans the counts into the layer's bin offsets and writes the 32-byte records
// in bin order.  The hits below its layer, counted in the same stream, give its
// first record, so no workgroup waits for another.  More hits go through two
// levels of counting sort (below): there the stream, once per layer, and the
// gathers, which use a few bytes of every line n_layers times over, cost more
// than seven launches and writing each record twice.  A pass by the one launch
// and by the two levels: one event of 4200 hits 197 and 220 us, of 56,000 241
// and 246, of 140,000 327 and 311; four of 56,000 378 and 331; thirty of 6800
// 312 and 326, ten of 20,400 397 and 404.  Only sums are known here, and one
// event may hold nearly all the hits, and layers of more than the LDS holds are
// left to one workgroup and global memory: so an average layer of such an event
// may have 16,384 hits, about what the LDS holds.  Ten layers, one event of
// 155,000 hits among twenty 456 and 367 us, one of 230,000 among twelve 552 and
// 368; thirty even events of 4200 228 and 246.
inline bool bin_direct(int64_t n_hits, int n_events, int n_layers)
{
    return n_hits <= 65536 || (n_hits <= 262144 && n_hits <= (int64_t)n_events * 24576 &&
                               n_hits <= (int64_t)n_layers * 16384);
}
constexpr int kDirectShare = 1024;  // hits that a workgroup writes, on average, at least
constexpr int kDirectSplit = 8;     // workgroups of an (event, layer), at most
constexpr int kBinThreads = 1024;
constexpr int kBinWaves = kBinThreads / 64;
constexpr int kBinStream = 8;       // layer numbers a lane loads together
constexpr int kBinBatch = 3;        // hits of a lane whose positions are gathered together
constexpr int kBinItems = 15;       // listed hits of a lane, at most, in LDS
constexpr int kBinCap = kBinItems * kBinThreads;   // with 4096 bins, two workgroups share a CU

// first phi row of share s of a layer's np rows; the share of row b is b * split / np
__host__ __device__ inline int share_row(int s, int np, int split) { return (s * np + split - 1) / split; }

__device__ inline int row_bin(const kf_layer& L, int bp, float hx, float hy, float hz)
{
    const float v = L.kind == 0 ? hz : sqrtf(hx * hx + hy * hy);
    return bp * L.nbin_2 + coord_bin_of(v, float(L.lo), float(L.hi), L.nbin_2);
}

__device__ inline int hit_bin(const kf_layer& L, float hx, float hy, float hz)
{
    return row_bin(L, phi_bin_of(atan2f(hy, hx), L.nbin_phi), hx, hy, hz);
}

struct HitView {
    const float *x, *y, *z, *su, *sv;
    const int32_t* layer;
};

__device__ inline BinnedHit binned_record(const HitView& h, int32_t i)
{
    BinnedHit r;
    r.x = h.x[i];
    r.y = h.y[i];
    r.z = h.z[i];
    r.su = h.su[i];
    r.sv = h.sv[i];
    r.idx = i;
    const float rho = sqrtf(r.x * r.x + r.y * r.y);
    r.cphi = r.x / rho;
    r.sphi = r.y / rho;
    return r;
}

// The hits [*lo, *hi) of n_hits that event e owns: those whose search
// (event_of) ends at it, which is the interval between the offsets that the
// search passes on the way, each loaded by a lane of its own.  With rising
// offsets these are off[e] and off[e + 1]; where the offsets decrease or lie
// outside the hits, every hit still has one event at most.  Called by whole
// waves.
__device__ inline void event_range(const int32_t* __restrict__ off, int n_events, int e, int32_t n_hits,
                                   uint32_t* lo, uint32_t* hi)
{
    const int ln = threadIdx.x & 63;
    int a = 0, b = n_events, mine = ln == 0 ? 0 : (ln == 1 ? n_events : -1);
    bool left = ln == 0;                    // an offset at or below the event's hits
    for (int step = 2; b - a > 1; ++step) {
        const int mid = (a + b) >> 1;
        if (ln == step) {
            mine = mid;
            left = e >= mid;
        }
        if (e >= mid) a = mid;
        else b = mid;
    }
    int v = mine >= 0 ? off[mine] : 0;
    v = v < 0 ? 0 : (v < n_hits ? v : n_hits);
    int l = mine >= 0 && left ? v : 0, h = mine >= 0 && !left ? v : n_hits;
    for (int o = 32; o > 0; o >>= 1) {
        const int lo2 = __shfl_xor(l, o), hi2 = __shfl_xor(h, o);
        l = lo2 > l ? lo2 : l;
        h = hi2 < h ? hi2 : h;
    }
    *lo = (uint32_t)__builtin_amdgcn_readfirstlane(l);
    h = __builtin_amdgcn_readfirstlane(h);
    *hi = *lo > (uint32_t)h ? *lo : (uint32_t)h;
}

// Streams layer[lo, hi): f(number in the list, hit) for every hit of layer l,
// in any order; *cnt (LDS, zero on entry) counts them.  Returns this lane's
// hits of lower layers.
template <typename F>
__device__ inline int stream_layer(const int32_t* __restrict__ layer, uint32_t lo, uint32_t hi, int l,
                                   int* cnt, F f)
{
    const int ln = threadIdx.x & 63;
    int less = 0;
    for (uint32_t i0 = lo; i0 < hi; i0 += kBinStream * kBinThreads) {
        int v[kBinStream];
#pragma unroll
        for (int q = 0; q < kBinStream; ++q) {
            const uint32_t i = i0 + q * kBinThreads + threadIdx.x;
            v[q] = i < hi ? layer[i] : -1;
        }
        uint64_t m[kBinStream];
        int c = 0;
#pragma unroll
        for (int q = 0; q < kBinStream; ++q) {
            m[q] = __ballot(v[q] == l);
            c += __popcll(m[q]);
            less += (uint32_t)v[q] < (uint32_t)l ? 1 : 0;
        }
        if (c == 0) continue;
        int base = 0;
        if (ln == 0) base = atomicAdd(cnt, c);
        base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
        for (int q = 0; q < kBinStream; ++q) {
            if (v[q] == l)
                f(base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m[q] >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m[q], 0u)),
                  (int32_t)(i0 + q * kBinThreads + threadIdx.x));
            base += __popcll(m[q]);
        }
    }
    return less;
}

__global__ __launch_bounds__(kBinThreads) void bin_kernel(
    HitView h, int64_t n_hits, const int32_t* __restrict__ event_off, int n_events, int stride,
    int split, const kf_layer* __restrict__ layers, int n_layers, int nb_max, BinLayout bl, int32_t* list_g,
    int32_t* bin_g, int32_t* perm_g, int32_t* __restrict__ bin_off, BinnedHit* __restrict__ out)
{
    extern __shared__ int bin_smem[];
    int* hist = bin_smem;                 // [nb_max]
    int* list = bin_smem + nb_max;        // [kBinCap]
    __shared__ int lds[kBinWaves];
    __shared__ int cnt[2];
    const int t = threadIdx.x;
    // the workgroups of one event on one XCD (workgroups go to the XCDs in turn)
    const int turn = blockIdx.x / stride, share = turn % split, l = turn / split % n_layers;
    const int e = (int)(blockIdx.x % stride) + stride * (turn / split / n_layers);
    if (e >= n_events) return;
    const kf_layer& L = layers[l];
    int first = share_row(share, L.nbin_phi, split) * L.nbin_2;
    int nb = share_row(share + 1, L.nbin_phi, split) * L.nbin_2 - first;
    uint32_t lo, hi;
    event_range(event_off, n_events, e, (int32_t)n_hits, &lo, &hi);
    for (int b = t; b < nb_max; b += kBinThreads) hist[b] = 0;
    if (t < 2) cnt[t] = 0;
    __syncthreads();
    const int less = stream_layer(h.layer, lo, hi, l, &cnt[0], [&](int k, int32_t i) {
        if (k < kBinCap) list[k] = i;
    });
    int before;                           // the layer's first record
    (void)block_scan_excl(less, &before, lds);   // (its barriers cover list and cnt)
    before += (int)lo;
    const int n = cnt[0];
    const bool in_lds = n <= kBinCap;
    uint32_t place[kBinItems];            // bin, and rank in it; ~0 in another share
    int lower = 0;                        // this lane's hits in the shares before
    if (in_lds) {
#pragma unroll
        for (int q0 = 0; q0 < kBinItems; q0 += kBinBatch) {
            if (q0 * kBinThreads >= n) break;
            float px[kBinBatch], py[kBinBatch], pz[kBinBatch];
#pragma unroll
            for (int q = 0; q < kBinBatch; ++q) {
                const int k = (q0 + q) * kBinThreads + t;
                const int i = list[k < n ? k : 0];
                px[q] = h.x[i];
                py[q] = h.y[i];
                pz[q] = L.kind == 0 ? h.z[i] : 0.0f;
            }
#pragma unroll
            for (int q = 0; q < kBinBatch; ++q) {
                place[q0 + q] = ~0u;
                if ((q0 + q) * kBinThreads + t < n) {
                    const int b = hit_bin(L, px[q], py[q], pz[q]) - first;
                    if (b >= 0 && b < nb) place[q0 + q] = ((uint32_t)b << 16) | (uint32_t)atomicAdd(&hist[b], 1);
                    lower += b < 0 ? 1 : 0;
                }
            }
        }
    } else {
        // too many for the LDS: the first share's workgroup takes the layer
        if (share != 0) return;
        nb = L.nbin_phi * L.nbin_2;
        stream_layer(h.layer, lo, hi, l, &cnt[1], [&](int k, int32_t i) { list_g[before + k] = i; });
        __syncthreads();
        for (int k = t; k < n; k += kBinThreads) {
            const int i = list_g[before + k];
            const int b = hit_bin(L, h.x[i], h.y[i], h.z[i]);
            atomicAdd(&hist[b], 1);
            bin_g[before + k] = b;
        }
    }
    int skip;
    (void)block_scan_excl(lower, &skip, lds);    // (its barriers cover hist)
    before += skip;
    // exclusive scan of the bin counts: lane t takes bins [t*per, (t+1)*per)
    const int per = (nb + kBinThreads - 1) / kBinThreads;
    const int b0 = t * per;
    int s = 0;
    for (int q = 0; q < per; ++q)
        if (b0 + q < nb) s += hist[b0 + q];
    int tot;
    int run = block_scan_excl(s, &tot, lds);
    int32_t* bo = bin_off + (int64_t)e * bl.per_event + bl.base[l] + first;
    for (int q = 0; q < per; ++q)
        if (b0 + q < nb) {
            const int c = hist[b0 + q];
            hist[b0 + q] = run;
            bo[b0 + q] = before + run;
            run += c;
        }
    // the event's last bin ends at an entry of its own
    if (l == n_layers - 1 && first + nb == L.nbin_phi * L.nbin_2 && t == 0) bo[nb] = before + tot;
    // the hits in bin order, written so that every line is filled at once
    int item[kBinItems];
    if (in_lds) {
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
            if (q * kBinThreads >= n) break;
            const int k = q * kBinThreads + t;
            item[q] = k < n ? list[k] : 0;
        }
    }
    __syncthreads();
    if (in_lds) {
#pragma unroll
        for (int q = 0; q < kBinItems; ++q) {
            if (q * kBinThreads >= n) break;
            if (place[q] != ~0u) list[hist[place[q] >> 16] + (int)(place[q] & 0xFFFFu)] = item[q];
        }
        __syncthreads();
        for (int j0 = t; j0 < tot; j0 += kBinBatch * kBinThreads) {
            BinnedHit r[kBinBatch];
#pragma unroll
            for (int q = 0; q < kBinBatch; ++q) {
                const int j = j0 + q * kBinThreads;
                r[q] = binned_record(h, list[j < tot ? j : j0]);
            }
#pragma unroll
            for (int q = 0; q < kBinBatch; ++q)
                if (j0 + q * kBinThreads < tot) out[before + j0 + q * kBinThreads] = r[q];
        }
    } else {
        for (int k = t; k < n; k += kBinThreads)
            perm_g[before + atomicAdd(&hist[bin_g[before + k]], 1)] = list_g[before + k];
        __syncthreads();
        for (int j = t; j < n; j += kBinThreads) out[before + j] = binned_record(h, perm_g[before + j]);
    }
}

// Two levels of counting sort, all hot counters in LDS.  A segment is a share
// of the phi rows of one (event, layer), `split` of them a layer.
// (1) Hits are grouped by segment: a workgroup counts a chunk of hits per
//     segment in LDS and adds the counts to the segments' (seg_count_kernel);
//     after their prefix sum, it reserves its chunk's share of every segment
//     with one atomic, sorts the chunk's hits by segment in LDS and writes
//     them in that order, so that full lines leave (seg_scatter_kernel).
// (2) One workgroup per segment reads its hits once, counts them per bin in
//     LDS, scans the counts into the bin offsets, sorts the hits in LDS and
//     writes the 32-byte records (bin_segment_kernel).
// Memory bounds each: 16, 48 and 56 bytes a hit, 37, 103 and 107 us for the
// 9,200,000 hits of 64 events.  (With complete records written from the
// registers as they came and gathered again in bin order: 187 and 243 us.)
constexpr int kSegThreads = 1024;
constexpr int kSegItems = 4;
constexpr int kSegChunk = kSegThreads * kSegItems;   // hits per workgroup in level 1
constexpr int kSegLocal = 2048;      // segments a level-1 workgroup counts in LDS
constexpr int kChunkEvents = 64;     // events of a chunk whose boundaries level 1 keeps in LDS
// (512 x 4: 107 us for the 64 events and 27 for the 2,300,000 hits of sixteen
// on ten layers; 1024 x 3 112 and 32, 256 x 8 110 and 30)
constexpr int kSortThreads = 512;
constexpr int kSortItems = 4;
constexpr int kSortCap = kSortThreads * kSortItems;   // hits a segment's workgroup holds in LDS

// A hit between the levels.
struct alignas(8) StagedHit {
    float x, y, z, su, sv;
    int32_t idx;
};

__device__ inline BinnedHit binned_record(const StagedHit& h)
{
    BinnedHit r;
    r.x = h.x;
    r.y = h.y;
    r.z = h.z;
    r.su = h.su;
    r.sv = h.sv;
    r.idx = h.idx;
    const float rho = sqrtf(r.x * r.x + r.y * r.y);
    r.cphi = r.x / rho;
    r.sphi = r.y / rho;
    return r;
}

__device__ inline int event_clamped(const int32_t* off, int n_events, int64_t i)
{
    if (i < off[0]) return 0;
    if (i >= off[n_events]) return n_events - 1;
    return event_of(off, n_events, i);
}

__global__ __launch_bounds__(256) void seg_count_kernel(int64_t n_hits, HitView hv,
                                                        const int32_t* __restrict__ event_off,
                                                        int n_events, const kf_layer* __restrict__ layers,
                                                        int n_layers, int split,
                                                        int32_t* __restrict__ seg_key,
                                                        int32_t* __restrict__ seg_cnt)
{
    __shared__ int h[kSegLocal];
    __shared__ int eoff[kChunkEvents + 2];
    __shared__ int nphi[kMaxLayers];
    const int64_t c0 = (int64_t)blockIdx.x * kSegChunk;
    const int64_t c1 = c0 + kSegChunk < n_hits ? c0 + kSegChunk : n_hits;
    const int e0 = event_clamped(event_off, n_events, c0);
    const int e1 = event_clamped(event_off, n_events, c1 - 1);
    const int per = n_layers * split;
    const int s0 = e0 * per;
    const int ns = (e1 + 1) * per - s0;
    const bool local = ns > 0 && ns <= kSegLocal;   // ns <= 0 only for a decreasing event_off
    // the chunk's event boundaries in LDS: each hit's event by a short search there
    const bool near = e1 >= e0 && e1 - e0 < kChunkEvents;
    if (near)
        for (int k = threadIdx.x; k <= e1 - e0 + 1; k += blockDim.x) eoff[k] = event_off[e0 + k];
    const int64_t all_lo = event_off[0], all_hi = event_off[n_events];
    if (local)
        for (int b = threadIdx.x; b < ns; b += blockDim.x) h[b] = 0;
    for (int l = threadIdx.x; l < n_layers; l += blockDim.x) nphi[l] = layers[l].nbin_phi;
    __syncthreads();
    for (int64_t i0 = c0 + threadIdx.x; i0 < c1; i0 += (int64_t)kSegItems * blockDim.x) {
        int lay[kSegItems];
        float x[kSegItems], y[kSegItems];
#pragma unroll
        for (int q = 0; q < kSegItems; ++q) {
            const int64_t i = i0 + (int64_t)q * blockDim.x;
            lay[q] = i < c1 ? hv.layer[i] : -1;
            x[q] = split > 1 && i < c1 ? hv.x[i] : 0.0f;
            y[q] = split > 1 && i < c1 ? hv.y[i] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < kSegItems; ++q) {
            const int64_t i = i0 + (int64_t)q * blockDim.x;
            if (i >= c1) continue;
            const int l = lay[q];
            int key = -1;
            if (l >= 0 && l < n_layers && i >= all_lo && i < all_hi) {
                int e;
                if (near) {
                    int lo = 0, hi = e1 - e0 + 1;
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        if (eoff[mid] <= i) lo = mid;
                        else hi = mid;
                    }
                    e = e0 + lo;
                } else {
                    e = event_of(event_off, n_events, i);
                }
                key = e * n_layers + l;
                if (split > 1)
                    key = key * split + phi_bin_of(atan2f(y[q], x[q]), nphi[l]) * split / nphi[l];
            }
            seg_key[i] = key;
            if (key >= 0) {
                // (a decreasing event_off could put a hit outside the chunk's
                // event range: such a hit takes the global counter)
                if (local && (unsigned)(key - s0) < (unsigned)ns) atomicAdd(&h[key - s0], 1);
                else atomicAdd(&seg_cnt[key], 1);
            }
        }
    }
    __syncthreads();
    if (local)
        for (int b = threadIdx.x; b < ns; b += blockDim.x)
            if (h[b]) atomicAdd(&seg_cnt[s0 + b], h[b]);
}

__global__ __launch_bounds__(kSegThreads) void seg_scatter_kernel(int64_t n_hits, HitView hv,
                                                                  const int32_t* __restrict__ event_off,
                                                                  int n_events, int per,
                                                                  const int32_t* __restrict__ seg_key,
                                                                  const int32_t* __restrict__ seg_off,
                                                                  int32_t* __restrict__ seg_left,
                                                                  StagedHit* __restrict__ staged)
{
    __shared__ StagedHit rec[kSegChunk];  // the chunk's hits by segment
    __shared__ int pos[kSegChunk];        // their places in `staged`
    __shared__ int h[kSegLocal], base[kSegLocal];
    __shared__ int lds[kSegThreads / 64];
    const int t = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * kSegChunk;
    const int64_t c1 = c0 + kSegChunk < n_hits ? c0 + kSegChunk : n_hits;
    int key[kSegItems], rank[kSegItems];
    StagedHit r[kSegItems];
#pragma unroll
    for (int q = 0; q < kSegItems; ++q) {
        const int64_t i = c0 + q * kSegThreads + t;
        key[q] = i < c1 ? seg_key[i] : -1;
        const int64_t j = i < c1 ? i : c0;
        r[q].x = hv.x[j];
        r[q].y = hv.y[j];
        r[q].z = hv.z[j];
        r[q].su = hv.su[j];
        r[q].sv = hv.sv[j];
        r[q].idx = (int32_t)j;
    }
    const int s0 = event_clamped(event_off, n_events, c0) * per;
    const int ns = (event_clamped(event_off, n_events, c1 - 1) + 1) * per - s0;
    const bool local = ns > 0 && ns <= kSegLocal;   // ns <= 0 only for a decreasing event_off
    if (local) {
        for (int b = t; b < ns; b += kSegThreads) h[b] = 0;
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < kSegItems; ++q) {
        rank[q] = -1;
        if (key[q] < 0) continue;
        if (local && (unsigned)(key[q] - s0) < (unsigned)ns)
            rank[q] = atomicAdd(&h[key[q] - s0], 1);
        else
            staged[seg_off[key[q]] + atomicSub(&seg_left[key[q]], 1) - 1] = r[q];
    }
    if (!local) return;
    __syncthreads();
    // the segments' places in the sorted chunk, lane t those of segments
    // [2 t, 2 t + 2), and a share of every segment for the chunk
    static_assert(kSegLocal == 2 * kSegThreads, "two segments a lane");
    const int b0 = 2 * t;
    const int n0 = b0 < ns ? h[b0] : 0, n1 = b0 + 1 < ns ? h[b0 + 1] : 0;
    int n;
    const int at = block_scan_excl(n0 + n1, &n, lds);
    if (n0) base[b0] = seg_off[s0 + b0] + atomicSub(&seg_left[s0 + b0], n0) - n0 - at;
    if (n1) base[b0 + 1] = seg_off[s0 + b0 + 1] + atomicSub(&seg_left[s0 + b0 + 1], n1) - n1 - at - n0;
    if (b0 < ns) h[b0] = at;
    if (b0 + 1 < ns) h[b0 + 1] = at + n0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSegItems; ++q) {
        if (rank[q] < 0) continue;
        const int j = h[key[q] - s0] + rank[q];
        rec[j] = r[q];
        pos[j] = base[key[q] - s0] + j;
    }
    __syncthreads();
    // three lanes a record
    const uint2* src = (const uint2*)rec;
    uint2* dst = (uint2*)staged;
    for (int d = t; d < 3 * n; d += kSegThreads) {
        const int j = (int)((uint32_t)d / 3u);
        dst[(int64_t)pos[j] * 3 + (d - 3 * j)] = src[d];
    }
}

// bin of a hit within its share; the share was chosen by the same row
__device__ inline int share_bin(const kf_layer& L, float x, float y, float z, int first, int nb)
{
    const int b = hit_bin(L, x, y, z) - first;
    return b < 0 ? 0 : (b < nb ? b : nb - 1);
}

__global__ __launch_bounds__(kSortThreads) void bin_segment_kernel(
    const int32_t* __restrict__ seg_off, const StagedHit* __restrict__ staged,
    const kf_layer* __restrict__ layers, int n_layers, int split, BinLayout bl,
    int32_t* __restrict__ bin_off, BinnedHit* __restrict__ out)
{
    __shared__ StagedHit rec[kSortCap];
    extern __shared__ int bin_smem[];
    int* hist = bin_smem;                 // [the most bins of a segment]
    __shared__ int lds[kSortThreads / 64];
    const int seg = blockIdx.x;
    const int el = seg / split, share = seg - el * split;
    const int e = el / n_layers, l = el - e * n_layers;
    const kf_layer& L = layers[l];
    const int first = share_row(share, L.nbin_phi, split) * L.nbin_2;
    const int nb = share_row(share + 1, L.nbin_phi, split) * L.nbin_2 - first;
    const int lo = seg_off[seg], n = seg_off[seg + 1] - lo;
    const int t = threadIdx.x;
    const bool in_lds = n <= kSortCap;
    // (the records' three parts as plain pairs: an array of records went to scratch)
    float2 xy[kSortItems] = {}, zu[kSortItems] = {}, vi[kSortItems] = {};
    if (in_lds && n > 0) {
#pragma unroll
        for (int q = 0; q < kSortItems; ++q) {
            const float2* p = (const float2*)&staged[lo + (q * kSortThreads + t < n ? q * kSortThreads + t : 0)];
            xy[q] = p[0];
            zu[q] = p[1];
            vi[q] = p[2];
        }
    }
    for (int b = t; b < nb; b += kSortThreads) hist[b] = 0;
    __syncthreads();
    uint32_t place[kSortItems];           // bin, and rank in it
    if (in_lds) {
#pragma unroll
        for (int q = 0; q < kSortItems; ++q)
            if (q * kSortThreads + t < n) {
                const int b = share_bin(L, xy[q].x, xy[q].y, zu[q].x, first, nb);
                place[q] = ((uint32_t)b << 16) | (uint32_t)atomicAdd(&hist[b], 1);
            }
    } else {
        for (int i = lo + t; i < lo + n; i += kSortThreads)
            atomicAdd(&hist[share_bin(L, staged[i].x, staged[i].y, staged[i].z, first, nb)], 1);
    }
    __syncthreads();
    // exclusive scan of the bin counts: lane t takes bins [t*per, (t+1)*per)
    const int per = (nb + kSortThreads - 1) / kSortThreads;
    const int b0 = t * per;
    int s = 0;
    for (int q = 0; q < per; ++q)
        if (b0 + q < nb) s += hist[b0 + q];
    int tot;
    int run = block_scan_excl(s, &tot, lds);
    int32_t* bo = bin_off + (int64_t)e * bl.per_event + bl.base[l] + first;
    for (int q = 0; q < per; ++q)
        if (b0 + q < nb) {
            const int c = hist[b0 + q];
            hist[b0 + q] = run;
            bo[b0 + q] = lo + run;
            run += c;
        }
    // the event's last bin ends at an entry of its own
    if (l == n_layers - 1 && share == split - 1 && t == 0) bo[nb] = lo + n;
    __syncthreads();
    if (in_lds) {
#pragma unroll
        for (int q = 0; q < kSortItems; ++q)
            if (q * kSortThreads + t < n) {
                float2* p = (float2*)&rec[hist[place[q] >> 16] + (int)(place[q] & 0xFFFFu)];
                p[0] = xy[q];
                p[1] = zu[q];
                p[2] = vi[q];
            }
        __syncthreads();
        for (int j = t; j < n; j += kSortThreads) out[lo + j] = binned_record(rec[j]);
    } else {
        // more hits than the LDS holds: straight to their places
        for (int i = lo + t; i < lo + n; i += kSortThreads) {
            const StagedHit h = staged[i];
            out[lo + atomicAdd(&hist[share_bin(L, h.x, h.y, h.z, first, nb)], 1)] = binned_record(h);
        }
    }
}

// ------------------------------------------------------------------ prefix sums
// Exclusive prefix sum of n int32 in three launches (no library scan, so that
// the pass contains kernels only and can be captured into a graph): per-chunk
// totals, an in-place scan of the totals by one workgroup, and a rescan of
// each chunk from its offset.
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanChunk = kScanThreads * kScanItems;

__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(const int32_t* __restrict__ in,
                                                                   int64_t n,
                                                                   int32_t* __restrict__ bsum)
{
    __shared__ int lds[kScanThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + threadIdx.x;
    int s = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const int64_t i = base + (int64_t)q * kScanThreads;
        s += i < n ? in[i] : 0;
    }
    int tot;
    (void)block_scan_excl(s, &tot, lds);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void scan_top_kernel(int32_t* __restrict__ bsum, int nb)
{
    __shared__ int lds[1024 / 64];
    int carry = 0;
    for (int b0 = 0; b0 < nb; b0 += 1024) {
        const int i = b0 + (int)threadIdx.x;
        const int v = i < nb ? bsum[i] : 0;
        int tot;
        const int ex = block_scan_excl(v, &tot, lds);
        if (i < nb) bsum[i] = carry + ex;
        carry += tot;
    }
}

__global__ __launch_bounds__(kScanThreads) void scan_apply_kernel(const int32_t* __restrict__ in,
                                                                  int64_t n,
                                                                  const int32_t* __restrict__ bsum,
                                                                  int32_t* __restrict__ out)
{
    __shared__ int lds[kScanThreads / 64];
    // lane t takes kScanItems consecutive values of the chunk
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
    int v[kScanItems];
    int s = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        v[q] = base + q < n ? in[base + q] : 0;
        s += v[q];
    }
    int tot;
    int run = bsum[blockIdx.x] + block_scan_excl(s, &tot, lds);
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        if (base + q < n) out[base + q] = run;
        run += v[q];
    }
}

// ------------------------------------------------------------------ seed order
constexpr int kSeedCells = 64 * 64;   // eta x phi cells per event
constexpr int kRankMaxEvents = 16384; // events ranked by size for the largest-first order

// Position of each event in the processing order: by hit count, largest
// first, ties by event index (a permutation of 0..n_events-1).
__global__ __launch_bounds__(256) void event_rank_kernel(const int32_t* __restrict__ event_off,
                                                         int n_events, int32_t* __restrict__ erank)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_events) return;
    const int ne = event_off[e + 1] - event_off[e];
    int r = 0;
    for (int q = 0; q < n_events; ++q) {
        const int nq = event_off[q + 1] - event_off[q];
        r += (nq > ne || (nq == ne && q < e)) ? 1 : 0;
    }
    erank[e] = r;
}

// eta over [-3, 3) and phi over [-pi, pi) in 64 bins each; a non-finite
// angle falls into bin 0
__device__ inline int seed_cell(float th, float ph)
{
    const float eta = -logf(tanf(0.5f * th));
    float fe = floorf((eta + 3.0f) * (64.0f / 6.0f));
    fe = fe >= 0.0f ? (fe < 63.0f ? fe : 63.0f) : 0.0f;
    float fp = floorf((ph + float(kPi)) * (64.0f / float(2.0 * kPi)));
    fp = fp >= 0.0f ? (fp < 63.0f ? fp : 63.0f) : 0.0f;
    return (int)fe * 64 + (int)fp;
}

__global__ __launch_bounds__(256) void seed_cell_kernel(int64_t n, int64_t ld, const float* __restrict__ par,
                                                        const int32_t* __restrict__ seed_event,
                                                        int n_events,
                                                        const int32_t* __restrict__ erank,
                                                        int32_t* __restrict__ cnt,
                                                        int32_t* __restrict__ cell)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float th = par[5 * ld + i], ph = par[4 * ld + i];
    int e = seed_event[i];
    e = e < 0 ? 0 : (e >= n_events ? n_events - 1 : e);
    if (erank) e = erank[e];
    const int c = e * kSeedCells + seed_cell(th, ph);
    atomicAdd(&cnt[c], 1);
    cell[i] = c;
}

__global__ __launch_bounds__(256) void seed_scatter_kernel(int64_t n, const int32_t* __restrict__ cell,
                                                           const int32_t* __restrict__ off,
                                                           int32_t* __restrict__ cnt,
                                                           int32_t* __restrict__ order)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int c = cell[i];
    order[off[c] + atomicSub(&cnt[c], 1) - 1] = (int32_t)i;
}

// The scatter leaves a cell's seeds in arbitrary order; sort each cell by
// seed index so that tiles are the same from run to run.  Cells above
// kCellSortMax seeds (only degenerate inputs pile up so) keep the scatter order.
constexpr int kCellSortMax = 256;
__global__ __launch_bounds__(256) void cell_sort_kernel(int64_t n_cells, const int32_t* __restrict__ off,
                                                        int32_t* __restrict__ order)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_cells) return;
    const int lo = off[c], hi = off[c + 1];
    if (hi - lo < 2 || hi - lo > kCellSortMax) return;
    for (int i = lo + 1; i < hi; ++i) {
        const int32_t v = order[i];
        int j = i - 1;
        while (j >= lo && order[j] > v) {
            order[j + 1] = order[j];
            --j;
        }
        order[j + 1] = v;
    }
}

// Tiles of seeds of like cost.  A tile runs as long as its slowest seed,
// and low-pT seeds in the central barrel (loopers, which curl back through
// the layers with ever wider windows) walk longest, so inside each tile
// queue's contiguous range of the processing order the seeds are
// partitioned, stably, by a cost class of |q/pT| and |eta|, costliest first:
// fewer tiles wait on one looper, and the long tiles start first instead of
// ending the pass.  The costliest class, the central loopers, comes in tiles
// of half the seeds: a tile's window scan is shared by its candidates, so
// such a tile ends in about half the time, and the few longest tiles no
// longer outlast the rest of the pass.
constexpr int kCostClasses = 4;

// seeds in a tile of the costliest class: half a tile
__host__ __device__ inline int looper_tile_seeds(int S)
{
    return S / 2 > 1 ? S / 2 : 1;
}
__device__ inline int cost_class(float c, float theta)
{
    // |theta - pi/2| < 0.4803: |eta| < 0.5; < 0.8658: |eta| < 1
    const float a = fabsf(c), e = fabsf(theta - 1.57079633f);
    if (a > 1.0f / 0.6f && e < 0.4803f) return 0;   // central loopers, pT < 0.6 GeV
    if (a > 1.0f / 0.7f && e < 0.8658f) return 1;   // pT < 0.7 GeV, |eta| < 1
    return a > 1.0f ? 2 : 3;                         // pT < 1 GeV, the rest
}

// Two passes over blocks of kCostBlock entries of each queue range [q chunk,
// (q + 1) chunk) of the cell order (chunk is a whole number of tiles): the
// blocks' class counts, then each block places its entries at the class's
// base in the range plus the class's entries in earlier blocks, lanes and
// waves (a stable partition).
constexpr int kCostBlock = 1024;

__device__ inline void cost_block_range(int64_t n, int64_t chunk, int nbq, int64_t* lo, int64_t* hi)
{
    const int q = blockIdx.x / nbq, b = blockIdx.x - q * nbq;
    const int64_t qhi = (int64_t)(q + 1) * chunk < n ? (int64_t)(q + 1) * chunk : n;
    *lo = (int64_t)q * chunk + (int64_t)b * kCostBlock;
    *hi = *lo + kCostBlock < qhi ? *lo + kCostBlock : qhi;
}

__global__ __launch_bounds__(kCostBlock) void cost_count_kernel(int64_t n, int64_t ld,
                                                                const float* __restrict__ par,
                                                                const int32_t* __restrict__ order,
                                                                int64_t chunk, int nbq,
                                                                int32_t* __restrict__ cnt)
{
    __shared__ int tot[kCostClasses];
    int64_t lo, hi;
    cost_block_range(n, chunk, nbq, &lo, &hi);
    const int t = threadIdx.x;
    if (t < kCostClasses) tot[t] = 0;
    __syncthreads();
    const int64_t i = lo + t;
    const int k = i < hi ? cost_class(par[3 * ld + order[i]], par[5 * ld + order[i]]) : -1;
    for (int c = 0; c < kCostClasses; ++c) {
        const unsigned long long m = __ballot(k == c);
        if ((t & 63) == 0 && m) atomicAdd(&tot[c], __popcll(m));
    }
    __syncthreads();
    if (t < kCostClasses) cnt[(size_t)blockIdx.x * kCostClasses + t] = tot[t];
}

__global__ __launch_bounds__(kCostBlock) void cost_place_kernel(int64_t n, int64_t ld,
                                                                const float* __restrict__ par,
                                                                const int32_t* __restrict__ order,
                                                                int64_t chunk, int nbq,
                                                                const int32_t* __restrict__ cnt,
                                                                int32_t* __restrict__ out,
                                                                int32_t* __restrict__ queue_loopers)
{
    __shared__ int wtot[kCostBlock / 64][kCostClasses];   // per wave and class
    __shared__ int base[kCostClasses];                      // class base of this block in the range
    int64_t lo, hi;
    cost_block_range(n, chunk, nbq, &lo, &hi);
    const int q = blockIdx.x / nbq, b = blockIdx.x - q * nbq;
    const int t = threadIdx.x, wave = t >> 6, ln = t & 63;
    if (b == 0 && t == 0) {
        // the range's costliest-class seeds (its head after the partition)
        int c0 = 0;
        for (int bb = 0; bb < nbq; ++bb) c0 += cnt[((size_t)q * nbq + bb) * kCostClasses];
        queue_loopers[q] = c0;
    }
    if (lo >= hi) return;
    if (t < kCostClasses) {
        // entries of the range in the costlier classes, then this class's in earlier blocks
        int before = 0, costlier = 0;
        for (int bb = 0; bb < nbq; ++bb) {
            const int32_t* c = cnt + ((size_t)q * nbq + bb) * kCostClasses;
            for (int k = 0; k < t; ++k) costlier += c[k];
            if (bb < b) before += c[t];
        }
        base[t] = costlier + before;
    }
    const int64_t i = lo + t;
    const int k = i < hi ? cost_class(par[3 * ld + order[i]], par[5 * ld + order[i]]) : -1;
    int below = 0;
    for (int c = 0; c < kCostClasses; ++c) {
        const unsigned long long m = __ballot(k == c);
        if (ln == 0) wtot[wave][c] = __popcll(m);
        if (k == c)
            below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    }
    __syncthreads();
    if (k >= 0) {
        int pos = base[k] + below;
        for (int w = 0; w < wave; ++w) pos += wtot[w][k];
        out[(int64_t)q * chunk + pos] = order[i];
    }
}

// A few seeds' tile order in one launch of one workgroup: the keys (event
// position, cell, seed) and then (queue, cost class, place) are sorted in
// registers, entry q kOrderThreads + t with lane t, by a bitonic network whose
// exchanges within a wave are shuffles.  Up to kOrderMax seeds: 56 seeds 150 us
// a pass by this one launch and 159 by the general way's ten, 744 seeds 229 and
// 239, 1700 seeds of 30 events 234 and 237; with four entries a lane 2800 seeds
// 385 and 370.
constexpr int kOrderThreads = 1024;
constexpr int kOrderItems = 2;
constexpr int kOrderMax = kOrderThreads * kOrderItems;   // seeds: 12 bits of a key
constexpr int kOrderEvents = 256;                        // events x kSeedCells: the other 20

template <int NQ>
__device__ inline void sort_keys(uint32_t (&v)[NQ], uint32_t* buf)
{
    const int t = threadIdx.x;
    for (int k = 2; k <= NQ * kOrderThreads; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            uint32_t o[NQ];
            if (j >= kOrderThreads) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    o[q] = v[q];
#pragma unroll
                    for (int r = 0; r < NQ; ++r) o[q] = r == (q ^ (j / kOrderThreads)) ? v[r] : o[q];
                }
            } else if (j >= 64) {
                __syncthreads();
#pragma unroll
                for (int q = 0; q < NQ; ++q) buf[q * kOrderThreads + t] = v[q];
                __syncthreads();
#pragma unroll
                for (int q = 0; q < NQ; ++q) o[q] = buf[q * kOrderThreads + (t ^ j)];
            } else {
#pragma unroll
                for (int q = 0; q < NQ; ++q) o[q] = __shfl_xor(v[q], j);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int i = q * kOrderThreads + t;
                const bool low = ((i & k) == 0) == ((i & j) == 0);
                v[q] = low ? (v[q] < o[q] ? v[q] : o[q]) : (v[q] < o[q] ? o[q] : v[q]);
            }
        }
}

template <int NQ>
__global__ __launch_bounds__(kOrderThreads) void small_order_kernel(
    int n, int64_t ld, const float* __restrict__ par, const int32_t* __restrict__ seed_event,
    const int32_t* __restrict__ event_off, int n_events, int largest_first, int chunk,
    int32_t* __restrict__ tile_order, int32_t* __restrict__ queue_loopers,
    int32_t* __restrict__ tile_counter)
{
    __shared__ uint32_t buf[NQ * kOrderThreads];
    __shared__ int32_t seed[NQ * kOrderThreads];
    __shared__ uint8_t cls[NQ * kOrderThreads];
    __shared__ int size[kOrderEvents], rank[kOrderEvents], loopers[kQueues];
    const int t = threadIdx.x;
    if (t < n_events) size[t] = event_off[t + 1] - event_off[t];
    if (t < kQueues) loopers[t] = 0;
    for (int k = t; k < kQueues * kQueueStride; k += kOrderThreads) tile_counter[k] = 0;
    __syncthreads();
    if (t < n_events) {
        int r = t;
        if (largest_first) {
            r = 0;
            for (int q = 0; q < n_events; ++q) r += (size[q] > size[t] || (size[q] == size[t] && q < t)) ? 1 : 0;
        }
        rank[t] = r;
    }
    __syncthreads();
    uint32_t v[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int i = q * kOrderThreads + t;
        v[q] = ~0u;
        if (i < n) {
            const float th = par[5 * ld + i], ph = par[4 * ld + i];
            int e = seed_event[i];
            e = e < 0 ? 0 : (e >= n_events ? n_events - 1 : e);
            v[q] = (uint32_t)(rank[e] * kSeedCells + seed_cell(th, ph)) << 12 | (uint32_t)i;
            cls[i] = (uint8_t)cost_class(par[3 * ld + i], th);
        }
    }
    sort_keys<NQ>(v, buf);
    __syncthreads();                       // cls, and the last reads of buf
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int p = q * kOrderThreads + t;
        if (p < n) {
            const int i = (int)(v[q] & 0xFFFu), c = cls[i], queue = p / chunk;
            seed[p] = i;
            v[q] = (uint32_t)(queue * kCostClasses + c) << 12 | (uint32_t)p;
            if (c == 0) atomicAdd(&loopers[queue], 1);
        }
    }
    sort_keys<NQ>(v, buf);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int p = q * kOrderThreads + t;
        if (p < n) tile_order[p] = seed[v[q] & 0xFFFu];
    }
    if (t < kQueues) queue_loopers[t] = loopers[t];
}

// ------------------------------------------------------------------ find
// LDS writes of one wave made visible to that wave's other lanes
__device__ inline void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A hit's place in a candidate's child list, (chi2, hit index) ascending, as
// one unsigned key: the float's bits made monotone (-0 taken as +0) above
// the non-negative index.
__device__ inline uint64_t child_key(float c2, int32_t id)
{
    uint32_t u = __float_as_uint(c2);
    if (u == 0x80000000u) u = 0u;
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((uint64_t)u << 32) | (uint32_t)id;
}

__device__ inline float child_key_chi2(uint64_t key)
{
    const uint32_t u = (uint32_t)(key >> 32);
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}

// A child's place in its seed's selection: more hits first, then lower chi2
// (as child_key's bits), then parent slot j and child c.
__device__ inline uint64_t merge_key(int nhits, float c2, int j, int c)
{
    uint32_t u = __float_as_uint(c2);
    if (u == 0x80000000u) u = 0u;
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    const uint32_t nh = nhits < 0 ? 0u : nhits > 255 ? 255u : (uint32_t)nhits;
    return ((uint64_t)(255u - nh) << 56) | ((uint64_t)u << 24) | ((uint64_t)j << 16) |
           ((uint64_t)c << 8);
}

// A 64-bit value of one lane (uniform), of the lane before (0 in a row's
// first), and the wave's smallest 32-bit value (uniform).
__device__ inline uint64_t readlane64(uint64_t v, int lane)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}

__device__ inline uint64_t lane_before64(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, 0x111, 0xf, 0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), 0x111, 0xf, 0xf, false);
    return ((uint64_t)hi << 32) | lo;
}

template <int CTRL, int ROWS>
__device__ inline uint32_t dpp_min_u32(uint32_t v)
{
    const uint32_t u = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, CTRL, ROWS, 0xf, false);
    return u < v ? u : v;
}

__device__ inline uint32_t wave_min_u32(uint32_t v, int lanes)
{
    // row shifts by 1, 2, 4, 8, then the rows' last lanes broadcast upwards
    v = dpp_min_u32<0x111, 0xf>(v);
    v = dpp_min_u32<0x112, 0xf>(v);
    v = dpp_min_u32<0x114, 0xf>(v);
    v = dpp_min_u32<0x118, 0xf>(v);
    v = dpp_min_u32<0x142, 0xa>(v);
    v = dpp_min_u32<0x143, 0xc>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lanes - 1);
}

template <int CTRL, int ROWS>
__device__ inline int dpp_max_i32(int v)
{
    const int u = __builtin_amdgcn_update_dpp(v, v, CTRL, ROWS, 0xf, false);
    return u > v ? u : v;
}

// running maximum over the lanes
__device__ inline int wave_max_scan(int v)
{
    v = dpp_max_i32<0x111, 0xf>(v);
    v = dpp_max_i32<0x112, 0xf>(v);
    v = dpp_max_i32<0x114, 0xf>(v);
    v = dpp_max_i32<0x118, 0xf>(v);
    v = dpp_max_i32<0x142, 0xa>(v);
    return dpp_max_i32<0x143, 0xc>(v);
}

// The chi2 in a selection key (its float bits made monotone).
__device__ inline float merge_key_chi2(uint64_t key)
{
    const uint32_t u = (uint32_t)(key >> 24);
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}

// Row stride of the window owners' position covariance in LDS: six values
// padded to whole 16-byte reads (three for FP64, two for FP32)
template <typename C> constexpr int kOwnCov = sizeof(C) == 8 ? 6 : 8;

template <typename C>
__device__ inline void load_owner_cov(const C* r, C pc[6])
{
    if constexpr (sizeof(C) == 8) {
        const double2 a = *(const double2*)r, b = *(const double2*)(r + 2), c = *(const double2*)(r + 4);
        pc[0] = a.x; pc[1] = a.y; pc[2] = b.x; pc[3] = b.y; pc[4] = c.x; pc[5] = c.y;
    } else {
        const float4 a = *(const float4*)r;
        const float2 b = *(const float2*)(r + 4);
        pc[0] = a.x; pc[1] = a.y; pc[2] = a.z; pc[3] = a.w; pc[4] = b.x; pc[5] = b.y;
    }
}

// A hit (record halves r0: x, y, z, su; r1: sv, cos phi, sin phi, index)
// against a window owner's record (oa, ob: see WaveLds::orec): inside the
// window's box.  |azimuth difference| <= dphi (< pi/2): same half-plane, |sin|
// bounded.
template <typename T>
__device__ inline bool window_test(const float4& oa, const float4& ob, const float4& r0, const float4& r1)
{
    const float hcp = r1.y, hsp = r1.z;
    const T ox = T(oa.x), oy = T(oa.y), oz = T(oa.z);
    const T cpp = T(oa.w), spp = T(ob.x);
    const T sin_dphi = T(ob.y), wv = T(ob.z);
    const int fl = __float_as_int(ob.w);
    const int kind = fl >> 1;
    bool pass = (fl & 1) || (T(hcp) * cpp + T(hsp) * spp > T(0) &&
                             !(Tr<T>::abs_(T(hsp) * cpp - T(hcp) * spp) > sin_dphi));
    if (pass) {
        const T rv = kind == 0 ? T(r0.z) - oz : T(hcp) * (T(r0.x) - ox) + T(hsp) * (T(r0.y) - oy);
        pass = !(Tr<T>::abs_(rv) > wv);
    }
    return pass;
}

// Its chi2 against the owner's position and position covariance pc: below the cut.
template <typename T, typename C, typename U>
__device__ inline bool chi2_test(const float4& oa, const float4& ob, const C pc[6], const float4& r0,
                                 const float4& r1, float cut, unsigned* n_chi2, float* c2f)
{
    HitFrame<U> f;
    f.hx = U(r0.x);
    f.hy = U(r0.y);
    f.hz = U(r0.z);
    f.c = U(r1.y);
    f.s = U(r1.z);
    f.vu = U(r0.w) * U(r0.w);
    f.vv = U(r1.x) * U(r1.x);
    const U c2u = hit_chi2_pos<U>(U(oa.x), U(oa.y), U(oa.z), U(pc[0]), U(pc[1]), U(pc[2]), U(pc[3]), U(pc[4]),
                                  U(pc[5]), f, __float_as_int(ob.w) >> 1);
    ++*n_chi2;
    *c2f = float(c2u);
    return c2u < U(cut);
}

constexpr int kSeg = 128;       // phi rows queued per wave per round
constexpr int kScanBatch = 4;   // hits per lane in flight in the scan
constexpr int kAcc = 64 * kScanBatch;
constexpr int kInsBatch = 4;    // accepted hits an owner loads together
// Bins from which a window is scanned with its seed's others.  The group scan
// costs its lists' set-up, and reads the union of windows that may differ; the
// queue one load per candidate and hit.  The line was drawn at 128 x 32 bins a
// layer: 64 events of 2100 tracks 2049 us by the queue alone, 1914 from 256 bins
// on, 1862 from 1024, 1926 from 4096; 16 events with overlapping seeds 1450,
// 1232, 1238, 1290.  It counts bins and not the hits in them; no call became
// slower for it on other grids (16 events with overlapping seeds by the queue and
// with it, a grid of 32 x 8, where no window is as long, 1508 and 1283 us; of 512
// x 32 1518 and 1269).
constexpr int kLongBins = 1024;
constexpr int kSelKeys = 64 * (kMaxCands + 1);   // children of a wave's candidates, at most

// Covariance entries beside the position block that a candidate leaves in LDS
// during the window scan and the selection (their packed indices): they need
// no registers there, and a surviving child reads them from its parent's
// column instead of by two shuffles each.  More would cost the eighth wave of
// a compute unit.
constexpr int kPark = 8;
__host__ __device__ constexpr int parked(int k)
{
    constexpr int at[kPark] = {pk(0, 3), pk(0, 4), pk(0, 5), pk(1, 3), pk(1, 4), pk(1, 5), pk(2, 3), pk(2, 4)};
    return at[k];
}

// LDS of one wave; arrays lane-minor unless noted.  The window scan's queues
// and the selection's keys are never live together.
template <typename C>
struct alignas(16) WaveLds {
    C ocov[64 * kOwnCov<C>];    // window owner's predicted position covariance
                                //          P00 P01 P02 P11 P12 P22 (16-byte rows)
    C park[kPark * 64];         // entries of the covariance that wait here for the selection
    float orec[64 * 8];         // window owner record: predicted x, y, z, cos and sin of its
                                //        azimuth, sin(dphi), wv, flags (two 16-byte reads)
    union {
        struct {
            int32_t seg[3 * kSeg];      // queued phi rows: owner lane, first hit, count
            int32_t segpre[kSeg + 4];   // prefix of the rows' hit counts
            int32_t acc[3 * kAcc];      // per owner lane its accepted hits' first and last entry
                                        // ([0, 64), [64, 128)); the entries' hit index; their
                                        // binned index
            float accc2[kAcc];          // their chi2
            int32_t rowp[5 * 64];       // per owner lane: row prefix, first row, bins, base, sizes
        };
        struct {
            uint64_t key[kSelKeys];     // [seeds][max_cands (max_cands + 1)] a seed's children
            uint64_t sel[64];           // [seeds][max_cands] its survivors, best first
            int32_t cbidx[kMaxCands * 64];   // binned index of each candidate's accepted hits
        };
    };
    int32_t finite;             // whether the tile's seeds have finite covariances (see transport)
};

// LDS of a workgroup: the layers, the navigation's surface orders, then each
// wave's own block
__host__ __device__ inline size_t find_layers_bytes(int nl)
{
    return (sizeof(FindLayer) * nl + nav_bytes(nl) + 15) & ~size_t(15);
}

template <typename C>
__host__ __device__ inline size_t find_shared_bytes(int W, int nl)
{
    return find_layers_bytes(nl) + sizeof(WaveLds<C>) * ((W + 63) / 64);
}

// wave-wide exclusive prefix sum (and total) of one int per lane
__device__ inline int wave_scan(int v, int wlanes, int* total)
{
    const int ln = (int)(threadIdx.x & 63);
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o);
        if (ln >= o) incl += u;
    }
    *total = __shfl(incl, wlanes - 1);
    return incl - v;
}

// prefix of nseg queued rows' hit counts, two rows per lane; the total
template <typename LEN, typename PRE>
__device__ inline int row_prefix(LEN len, PRE pre, int nseg, int wlanes)
{
    const int ln = (int)(threadIdx.x & 63);
    const int la = 2 * ln < nseg ? len[2 * ln] : 0;
    const int lb = 2 * ln + 1 < nseg ? len[2 * ln + 1] : 0;
    int H = 0;
    const int p = wave_scan(la + lb, wlanes, &H);
    if (2 * ln < nseg) pre[2 * ln] = p;
    if (2 * ln + 1 < nseg) pre[2 * ln + 1] = p + la;
    if (ln == 0) pre[nseg] = H;
    wave_fence();
    return H;
}

// Scan of the long windows of a seed's candidates on one layer (the lanes of
// `group`, at most an eighth of the wave's): rows u_lo .. u_lo + u_rows - 1
// (modulo np) times second bins u_v0 .. u_v1 of the layer whose first bin in
// the event is row0, the union of the windows.  64 consecutive hits at a time
// are tested against each window; the windows' best hits are sorted lists over
// eight lanes each, which only hits below a list's entry MC - 1 enter, best
// first.  A function of its own: the finding kernel has no registers to spare
// for it, and it runs for a few seeds in a thousand.
struct LongList {
    uint64_t best;      // lane 8 k + q: entry q of the k-th window
    int bi;             // its binned index
    int count;          // lanes 8 k ..: hits below the cut in the k-th window
    unsigned tests;     // chi2 tests of this lane
};

template <typename C>
using LdsPtr = __attribute__((address_space(3))) WaveLds<C>*;

template <typename T, typename C, typename U>
__device__ __attribute__((noinline)) LongList long_scan(LdsPtr<C> w, const BinnedHit* bh, const int32_t* bin_off,
                                                        uint64_t group_, int u_lo_, int u_rows_, int u_v0_,
                                                        int u_v1_, int np_, int n2_, int row0_, int MC_,
                                                        int wlanes_, float cut)
{
    // (arguments arrive in vector registers; these are uniform)
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int u_lo = uni(u_lo_), u_rows = uni(u_rows_), u_v0 = uni(u_v0_), u_v1 = uni(u_v1_);
    const int np = uni(np_), n2 = uni(n2_), row0 = uni(row0_), MC = uni(MC_), wlanes = uni(wlanes_);
    const uint64_t group = ((uint64_t)(uint32_t)uni((int)(group_ >> 32)) << 32) | (uint32_t)uni((int)(uint32_t)group_);
    const int ln = (int)(threadIdx.x & 63);
    auto* h0s = w->seg + kSeg;
    auto* lens = w->seg + 2 * kSeg;
    auto* pre = w->segpre;
    auto* mark = w->acc;
    LongList L{~0ull, -1, 0, 0u};
    const int segcap = 2 * wlanes < kSeg ? 2 * wlanes : kSeg;
    for (int rr0 = 0; rr0 < u_rows; rr0 += segcap) {
        const int nseg = u_rows - rr0 < segcap ? u_rows - rr0 : segcap;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int j = r * wlanes + ln;
            if (j < nseg) {
                const int bb = u_lo + rr0 + j;
                const uint32_t rb = (uint32_t)row0 + (uint32_t)((((bb % np) + np) % np) * n2);
                const int h0 = bin_off[rb + u_v0];
                const int h1 = bin_off[rb + u_v1 + 1];
                h0s[j] = h0;
                lens[j] = h1 - h0;
            }
        }
        wave_fence();
        const int H = uni(row_prefix(lens, pre, nseg, wlanes));
        int row_at = 0;                     // the row of the batch's first hit, or before it
        for (int g0 = 0; g0 < H; g0 += wlanes * kScanBatch) {
            float4 r0[kScanBatch], r1[kScanBatch];
            int bix[kScanBatch];
            // the row of each hit: rows that start in the batch leave their number
            // at their first hit, and a running maximum carries it on
#pragma unroll
            for (int q = 0; q < kScanBatch; ++q) mark[q * wlanes + ln] = row_at;
            wave_fence();
            for (int r = row_at + 1 + ln; __ballot(r < nseg); r += wlanes) {
                const int p0 = r < nseg ? pre[r] : 0x7fffffff;
                if (p0 < g0 + wlanes * kScanBatch && p0 >= g0 && pre[r + 1] > p0) mark[p0 - g0] = r;
            }
            wave_fence();
#pragma unroll
            for (int q = 0; q < kScanBatch; ++q) {
                const int g = g0 + q * wlanes + ln;
                int row = wave_max_scan(mark[q * wlanes + ln]);
                row = row > row_at ? row : row_at;
                row_at = __builtin_amdgcn_readlane(row, wlanes - 1);
                bix[q] = g < H ? h0s[row] - pre[row] + g : -1;
                const int b = bix[q] < 0 ? 0 : bix[q];
                r0[q] = *(const float4*)&bh[b].x;
                r1[q] = *(const float4*)&bh[b].sv;
            }
            int k = 0;
            for (uint64_t g = group; g; g &= g - 1, ++k) {
                const int l = __builtin_ctzll(g);
                float rec[8];
                C pc[6];
#pragma unroll
                for (int q = 0; q < 8; ++q) rec[q] = w->orec[l * 8 + q];
#pragma unroll
                for (int q = 0; q < 6; ++q) pc[q] = w->ocov[l * kOwnCov<C> + q];
                const float4 oa = make_float4(rec[0], rec[1], rec[2], rec[3]);
                const float4 ob = make_float4(rec[4], rec[5], rec[6], rec[7]);
                const bool mine = ln >> 3 == k;
                uint64_t kth = readlane64(L.best, 8 * k + MC - 1);
#pragma unroll
                for (int q = 0; q < kScanBatch; ++q) {
                    float c2f = 0.0f;
                    bool ok = bix[q] >= 0 && window_test<T>(oa, ob, r0[q], r1[q]);
                    if (ok) ok = chi2_test<T, C, U>(oa, ob, pc, r0[q], r1[q], cut, &L.tests, &c2f);
                    const int n_ok = __popcll(__ballot(ok));
                    L.count += mine ? n_ok : 0;
                    uint64_t e = ok ? child_key(c2f, __float_as_int(r1[q].w)) : ~0ull;
                    // the best remaining hit, by its key's high word (by the low one
                    // among equals), until none is below the last entry
                    while (__ballot(e < kth)) {
                        const uint32_t hi = wave_min_u32((uint32_t)(e >> 32), wlanes);
                        uint64_t at = __ballot((uint32_t)(e >> 32) == hi);
                        if (at & (at - 1)) {
                            const uint32_t lo = wave_min_u32((uint32_t)(e >> 32) == hi ? (uint32_t)e : ~0u, wlanes);
                            at = __ballot((uint32_t)(e >> 32) == hi && (uint32_t)e == lo);
                        }
                        const int from = __builtin_ctzll(at);
                        const uint64_t ee = readlane64(e, from);
                        const int e_bi = __builtin_amdgcn_readlane(bix[q], from);
                        // the lane before's entry (a list's first: below everything)
                        uint64_t up = lane_before64(L.best);
                        up = (ln & 7) ? up : 0;
                        const int up_bi = __builtin_amdgcn_update_dpp(0, L.bi, 0x111, 0xf, 0xf, false);
                        const bool here = mine && ee < L.best, before = ee < up;
                        L.best = here ? (before ? up : ee) : L.best;
                        L.bi = here ? (before ? up_bi : e_bi) : L.bi;
                        kth = readlane64(L.best, 8 * k + MC - 1);
                        if (ln == from) e = ~0ull;
                    }
                }
            }
        }
        wave_fence();                       // the queue is rewritten next
    }
    return L;
}

// waves per SIMD the register allocation is held to (a build-time tuning knob)
#ifndef KF_FIND_WAVES
#define KF_FIND_WAVES 2
#endif

template <typename T, typename C, typename U, bool LEARN, bool MAT, bool STEER, bool FIELD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KF_FIND_WAVES))) void find_kernel(
    FindArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int W = blockDim.x;
    const int S = a.seeds_per_tile;
    const int MC = a.prm.max_cands;
    const int SPW = seeds_per_wave(W, MC);
    const int nl = a.n_layers;
    // seeds and outputs are stored in T; in registers a candidate's state is
    // held in T and its covariance in C (the update runs in U)
    const T* scov = (const T*)a.scov;
    T* ocov = (T*)a.ocov;
    const int nw = (W + 63) / 64;
    const int t = threadIdx.x;
    FindLayer* layers = (FindLayer*)smem;
    void* nav_mem = smem + sizeof(FindLayer) * nl;
    WaveLds<C>& w = ((WaveLds<C>*)(smem + find_layers_bytes(nl)))[t >> 6];
    int nbarrel = 0;
    for (int l = 0; l < nl; ++l) nbarrel += a.layers[l].kind == 0 ? 1 : 0;
    for (int l = t; l < ((nl + 3) & ~3); l += W) {
        nav_place(a.layers, nl, l, nav_mem);
        if (l < nl) {
            const kf_layer L = a.layers[l];
            FindLayer f{};
            f.r_or_z = float(L.r_or_z);
            f.lo = float(L.lo);
            f.hi = float(L.hi);
            f.x0 = float(L.x0);
            f.win_su = float(L.win_su);
            f.win_sv = float(L.win_sv);
            f.kind = L.kind;
            f.nbin_phi = L.nbin_phi;
            f.nbin_2 = L.nbin_2;
            f.base = a.bl.base[l];
            layers[l] = f;
        }
    }
    const NavOrder nav = nav_view(nav_mem, nl, nbarrel);
    __syncthreads();
    // From here on the workgroup's waves never meet: a wave takes its own tiles
    // and its lanes exchange through LDS and shuffles under wave-level fences,
    // so that no wave waits for another's step and no step waits, as a
    // workgroup barrier does, for its stores (the back-pointers) to be
    // acknowledged.
    const int ln64 = t & 63;
    const int s_loc = ln64 / MC;            // seed within the wave's tile
    const int slot = ln64 % MC;
    const bool lane_ok = s_loc < SPW;
    const int lbase = ln64 - slot;          // lane of this seed's slot 0
    const T kb = T(kKappa) * T(a.prm.bz);
    const float cut = float(a.prm.chi2_cut);
    unsigned n_prop = 0, n_upd = 0, n_chi2 = 0, n_kept = 0;   // per lane: far below 2^32
    int n_newton = 0, n_disk = 0, n_guess = 0, n_fallback = 0;
    int2* bp_base = a.bp + ((size_t)blockIdx.x * nw + (t >> 6)) * nl * S * kMaxCands;

    // The processing order is split into kQueues contiguous ranges of whole
    // tiles, one per XCD (workgroups are dispatched to the XCDs round-robin), so
    // that a range's neighbouring eta-phi tiles share that XCD's L2.  A range's
    // costliest-class seeds, at its head, come in tiles of SL seeds, the rest in
    // tiles of S.  The waves of a range's workgroups take its first tiles by
    // their place, the others from the range's counter (one cache line each),
    // and a wave whose range is exhausted takes tiles from the others; no
    // counter is touched for a range whose tiles are all taken by place.
    const int64_t cs = (int64_t)((a.n_tiles + kQueues - 1) / kQueues) * S;
    const int SL = looper_tile_seeds(S);
    const int home = blockIdx.x % kQueues;
    bool first = true;
    for (;;) {
        int tstart = -1, tcount = 0;
        if (ln64 == 0) {
            for (int d = 0; d < kQueues; ++d) {
                const int q = (home + d) % kQueues;
                const int64_t lo = q * cs;
                const int64_t hi = lo + cs < a.n_seeds ? lo + cs : a.n_seeds;
                if (lo >= hi) continue;
                const int nq = (int)(hi - lo);
                int c0 = a.queue_loopers[q];
                c0 = c0 < 0 ? 0 : (c0 > nq ? nq : c0);
                const int nlt = (c0 + SL - 1) / SL;
                const int ntq = nlt + (nq - c0 + S - 1) / S;
                // waves at home in this range, and the tile of this one's place
                const int placed = ((int)gridDim.x - q + kQueues - 1) / kQueues * nw;
                int i = ((int)blockIdx.x / kQueues) * nw + (t >> 6);
                if (!(first && d == 0)) {
                    if (placed >= ntq) continue;
                    i = placed + atomicAdd(&a.tile_counter[q * kQueueStride], 1);
                }
                if (i < nlt) {
                    tstart = (int)lo + i * SL;
                    tcount = c0 - i * SL < SL ? c0 - i * SL : SL;
                    break;
                }
                const int64_t j0 = c0 + (int64_t)(i - nlt) * S;   // first seed of a full tile
                if (j0 < nq) {
                    tstart = (int)(lo + j0);
                    tcount = nq - j0 < S ? (int)(nq - j0) : S;
                    break;
                }
            }
        }
        first = false;
        tstart = __builtin_amdgcn_readfirstlane(tstart);
        tcount = __builtin_amdgcn_readfirstlane(tcount);
        if (tstart < 0) break;

        const bool valid = lane_ok && s_loc < tcount;
        const int sid = valid ? a.order[tstart + s_loc] : 0;
        int ev = valid ? a.seed_event[sid] : 0;
        const bool bad_event = ev < 0 || ev >= a.n_events;
        if (bad_event) ev = 0;
        // candidate registers
        T p[6];
        C P[21];
        float chi2 = 0.0f;
        int nhits = 0, misses = 0;
        uint32_t status = 0;
        bool occupied = valid && slot == 0;
        bool done = true;
        if (occupied) {
#pragma unroll
            for (int k = 0; k < 6; ++k) p[k] = T(a.spar[k * a.sld + sid]);
#pragma unroll
            for (int k = 0; k < 21; ++k) P[k] = C(scov[k * a.sld + sid]);
            chi2 = a.schi2[sid];
            nhits = (a.sndf[sid] + 5) / 2;
            status = a.sstatus[sid] | (bad_event ? (uint32_t)KF_ST_BADINPUT : 0u);
            done = (status & kFreezeMask) != 0;
        } else {
#pragma unroll
            for (int k = 0; k < 6; ++k) p[k] = T(0);
#pragma unroll
            for (int k = 0; k < 21; ++k) P[k] = C(0);
        }
        if (ln64 == 0) w.finite = 1;
        wave_fence();
        if (!all_finite(P)) w.finite = 0;
        wave_fence();
        // steering: the seed's region and the plan entry after its last seed
        // layer (every lane of the seed computes the same)
        int rg = 0, pos = 0;
        if constexpr (STEER) {
            if (valid) {
                const double eta = -log(tan(0.5 * (double)a.spar[5 * a.sld + sid]));
                rg = -1;
                for (int g = 0; g < a.steer->n; ++g)
                    if (eta >= a.steer->eta_lo[g] && eta < a.steer->eta_hi[g]) {
                        rg = g;
                        break;
                    }
                int start = -1;
                if (rg >= 0) {
                    for (int q = 0; q < 3; ++q) {
                        const int hi = a.seed_hits[q * a.sld + sid];
                        if (hi < 0 || hi >= a.n_hits) continue;
                        const int hl = a.hit_layer[hi];
                        for (int j = 0; j < a.steer->len[rg]; ++j)
                            if (a.steer->layers[rg][j] == hl && j + 1 > start) start = j + 1;
                    }
                }
                if (start < 0) {
                    if (occupied && !done) {
                        status |= KF_ST_UNREACHABLE;
                        done = true;
                    }
                    rg = 0;
                    start = 0;
                }
                pos = start;
            }
        }
        int nsteps = 0;
        for (int step = 0; step < nl; ++step) {
            const bool live = occupied && !done;
            if (__ballot(live) == 0) break;
            // ---- a3: navigate and propagate (LEARN: the whole wave first
            // evaluates the learned start of its candidates' barrel solves)
            T s_guess = T(-1);
            if (LEARN) {
                float f[kMlpIn] = {0, 0, 0, 0, 0, 0, 0, 0};
                const int bl = live ? next_barrel(p, nav) : -1;
                if (bl >= 0) mlp_features(p, layers[bl], a.prm, f);
                const float y = mlp_wave(a.mlp, f, __ballot(bl >= 0));
                if (bl >= 0) {
                    s_guess = T(mlp_guess(f, y));
                    ++n_guess;
                }
            }
            int pl = -1;
            if (live) {
                T s;
                int layer;
                T sth = T(0), cth = T(0);     // theta stays along the helix
                if constexpr (!FIELD) Tr<T>::sincos_(p[5], &sth, &cth);
                T fl = T(0);
                T fq[6];
                if constexpr (FIELD && STEER)
                    layer = steer_next_field(p, layers, a.steer->layers[rg], a.steer->len[rg], &pos,
                                             a.prm, &fl, fq, &status, &n_newton, &n_disk);
                else if constexpr (FIELD)
                    layer = navigate_field(p, layers, nl, a.prm, &fl, fq, &status, &n_newton,
                                           &n_disk, s_guess >= T(0) ? s_guess / Tr<T>::sin_(p[5]) : T(-1),
                                           LEARN ? a.prm.mlp_max_iter : 0, &n_fallback);
                else if constexpr (STEER)
                    layer = steer_next(p, layers, a.steer->layers[rg], a.steer->len[rg], &pos,
                                       a.prm, kb, sth, cth, &s, &status, &n_newton, &n_disk);
                else
                    layer = navigate(p, layers, nav, a.prm, kb, sth, cth, &s, &status, &n_newton,
                                     &n_disk, s_guess, LEARN ? a.prm.mlp_max_iter : 0, &n_fallback);
                if (layer < 0) {
                    done = true;
                } else {
                    ++n_prop;
                    const FindLayer L = layers[layer];
                    if constexpr (FIELD)
                        field_transport(p, P, fq, fl, a.prm, L.kind, T(L.r_or_z),
                                        w.finite != 0);
                    else
                        transport(p, P, s, kb, L.kind, T(L.r_or_z), sth, cth,
                                  w.finite != 0);
                    if (a.material) {
                        if constexpr (MAT)
                            add_material(p, P, L, a.mat, T(a.prm.mass));
                        else if constexpr (FIELD)
                            add_scatter(p, P, L.kind, T(L.x0), T(a.prm.mass));
                        else
                            add_scatter(p, P, L.kind, T(L.x0), T(a.prm.mass), sth, cth);
                    }
                    bool fin = true;
#pragma unroll
                    for (int k = 0; k < 6; ++k) fin &= isfinite(p[k]);
                    if (fin) {
                        pl = layer;
                    } else {
                        status |= KF_ST_NAN;
                        done = true;
                    }
                }
            }
            // ---- a4: hit-search window, then the window's bins scanned by the
            // whole wave together.  Per-candidate windows differ widely (a diffuse
            // state can cover many rows of bins), so lanes queue their rows and
            // the wave walks the flattened (row, hit) list 64 x kScanBatch hits at
            // a time; accepted hits are compacted with a ballot and each owner
            // lane inserts its own into its sorted list.
            if (lane_ok) {
#pragma unroll
                for (int k = 0; k < 3; ++k) w.orec[ln64 * 8 + k] = float(p[k]);
                C* oc = w.ocov + ln64 * kOwnCov<C>;
                oc[0] = P[pk(0, 0)];
                oc[1] = P[pk(0, 1)];
                oc[2] = P[pk(0, 2)];
                oc[3] = P[pk(1, 1)];
                oc[4] = P[pk(1, 2)];
                oc[5] = P[pk(2, 2)];
#pragma unroll
                for (int k = 0; k < kPark; ++k) w.park[k * 64 + ln64] = P[parked(k)];
            }
            // this candidate's accepted hits, best first: key and binned index
            uint64_t lk[kMaxCands];
            int32_t lbi[kMaxCands];
#pragma unroll
            for (int k = 0; k < kMaxCands; ++k) {
                lk[k] = ~0ull;
                lbi[k] = -1;
            }
            int nacc = 0;
            int nrow = 0, row_lo = 0, v0 = 0, v1 = 0, np = 1, n2 = 1, row0 = 0;
            if (pl >= 0) {
                const FindLayer L = layers[pl];
                const Window<T> Wn = make_window<T, C>(p, P, L, T(cut));
                if (Wn.ok) {
                    np = L.nbin_phi;
                    n2 = L.nbin_2;
                    int b_lo = 0, b_hi = np - 1;
                    if (!Wn.all_phi) {
                        const T phi = Tr<T>::atan2_(p[1], p[0]);
                        b_lo = (int)Tr<T>::floor_((phi - Wn.dphi + T(kPi)) * T(np) / T(2.0 * kPi));
                        b_hi = (int)Tr<T>::floor_((phi + Wn.dphi + T(kPi)) * T(np) / T(2.0 * kPi));
                        if (b_hi - b_lo + 1 >= np || b_hi < b_lo) {
                            b_lo = 0;
                            b_hi = np - 1;
                        }
                    }
                    nrow = b_hi - b_lo + 1;
                    row_lo = b_lo;
                    v0 = coord_bin_of(float(Wn.vlo), float(L.lo), float(L.hi), n2);
                    v1 = coord_bin_of(float(Wn.vhi), float(L.lo), float(L.hi), n2);
                    row0 = (int)((uint32_t)ev * (uint32_t)a.bl.per_event + (uint32_t)L.base);
                    const T rho = Tr<T>::sqrt_(p[0] * p[0] + p[1] * p[1]);
                    w.orec[ln64 * 8 + 3] = float(p[0] / rho);
                    w.orec[ln64 * 8 + 4] = float(p[1] / rho);
                    w.orec[ln64 * 8 + 5] = float(Wn.sin_dphi);
                    w.orec[ln64 * 8 + 6] = float(Wn.wv);
                    w.orec[ln64 * 8 + 7] = __int_as_float((Wn.all_phi ? 1 : 0) | (L.kind << 1));
                }
            }
            {
                const int ln = ln64;
                const int wlanes = W < 64 ? W : 64;
                int32_t* sg_own = w.seg;
                int32_t* sg_h0 = sg_own + kSeg;
                int32_t* sg_len = sg_h0 + kSeg;
                int32_t* sg_pre = w.segpre;
                // accepted hits are compacted in hit order, and the flattened hits
                // run owner by owner, so each owner's accepted hits of a round form
                // one range [ac_first, ac_last]
                int32_t* ac_first = w.acc;
                int32_t* ac_last = ac_first + 64;
                int32_t* ac_id = ac_first + kAcc;
                int32_t* ac_bi = ac_id + kAcc;
                float* ac_c2 = w.accc2;
                const int segcap = 2 * wlanes < kSeg ? 2 * wlanes : kSeg;
                // (0) windows of kLongBins bins or more, first: the candidates of one
                // seed on one layer look at nearly the same hits, so the union of
                // their windows is read once, 64 consecutive hits at a time, and
                // every hit is tested against each of them.  Their best hits are
                // sorted lists over eight lanes each, which a hit enters at once, and
                // only the hits below a list's last entry do, best first.  A few
                // low-pT seeds of a large event test 30,000 to 60,000 hits; by the
                // queue below their hits are loaded once per candidate, 256 at a
                // time and waited for, and inserted one by one by the owner lane,
                // and the longest such seed ends the pass (times at kLongBins).
                // Steered kernels keep to the queue, which their plans' shorter
                // windows seldom fill: 24 events 661 us with the call, 649 without.
                uint64_t longs = 0;
                if constexpr (!STEER) longs = __ballot(pl >= 0 && (int64_t)nrow * (v1 - v0 + 1) >= kLongBins);
                if (__builtin_expect_with_probability(longs != 0, 0, 0.999))
                while (longs) {
                    const int o = __builtin_ctzll(longs);
                    const int o_pl = __builtin_amdgcn_readlane(pl, o);
                    const int o_base = __builtin_amdgcn_readlane(lbase, o);
                    // the group: this seed's long windows on this layer, eight lanes each
                    uint64_t group = longs & __ballot(pl == o_pl && lbase == o_base);
                    while (__popcll(group) > wlanes / 8) group &= ~(1ull << (63 - __builtin_clzll(group)));
                    longs &= ~group;
                    int u_lo = 0x7fffffff, u_hi = -0x7fffffff, u_v0 = 0x7fffffff, u_v1 = 0;
                    for (uint64_t g = group; g; g &= g - 1) {
                        const int l = __builtin_ctzll(g);
                        const int r_lo = __builtin_amdgcn_readlane(row_lo, l);
                        const int r_hi = r_lo + __builtin_amdgcn_readlane(nrow, l) - 1;
                        const int b0 = __builtin_amdgcn_readlane(v0, l), b1 = __builtin_amdgcn_readlane(v1, l);
                        u_lo = r_lo < u_lo ? r_lo : u_lo;
                        u_hi = r_hi > u_hi ? r_hi : u_hi;
                        u_v0 = b0 < u_v0 ? b0 : u_v0;
                        u_v1 = b1 > u_v1 ? b1 : u_v1;
                    }
                    const int o_np = __builtin_amdgcn_readlane(np, o), o_n2 = __builtin_amdgcn_readlane(n2, o);
                    const int o_row0 = __builtin_amdgcn_readlane(row0, o);
                    int u_rows = u_hi - u_lo + 1;
                    if (u_rows >= o_np || u_rows <= 0) {
                        u_lo = 0;
                        u_rows = o_np;
                    }
                    const LongList ll = long_scan<T, C, U>(
                        (LdsPtr<C>)(&w), a.bh, a.bin_off, group, u_lo, u_rows, u_v0, u_v1, o_np, o_n2, o_row0,
                        MC, wlanes, cut);
                    n_chi2 += ll.tests;
                    int k = 0;
                    for (uint64_t g = group; g; g &= g - 1, ++k) {
                        const int l = __builtin_ctzll(g);
                        const int n_acc = __builtin_amdgcn_readlane(ll.count, 8 * k);
                        if (ln == l) {
                            nacc = n_acc;
                            nrow = 0;                       // nothing left for the queue
                        }
#pragma unroll
                        for (int q = 0; q < kMaxCands; ++q) {
                            const uint64_t x = readlane64(ll.best, 8 * k + q);
                            const int z = __builtin_amdgcn_readlane(ll.bi, 8 * k + q);
                            lk[q] = ln == l ? x : lk[q];
                            lbi[q] = ln == l ? z : lbi[q];
                        }
                    }
                }
                // rows of every lane, flattened: lane o owns rows [rowpre[o],
                // rowpre[o] + nrow_o) of the wave's row list
                ac_first[ln] = 0x7fffffff;
                ac_last[ln] = -1;
                int R = 0;
                const int rpre = wave_scan(nrow, wlanes, &R);
                // the row parameters of each owner, for the lanes that expand its rows
                int32_t* rw_par = w.rowp;
                rw_par[ln] = rpre;
                rw_par[64 + ln] = row_lo;
                rw_par[128 + ln] = v0 | (v1 << 16);
                rw_par[192 + ln] = row0;
                rw_par[256 + ln] = np | (n2 << 16);
                wave_fence();
                for (int rr0 = 0; rr0 < R; rr0 += segcap) {
                    // (1) queue rows rr0 .. rr0 + segcap - 1, two per lane; their bin
                    //     ranges are loaded together
                    const int nseg = R - rr0 < segcap ? R - rr0 : segcap;
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const int j = r * wlanes + ln;
                        if (j < nseg) {
                            const int g = rr0 + j;
                            int lo = 0, hi = wlanes;      // rowpre[lo] <= g < rowpre[hi]
                            while (hi - lo > 1) {
                                const int mid = (lo + hi) >> 1;
                                if (rw_par[mid] <= g) lo = mid;
                                else hi = mid;
                            }
                            const int o = lo;
                            const int bb = rw_par[64 + o] + (g - rw_par[o]);
                            const int vv = rw_par[128 + o], pp = rw_par[256 + o];
                            const int onp = pp & 0xFFFF, on2 = pp >> 16;
                            const uint32_t rb = (uint32_t)rw_par[192 + o] + (uint32_t)((((bb % onp) + onp) % onp) * on2);
                            const int h0 = a.bin_off[rb + (vv & 0xFFFF)];
                            const int h1 = a.bin_off[rb + (vv >> 16) + 1];
                            sg_own[j] = o;
                            sg_h0[j] = h0;
                            sg_len[j] = h1 - h0;
                        }
                    }
                    wave_fence();
                    // (2) prefix of the queued rows' hit counts, two rows per lane
                    const int H = row_prefix(sg_len, sg_pre, nseg, wlanes);
                    // (3) the flattened hits, 64 x kScanBatch per round.  Lane ln
                    //     walks its own contiguous segment of the list, kScanBatch
                    //     hits per round, so that a round holds hits of many owners
                    //     and their insertions below run side by side.  Owners
                    //     still rise with the lane, so a round's accepted hits of
                    //     one owner stay one range of the compaction.
                    const int nround = (H + wlanes * kScanBatch - 1) / (wlanes * kScanBatch);
                    const int gseg = ln * kScanBatch * nround;   // first hit of the segment
                    // the lane's current row, held in registers: its end in the
                    // list, owner, and binned index minus list position
                    int row = 0, r_end = H, r_own = -1, r_base = 0;
                    if (gseg < H) {
                        int hi = nseg;                            // sg_pre[row] <= gseg < sg_pre[hi]
                        while (hi - row > 1) {
                            const int mid = (row + hi) >> 1;
                            if (sg_pre[mid] <= gseg) row = mid;
                            else hi = mid;
                        }
                        r_end = sg_pre[row + 1];
                        r_own = sg_own[row];
                        r_base = sg_h0[row] - sg_pre[row];
                    }
                    for (int ir = 0; ir < nround; ++ir) {
                        float4 r0[kScanBatch], r1[kScanBatch];
                        int own[kScanBatch], bix[kScanBatch];
                        const int gb = gseg + ir * kScanBatch;
#pragma unroll
                        for (int q = 0; q < kScanBatch; ++q) {
                            const int g = gb + q;
                            own[q] = -1;
                            bix[q] = 0;
                            if (g < H) {
                                while (g >= r_end) {                 // sg_pre[nseg] = H > g
                                    ++row;
                                    r_end = sg_pre[row + 1];
                                    r_own = sg_own[row];
                                    r_base = sg_h0[row] - sg_pre[row];
                                }
                                own[q] = r_own;
                                bix[q] = r_base + g;
                            }
                            r0[q] = *(const float4*)&a.bh[bix[q]].x;
                            r1[q] = *(const float4*)&a.bh[bix[q]].sv;
                        }
                        bool okq[kScanBatch];
                        float c2q[kScanBatch];
#pragma unroll
                        for (int q = 0; q < kScanBatch; ++q) {
                            bool ok = false;
                            float c2f = 0.0f;
                            const int o = own[q];
                            if (o >= 0) {
                                const float4 oa = *(const float4*)&w.orec[o * 8];
                                const float4 ob = *(const float4*)&w.orec[o * 8 + 4];
                                if (window_test<T>(oa, ob, r0[q], r1[q])) {
                                    C pc[6];
                                    load_owner_cov(w.ocov + o * kOwnCov<C>, pc);
                                    ok = chi2_test<T, C, U>(oa, ob, pc, r0[q], r1[q], cut, &n_chi2, &c2f);
                                }
                            }
                            okq[q] = ok;
                            c2q[q] = c2f;
                        }
                        // compaction in hit order (lane-major: a lane's hits are
                        // consecutive), each entry widening its owner's range
                        int nok = 0;
#pragma unroll
                        for (int q = 0; q < kScanBatch; ++q) nok += okq[q] ? 1 : 0;
                        // exclusive prefix of nok (< 8) over the lanes, bit by bit
                        static_assert(kScanBatch < 8, "nok takes three bits");
                        int pos = 0;
#pragma unroll
                        for (int b = 0; b < 3; ++b) {
                            const uint64_t m = __ballot((nok >> b) & 1);
                            pos += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))
                                   << b;
                        }
#pragma unroll
                        for (int q = 0; q < kScanBatch; ++q)
                            if (okq[q]) {
                                ac_id[pos] = __float_as_int(r1[q].w);
                                ac_bi[pos] = bix[q];
                                ac_c2[pos] = c2q[q];
                                atomicMin(&ac_first[own[q]], pos);
                                atomicMax(&ac_last[own[q]], pos);
                                ++pos;
                            }
                        wave_fence();
                        // (4) owners take their accepted hits; one that cannot enter
                        // the sorted list (not below its last entry) is only counted
                        const int j1 = ac_last[ln];
                        for (int jb = ac_first[ln]; jb <= j1; jb += kInsBatch) {
                            // the batch's entries are loaded together
                            float cb[kInsBatch];
                            int32_t ib[kInsBatch], bb[kInsBatch];
#pragma unroll
                            for (int u = 0; u < kInsBatch; ++u) {
                                const int j = jb + u <= j1 ? jb + u : j1;
                                cb[u] = ac_c2[j];
                                ib[u] = ac_id[j];
                                bb[u] = ac_bi[j];
                            }
#pragma unroll
                            for (int u = 0; u < kInsBatch; ++u) {
                                if (jb + u > j1) break;
                                uint64_t e = child_key(cb[u], ib[u]);
                                int32_t bi = bb[u];
                                ++nacc;
                                if (!(e < lk[kMaxCands - 1])) continue;
                                // the list is ascending, so "e below entry q" holds
                                // from the insertion point on: every slot takes
                                // its own, its predecessor's or the new entry,
                                // all decided from the old entries at once
                                bool lt[kMaxCands];
#pragma unroll
                                for (int q = 0; q < kMaxCands; ++q) lt[q] = e < lk[q];
#pragma unroll
                                for (int q = kMaxCands - 1; q > 0; --q) {
                                    lk[q] = lt[q] ? (lt[q - 1] ? lk[q - 1] : e) : lk[q];
                                    lbi[q] = lt[q] ? (lt[q - 1] ? lbi[q - 1] : bi) : lbi[q];
                                }
                                lk[0] = lt[0] ? e : lk[0];
                                lbi[0] = lt[0] ? bi : lbi[0];
                            }
                        }
                        ac_first[ln] = 0x7fffffff;
                        ac_last[ln] = -1;
                        wave_fence();
                    }
                    // the queue is rewritten next round: every lane is done reading it
                    wave_fence();
                }
            }
            // ---- a5: per-seed selection.  The candidates of a seed write their
            // children's merge keys (all different) into one list in LDS: each its
            // accepted hits, best first, and the child without a hit.  The seed's
            // lanes then take the list's keys in turn, and a key's rank is the
            // number of smaller ones in the list; ranks below max_cands survive.
            // (One lane merging its seed's sorted lists waits on LDS for every
            // pick; every lane comparing its own keys with all places of the other
            // lanes' lists mostly compares with empty places.)
            const int nk = nacc < MC ? nacc : MC;       // hit children
            wave_fence();                               // the scan's LDS is free
            if (lane_ok) w.sel[s_loc * MC + slot] = ~0ull;
            int n_key, n_key_max;      // the seed's keys, and the most of any seed of the wave
            {
                // where this candidate's keys start: the counts (at most
                // kMaxCands + 1, so four bits) of the seed's lower slots
                const int cnt = occupied ? nk + 1 : 0;
                const uint64_t lower = lane_ok ? ((1ull << slot) - 1) << lbase : 0;
                const uint64_t mine = lane_ok ? ((1ull << MC) - 1) << lbase : 0;
                int at = 0;
                n_key = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const uint64_t m = __ballot((cnt >> b) & 1);
                    at += __popcll(m & lower) << b;
                    n_key += __popcll(m & mine) << b;
                }
                n_key_max = 0;
                while (__ballot(n_key > n_key_max)) n_key_max += 4;
                uint64_t* keys = w.key + s_loc * MC * (MC + 1);
                if (occupied) {
#pragma unroll
                    for (int c = 0; c < kMaxCands; ++c)
                        if (c < nk) {
                            keys[at + c] = merge_key(nhits + 1, chi2 + child_key_chi2(lk[c]), slot, c);
                            w.cbidx[c * 64 + ln64] = lbi[c];
                        }
                    keys[at + nk] = merge_key(nhits, chi2, slot, nk);
                }
                wave_fence();
                constexpr int kOwn = 3;                 // keys a lane ranks at once
                for (int i0 = slot; __ballot(lane_ok && i0 < n_key); i0 += kOwn * MC) {
                    uint64_t own[kOwn];
                    int rank[kOwn];
#pragma unroll
                    for (int u = 0; u < kOwn; ++u) {
                        const int i = i0 + u * MC;
                        own[u] = lane_ok && i < n_key ? keys[i] : 0ull;
                        rank[u] = 0;
                    }
                    for (int j = 0; j < n_key_max; j += 4) {
                        uint64_t k2[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) k2[v] = j + v < n_key ? keys[j + v] : ~0ull;
#pragma unroll
                        for (int v = 0; v < 4; ++v)
#pragma unroll
                            for (int u = 0; u < kOwn; ++u) rank[u] += k2[v] < own[u] ? 1 : 0;
                    }
#pragma unroll
                    for (int u = 0; u < kOwn; ++u)
                        if (lane_ok && i0 + u * MC < n_key && rank[u] < MC) w.sel[s_loc * MC + rank[u]] = own[u];
                }
            }
            wave_fence();
            // ---- a6: materialise the surviving children (Kalman update for hit
            // children).  A child copies its parent's predicted state from the
            // parent's registers (same wave); every lane takes part in the copy.
            int sel_j = 0, sel_c = 0, src = ln64;
            bool occ_new = false;
            uint64_t sel_key = ~0ull;
            if (valid) {
                sel_key = w.sel[s_loc * MC + slot];
                occ_new = sel_key != ~0ull;
                if (occ_new) {
                    sel_j = (int)(sel_key >> 16) & 0xFF;
                    sel_c = (int)(sel_key >> 8) & 0xFF;
                    src = lbase + sel_j;
                }
            }
            {
                // position and its covariance from the parent's owner record, the
                // parked entries, and the rest from its registers
                C pc[6];
                load_owner_cov(w.ocov + src * kOwnCov<C>, pc);
                const float4 x = *(const float4*)&w.orec[src * 8];
                p[0] = T(x.x);
                p[1] = T(x.y);
                p[2] = T(x.z);
#pragma unroll
                for (int k = 3; k < 6; ++k) p[k] = __shfl(p[k], src);
                P[pk(0, 0)] = pc[0];
                P[pk(0, 1)] = pc[1];
                P[pk(0, 2)] = pc[2];
                P[pk(1, 1)] = pc[3];
                P[pk(1, 2)] = pc[4];
                P[pk(2, 2)] = pc[5];
#pragma unroll
                for (int k = 0; k < kPark; ++k) P[parked(k)] = w.park[k * 64 + src];
                P[pk(2, 5)] = __shfl(P[pk(2, 5)], src);
#pragma unroll
                for (int k = pk(3, 3); k < 21; ++k) P[k] = __shfl(P[k], src);
            }
            nhits = __shfl(nhits, src);
            misses = __shfl(misses, src);
            status = __shfl(status, src);
            // the parent's outcome: done, its layer + 1, its hit children, its plan position
            const int m3 = __shfl((done ? 1 : 0) | ((pl + 1) << 1) | (nk << 8) | (pos << 16), src);
            if (valid) {
                occupied = occ_new;
                int2 bpe = make_int2(-1, 0xFF00);
                if (occupied) {
                    const int j = sel_j;
                    const int c = sel_c;
                    // the child's chi2, with its hit's where it has one
                    chi2 = merge_key_chi2(sel_key);
                    done = (m3 & 1) != 0;
                    const int ppl = ((m3 >> 1) & 0x7F) - 1;
                    if constexpr (STEER) pos = (m3 >> 16) & 0xFF;
                    if (ppl >= 0) {
                        ++n_kept;
                        if (c < ((m3 >> 8) & 0xFF)) {
                            const int bi = w.cbidx[c * 64 + lbase + j];
                            const BinnedHit hh = a.bh[bi];
                            HitFrame<U> f;
                            f.hx = U(hh.x);
                            f.hy = U(hh.y);
                            f.hz = U(hh.z);
                            f.c = U(hh.cphi);
                            f.s = U(hh.sphi);
                            f.vu = U(hh.su) * U(hh.su);
                            f.vv = U(hh.sv) * U(hh.sv);
                            U c2 = U(0);
                            const int r = kf_update<T, C, U>(p, P, f, layers[ppl].kind, &c2);
                            ++n_upd;
                            if (r) {
                                status |= (uint32_t)r;
                                done = true;
                            }
                            nhits += 1;
                            misses = 0;
                            bpe = make_int2(hh.idx, j | (ppl << 8));
                        } else {
                            misses += 1;
                            if (misses > a.prm.max_miss) done = true;
                            bpe = make_int2(-1, j | (ppl << 8));
                        }
                    } else {
                        bpe = make_int2(-1, j | 0xFF00);
                    }
                    bp_base[((size_t)step * S + s_loc) * kMaxCands + slot] = bpe;
                }
            }
            // (the next step's LDS writes come after every lane's reads above)
            wave_fence();
            ++nsteps;
        }
        // ---- a7: best candidate (slot 0, candidates are kept sorted) and its hit list.
        // A layer visited more than once (a looper curling back) reports its
        // latest hit: the back-pointers are walked from the last step and the
        // first hit met per layer is kept, then the seed hits where nothing came
        // later.  Each lane loads the entries that its own slot wrote, several
        // steps at once, and the walk follows the chain by shuffles; the layers
        // already filled are a bit mask.  (One lane would chase the entries and the
        // filled layers through memory, a round trip each.)
        {
            int32_t* oh = a.out_hits + (int64_t)sid * nl;
            if (valid)
                for (int l = slot; l < nl; l += MC) oh[l] = -1;
            int32_t sh_hit[3], sh_lay[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                sh_hit[q] = valid ? a.seed_hits[q * a.sld + sid] : -1;
                const bool in = sh_hit[q] >= 0 && sh_hit[q] < a.n_hits;
                sh_lay[q] = in ? a.hit_layer[sh_hit[q]] : -1;
            }
            wave_fence();                       // the -1s come before the hits
            uint64_t seen = 0;
            int k = 0;
            constexpr int kWalk = 4;            // steps loaded at once
            for (int s1 = nsteps; s1 > 0; s1 -= kWalk) {
                int2 e[kWalk];
#pragma unroll
                for (int u = 0; u < kWalk; ++u) {
                    const int st = s1 - 1 - u;
                    e[u] = make_int2(-1, 0xFF00);
                    if (valid && st >= 0) e[u] = bp_base[((size_t)st * S + s_loc) * kMaxCands + slot];
                }
#pragma unroll
                for (int u = 0; u < kWalk; ++u) {
                    if (s1 - 1 - u < 0) break;
                    const int from = lbase + k;
                    const int ex = __shfl(e[u].x, from), ey = __shfl(e[u].y, from);
                    const int lay = (ey >> 8) & 0xFF;
                    if (valid && ex >= 0 && lay < nl && !((seen >> lay) & 1)) {
                        seen |= 1ull << lay;
                        if (slot == 0) oh[lay] = ex;
                    }
                    k = ey & 0xFF;
                }
            }
#pragma unroll
            for (int q = 2; q >= 0; --q) {
                const int hl = sh_lay[q];
                if (valid && hl >= 0 && hl < nl && !((seen >> hl) & 1)) {
                    seen |= 1ull << hl;
                    if (slot == 0) oh[hl] = sh_hit[q];
                }
            }
        }
        if (valid && slot == 0) {
#pragma unroll
            for (int q = 0; q < 6; ++q) a.opar[q * a.old + sid] = float(p[q]);
#pragma unroll
            for (int q = 0; q < 21; ++q) ocov[q * a.old + sid] = T(P[q]);
            a.ochi2[sid] = chi2;
            a.ondf[sid] = 2 * nhits - 5;
            a.ostatus[sid] = status;
        }
    }
    if (a.counters) {
        // wave-level reduction of the per-lane counts, added by one atomic
        // instruction of eight lanes (their counters share a line)
        unsigned long long c[kFindCounters] = {(unsigned long long)n_prop, (unsigned long long)n_upd,
                                               (unsigned long long)n_chi2, (unsigned long long)n_newton,
                                               (unsigned long long)n_disk, (unsigned long long)n_guess,
                                               (unsigned long long)n_fallback, (unsigned long long)n_kept};
        unsigned long long mine = 0;
#pragma unroll
        for (int q = 0; q < kFindCounters; ++q) {
            for (int o = 32; o > 0; o >>= 1) c[q] += __shfl_xor(c[q], o);
            if (ln64 == q) mine = c[q];
        }
        if (ln64 < kFindCounters && mine) atomicAdd(&a.counters[ln64], mine);
    }
}

// ------------------------------------------------------------------ host side
namespace {
inline unsigned blocks_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }
}

size_t find_shared_size(int W, int nl, int prec)
{
    return prec == KF_PREC_FP32 ? find_shared_bytes<float>(W, nl) : find_shared_bytes<double>(W, nl);
}

// Instantiations: (precision) x (plain, learned, steered; each also in the
// parametrised field) x (material map); learned and steered exclude each other.
template <typename T, typename C, typename U, bool LEARN, bool MAT>
static hipError_t find_occ2(bool steer, bool field, int W, size_t lds, int* out)
{
    if (field) {
        if constexpr (!LEARN)
            if (steer)
                return hipOccupancyMaxActiveBlocksPerMultiprocessor(
                    out, find_kernel<T, C, U, false, MAT, true, true>, W, lds);
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(out, find_kernel<T, C, U, LEARN, MAT, false, true>,
                                                            W, lds);
    }
    if constexpr (!LEARN)
        if (steer)
            return hipOccupancyMaxActiveBlocksPerMultiprocessor(
                out, find_kernel<T, C, U, false, MAT, true, false>, W, lds);
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(out, find_kernel<T, C, U, LEARN, MAT, false, false>,
                                                        W, lds);
}

template <typename T, typename C, typename U, bool LEARN>
static hipError_t find_occ(bool mat, bool steer, bool field, int W, size_t lds, int* out)
{
    return mat ? find_occ2<T, C, U, LEARN, true>(steer, field, W, lds, out)
               : find_occ2<T, C, U, LEARN, false>(steer, field, W, lds, out);
}

hipError_t find_max_blocks_per_cu(int W, int nl, int prec, bool learn, bool mat, bool steer,
                                  bool field, int* out)
{
    const size_t lds = find_shared_size(W, nl, prec);
    if (prec == KF_PREC_FP32)
        return learn ? find_occ<float, float, float, true>(mat, steer, field, W, lds, out)
                     : find_occ<float, float, float, false>(mat, steer, field, W, lds, out);
    return learn ? find_occ<float, double, double, true>(mat, steer, field, W, lds, out)
                 : find_occ<float, double, double, false>(mat, steer, field, W, lds, out);
}

hipError_t launch_fill(int32_t* p, int64_t n, int32_t v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    unsigned g = blocks_for(n, 256);
    if (g > 4096) g = 4096;
    fill_i32_kernel<<<g, 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_scan(const int32_t* in, int32_t* out, int64_t n, int32_t* bsum, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const unsigned nb = blocks_for(n, kScanChunk);
    scan_reduce_kernel<<<nb, kScanThreads, 0, s>>>(in, n, bsum);
    scan_top_kernel<<<1, 1024, 0, s>>>(bsum, (int)nb);
    scan_apply_kernel<<<nb, kScanThreads, 0, s>>>(in, n, bsum, out);
    return hipGetLastError();
}

// Shares of a layer's phi rows that level 2 sorts by themselves: on average
// half of what a workgroup's LDS holds (events differ), as long as a level-1
// workgroup can count all of an event's.
static int bin_split(int64_t n_hits, int n_events, int n_layers)
{
    const int64_t segs = (int64_t)n_events * (n_layers > 0 ? n_layers : 1);
    int64_t k = (n_hits + segs * (kSortCap / 2) - 1) / (segs * (kSortCap / 2));
    const int64_t most = kSegLocal / 2 / (n_layers > 0 ? n_layers : 1);
    k = k < most ? k : most;
    return (int)(k < 1 ? 1 : k);
}

hipError_t launch_bin(const FindPlan& pl, const kf_hits* h, const int32_t* event_off, int n_events,
                      const kf_layer* layers, const kf_layer* d_layers, int n_layers, hipStream_t s)
{
    hipError_t e;
    const HitView v{h->x, h->y, h->z, h->su, h->sv, h->layer};
    if (bin_direct(h->n, n_events, n_layers)) {
        int nb_max = 1;
        for (int l = 0; l < n_layers; ++l) {
            const int nb = layers[l].nbin_phi * layers[l].nbin_2;
            nb_max = nb > nb_max ? nb : nb_max;
        }
        // shares of a layer of kDirectShare hits on average: a workgroup's
        // gathers, a line a clock, are what the call waits for
        const int64_t segs = (int64_t)n_events * n_layers;
        int split = (int)(h->n / (segs * kDirectShare));
        split = split < 1 ? 1 : (split < kDirectSplit ? split : kDirectSplit);
        const size_t lds = sizeof(int) * ((size_t)nb_max + kBinCap);
        // an event's workgroups run on kQueues / stride of the XCDs: four for a
        // single event (56,000 hits: 27 us; 32 on two, 58 on one, where they
        // stream at once); a grid takes fewer than 2^32 threads
        int stride = n_events > 2 ? kQueues : 2 * n_events;
        int64_t grid = (int64_t)((n_events + stride - 1) / stride) * stride * n_layers * split;
        if (grid * kBinThreads > 0xffffffffLL) {
            stride = 1;
            grid = segs * split;
        }
        bin_kernel<<<(unsigned)grid, kBinThreads, lds, s>>>(v, h->n, event_off, n_events, stride, split, d_layers,
                                                            n_layers, nb_max, pl.bl, pl.hit_key,
                                                            pl.hit_bin, pl.hit_perm, pl.off,
                                                            (BinnedHit*)pl.binned);
        return hipGetLastError();
    }
    const int split = bin_split(h->n, n_events, n_layers);
    const int64_t n_seg = (int64_t)n_events * n_layers * split;
    int nb_max = 1;
    for (int l = 0; l < n_layers; ++l) {
        const int nb = share_row(1, layers[l].nbin_phi, split) * layers[l].nbin_2;   // the first share's: the most
        nb_max = nb > nb_max ? nb : nb_max;
    }
    if ((e = launch_fill(pl.seg_cnt, n_seg + 1, 0, s)) != hipSuccess) return e;
    const unsigned nchunk = blocks_for(h->n, kSegChunk);
    seg_count_kernel<<<nchunk, 256, 0, s>>>(h->n, v, event_off, n_events, d_layers, n_layers, split,
                                            pl.hit_key, pl.seg_cnt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_scan(pl.seg_cnt, pl.seg_off, n_seg + 1, pl.bsum, s)) != hipSuccess) return e;
    // (seg_cnt then counts down the places left in every segment)
    seg_scatter_kernel<<<nchunk, kSegThreads, 0, s>>>(h->n, v, event_off, n_events, n_layers * split,
                                                      pl.hit_key, pl.seg_off, pl.seg_cnt,
                                                      (StagedHit*)pl.staged);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    bin_segment_kernel<<<(unsigned)n_seg, kSortThreads, sizeof(int) * (size_t)nb_max, s>>>(
        pl.seg_off, (const StagedHit*)pl.staged, d_layers, n_layers, split, pl.bl, pl.off,
        (BinnedHit*)pl.binned);
    return hipGetLastError();
}

hipError_t launch_cost_order(const FindPlan& pl, const kf_tracks* seeds, int n_tiles,
                             int seeds_per_tile, hipStream_t s)
{
    if (seeds->n == 0) return launch_fill(pl.queue_loopers, kQueues, 0, s);
    const int64_t chunk = (int64_t)((n_tiles + kQueues - 1) / kQueues) * seeds_per_tile;
    const int nbq = (int)((chunk + kCostBlock - 1) / kCostBlock);
    cost_count_kernel<<<kQueues * nbq, kCostBlock, 0, s>>>(seeds->n, seeds->ld, (const float*)seeds->par,
                                                          pl.order, chunk, nbq, pl.cost_cnt);
    cost_place_kernel<<<kQueues * nbq, kCostBlock, 0, s>>>(seeds->n, seeds->ld, (const float*)seeds->par,
                                                          pl.order, chunk, nbq, pl.cost_cnt, pl.tile_order,
                                                          pl.queue_loopers);
    return hipGetLastError();
}

bool small_order(int64_t n_seeds, int n_events)
{
    return n_seeds > 0 && n_seeds <= kOrderMax && n_events <= kOrderEvents;
}

hipError_t launch_small_order(const FindPlan& pl, const kf_tracks* seeds, const int32_t* seed_event,
                              const int32_t* event_off, int n_events, int largest_first, int n_tiles,
                              int seeds_per_tile, hipStream_t s)
{
    const int n = (int)seeds->n;
    const int chunk = (n_tiles + kQueues - 1) / kQueues * seeds_per_tile;
    auto* k = n <= kOrderThreads ? small_order_kernel<1> : small_order_kernel<kOrderItems>;
    k<<<1, kOrderThreads, 0, s>>>(n, seeds->ld, (const float*)seeds->par, seed_event, event_off, n_events,
                                  largest_first, chunk, pl.tile_order, pl.queue_loopers, pl.tile_counter);
    return hipGetLastError();
}

hipError_t launch_seed_order(const FindPlan& pl, const kf_tracks* seeds, const int32_t* seed_event,
                             const int32_t* event_off, int n_events, int largest_first,
                             hipStream_t s)
{
    if (seeds->n == 0) return hipSuccess;
    hipError_t e;
    const int64_t total = (int64_t)n_events * kSeedCells;
    if ((e = launch_fill(pl.scnt, total + 1, 0, s)) != hipSuccess) return e;
    // the ranking compares every pair of events: beyond kRankMaxEvents the
    // events keep their input order
    if (n_events > kRankMaxEvents) largest_first = 0;
    if (largest_first) {
        event_rank_kernel<<<blocks_for(n_events, 256), 256, 0, s>>>(event_off, n_events, pl.erank);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    seed_cell_kernel<<<blocks_for(seeds->n, 256), 256, 0, s>>>(
        seeds->n, seeds->ld, (const float*)seeds->par, seed_event, n_events,
        largest_first ? pl.erank : nullptr, pl.scnt, pl.cell);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_scan(pl.scnt, pl.soff, total + 1, pl.bsum, s)) != hipSuccess) return e;
    seed_scatter_kernel<<<blocks_for(seeds->n, 256), 256, 0, s>>>(seeds->n, pl.cell, pl.soff,
                                                                  pl.scnt, pl.order);
    cell_sort_kernel<<<blocks_for(total, 256), 256, 0, s>>>(total, pl.soff, pl.order);
    return hipGetLastError();
}

// ---------------------------------------------------------------- seed cleaning
// Duplicate seeds (same event; a shared hit, or eta, phi and q/pT all within
// the thresholds) and the order-free rule: a seed is removed iff a better
// duplicate exists.  Three passes: clear the claim slot of every hit a
// taking-part seed holds; in cell order, every seed writes a compact record
// (key, eta, phi, q/pT) at its position and claims its hits with an atomic
// minimum of its key; then, again in cell order, each seed checks its hits'
// claims (a lower key there is a better seed sharing that hit) and the
// records of its own and the eight neighbouring (eta, phi) cells, which are
// contiguous ranges (the thresholds are below a cell's width, so every
// parameter duplicate is there).

// (chi2 as float, then index), ascending = better; ~0 = takes no part
__device__ inline unsigned long long clean_key(float chi2, int64_t i)
{
    uint32_t u = __float_as_uint(chi2);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return ((unsigned long long)u << 32) | (unsigned long long)(uint32_t)i;
}

__device__ inline bool clean_part(uint32_t st, int32_t e, int n_events)
{
    return (st & kFreezeMask & ~(uint32_t)KF_ST_DUPLICATE) == 0 && e >= 0 && e < n_events;
}

__global__ __launch_bounds__(256) void clean_reset_kernel(int64_t n, int64_t ld,
                                                          const uint32_t* __restrict__ status,
                                                          const int32_t* __restrict__ seed_event,
                                                          int n_events,
                                                          const int32_t* __restrict__ seed_hits,
                                                          int64_t n_hits,
                                                          unsigned long long* __restrict__ best)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || !clean_part(status[i], seed_event[i], n_events)) return;
    for (int k = 0; k < 3; ++k) {
        const int32_t h = seed_hits[k * ld + i];
        if (h >= 0 && h < n_hits) best[h] = ~0ull;
    }
}

__global__ __launch_bounds__(256) void clean_claim_kernel(
    int64_t n, int64_t ld, const float* __restrict__ par, const float* __restrict__ chi2,
    const uint32_t* __restrict__ status, const int32_t* __restrict__ seed_event, int n_events,
    const int32_t* __restrict__ seed_hits, int64_t n_hits, const int32_t* __restrict__ order,
    unsigned long long* __restrict__ best, CleanRec* __restrict__ rec)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const int32_t i = order[t];
    CleanRec r;
    if (!clean_part(status[i], seed_event[i], n_events)) {
        r.key = ~0ull;
        r.eta = 0.0;
        r.phi = 0.0f;
        r.c = 0.0f;
        rec[t] = r;
        return;
    }
    r.key = clean_key(chi2[i], i);
    r.eta = -log(tan(0.5 * (double)par[5 * ld + i]));
    r.phi = par[4 * ld + i];
    r.c = par[3 * ld + i];
    rec[t] = r;
    for (int k = 0; k < 3; ++k) {
        const int32_t h = seed_hits[k * ld + i];
        if (h >= 0 && h < n_hits) atomicMin(&best[h], r.key);
    }
}

__global__ __launch_bounds__(256) void clean_mark_kernel(
    int64_t n, int64_t ld, uint32_t* __restrict__ status, const int32_t* __restrict__ seed_hits,
    int64_t n_hits, const unsigned long long* __restrict__ best, const CleanRec* __restrict__ rec,
    const int32_t* __restrict__ cell, const int32_t* __restrict__ soff,
    const int32_t* __restrict__ order, double deta, double dphi, double dc)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const CleanRec me = rec[t];
    if (me.key == ~0ull) return;
    const int32_t j = order[t];
    bool dup = false;
    for (int k = 0; k < 3; ++k) {
        const int32_t h = seed_hits[k * ld + j];
        if (h >= 0 && h < n_hits && best[h] < me.key) dup = true;
    }
    if (!dup) {
        const double ej = me.eta, pj = me.phi, cj = me.c;
        const int c = cell[j];
        const int base = c - c % kSeedCells;
        const int fe = (c % kSeedCells) / 64, fp = c % 64;
        for (int de = -1; de <= 1 && !dup; ++de) {
            const int e2 = fe + de;
            if (e2 < 0 || e2 > 63) continue;
            for (int dp = -1; dp <= 1 && !dup; ++dp) {
                const int cc = base + e2 * 64 + ((fp + dp + 64) & 63);
                const int q1 = soff[cc + 1];
                for (int q = soff[cc]; q < q1; ++q) {
                    const CleanRec o = rec[q];
                    if (o.key >= me.key) continue;     // not better, itself, or no part
                    double d = (double)o.phi - pj;
                    if (d > kPi) d -= 2.0 * kPi;
                    if (d < -kPi) d += 2.0 * kPi;
                    if (fabs(o.eta - ej) < deta && fabs(d) < dphi && fabs((double)o.c - cj) < dc) {
                        dup = true;
                        break;
                    }
                }
            }
        }
    }
    const uint32_t st = status[j];
    status[j] = dup ? (st | (uint32_t)KF_ST_DUPLICATE) : (st & ~(uint32_t)KF_ST_DUPLICATE);
}

hipError_t launch_clean(const FindPlan& pl, const kf_tracks* seeds, const int32_t* seed_event,
                        int n_events, const int32_t* seed_hits, int64_t n_hits,
                        const kf_params& prm, hipStream_t s)
{
    if (seeds->n == 0) return hipSuccess;
    const unsigned nb = blocks_for(seeds->n, 256);
    clean_reset_kernel<<<nb, 256, 0, s>>>(seeds->n, seeds->ld, seeds->status, seed_event, n_events,
                                          seed_hits, n_hits, pl.clean_best);
    clean_claim_kernel<<<nb, 256, 0, s>>>(seeds->n, seeds->ld, (const float*)seeds->par,
                                          (const float*)seeds->chi2, seeds->status, seed_event,
                                          n_events, seed_hits, n_hits, pl.order, pl.clean_best,
                                          pl.clean_rec);
    clean_mark_kernel<<<nb, 256, 0, s>>>(seeds->n, seeds->ld, seeds->status, seed_hits, n_hits,
                                         pl.clean_best, pl.clean_rec, pl.cell, pl.soff, pl.order,
                                         prm.clean_deta, prm.clean_dphi, prm.clean_dc);
    return hipGetLastError();
}

// ---------------------------------------------------------------- duplicate removal
// Found tracks sharing at least frac of the shorter one's hits; the better by
// (more hits, lower float chi2, lower index) removes the other, each track
// decided independently.  A hit -> tracks index (count, prefix, scatter)
// limits the comparisons to tracks that meet in a hit; a pair's shared hits
// are counted layer by layer (a hit sits only in its own layer's column).

__device__ inline bool dedup_part(uint32_t st)
{
    return (st & kFreezeMask & ~(uint32_t)KF_ST_DUPTRACK) == 0;
}

__global__ __launch_bounds__(256) void dedup_count_kernel(int64_t n, int nl,
                                                          const int32_t* __restrict__ rows,
                                                          const uint32_t* __restrict__ status,
                                                          int64_t n_hits, int32_t* __restrict__ cnt,
                                                          int32_t* __restrict__ nh)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    if (!dedup_part(status[j])) {
        nh[j] = -1;
        return;
    }
    int c = 0;
    for (int l = 0; l < nl; ++l) {
        const int32_t h = rows[j * nl + l];
        if (h >= 0 && h < n_hits) {
            atomicAdd(&cnt[h], 1);
            ++c;
        }
    }
    nh[j] = c;
}

__global__ __launch_bounds__(256) void dedup_fill_kernel(int64_t n, int nl,
                                                         const int32_t* __restrict__ rows,
                                                         const int32_t* __restrict__ nh,
                                                         int64_t n_hits,
                                                         const int32_t* __restrict__ off,
                                                         int32_t* __restrict__ cnt,
                                                         int32_t* __restrict__ users)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n || nh[j] < 0) return;
    for (int l = 0; l < nl; ++l) {
        const int32_t h = rows[j * nl + l];
        if (h >= 0 && h < n_hits) users[off[h] + atomicSub(&cnt[h], 1) - 1] = (int32_t)j;
    }
}

// A track's shared-hit count with each partner is accumulated while walking
// its hits' user lists (a partner appears once per hit it shares); up to
// kDedupPartners better partners are tracked in registers, and a track with
// more falls back to counting each pair's shared hits layer by layer.
constexpr int kDedupPartners = 8;

__global__ __launch_bounds__(256) void dedup_mark_kernel(int64_t n, int nl,
                                                         const int32_t* __restrict__ rows,
                                                         const float* __restrict__ chi2,
                                                         uint32_t* __restrict__ status,
                                                         const int32_t* __restrict__ event,
                                                         const int32_t* __restrict__ nh,
                                                         int64_t n_hits,
                                                         const int32_t* __restrict__ off,
                                                         const int32_t* __restrict__ users,
                                                         double frac)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int nj = nh[j];
    if (nj < 0) return;
    const float fj = chi2[j];
    const int32_t ej = event[j];
    auto better = [&](int32_t i) {
        const int ni = nh[i];
        const float fi = chi2[i];
        return event[i] == ej && (ni > nj || (ni == nj && (fi < fj || (fi == fj && i < j))));
    };
    auto is_dup = [&](int32_t i, int shared) {
        const int ni = nh[i];
        const int mn = ni < nj ? ni : nj;
        return mn > 0 && (double)shared >= frac * (double)mn;
    };
    int32_t pid[kDedupPartners];
    int pcnt[kDedupPartners];
    int np = 0;
    bool overflow = false;
    for (int l = 0; l < nl; ++l) {
        const int32_t h = rows[j * nl + l];
        if (h < 0 || h >= n_hits) continue;
        for (int u = off[h]; u < off[h + 1]; ++u) {
            const int32_t i = users[u];
            if (i == j || !better(i)) continue;
            int q = 0;
#pragma unroll
            for (int r = 0; r < kDedupPartners; ++r)
                if (r < np && pid[r] == i) q = r + 1;
            if (q > 0) {
#pragma unroll
                for (int r = 0; r < kDedupPartners; ++r)
                    if (r == q - 1) ++pcnt[r];
            } else if (np < kDedupPartners) {
#pragma unroll
                for (int r = 0; r < kDedupPartners; ++r)
                    if (r == np) {
                        pid[r] = i;
                        pcnt[r] = 1;
                    }
                ++np;
            } else {
                overflow = true;
            }
        }
    }
    bool dup = false;
#pragma unroll
    for (int r = 0; r < kDedupPartners; ++r)
        if (r < np && is_dup(pid[r], pcnt[r])) dup = true;
    if (!dup && overflow) {
        // more better partners than tracked: count every pair directly
        for (int l = 0; l < nl && !dup; ++l) {
            const int32_t h = rows[j * nl + l];
            if (h < 0 || h >= n_hits) continue;
            for (int u = off[h]; u < off[h + 1] && !dup; ++u) {
                const int32_t i = users[u];
                if (i == j || !better(i)) continue;
                int shared = 0;
                for (int m = 0; m < nl; ++m) {
                    const int32_t hj = rows[j * nl + m];
                    shared += (hj >= 0 && hj < n_hits && rows[(int64_t)i * nl + m] == hj) ? 1 : 0;
                }
                dup = is_dup(i, shared);
            }
        }
    }
    const uint32_t st = status[j];
    status[j] = dup ? (st | (uint32_t)KF_ST_DUPTRACK) : (st & ~(uint32_t)KF_ST_DUPTRACK);
}

hipError_t launch_dedup(const FindPlan& pl, int64_t n, int nl, const int32_t* rows,
                        const float* chi2, uint32_t* status, const int32_t* event, int64_t n_hits,
                        double frac, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipError_t e;
    if ((e = launch_fill(pl.dup_cnt, n_hits + 1, 0, s)) != hipSuccess) return e;
    const unsigned nb = blocks_for(n, 256);
    dedup_count_kernel<<<nb, 256, 0, s>>>(n, nl, rows, status, n_hits, pl.dup_cnt, pl.dup_nh);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_scan(pl.dup_cnt, pl.dup_off, n_hits + 1, pl.bsum, s)) != hipSuccess) return e;
    dedup_fill_kernel<<<nb, 256, 0, s>>>(n, nl, rows, pl.dup_nh, n_hits, pl.dup_off, pl.dup_cnt,
                                         pl.dup_users);
    dedup_mark_kernel<<<nb, 256, 0, s>>>(n, nl, rows, chi2, status, event, pl.dup_nh, n_hits,
                                         pl.dup_off, pl.dup_users, frac);
    return hipGetLastError();
}

size_t plan_find(FindPlan* pl, void* base, int64_t n_hits, int n_events, int64_t n_seeds,
                 int n_layers, int n_waves, int seeds_per_tile)
{
    size_t off = 0;
    auto take = [&](size_t bytes) -> void* {
        void* p = base ? (void*)((char*)base + off) : nullptr;
        off += (bytes + 255) & ~size_t(255);
        return p;
    };
    const int64_t nb = (int64_t)n_events * pl->bl.per_event;
    const int64_t nc = (int64_t)n_events * kSeedCells + 1;
    const int64_t ns = n_seeds > 0 ? n_seeds : 1;
    const int64_t nh = n_hits > 0 ? n_hits : 1;
    const bool direct = bin_direct(n_hits, n_events, n_layers);
    const int64_t nseg = direct ? 0 : (int64_t)n_events * n_layers * bin_split(n_hits, n_events, n_layers) + 1;
    int64_t nsmax = nseg > nc ? nseg : nc;
    if (nh + 1 > nsmax) nsmax = nh + 1;
    const int64_t nsum = (nsmax + kScanChunk - 1) / kScanChunk;
    pl->off = (int32_t*)take(sizeof(int32_t) * nb);
    pl->hit_key = (int32_t*)take(sizeof(int32_t) * nh);
    if (direct) {
        pl->hit_bin = (int32_t*)take(sizeof(int32_t) * nh);
        pl->hit_perm = (int32_t*)take(sizeof(int32_t) * nh);
    } else {
        pl->seg_cnt = (int32_t*)take(sizeof(int32_t) * nseg);
        pl->seg_off = (int32_t*)take(sizeof(int32_t) * nseg);
        pl->staged = take(sizeof(StagedHit) * nh);
    }
    pl->binned = take(sizeof(BinnedHit) * nh);
    pl->scnt = (int32_t*)take(sizeof(int32_t) * nc);
    pl->soff = (int32_t*)take(sizeof(int32_t) * nc);
    pl->erank = (int32_t*)take(sizeof(int32_t) * n_events);
    pl->cell = (int32_t*)take(sizeof(int32_t) * ns);
    pl->order = (int32_t*)take(sizeof(int32_t) * ns);
    pl->tile_order = (int32_t*)take(sizeof(int32_t) * ns);
    {
        // class counts per block of the cost order, blocks as launch_cost_order makes them
        const int64_t S = seeds_per_tile > 0 ? seeds_per_tile : 1;
        const int64_t n_tiles = (ns + S - 1) / S;
        const int64_t chunk = (n_tiles + kQueues - 1) / kQueues * S;
        const int64_t nbq = (chunk + kCostBlock - 1) / kCostBlock;
        pl->cost_cnt = (int32_t*)take(sizeof(int32_t) * kCostClasses * kQueues * (size_t)nbq);
    }
    pl->queue_loopers = (int32_t*)take(sizeof(int32_t) * kQueues);
    pl->bsum = (int32_t*)take(sizeof(int32_t) * nsum);
    pl->bp = (int2*)take(sizeof(int2) * (size_t)n_waves * n_layers * seeds_per_tile * kMaxCands);
    // the cells' counters, which the order leaves at zero
    static_assert(kQueues * kQueueStride <= kSeedCells, "an event's cells hold the tile counters");
    pl->tile_counter = pl->scnt;
    pl->clean_best = (unsigned long long*)take(sizeof(unsigned long long) * nh);
    pl->clean_rec = (CleanRec*)take(sizeof(CleanRec) * ns);
    pl->dup_cnt = (int32_t*)take(sizeof(int32_t) * (nh + 1));
    pl->dup_off = (int32_t*)take(sizeof(int32_t) * (nh + 1));
    pl->dup_users = (int32_t*)take(sizeof(int32_t) * ns * (n_layers > 0 ? n_layers : 1));
    pl->dup_nh = (int32_t*)take(sizeof(int32_t) * ns);
    return off;
}

template <typename T, typename C, typename U, bool LEARN, bool MAT>
static void find_launch2(const FindArgs& a, int W, int grid, size_t lds, hipStream_t s)
{
    if (a.prm.field_z0 > 0.0) {
        if constexpr (!LEARN)
            if (a.steer) {
                find_kernel<T, C, U, false, MAT, true, true><<<grid, W, lds, s>>>(a);
                return;
            }
        find_kernel<T, C, U, LEARN, MAT, false, true><<<grid, W, lds, s>>>(a);
        return;
    }
    if constexpr (!LEARN)
        if (a.steer) {
            find_kernel<T, C, U, false, MAT, true, false><<<grid, W, lds, s>>>(a);
            return;
        }
    find_kernel<T, C, U, LEARN, MAT, false, false><<<grid, W, lds, s>>>(a);
}

template <typename T, typename C, typename U, bool LEARN>
static void find_launch(const FindArgs& a, int W, int grid, size_t lds, hipStream_t s)
{
    if (a.mat.x0)
        find_launch2<T, C, U, LEARN, true>(a, W, grid, lds, s);
    else
        find_launch2<T, C, U, LEARN, false>(a, W, grid, lds, s);
}

hipError_t launch_find_kernel(const FindArgs& a, int W, int grid, int prec, bool learn, hipStream_t s)
{
    const size_t lds = find_shared_size(W, a.n_layers, prec);
    if (prec == KF_PREC_FP32)
        learn ? find_launch<float, float, float, true>(a, W, grid, lds, s)
              : find_launch<float, float, float, false>(a, W, grid, lds, s);
    else
        learn ? find_launch<float, double, double, true>(a, W, grid, lds, s)
              : find_launch<float, double, double, false>(a, W, grid, lds, s);
    return hipGetLastError();
}

}  // namespace kfmi
