// wsgrid device kernels (gfx950).  See wsgrid.hip for the launch sequence.
// The header is included by several compilation units: kernels that are not
// templates are static (one copy per unit that launches them).
#pragma once
#include <type_traits>

#include "common.hpp"
#include "fft.hpp"

namespace wsg {

// ---------------------------------------------------------------- utilities --

// Streaming copy for the bandwidth probe: each block walks kProbeUnroll
// consecutive 16-byte vectors per thread per round (all loads issued before
// the stores, non-temporal both ways), rounds strided by the whole grid.  Of
// the shapes measured (128-1024 threads, 4-16 vectors, 512-16384 blocks,
// temporal or not) this one streamed fastest.
constexpr int kProbeThreads = 256;
constexpr int kProbeUnroll = 8;
typedef unsigned int probe_vec __attribute__((ext_vector_type(4)));
static __global__ void __launch_bounds__(kProbeThreads) k_copy_probe(const probe_vec* __restrict__ src,
                                                                   probe_vec* __restrict__ dst, size_t n) {
    const size_t step = size_t(gridDim.x) * kProbeThreads * kProbeUnroll;
    for (size_t base = size_t(blockIdx.x) * kProbeThreads * kProbeUnroll + threadIdx.x; base < n; base += step) {
        probe_vec v[kProbeUnroll];
#pragma unroll
        for (int u = 0; u < kProbeUnroll; ++u) {
            const size_t i = base + size_t(u) * kProbeThreads;
            if (i < n) v[u] = __builtin_nontemporal_load(src + i);
        }
#pragma unroll
        for (int u = 0; u < kProbeUnroll; ++u) {
            const size_t i = base + size_t(u) * kProbeThreads;
            if (i < n) __builtin_nontemporal_store(v[u], dst + i);
        }
    }
}

// ------------------------------------------------------ visibility binning --
//
// Hermitian fold (Sec. 5.4), normalised coordinates u' = (l_max/x0) u,
// v' = (m_max/y0) v, w' = n_scale w (Sec. 5.2), and for each axis the first
// support index F - W + 1 with F = floor(xi + W/2) and the offset
// nu = xi + W/2 - F - 1/2 (Sec. 3.3).  Products and sums are rounded one by one
// (contraction off: __dmul_rn and __dadd_rn are plain operators here, which the
// compiler may fuse) so that the support decision matches a plain evaluation of
// the same formulas, in every kernel that makes it.
struct VisCoords {
    int ru, rv, rt;
    double nu_u, nu_v, nu_w;
    double w;          // folded w
    bool folded;
};

__device__ __forceinline__ bool axis_support(double xi, int W, double& nu, long long& first) {
#pragma clang fp contract(off)
    double hw = 0.5 * W;
    double t = xi + hw;
    double F = floor(t);
    nu = (t - F) - 0.5;
    first = (long long)F - W + 1;
    return true;
}

// The non-negative residue of the integer-valued f (|f| < 2^53) modulo n, in
// FP64: the quotient's floor may be one off after rounding, which the two
// corrections undo; q n and f - q n are exact.
__device__ __forceinline__ int residue(double f, int n) {
    const double dn = double(n);
    const double q = floor(__ddiv_rn(f, dn));
    double r = __dadd_rn(f, -__dmul_rn(q, dn));
    if (r < 0.0) r += dn;
    if (r >= dn) r -= dn;
    return int(r);
}

// ch: the visibility's channel (virtual layer offset ch nbt kTileT)
__device__ __forceinline__ bool vis_coords_of(double u, double v, double w, int ch, const DevParams& P,
                                              VisCoords& c) {
#pragma clang fp contract(off)
    if (!isfinite(u) || !isfinite(v) || !isfinite(w)) return false;
    c.folded = w < 0.0;
    if (c.folded) {
        u = -u;
        v = -v;
        w = -w;
    }
    if (w > P.wmax) return false;
    const double up = P.umul * u, vp = P.umul * v, wp = P.nscale * w + P.wshift;
    if (fabs(up) > 1e15 || fabs(vp) > 1e15) return false;
    long long fu, fv, ft;
    axis_support(up, P.W, c.nu_u, fu);
    axis_support(vp, P.W, c.nu_v, fv);
    axis_support(wp, P.Wz, c.nu_w, ft);
    // the non-negative residues modulo N' (|first| < 2^51 after the check above)
    c.ru = residue(double(fu), P.Np);
    c.rv = residue(double(fv), P.Np);
    long long it = ft - P.t_lo;
    if (P.tclamp && it == P.n_layers) it = P.n_layers - 1;      // w = wmax: the last bin is closed
    if (it < 0 || it > P.n_layers - P.Wz) return false;
    c.rt = int(it) + ch * P.nbt * kTileT;
    c.w = w;
    return true;
}

__device__ __forceinline__ bool vis_coords(const double* __restrict__ uvw, long long k, int ch,
                                           const DevParams& P, VisCoords& c) {
    return vis_coords_of(uvw[3 * k], uvw[3 * k + 1], uvw[3 * k + 2], ch, P, c);
}

__device__ __forceinline__ int bin_of(const VisCoords& c, const DevParams& P) {
    return (c.rt / kTileT * P.nbs + c.rv / kTileS) * P.nbr + c.ru / kTileR;
}

// Bin counts are updated with device-scope atomics, whose cost is per operation
// and, on one address, serial.  A block of k_bin_count therefore takes a chunk of
// kAggChunk consecutive visibilities (a run of time steps of every baseline, whose
// tracks stay in few bins) and aggregates them per bin in an LDS table (open
// addressing, bounded probing) before one global update per distinct bin; a
// visibility whose bin finds no table slot updates the global counter directly.
// Either way the counter's value and the place in the table give each visibility
// its place in its bin (`rank`), so that the records need no second table
// (scatter kernel, 10M visibilities: 358 -> 257 us, 16M of 128 antennas 1129 ->
// 448).  Chunks of 1,024 make the fullest bins' counters wait for each other
// (301,717 visibilities: 48 us against 28).
constexpr int kAggThreads = 1024;
constexpr int kAggPer = 8;
constexpr int kAggChunk = kAggThreads * kAggPer;
constexpr int kAggSlots = 4096;
constexpr int kAggProbes = 32;

struct AggTable {
    int key[kAggSlots];
    uint32_t cnt[kAggSlots];
    uint32_t skipped;
};

// Binning blocks of a batched call: channel c's visibilities are
// [coff[c], coff[c + 1]) of the concatenated arrays, CHUNK of them per block (one
// channel per block, so the lookup is wave-uniform).
struct ChunkRange {
    long long k0, k1;
    int ch;
};
template <int CHUNK>
__device__ __forceinline__ ChunkRange chunk_of_block(const long long* __restrict__ coff, int nch) {
    ChunkRange r;
    r.ch = 0;
    for (long long b = blockIdx.x;; ++r.ch) {
        r.k0 = coff[r.ch] + b * CHUNK;
        r.k1 = coff[r.ch + 1];
        if (r.ch + 1 >= nch || r.k0 < r.k1) break;
        b -= (r.k1 - coff[r.ch] + CHUNK - 1) / CHUNK;
    }
    r.k1 = min(r.k1, r.k0 + CHUNK);
    return r;
}

__device__ __forceinline__ void agg_init(AggTable& T) {
    for (int i = threadIdx.x; i < kAggSlots; i += blockDim.x) {
        T.key[i] = -1;
        T.cnt[i] = 0u;
    }
    if (threadIdx.x == 0) T.skipped = 0u;
}

// slot of key (inserted if absent), or -1 when the probe sequence is full
__device__ __forceinline__ int agg_slot(AggTable& T, int key) {
    int h = int((uint32_t(key) * 2654435761u) >> (32 - 12)) & (kAggSlots - 1);
    for (int p = 0; p < kAggProbes; ++p) {
        const int k = T.key[h];
        if (k == key) return h;
        if (k == -1) {
            const int old = atomicCAS(&T.key[h], -1, key);
            if (old == -1 || old == key) return h;
        }
        h = (h + 1) & (kAggSlots - 1);
    }
    return -1;
}

static __global__ void __launch_bounds__(kAggThreads) k_bin_count(const double* __restrict__ uvw,
                                                           const long long* __restrict__ coff, DevParams P,
                                                           uint32_t* __restrict__ count,
                                                           uint32_t* __restrict__ skipped, uint32_t* __restrict__ rank) {
    __shared__ AggTable T;
    agg_init(T);
    __syncthreads();
    const ChunkRange cr = chunk_of_block<kAggChunk>(coff, P.nch);
    uint32_t my_skipped = 0;
    // the thread's coordinates, all loads in flight at once
    double xu[kAggPer], xv[kAggPer], xw[kAggPer];
#pragma unroll
    for (int i = 0; i < kAggPer; ++i) {
        const long long k = cr.k0 + (long long)i * kAggThreads + threadIdx.x;
        const bool in = k < cr.k1;
        xu[i] = in ? uvw[3 * k] : 0.0;
        xv[i] = in ? uvw[3 * k + 1] : 0.0;
        xw[i] = in ? uvw[3 * k + 2] : 0.0;
    }
    uint32_t tag[kAggPer];       // slot << 16 | place among the block's; 0xffffffff: rank written already
#pragma unroll
    for (int i = 0; i < kAggPer; ++i) {
        tag[i] = 0xffffffffu;
        const long long k = cr.k0 + (long long)i * kAggThreads + threadIdx.x;
        if (k >= cr.k1) continue;
        VisCoords c;
        if (!vis_coords_of(xu[i], xv[i], xw[i], cr.ch, P, c)) {
            ++my_skipped;
            continue;
        }
        const int b = bin_of(c, P);
        const int sl = agg_slot(T, b);
        if (sl >= 0) tag[i] = (uint32_t(sl) << 16) | atomicAdd(&T.cnt[sl], 1u);
        else rank[k] = atomicAdd(&count[b], 1u);
    }
    if (my_skipped) atomicAdd(&T.skipped, my_skipped);
    __syncthreads();
    for (int i = threadIdx.x; i < kAggSlots; i += kAggThreads)
        if (T.key[i] >= 0) T.cnt[i] = atomicAdd(&count[T.key[i]], T.cnt[i]);
    if (threadIdx.x == 0 && T.skipped) atomicAdd(skipped, T.skipped);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kAggPer; ++i)
        if (tag[i] != 0xffffffffu)
            rank[cr.k0 + (long long)i * kAggThreads + threadIdx.x] = T.cnt[tag[i] >> 16] + (tag[i] & 0xffffu);
}

// Clears the counters and marks of a binning, which sit side by side in the
// workspace, and writes the channel table (one launch for what were six).
template <typename Args>
__global__ void k_bin_init(Args ca, int nch, long long* __restrict__ coff, uint32_t* __restrict__ zero, size_t words) {
    if (blockIdx.x == 0 && int(threadIdx.x) <= nch) coff[threadIdx.x] = ca.off[threadIdx.x];
    for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < words; i += size_t(gridDim.x) * blockDim.x)
        zero[i] = 0u;
}

// The wave's next places of a counter for its lanes with `want` (one atomic per wave).
__device__ __forceinline__ uint32_t wave_reserve(uint32_t* counter, bool want) {
    const unsigned long long m = __ballot(want);
    if (m == 0) return 0u;
    const int lane = threadIdx.x & 63, first = __builtin_ctzll(m);
    uint32_t base = 0;
    if (lane == first) base = atomicAdd(counter, uint32_t(__popcll(m)));
    return __shfl(base, first, 64) + uint32_t(__popcll(m & ((1ull << lane) - 1ull)));
}

// Counts of few visibilities: a thread each, its place in its bin straight from
// the bin's counter (5,000 visibilities: 11 -> 4 us, 46,332: 17 -> 8).  With more
// the atomics on the fullest bins wait for each other (120,011: 34 us, 2M: 224).
// So they do, 11 ns each, where the visibilities lie in few bins (short baselines,
// small maps: 65,536 in one bin 720 us), so a wave first joins its lanes of one bin,
// for eight bins, and goes on where these held enough of its lanes (join_lanes):
// the rest of a wave takes up to 2 us, as long as 150 updates of one counter, which
// M visibilities bring when eight bins hold 8 + 64 8 150 / M of its lanes.
constexpr int kDirectThreads = 256;
static __global__ void __launch_bounds__(kDirectThreads) k_bin_count_direct(const double* __restrict__ uvw,
                                                           const long long* __restrict__ coff, DevParams P,
                                                           uint32_t* __restrict__ count,
                                                           uint32_t* __restrict__ skipped, uint32_t* __restrict__ rank,
                                                           int join_lanes) {
    const ChunkRange cr = chunk_of_block<kDirectThreads>(coff, P.nch);
    const long long k = cr.k0 + threadIdx.x;
    VisCoords c;
    const bool in = k < cr.k1, ok = in && vis_coords(uvw, k, cr.ch, P, c);
    const int lane = threadIdx.x & 63, b = ok ? bin_of(c, P) : -1;
    unsigned long long todo = __ballot(ok), group = 1ull << lane;        // the lanes of this lane's bin
    const int kept = __popcll(todo);
    auto join = [&]() {                  // the first such lane's bin (none left: no change)
        const int key = __builtin_amdgcn_readlane(b, int(__builtin_ctzll(todo | (1ull << 63))));
        const unsigned long long same = __ballot(b == key);
        if (b == key) group = same;
        todo &= ~same;
    };
#pragma unroll
    for (int n = 0; n < 8; ++n) join();
    if (kept - __popcll(todo) >= join_lanes)
        while (todo != 0ull) join();
    const int first = __builtin_ctzll(group);
    uint32_t place = 0;
    if (ok && lane == first) place = atomicAdd(&count[b], uint32_t(__popcll(group)));
    place = __shfl(place, first, 64) + uint32_t(__popcll(group & ((1ull << lane) - 1ull)));
    if (ok) rank[k] = place;
    wave_reserve(skipped, in && !ok);
}

// Exclusive scan of n uint32 counts: per-block scan (1024 items per block of
// 256 threads), scan of the block sums in one block, then add; n up to
// kScanSmall in one block of 1024 threads, four items each at a time (5 us at
// 4,096 items, 22 at 32,768; the three launches 14 us up to there).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* sh, uint32_t& total) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    uint32_t inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) sh[wv] = inc;
    __syncthreads();
    uint32_t woff = 0;
    const int nw = blockDim.x >> 6;
    for (int i = 0; i < wv; ++i) woff += sh[i];
    total = 0;
    for (int i = 0; i < nw; ++i) total += sh[i];
    __syncthreads();
    return woff + inc - x;
}

static __global__ void k_scan_local(const uint32_t* __restrict__ in, uint32_t* __restrict__ out, int n,
                             uint32_t* __restrict__ block_sums) {
    __shared__ uint32_t sh[16];
    const int base = blockIdx.x * 1024 + threadIdx.x * 4;
    uint32_t v[4], s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = (base + i < n) ? in[base + i] : 0u;
        s += v[i];
    }
    uint32_t total;
    uint32_t off = block_exclusive_scan(s, sh, total);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (base + i < n) out[base + i] = off;
        off += v[i];
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

constexpr int kScanSmall = 8192;
static __global__ void __launch_bounds__(1024) k_scan_small(const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                                                            int n, uint32_t* __restrict__ grand) {
    __shared__ uint32_t sh[16];
    uint32_t carry = 0;
    for (int i0 = 0; i0 < n; i0 += 4096) {
        const int base = i0 + threadIdx.x * 4;
        uint32_t v[4], s = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = (base + i < n) ? in[base + i] : 0u;
            s += v[i];
        }
        uint32_t total;
        uint32_t off = carry + block_exclusive_scan(s, sh, total);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (base + i < n) out[base + i] = off;
            off += v[i];
        }
        carry += total;
    }
    if (threadIdx.x == 0) *grand = carry;
}

// single block of 1024 threads; each thread scans ceil(nb / 1024) consecutive sums
static __global__ void k_scan_sums(uint32_t* __restrict__ block_sums, int nb, uint32_t* __restrict__ grand) {
    __shared__ uint32_t sh[16];
    const int per = (nb + 1023) / 1024;
    const int base = threadIdx.x * per;
    uint32_t s = 0;
    for (int i = 0; i < per; ++i)
        if (base + i < nb) s += block_sums[base + i];
    uint32_t total;
    uint32_t off = block_exclusive_scan(s, sh, total);
    for (int i = 0; i < per; ++i) {
        if (base + i < nb) {
            const uint32_t v = block_sums[base + i];
            block_sums[base + i] = off;
            off += v;
        }
    }
    if (threadIdx.x == 0) *grand = total;
}

static __global__ void k_scan_add(uint32_t* __restrict__ out, int n, const uint32_t* __restrict__ block_sums) {
    const int base = blockIdx.x * 1024 + threadIdx.x * 4;
    const uint32_t add = block_sums[blockIdx.x];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (base + i < n) out[base + i] += add;
}

// The record of visibility k.
// grid: v = V exp(+i 2 pi w (n0 - 1)) with n0 - 1 = -zshift n_scale (eq. n_params:
// zshift = z0; zero without z offset, eq. n_params_no_offset),
// V conjugated for a folded visibility.  degrid: v = exp(-i 2 pi w (n0 - 1)).
template <typename R, bool GRID>
__device__ __forceinline__ Rec<R> make_rec(const VisCoords& c, long long k, const cpx<R>* __restrict__ vis,
                                           const DevParams& P) {
    Rec<R> r;
    r.ruv = uint32_t(c.ru) | (uint32_t(c.rv) << 16);
    r.rt = uint32_t(c.rt);
    r.nu[0] = R(c.nu_u);
    r.nu[1] = R(c.nu_v);
    r.nu[2] = R(c.nu_w);
    double turns = c.w * (-P.zshift * P.nscale);     // w (n0 - 1)
    double sn, co;
    phase_turns(GRID ? turns : -turns, &sn, &co);
    if (GRID) {
        cpx<R> V = vis[k];
        double vx = double(V.x), vy = c.folded ? -double(V.y) : double(V.y);
        r.v[0] = R(vx * co - vy * sn);
        r.v[1] = R(vx * sn + vy * co);
        r.idx = 0;
    } else {
        r.v[0] = R(co);
        r.v[1] = R(sn);
        r.idx = uint32_t(k) | (c.folded ? 0x80000000u : 0u);
    }
    return r;
}

// The records, binned.  degrid: a skipped visibility leaves its index behind the
// last record (counted down from the end of `tail`), for k_degrid_finish.
template <typename R, bool GRID>
__global__ void __launch_bounds__(kDirectThreads) k_bin_scatter(const double* __restrict__ uvw,
                                                             const cpx<R>* __restrict__ vis,
                                                             const long long* __restrict__ coff, DevParams P,
                                                             const uint32_t* __restrict__ start,
                                                             const uint32_t* __restrict__ rank,
                                                             uint32_t* __restrict__ spare, Rec<R>* __restrict__ rec,
                                                             Rec<R>* __restrict__ tail) {
    const ChunkRange cr = chunk_of_block<kDirectThreads>(coff, P.nch);
    const long long k = cr.k0 + threadIdx.x;
    VisCoords c;
    const bool in = k < cr.k1, ok = in && vis_coords(uvw, k, cr.ch, P, c);
    if (ok) rec[start[bin_of(c, P)] + rank[k]] = make_rec<R, GRID>(c, k, vis, P);
    if constexpr (!GRID) {
        const uint32_t at = wave_reserve(spare, in && !ok);
        if (in && !ok) tail[coff[P.nch] - 1 - at].idx = uint32_t(k);
    }
}

// Second-level sort and touch classes.  With B = 17 - W, a record whose first
// support index inside its tile is >= B along an axis also reaches the next
// tile along that axis (W <= 16: never the one after).  Its touch class is the
// 3-bit set c = (layer >= B) | (u >= B) << 1 | (v >= B) << 2.  A tile reads,
// from the bin one tile back along the axes of a set m, exactly the records
// whose class contains m.  Classes are stored in Gray-code order (position q
// holds class q ^ (q >> 1)): the records a tile needs from one bin are then at
// most two contiguous ranges, ten over the eight bins.  Inside a class, records
// are ordered by their first support index, so that records with the same or a
// near support box are adjacent (long runs along Earth-rotation tracks).
// With separate widths, the layer axis uses Bt = 17 - W_z and the u, v axes
// Buv = 17 - W.
__device__ __forceinline__ int class_part(int hi, int B) { return hi ? kTileT - B : B; }
__device__ __forceinline__ int class_position(int c) { return c ^ (c >> 1) ^ (c >> 2); }   // inverse Gray code
__device__ __forceinline__ int class_of(int lt, int lr, int ls, int Bt, int Buv) {
    return int(lt >= Bt) | (int(lr >= Buv) << 1) | (int(ls >= Buv) << 2);
}
// rank of the first key of class position q (q = 0..8) among the 4096 keys
__device__ __forceinline__ int class_base(int q, int Bt, int Buv) {
    int b = 0;
    for (int k = 0; k < q; ++k) {
        const int c = k ^ (k >> 1);
        b += class_part(c & 1, Bt) * class_part(c & 2, Buv) * class_part(c & 4, Buv);
    }
    return b;
}

// first start of the block of start i (of its class's part), and its size
__device__ __forceinline__ int block_start(int i, int edge) { return i / edge * edge; }

// One block per bin: LDS histogram over the 4096 in-tile positions enumerated
// in (class position, window block, start) order, exclusive scan, scatter to
// `out` (order among equal keys is arbitrary).  cls[8 bin + q] receives the
// start of class position q in `out`.
template <typename R>
__global__ void __launch_bounds__(256) k_bin_local_sort(const Rec<R>* __restrict__ in, Rec<R>* __restrict__ out,
                                                        const uint32_t* __restrict__ start,
                                                        uint32_t* __restrict__ cls, DevParams P) {
    constexpr int NK = kTileT * kTileR * kTileS;
    __shared__ uint32_t hist[NK];
    __shared__ uint32_t sh[16];
    __shared__ int cbase[9];
    __shared__ int blk[2][16];       // start l of the layer and the u, v axes: its block's start, size << 8, offset << 16
    const int bin = blockIdx.x;
    const uint32_t b0 = start[bin], b1 = start[bin + 1];
    if (b1 == b0) return;
    const int br = bin % P.nbr, bs = (bin / P.nbr) % P.nbs, bt = bin / (P.nbr * P.nbs);
    const int tid = threadIdx.x;
    const int Buv = 17 - P.W, Bt = 17 - P.Wz;
    if (tid < 9) cbase[tid] = class_base(tid, Bt, Buv);
    if (tid >= 32 && tid < 64) {
        const int ax = (tid >> 4) & 1, l = tid & 15, B = ax ? Buv : Bt;
        const int edge = ax ? P.euv : P.et;
        const int hi = l >= B, i = hi ? l - B : l, b = block_start(i, edge);
        blk[ax][l] = b | min(edge, class_part(hi, B) - b) << 8 | (i - b) << 16;
    }
    for (int i = tid; i < NK; i += 256) hist[i] = 0u;
    __syncthreads();
    auto key_of = [&](const Rec<R>& r) {
        const int lr = int(r.ruv & 0xffffu) - br * kTileR, ls = int(r.ruv >> 16) - bs * kTileS;
        const int lt = int(r.rt) - bt * kTileT;
        const int c = class_of(lt, lr, ls, Bt, Buv);
        const int t = blk[0][lt], u = blk[1][lr], v = blk[1][ls];
        const int nt = (t >> 8) & 255, nu = (u >> 8) & 255, nv = (v >> 8) & 255;
        const int pu = class_part(c & 2, Buv), pv = class_part(c & 4, Buv);
        // positions of the blocks before, then inside the block
        return cbase[class_position(c)] + ((t & 255) * pu + nt * (u & 255)) * pv + nt * nu * (v & 255) +
               ((t >> 16) * nu + (u >> 16)) * nv + (v >> 16);
    };
    for (uint32_t i = b0 + tid; i < b1; i += 256) atomicAdd(&hist[key_of(in[i])], 1u);
    __syncthreads();
    // exclusive scan: 16 consecutive keys per thread
    uint32_t v[NK / 256], sum = 0;
#pragma unroll
    for (int k = 0; k < NK / 256; ++k) {
        v[k] = hist[tid * (NK / 256) + k];
        sum += v[k];
    }
    uint32_t total;
    uint32_t off = block_exclusive_scan(sum, sh, total);
#pragma unroll
    for (int k = 0; k < NK / 256; ++k) {
        hist[tid * (NK / 256) + k] = off;
        off += v[k];
    }
    __syncthreads();
    if (tid < 8) cls[8 * size_t(bin) + tid] = b0 + (cbase[tid] < NK ? hist[cbase[tid]] : total);
    __syncthreads();
    for (uint32_t i = b0 + tid; i < b1; i += 256) {
        const Rec<R> r = in[i];
        out[b0 + atomicAdd(&hist[key_of(r)], 1u)] = r;
    }
}

// Tile occupancy: a tile is marked when some visibility reaches it: its own bin
// is non-empty, or the bin one tile back along the axes of a set m holds
// visibilities whose touch class contains m (from the class starts of the
// per-bin sort).  Only marked tiles of the stack are written (grid) or filled
// (degrid); the FFT passes treat unmarked tiles as zero (grid) or skip them
// (degrid).  A row of tiles (t tile, u tile) is marked in `rows` when one of
// its tiles is (`rows` zero on entry; racing stores all write 1), and its tiles
// are bits of the row's words of `mask` (mask_words(nbs) words, zero on entry).
static __global__ void k_tile_occupancy(const uint32_t* __restrict__ start, const uint32_t* __restrict__ cls, DevParams P,
                                 uint8_t* __restrict__ occ, uint8_t* __restrict__ rows, uint32_t* __restrict__ mask,
                                 uint32_t* __restrict__ flag) {
    const int tile = blockIdx.x * blockDim.x + threadIdx.x;
    const int nt = P.nch * P.nbt * P.nbs * P.nbr;
    if (tile >= nt) return;
    const int br = tile % P.nbr, bs = (tile / P.nbr) % P.nbs, bt = tile / (P.nbr * P.nbs);
    bool any = false;
    for (int nb = 0; nb < 8 && !any; ++nb) {
        const int it = (nb >> 2) & 1, is = (nb >> 1) & 1, ir = nb & 1;
        if (bt % P.nbt - it < 0) continue;      // not across a channel start
        const int bin = ((bt - it) * P.nbs + (bs - is + P.nbs) % P.nbs) * P.nbr + (br - ir + P.nbr) % P.nbr;
        const uint32_t b0 = start[bin], b1 = start[bin + 1];
        if (b1 == b0) continue;
        const int m = it | (ir << 1) | (is << 2);
        for (int q = 0; q < 8; ++q) {
            const int c = q ^ (q >> 1);
            if ((c & m) != m) continue;
            const uint32_t lo = cls[8 * size_t(bin) + q], hi = q < 7 ? cls[8 * size_t(bin) + q + 1] : b1;
            if (hi > lo) {
                any = true;
                break;
            }
        }
    }
    occ[tile] = any ? 1 : 0;
    flag[tile] = any ? 1u : 0u;
    if (any) {
        rows[bt * P.nbr + br] = 1;
        atomicOr(&mask[size_t(bt * P.nbr + br) * mask_words(P.nbs) + (bs >> 5)], 1u << (bs & 31));
    }
}

// The marked tiles among [first, first + n) in tile order: list[pos[t] -
// pos[first]] for every marked tile t, pos the exclusive scan of the flags.  A
// tile's ranges are gathered here, so that a tile block needs one load before its
// records.  pass: null, or where the tile kernels find the bounds of a list that
// starts with tile `first`, as in pos.
static __global__ void k_tile_list(const uint8_t* __restrict__ occ, const uint32_t* __restrict__ pos,
                            const uint32_t* __restrict__ start, const uint32_t* __restrict__ cls, DevParams P,
                            int first, int n_tiles, uint32_t* __restrict__ pass, TileRec* __restrict__ list) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, t = first + i;
    if (i == 0 && pass) {
        pass[first] = 0u;
        pass[first + n_tiles] = pos[first + n_tiles] - pos[first];
    }
    if (i >= n_tiles || !occ[t]) return;
    const int br = t % P.nbr, bs = (t / P.nbr) % P.nbs, bt = t / (P.nbr * P.nbs);
    TileRec& T = list[pos[t] - pos[first]];
    uint32_t total = 0, nbrs = 0;
    int n = 0;
    for (int nb = 0; nb < 8; ++nb) {
        const int it = (nb >> 2) & 1, is = (nb >> 1) & 1, ir = nb & 1;
        if (bt % P.nbt - it < 0) continue;      // not across a channel start
        const int bin = ((bt - it) * P.nbs + (bs - is + P.nbs) % P.nbs) * P.nbr + (br - ir + P.nbr) % P.nbr;
        const uint32_t b0 = start[bin], b1 = start[bin + 1];
        if (b1 == b0) continue;
        const int m = it | (ir << 1) | (is << 2);
        uint32_t at[9];
#pragma unroll
        for (int q = 0; q < 8; ++q) at[q] = cls[8 * size_t(bin) + q];
        at[8] = b1;
        uint32_t lo = 0;
        bool in = false;
#pragma unroll
        for (int q = 0; q <= 8; ++q) {          // at most two runs of classes that contain m
            const bool need = q < 8 && ((q ^ (q >> 1)) & m) == m;
            if (need && !in) lo = at[q];
            if (!need && in && at[q] > lo) {
                T.off[n] = total;
                T.delta[n] = lo - total;
                nbrs |= uint32_t(m) << (3 * n);
                total += at[q] - lo;
                ++n;
            }
            in = need;
        }
    }
    T.tile = uint32_t(t);
    T.total = total;
    T.nbrs = nbrs;
    for (; n < 10; ++n) T.off[n] = 0xffffffffu;
}

// ------------------------------------------------ 3-D scatter / gather tiles --
//
// A block holds one tile of kTileT layers x kTileR u-cells x kTileS v-cells of the
// stack at a time in LDS; the matrix kernels take several tiles one after the
// other (tiles_of_block).  The records that reach the tile (from its own bin and
// the seven bins one tile back, selected by touch class) form a virtual list of
// at most ten ranges of the record array (TileRec).  The list is cut into
// contiguous parts, one per wave (eight waves in the FP32 matrix scatter, four
// elsewhere); the waves work independently between the tile's set-up and its
// write-out, and each holds its next records in registers while it works on the
// current ones.  Each tile is read or written to HBM once.

// Kernel polynomial degree in nu per precision (the host fits both).
template <typename R>
struct KernelDegree {
    static constexpr int value = sizeof(R) == 8 ? 16 : 8;
};

// Record array index of virtual position v of the tile's list; m: its bin's set
// of axes.  T is wave-uniform, so the ranges come from scalar registers.
__device__ __forceinline__ uint32_t tile_record(const TileRec& T, uint32_t v, uint32_t& m) {
    uint32_t d = T.delta[0], k = 0;
#pragma unroll
    for (int g = 1; g < 10; ++g) {
        const bool past = v >= T.off[g];
        d = past ? T.delta[g] : d;
        k = past ? 3 * g : k;
    }
    m = (T.nbrs >> k) & 7u;
    return v + d;
}
__device__ __forceinline__ uint32_t tile_record(const TileRec& T, uint32_t v) {
    uint32_t m;
    return tile_record(T, v, m);
}

// The ranges of a tile's list, kept in scalar registers: read again for each batch
// of records, as the compiler has it, they held up every batch of a long list (the
// FP32 gather of 200,000 visibilities in few bins: 3.39 -> 3.23 ms).
struct HeldRanges {
    uint32_t off[10], delta[10], nbrs;
    static __device__ __forceinline__ uint32_t hold(uint32_t x) {
        int y = __builtin_amdgcn_readfirstlane(int(x));
        asm volatile("" : "+s"(y));
        return uint32_t(y);
    }
    __device__ __forceinline__ explicit HeldRanges(const TileRec& T) {
#pragma unroll
        for (int g = 0; g < 10; ++g) {
            off[g] = hold(T.off[g]);
            delta[g] = hold(T.delta[g]);
        }
        nbrs = hold(T.nbrs);
    }
    __device__ __forceinline__ uint32_t record(uint32_t v, uint32_t& m) const {      // tile_record
        uint32_t d = delta[0], k = 0;
#pragma unroll
        for (int g = 1; g < 10; ++g) {
            const bool past = v >= off[g];
            const uint32_t here = delta[g];
            d = past ? here : d;
            k = past ? 3 * g : k;
        }
        m = (nbrs >> k) & 7u;
        return v + d;
    }
};
struct ReadRanges {
    const TileRec& T;
    __device__ __forceinline__ explicit ReadRanges(const TileRec& t) : T(t) {}
    __device__ __forceinline__ uint32_t record(uint32_t v, uint32_t& m) const { return tile_record(T, v, m); }
};

// Signed offset of a support start from the tile origin along a periodic axis.
__device__ __forceinline__ int wrap_offset(int first, int origin, int Np) {
    int d = first - origin;
    if (d >= Np / 2) d -= Np;
    if (d < -Np / 2) d += Np;
    return d;
}

// x mod W in [0, W) for x > -16 W
template <int W>
__device__ __forceinline__ int mod_w(int x) {
    return (x + 16 * W) % W;
}

// The launch has one block per tile of the current layer pass (tile layers
// pl0 / kTileT onwards), and the blocks take the pass's occupied tiles from the
// ordered list (groups of 4 neighbours per XCD); the result is the place in the
// list, or -1 for a block beyond the occupied tiles (it exits at once).
__device__ __forceinline__ int tile_of_block(const DevParams& P, const uint32_t* __restrict__ tpos) {
    const int per_layer = P.nbs * P.nbr;
    const int nbt_pass = (P.pln + kTileT - 1) / kTileT;
    const int a = (P.pl0 / kTileT) * per_layer, e = a + nbt_pass * per_layer;
    const int first = int(tpos[a]), cnt = int(tpos[e]) - first;
    if (int(blockIdx.x) >= cnt) return -1;
    return first + xcd_interleave<4>(blockIdx.x, cnt);
}

// Kernel weights of one record on the three axes by Horner's rule: u and v
// from coef (width W), the layer axis from coefz (width WZ).  SAME: the w-axis
// design is the u, v one (WZ == W), so each coefficient read feeds three chains.
template <typename R, int W, int WZ, bool SAME>
__device__ __forceinline__ void record_weights(const Rec<R>& r, const R* __restrict__ coef, const R* __restrict__ coefz,
                                               R (&wu)[W], R (&wv)[W], R (&wt)[WZ]) {
    constexpr int D = KernelDegree<R>::value;
    static_assert(!SAME || WZ == W, "one design on all axes needs equal widths");
#pragma unroll
    for (int a = 0; a < W; ++a) {
        const R* c = coef + a * (D + 1);
        const R* cz = (SAME ? coef : coefz) + (a < WZ ? a : 0) * (D + 1);
        R hu = c[D], hv = c[D], ht = cz[D];
#pragma unroll
        for (int k = D - 1; k >= 0; --k) {
            const R ck = c[k];
            hu = hu * r.nu[0] + ck;
            hv = hv * r.nu[1] + ck;
            ht = ht * r.nu[2] + (SAME ? ck : cz[k]);
        }
        wu[a] = hu;
        wv[a] = hv;
        if (a < WZ) wt[a] = ht;
    }
}

__device__ __forceinline__ float bits_to_word(int v, float) { return __int_as_float(v); }
__device__ __forceinline__ double bits_to_word(int v, double) { return __hiloint2double(0, v); }
__device__ __forceinline__ int word_bits(float v) { return __float_as_int(v); }
__device__ __forceinline__ int word_bits(double v) { return __double2loint(v); }

// Scatter where the matrix kernel is not the better one (mat_scatter), or a window
// of 8 cells does not hold the support (W > 8): residue classes (Romein 2012,
// extended to three axes).  Lane (x, y)
// owns, among the W x W x WZ support cells of a record, the WZ cells whose u
// and v indices are congruent to x and y modulo W, one per layer residue a: for
// support start (dr, ds, dt) the u-cell dr + ((x - dr) mod W), the v-cell
// ds + ((y - ds) mod W) and the layer dt + ((a - dt) mod WZ).  Each round a wave
// stages 16 or 32 records into its slots (four or two lanes per record): the u
// weights times the value and the v weights rotated by the support start (so lane x reads position x
// whatever the record), and the layer weights rotated by dt with the packed
// support start, read by the whole wave as broadcasts.  Sums stay in registers
// while the owned cell stays the same; when the support moves, the lanes (or
// layer residues) whose owned cell changed add their sums to the LDS tile
// (atomics: the four waves share it) and restart from zero.  Records are sorted
// by support start inside each touch class, so supports mostly coincide or
// move by one cell.
template <typename R, int W, int WZ>
struct ScatterCfg {
    // records per wave round: 16 (four lanes stage each) for W <= 7, where the
    // block then fits in 40 KB of LDS (FP32: four blocks per CU) or 80 KB
    // (FP64: two), else 32 (two lanes each; at W = 7 that measured 8 % slower)
    static constexpr int kWaveBatch = W <= 7 ? 16 : 32;
    static constexpr int kLanesPerRecord = 64 / kWaveBatch;
    // waves per block, each on its own part of the tile's record list (eight
    // waves at three blocks per CU measured 13 % slower than four at four)
    static constexpr int kWaves = 4;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kSlots = kWaves * kWaveBatch;
    static constexpr int kPairs = W * W;
    static constexpr int kPI = (kPairs + 63) / 64;                // (x, y) residue pairs per lane
    static constexpr int kCells = kTileT * kTileR * kTileS;
    static constexpr int kWords = (WZ * sizeof(R) + 15) / 16 * 16 / sizeof(R);   // 16-byte rows
};

template <typename R, int W, int WZ>
struct __align__(16) ScatterStage {
    // layer weights rotated (position (a + dt) mod WZ holds C_z(s_a - nu_w))
    R words[ScatterCfg<R, W, WZ>::kSlots][ScatterCfg<R, W, WZ>::kWords];
    // value times u weights (real, imaginary), rotated by dr; v weights rotated by ds
    R wuv[ScatterCfg<R, W, WZ>::kSlots][3 * W];
};

// PREP: the records are those of a shared binning (degridding records: the
// phase e^{-i 2 pi w (n0 - 1)} and the visibility index with the fold flag);
// each record's value is then the visibility it names, conjugated when folded,
// times the conjugate phase (formed in FP64), and the lane keeps two records
// in flight so that the value's load (which needs the record's index) is
// issued a round before its staging.
template <typename R, int W, int WZ, bool SAME, bool PREP>
__global__ void __launch_bounds__((ScatterCfg<R, W, WZ>::kThreads)) k_grid_tiles(const Rec<R>* __restrict__ rec,
                                                    const TileRec* __restrict__ tlist,
                                                    const uint32_t* __restrict__ tpos, DevParams P,
                                                    const R* __restrict__ coef_g, const R* __restrict__ coefz_g,
                                                    const cpx<R>* __restrict__ vis, cpx<R>* __restrict__ stack) {
    using Cfg = ScatterCfg<R, W, WZ>;
    constexpr int PI = Cfg::kPI, WB = Cfg::kWaveBatch, D = KernelDegree<R>::value;
    __shared__ R tre[Cfg::kCells];
    __shared__ R tim[Cfg::kCells];
    __shared__ ScatterStage<R, W, WZ> st;

    const int place = tile_of_block(P, tpos);
    if (place < 0) return;     // unoccupied tiles are left unwritten and read as zero
    const TileRec& T = tlist[place];
    const int tile = int(T.tile);
    const int br = tile % P.nbr, bs = (tile / P.nbr) % P.nbs, bt = tile / (P.nbr * P.nbs);
    const int r0 = br * kTileR, s0 = bs * kTileS, t0 = bt * kTileT;
    const int nt_valid = min(kTileT, P.n_layers - t0 % (P.nbt * kTileT));   // layers of its channel
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

    constexpr int NT = Cfg::kThreads, NW = Cfg::kWaves;
    for (int i = tid; i < Cfg::kCells; i += NT) tre[i] = tim[i] = R(0);
    __syncthreads();
    const uint32_t total = T.total;
    // this wave's part of the list
    const uint32_t part = (total + NW - 1) / NW;
    const uint32_t q0 = min(total, part * uint32_t(wv)), q1 = min(total, q0 + part);

    if (q1 > q0) {
        // the lane's residue pairs, owned cells and register sums
        int px[PI], py[PI], cr[PI], cs[PI];
        bool pv[PI];
#pragma unroll
        for (int i = 0; i < PI; ++i) {
            const int p = lane + 64 * i;
            pv[i] = p < Cfg::kPairs;
            const int pc = min(p, Cfg::kPairs - 1);
            px[i] = pc / W;
            py[i] = pc % W;
            cr[i] = cs[i] = -1000;
        }
        int ct[WZ];                                  // owned layer per residue (wave-uniform)
        R ax[PI][WZ], ay[PI][WZ];
#pragma unroll
        for (int a = 0; a < WZ; ++a) ct[a] = -1000;
#pragma unroll
        for (int i = 0; i < PI; ++i)
#pragma unroll
            for (int a = 0; a < WZ; ++a) ax[i][a] = ay[i][a] = R(0);
        // add sum (i, a) to its owned cell if that cell is in the tile
        auto add_cell = [&](int i, int a) {
            const int t = ct[a];
            if (pv[i] && unsigned(cr[i]) < unsigned(kTileR) && unsigned(cs[i]) < unsigned(kTileS) &&
                unsigned(t) < unsigned(nt_valid)) {
                const int cell = (t * kTileR + cr[i]) * kTileS + cs[i];
                atomicAdd(&tre[cell], ax[i][a]);
                atomicAdd(&tim[cell], ay[i][a]);
            }
            ax[i][a] = ay[i][a] = R(0);
        };
        int prev = -1, prev_dt = -1000;
        // the support starts at packed d: flush the sums of owned cells that change
        auto move_to = [&](int d) {
            prev = d;
            const int dr = (d & 255) - 128, ds = ((d >> 8) & 255) - 128, dt = ((d >> 16) & 255) - 128;
            const int mr = mod_w<W>(-dr), ms = mod_w<W>(-ds);
#pragma unroll
            for (int i = 0; i < PI; ++i) {
                int xr = px[i] + mr, ys = py[i] + ms;
                xr -= xr >= W ? W : 0;
                ys -= ys >= W ? W : 0;
                const int nr = dr + xr, ns = ds + ys;
                if (nr != cr[i] || ns != cs[i]) {
#pragma unroll
                    for (int a = 0; a < WZ; ++a) add_cell(i, a);
                    cr[i] = nr;
                    cs[i] = ns;
                }
            }
            if (dt != prev_dt) {
                prev_dt = dt;
                const int mt = mod_w<WZ>(-dt);
#pragma unroll
                for (int a = 0; a < WZ; ++a) {
                    int k = a + mt;
                    k -= k >= WZ ? WZ : 0;
                    const int nt = dt + k;
                    if (nt != ct[a]) {
#pragma unroll
                        for (int i = 0; i < PI; ++i) add_cell(i, a);
                        ct[a] = nt;
                    }
                }
            }
        };

        const int slot0 = wv * WB;
        // staging: the lanes rl + WB h (h = 0 .. LPR - 1) take record rl, lane h
        // the kernel segments [h A0, (h + 1) A0), so the Horner work is spread
        // over the whole wave; the coefficients come from global memory (the
        // whole wave reads the same few, so the vector cache serves them)
        constexpr int LPR = Cfg::kLanesPerRecord;
        static_assert(WB * LPR == 64, "the wave stages WB records with LPR lanes each");
        constexpr int A0 = (W + LPR - 1) / LPR;
        static_assert(WZ <= W, "the w-axis function is at most as wide as the u, v one");
        const int rl = lane & (WB - 1), half = lane / WB;
        // The lane's coefficients, loaded once into registers when they fit in
        // 40 of them (else read from global memory at each staging).
        constexpr bool kRegCoef = A0 * (D + 1) * (SAME ? 1 : 2) * int(sizeof(R)) <= 160;
        R creg[kRegCoef ? A0 : 1][D + 1], czreg[(kRegCoef && !SAME) ? A0 : 1][D + 1];
        if constexpr (kRegCoef) {
#pragma unroll
            for (int i = 0; i < A0; ++i) {
                const int a = i + half * A0;
#pragma unroll
                for (int k = 0; k <= D; ++k) {
                    creg[i][k] = coef_g[min(a, W - 1) * (D + 1) + k];
                    if constexpr (!SAME) czreg[i][k] = coefz_g[min(a, WZ - 1) * (D + 1) + k];
                }
            }
        }
        // the lane's next record: virtual position vn
        uint32_t vn = q0 + uint32_t(rl);
        Rec<R> nxt{}, nxt2{};
        cpx<R> nval{R(0), R(0)};
        if (vn < q1) nxt = rec[tile_record(T, vn)];
        if constexpr (PREP) {
            if (vn < q1) nval = vis[nxt.idx & 0x7fffffffu];
            if (vn + WB < q1) nxt2 = rec[tile_record(T, vn + WB)];
        }
        for (uint32_t base = q0; base < q1; base += WB) {
            const int n = __builtin_amdgcn_readfirstlane(int(min(uint32_t(WB), q1 - base)));
            // support start of this lane's record, relative to the tile, packed
            const int dr = wrap_offset(int(nxt.ruv & 0xffffu), r0, P.Np);
            const int ds = wrap_offset(int(nxt.ruv >> 16), s0, P.Np);
            const int dt = int(nxt.rt) - t0;
            const int d = (dr + 128) | ((ds + 128) << 8) | ((dt + 128) << 16);
            if (rl < n) {
                // stage: rotated weights, value folded into the u weights
                const int pr = mod_w<W>(dr), ps = mod_w<W>(ds), pt = mod_w<WZ>(dt);
                const int slot = slot0 + rl;
                R v0 = nxt.v[0], v1 = nxt.v[1];
                if constexpr (PREP) {
                    const double vx = double(nval.x), vy = (nxt.idx & 0x80000000u) ? -double(nval.y) : double(nval.y);
                    const double co = double(nxt.v[0]), sn = -double(nxt.v[1]);
                    v0 = R(vx * co - vy * sn);
                    v1 = R(vx * sn + vy * co);
                }
#pragma unroll
                for (int i = 0; i < A0; ++i) {
                    const int a = i + half * A0;
                    const R* c = coef_g + min(a, W - 1) * (D + 1);
                    const R* cz = (SAME ? coef_g : coefz_g) + min(a, WZ - 1) * (D + 1);
                    auto cu = [&](int k) { if constexpr (kRegCoef) return creg[i][k]; else return c[k]; };
                    auto cw = [&](int k) {
                        if constexpr (SAME) return cu(k);
                        else if constexpr (kRegCoef) return czreg[i][k];
                        else return cz[k];
                    };
                    R hu = cu(D), hv = cu(D), ht = cw(D);
#pragma unroll
                    for (int k = D - 1; k >= 0; --k) {
                        const R ck = cu(k);
                        hu = hu * nxt.nu[0] + ck;
                        hv = hv * nxt.nu[1] + ck;
                        ht = ht * nxt.nu[2] + cw(k);
                    }
                    if (a < W) {
                        int ku = pr + a, kv = ps + a;
                        ku -= ku >= W ? W : 0;
                        kv -= kv >= W ? W : 0;
                        st.wuv[slot][ku] = v0 * hu;
                        st.wuv[slot][W + ku] = v1 * hu;
                        st.wuv[slot][2 * W + kv] = hv;
                    }
                    if (a < WZ) {
                        int kt = pt + a;
                        kt -= kt >= WZ ? WZ : 0;
                        st.words[slot][kt] = ht;
                    }
                }
            }
            // slots whose support start differs from the previous slot's (slot 0:
            // from the wave's current one): a scalar bit mask, so that the
            // per-record check below costs no vector instruction
            const int d_before = __shfl_up(d, 1, 64);
            const bool moved = half == 0 && rl < n && (rl == 0 ? d != prev : d != d_before);
            const uint64_t move_mask = __ballot(moved);
            wave_sync();
            vn += WB;
            if constexpr (PREP) {
                nxt = nxt2;
                if (vn < q1) nval = vis[nxt.idx & 0x7fffffffu];
                if (vn + WB < q1) nxt2 = rec[tile_record(T, vn + WB)];
            } else {
                if (vn < q1) nxt = rec[tile_record(T, vn)];
            }

            // groups of four slots with fixed offsets (one address update per
            // group); each slot's stage values are read while the previous
            // slot's products are formed
            struct Slot {
                R wt[WZ], fx[PI], fy[PI], fv[PI];
            };
            auto read_slot = [&](int slot, Slot& q) {
#pragma unroll
                for (int a = 0; a < WZ; ++a) q.wt[a] = st.words[slot][a];      // broadcast
#pragma unroll
                for (int i = 0; i < PI; ++i) {
                    q.fx[i] = st.wuv[slot][px[i]];
                    q.fy[i] = st.wuv[slot][W + px[i]];
                    q.fv[i] = st.wuv[slot][2 * W + py[i]];
                }
            };
            Slot q[2];            // slot j in q[j & 1]: two register sets, no copies
            read_slot(slot0, q[0]);
            for (int j0 = 0; j0 < n; j0 += 4) {
                const uint32_t m4 = uint32_t(move_mask >> j0) & 15u;
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int j = j0 + jj;
                    if (j >= n) break;
                    if (j + 1 < n) read_slot(slot0 + j + 1, q[(jj + 1) & 1]);
                    if (m4 & (1u << jj)) move_to(__builtin_amdgcn_readlane(d, j));
                    const Slot& c = q[jj & 1];
#pragma unroll
                    for (int i = 0; i < PI; ++i) {
                        const R gx = c.fx[i] * c.fv[i], gy = c.fy[i] * c.fv[i];
#pragma unroll
                        for (int a = 0; a < WZ; ++a) {
                            ax[i][a] += gx * c.wt[a];
                            ay[i][a] += gy * c.wt[a];
                        }
                    }
                }
            }
            wave_sync();
        }
#pragma unroll
        for (int i = 0; i < PI; ++i)
#pragma unroll
            for (int a = 0; a < WZ; ++a) add_cell(i, a);
    }
    __syncthreads();
    // write the tile: rows of kTileS cells
    for (int i = tid; i < nt_valid * kTileR * kTileS; i += NT) {
        const int ss = i % kTileS, rr = (i / kTileS) % kTileR, tt = i / (kTileR * kTileS);
        stack[tile_base(P, t0 - P.pl0 + tt, br, bs) * (kTileR * kTileS) + rr * kTileS + ss] = cpx<R>{tre[i], tim[i]};
    }
}

// Matrix products of the tile kernels: D (16 x 16) += A (16 x 4) B (4 x 16),
// lane l holding A[l % 16][l / 16], B[l / 16][l % 16] and, in element v, row
// mfma_row(v) of column l % 16 of D.
typedef float mfma_f4 __attribute__((ext_vector_type(4)));
typedef double mfma_d4 __attribute__((ext_vector_type(4)));
template <typename R>
struct Mfma;
template <>
struct Mfma<float> {
    using V = mfma_f4;
    static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
    static __device__ __forceinline__ V mul(float a, float b, V c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};
template <>
struct Mfma<double> {
    using V = mfma_d4;
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
    static __device__ __forceinline__ V mul(double a, double b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
};

// Scatter for W <= 8 (mat_scatter): over the records of one window the sums
//     cell (x, y, a) += sum_k [wu_k(x) wv_k(y)] [wt_k(a) V_k]
// are a product of a 64 x K matrix (rows the window's 8 x 8 pairs (x, y)) with a
// K x 16 one (columns the 8 layers a times real and imaginary), four 16 x 16 x 4
// matrix instructions per four records, summed in FP32 (FP64) as the vector
// instructions were.  A wave stages 8 records at a time, lane (record, h)
// evaluating segment h of the three kernel functions; each lands at its place of
// the window (the places off the support are zero).  The sums stay in the
// accumulators while the window does and are then added to the LDS tile, which
// holds doubles for both precisions: ds_add_f32 takes 3 clocks per active lane
// (192 for a full wave), ds_add_f64 8 for the wave.  On Earth-rotation tracks a
// window holds 28 visits at wide field (a start of one cell 14), so that 95 % of
// the matrix rows k carry a record.  Measured against the kernel of residue
// classes (k_grid_tiles), per call: wide field 2.12 -> 1.61 ms (FP32, shared
// binning) and 1.87 -> 1.55 (FP64), four channels at 1024^2 1.91 -> 0.95, W = 4
// 0.295 -> 0.249, W = 8 FP64 0.121 -> 0.085, 5,000 scattered visibilities
// 35 -> 21 us.
template <typename R, int W, int WZ>
struct MatScatterCfg {
    static constexpr int kWaves = sizeof(R) == 4 ? 8 : 4;        // two blocks per CU (80 KB of LDS)
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kBatch = 8;                             // records staged at a time
    static constexpr int kLT = 2 * kTileR * kTileS + 2;          // doubles between layers (skews them over the banks)
    static constexpr int kSlot = 48;                             // values between slots (8 wu, 8 wv, 16 b, padding)
};

// b of lane `from` (a value of the batch's record) for the lane's own record
__device__ __forceinline__ int lane_read(int v, int from) { return __builtin_amdgcn_ds_bpermute(from << 2, v); }
__device__ __forceinline__ float lane_read(float v, int from) {
    return __int_as_float(lane_read(__float_as_int(v), from));
}
__device__ __forceinline__ double lane_read(double v, int from) {
    return __hiloint2double(lane_read(__double2hiint(v), from), lane_read(__double2loint(v), from));
}

// Tiles a block of a matrix kernel takes one after the other: a block's start (its
// arguments, the list, the first records: four loads that wait for each other)
// took a quarter of its time, so a launch of many tiles gives each block several,
// a stride of the launch apart (neighbours, which differ little in work, then go
// to different blocks), the next one's records loaded during the current one.
// Below two rounds of resident blocks each block keeps one tile.  With the ranges
// from k_tile_list, wide field: FP32 scatter 1.61 -> 1.47 ms, FP64 1.55 -> 1.37;
// four channels at 1024^2 0.95 -> 0.86; three passes at 4096^2 8.43 -> 7.66.  The
// rest is issue: 18 vector and 13 scalar instructions per visit and a quarter of
// the time in the matrix units.
constexpr int kMostTiles = 16;
struct TileRun {
    int place, step, end;      // places of the list: place, place + step, ... < end
};
__device__ __forceinline__ bool tiles_of_block(const DevParams& P, const uint32_t* __restrict__ tpos, int resident,
                                               TileRun& run) {
    const int per_layer = P.nbs * P.nbr, a = (P.pl0 / kTileT) * per_layer;
    const int first = int(tpos[a]), cnt = int(tpos[a + (P.pln + kTileT - 1) / kTileT * per_layer]) - first;
    const int each = min(kMostTiles, max(1, cnt / (2 * resident)));
    run.step = (cnt + each - 1) / each;
    run.place = first + xcd_interleave<4>(blockIdx.x, run.step);
    run.end = first + cnt;
    return int(blockIdx.x) < run.step;
}

template <typename R, int W, int WZ, bool SAME, bool PREP>
__global__ void __launch_bounds__((MatScatterCfg<R, W, WZ>::kThreads)) k_grid_tiles_mat(const Rec<R>* __restrict__ rec,
                                                    const TileRec* __restrict__ tlist,
                                                    const uint32_t* __restrict__ tpos, DevParams P,
                                                    const R* __restrict__ coef_g, const R* __restrict__ coefz_g,
                                                    const cpx<R>* __restrict__ vis, cpx<R>* __restrict__ stack) {
    using Cfg = MatScatterCfg<R, W, WZ>;
    using M = Mfma<R>;
    constexpr int D = KernelDegree<R>::value, NW = Cfg::kWaves, NT = Cfg::kThreads, WB = Cfg::kBatch, LT = Cfg::kLT;
    constexpr int EUV = window_edge(W), ET = window_edge(WZ), BUV = 17 - W, BT = 17 - WZ;
    static_assert(W <= kWin && WZ <= W && WB * 8 == 64, "a wave stages 8 records, 8 segments each");
    __shared__ __align__(16) double cells[kTileT * LT];        // [t][r][s] real, imaginary
    __shared__ __align__(16) R stage[NW * WB * Cfg::kSlot];

    TileRun run;
    if (!tiles_of_block(P, tpos, 512, run)) return;     // unoccupied tiles are left unwritten and read as zero
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this wave's part of a tile's list: [q0, q1)
    auto part_of = [&](uint32_t total, uint32_t& q0, uint32_t& q1) {
        const uint32_t part = (total + NW - 1) / NW;
        q0 = min(total, part * uint32_t(wv));
        q1 = min(total, q0 + part);
    };
    // staging: lane (record lane % 8, segment h); segments past the width are zero
    const int slot = lane & 7, h = lane >> 3;
    R creg[D + 1], czreg[SAME ? 1 : D + 1];
#pragma unroll
    for (int k = 0; k <= D; ++k) {
        creg[k] = h < W ? coef_g[h * (D + 1) + k] : R(0);
        if constexpr (!SAME) czreg[k] = h < WZ ? coefz_g[h * (D + 1) + k] : R(0);
    }
    uint32_t q0, q1;
    part_of(tlist[run.place].total, q0, q1);
    Rec<R> nxt{};              // the lane's record of the next 64, and (PREP) its value
    cpx<R> nval{R(0), R(0)};
    if (q0 + uint32_t(lane) < q1) nxt = rec[tile_record(tlist[run.place], q0 + uint32_t(lane))];
    for (int i = tid; i < kTileT * LT; i += NT) cells[i] = 0.0;
    R* st = stage + wv * (WB * Cfg::kSlot);
    for (int i = lane; i < WB * Cfg::kSlot; i += 64) st[i] = R(0);
    if constexpr (PREP) {
        if (q0 + uint32_t(lane) < q1) nval = vis[nxt.idx & 0x7fffffffu];
    }
    R* my = st + slot * Cfg::kSlot;
    // operands: row i = 8 xb + y of block q is the pair (x, y), x = 4 xb + q
    const int kk = lane >> 4;
    const R* op = st + kk * Cfg::kSlot;
    const int at_u = ((lane >> 3) & 1) * 4, at_v = 8 + (lane & 7), at_b = 16 + (lane & 15);
    typename M::V acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = typename M::V{R(0), R(0), R(0), R(0)};
    __syncthreads();

    for (;;) {
        const TileRec& T = tlist[run.place];
        const int tile = int(T.tile);
        const int br = tile % P.nbr, bs = (tile / P.nbr) % P.nbs, bt = tile / (P.nbr * P.nbs);
        const int r0 = br * kTileR, s0 = bs * kTileS, t0 = bt * kTileT;
        const int nt_valid = min(kTileT, P.n_layers - t0 % (P.nbt * kTileT));   // layers of its channel
        const bool more = run.place + run.step < run.end;
        const TileRec& T2 = tlist[more ? run.place + run.step : run.place];
        uint32_t n0 = 0, n1 = 0;
        if (more) part_of(T2.total, n0, n1);
        int cur = -1;           // the window, packed
        auto flush = [&]() {
            const int wr = (cur & 255) - 128, ws = ((cur >> 8) & 255) - 128, wt = ((cur >> 16) & 255) - 128;
            const int t = wt + ((lane & 15) >> 1);
            if (unsigned(t) < unsigned(nt_valid)) {
                // the cells outside the tile go to the padding behind the layer, without a branch per cell
                double* base = cells + t * LT + (lane & 1);
                const int c0 = wr * kTileS + ws;
                bool sok[4];
                int off[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = M::row(lane, v), y = i & 7;
                    sok[v] = unsigned(ws + y) < unsigned(kTileS);
                    off[v] = c0 + (i >> 3) * 4 * kTileS + y;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int r = wr + 4 * (M::row(lane, v) >> 3) + q;
                        const int c = sok[v] && unsigned(r) < unsigned(kTileR) ? off[v] + q * kTileS : kTileR * kTileS;
                        atomicAdd(base + 2 * c, double(acc[q][v]));
                    }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = typename M::V{R(0), R(0), R(0), R(0)};
        };
        // the first records of the next tile, when this one's are all loaded
        auto load_next = [&]() {
            if (n0 + uint32_t(lane) < n1) nxt = rec[tile_record(T2, n0 + uint32_t(lane))];
        };
        if (q0 >= q1) {
            load_next();
            if constexpr (PREP) {
                if (n0 + uint32_t(lane) < n1) nval = vis[nxt.idx & 0x7fffffffu];
            }
        }
        for (uint32_t base = q0; base < q1; base += 64) {
            const int n = __builtin_amdgcn_readfirstlane(int(min(64u, q1 - base)));
            // the lane's record: window, place in it, value
            const int dr = wrap_offset(int(nxt.ruv & 0xffffu), r0, P.Np);
            const int ds = wrap_offset(int(nxt.ruv >> 16), s0, P.Np);
            const int dt = int(nxt.rt) - t0;
            auto place = [](int d, int B, int edge) {
                const int l = d & (kTileR - 1);
                return (l >= B ? l - B : l) % edge;
            };
            const int ou = place(dr, BUV, EUV), ov = place(ds, BUV, EUV), ot = place(dt, BT, ET);
            const int win = (dr - ou + 128) | ((ds - ov + 128) << 8) | ((dt - ot + 128) << 16);
            const int places = ou | (ov << 8) | (ot << 16);
            R nu0 = nxt.nu[0], nu1 = nxt.nu[1], nu2 = nxt.nu[2], v0 = nxt.v[0], v1 = nxt.v[1];
            if constexpr (PREP) {
                const double vx = double(nval.x), vy = (nxt.idx & 0x80000000u) ? -double(nval.y) : double(nval.y);
                const double co = double(nxt.v[0]), sn = -double(nxt.v[1]);
                v0 = R(vx * co - vy * sn);
                v1 = R(vx * sn + vy * co);
            }
            if (lane >= n) nu0 = nu1 = nu2 = v0 = v1 = R(0);        // finite weights, no value
            const int before = __shfl_up(win, 1, 64);
            const uint64_t moved = __ballot(lane < n && win != (lane == 0 ? cur : before));
            const bool last = base + 64 >= q1;
            const bool load = last ? n0 + uint32_t(lane) < n1 : base + 64 + uint32_t(lane) < q1;
            if (last) load_next();
            else if (load) nxt = rec[tile_record(T, base + 64 + uint32_t(lane))];
            // the values of those records are asked for once they have come
            const int vis_at = (min(n, 32) - 1) & ~7;
            for (int b0 = 0; b0 < n; b0 += WB) {
                {
                    const int from = b0 + slot;
                    const R a0 = lane_read(nu0, from), a1 = lane_read(nu1, from), a2 = lane_read(nu2, from);
                    const R x = lane_read(v0, from), y = lane_read(v1, from);
                    const int pl = (lane_read(places, from) + h * 0x010101) & 0x070707;
                    R hu = creg[D], hv = creg[D], ht = SAME ? creg[D] : czreg[D];
#pragma unroll
                    for (int k = D - 1; k >= 0; --k) {
                        hu = hu * a0 + creg[k];
                        hv = hv * a1 + creg[k];
                        ht = ht * a2 + (SAME ? creg[k] : czreg[k]);
                    }
                    my[pl & 255] = hu;
                    my[8 + ((pl >> 8) & 255)] = hv;
                    R* mb = my + 16 + 2 * (pl >> 16);
                    mb[0] = x * ht;
                    mb[1] = y * ht;
                }
                wave_sync();
#pragma unroll
                for (int g4 = 0; g4 < WB; g4 += 4) {
                    const int first = b0 + g4;
                    if (first >= n) break;
                    const R* o = op + g4 * Cfg::kSlot;
                    const R b = o[at_b], fv = o[at_v];
                    R fu[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) fu[q] = o[at_u + q] * fv;
                    const uint32_t m = uint32_t(moved >> first) & 15u;
                    if (m == 0) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[q] = M::mul(fu[q], b, acc[q]);
                        continue;
                    }
                    // the window moves inside the four: one product per window
                    for (int lo = 0; lo < 4;) {
                        if (m & (1u << lo)) {
                            if (cur >= 0) flush();
                            cur = __builtin_amdgcn_readlane(win, first + lo);
                        }
                        const uint32_t rest = m >> (lo + 1);
                        const int hi = rest ? lo + 1 + __builtin_ctz(rest) : 4;
                        const R bb = kk >= lo && kk < hi ? b : R(0);
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[q] = M::mul(fu[q], bb, acc[q]);
                        lo = hi;
                    }
                }
                wave_sync();
                if constexpr (PREP) {
                    if (b0 == vis_at && load) nval = vis[nxt.idx & 0x7fffffffu];
                }
            }
        }
        if (cur >= 0) flush();
        __syncthreads();
        // write the tile and clear it for the next one
        cpx<R>* dst = stack + tile_base(P, t0 - P.pl0, br, bs) * (kTileR * kTileS);
        const size_t layer = size_t(P.nbr) * P.nbs * (kTileR * kTileS);
        constexpr int LAYERS = NT / (kTileR * kTileS);       // layers written at a time
        static_assert(NT % (kTileR * kTileS) == 0, "a thread keeps its cell of every layer");
        const int c = tid % (kTileR * kTileS);
        for (int tt = tid / (kTileR * kTileS); tt < nt_valid; tt += LAYERS) {
            double2* at = reinterpret_cast<double2*>(cells + tt * LT + 2 * c);
            const double2 z = *at;
            dst[tt * layer + c] = cpx<R>{R(z.x), R(z.y)};
            *at = double2{0.0, 0.0};
        }
        if (!more) break;
        run.place += run.step;
        q0 = n0;
        q1 = n1;
        __syncthreads();
    }
}

// FP64 gather for W = 6 to 8 (mat_gather): for the records k of one window
//     out_k = sum_a wt_k(a) sum_(x, y) [wu_k(x) wv_k(y)] cell(x, y, a)
// the inner sums are a product of a K x 64 matrix (rows 16 records, columns the
// window's pairs (x, y)) with a 64 x 16 one (columns the 8 layers times real and
// imaginary), at most 16 matrix instructions of 16 x 16 x 4 per 16 records of a
// window; rows x of the window outside the tile are left out (a window at a
// tile's edge belongs to several tiles).  Rows that hold another window's record
// are computed and dropped.  The weights by layer and the sum over the layers
// follow on the vector units.  A wave stages kSlots records at a time as the
// scatter does.  Against a lane per record (k_degrid_tiles): wide field 2.80 ->
// 1.59 ms, 46,332 visibilities at 512^2 102 -> 63 us, 1,531 scattered ones 27 ->
// 16 us.  In FP32 a lane per record stays: half the LDS bytes and twice the
// vector rate make it the better one wherever a window holds few records
// (4096^2, 3 per window: 6.0 against 8.8 ms; 768^2, W = 6: 0.09 against 0.16)
// and as good where it holds 28 (wide field: 1.41 against 1.46).
template <typename R>
struct MatGatherCfg {
    static constexpr int kWaves = 4;                             // two blocks per CU (80 KB of LDS)
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kSlots = 16;                            // records staged at a time
    static constexpr int kSlot = 26;                             // values between slots (8 wu, 8 wv, 8 wt, padding)
    static constexpr int kLT = kTileR * kTileS + 2;              // cells between layers: a window's layers meet
                                                                 // distinct banks
};
// x of the lane n places back in its row of 16 (rotating)
template <int N>
__device__ __forceinline__ double row_ror(double x) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x120 + N, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x120 + N, 0xf, 0xf, true));
}

template <typename R, int W, int WZ, bool SAME>
__global__ void __launch_bounds__((MatGatherCfg<R>::kThreads)) __attribute__((amdgpu_waves_per_eu(2)))
    k_degrid_tiles_mat(const Rec<R>* __restrict__ rec, const TileRec* __restrict__ tlist,
                       const uint32_t* __restrict__ tpos, DevParams P, const R* __restrict__ coef_g,
                       const R* __restrict__ coefz_g, const cpx<R>* __restrict__ stack, cpx<R>* __restrict__ part,
                       size_t part_stride) {
    using Cfg = MatGatherCfg<R>;
    using M = Mfma<R>;
    constexpr int D = KernelDegree<R>::value, NW = Cfg::kWaves, NT = Cfg::kThreads, NS = Cfg::kSlots, LT = Cfg::kLT;
    constexpr int EUV = window_edge(W), ET = window_edge(WZ), BUV = 17 - W, BT = 17 - WZ;
    constexpr int STEP = NT / (kTileR * kTileS), PER = kTileT / STEP;        // a thread's cells: layers tl + STEP i
    static_assert(W <= kWin && WZ <= W && NT % (kTileR * kTileS) == 0, "a thread keeps its cell of every layer");
    __shared__ __align__(16) cpx<R> cells[kTileT * LT];          // [t][r][s]
    __shared__ __align__(16) R stage[NW * NS * Cfg::kSlot];

    TileRun run;
    if (!tiles_of_block(P, tpos, 512, run)) return;      // only occupied tiles are visited
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto part_of = [&](uint32_t total, uint32_t& q0, uint32_t& q1) {         // this wave's part of a tile's list
        const uint32_t each = (total + NW - 1) / NW;
        q0 = min(total, each * uint32_t(wv));
        q1 = min(total, q0 + each);
    };
    // staging: lane (record lane % 8, segment h); segments past the width are zero
    const int slot = lane & 7, h = lane >> 3;
    R creg[D + 1], czreg[SAME ? 1 : D + 1];
#pragma unroll
    for (int k = 0; k <= D; ++k) {
        creg[k] = h < W ? coef_g[h * (D + 1) + k] : R(0);
        if constexpr (!SAME) czreg[k] = h < WZ ? coefz_g[h * (D + 1) + k] : R(0);
    }
    // the tile's cells in the order pass A stored them
    const int e = tid % (kTileR * kTileS), tl = tid / (kTileR * kTileS);
    const size_t layer = size_t(P.nbr) * P.nbs * (kTileR * kTileS);
    cpx<R> cr[PER];
    auto load_cells = [&](int tile) {
        const int br = tile % P.nbr, bs = (tile / P.nbr) % P.nbs, t0 = tile / (P.nbr * P.nbs) * kTileT;
        const int nt_valid = min(kTileT, P.n_layers - t0 % (P.nbt * kTileT));
        const cpx<R>* src = stack + tile_base(P, t0 - P.pl0, br, bs) * (kTileR * kTileS) + e;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int tt = tl + STEP * i;
            cr[i] = tt < nt_valid ? src[tt * layer] : cpx<R>{R(0), R(0)};
        }
    };
    uint32_t q0, q1;
    part_of(tlist[run.place].total, q0, q1);
    Rec<R> nxt{};              // the lane's record of the next 64, its index and tile set
    uint32_t nxt_p = 0, nxt_m = 0;
    auto load_rec = [&](const TileRec& T, uint32_t v) {
        nxt_p = tile_record(T, v, nxt_m);
        nxt = rec[nxt_p];
    };
    if (q0 + uint32_t(lane) < q1) load_rec(tlist[run.place], q0 + uint32_t(lane));
    load_cells(int(tlist[run.place].tile));
    R* st = stage + wv * (NS * Cfg::kSlot);
    for (int i = lane; i < NS * Cfg::kSlot; i += 64) st[i] = R(0);
    // operands: lane (g, i) holds A row i (record), and B column i = 2 a + c; the
    // matrix step (x, half) joins the pairs (x, 4 half + g)
    const int g = lane >> 4, i16 = lane & 15;

    for (;;) {
        const TileRec& T = tlist[run.place];
        const int tile = int(T.tile);
        const int br = tile % P.nbr, bs = (tile / P.nbr) % P.nbs, bt = tile / (P.nbr * P.nbs);
        const int r0 = br * kTileR, s0 = bs * kTileS, t0 = bt * kTileT;
        const bool more = run.place + run.step < run.end;
        const TileRec& T2 = tlist[more ? run.place + run.step : run.place];
        uint32_t n0 = 0, n1 = 0;
        if (more) part_of(T2.total, n0, n1);
        {
            int rr, ss;
            degrid_place(e, bs, P.classes, rr, ss);
            cpx<R>* dst = cells + rr * kTileS + ss - s0;
#pragma unroll
            for (int i = 0; i < PER; ++i) dst[(tl + STEP * i) * LT] = cr[i];
        }
        __syncthreads();
        if (more) load_cells(int(T2.tile));
        if (q0 >= q1 && n0 + uint32_t(lane) < n1) load_rec(T2, n0 + uint32_t(lane));
        int cur = -1;                // the window whose cells are in b, packed
        R b[2 * kWin];
        for (uint32_t base = q0; base < q1; base += 64) {
            const int n = __builtin_amdgcn_readfirstlane(int(min(64u, q1 - base)));
            const int dr = wrap_offset(int(nxt.ruv & 0xffffu), r0, P.Np);
            const int ds = wrap_offset(int(nxt.ruv >> 16), s0, P.Np);
            const int dt = int(nxt.rt) - t0;
            auto place = [](int d, int B, int edge) {
                const int l = d & (kTileR - 1);
                return (l >= B ? l - B : l) % edge;
            };
            const int ou = place(dr, BUV, EUV), ov = place(ds, BUV, EUV), ot = place(dt, BT, ET);
            const int win = (dr - ou + 128) | ((ds - ov + 128) << 8) | ((dt - ot + 128) << 16);
            const int places = ou | (ov << 8) | (ot << 16);
            R nu0 = nxt.nu[0], nu1 = nxt.nu[1], nu2 = nxt.nu[2];
            if (lane >= n) nu0 = nu1 = nu2 = R(0);                  // finite weights
            // where this tile's part of the record goes: the slot of the tile's offset
            // from the record's own bin (no two tiles share a slot)
            const unsigned long long to = (unsigned long long)nxt_m * part_stride + nxt_p;
            const int to_lo = int(uint32_t(to)), to_hi = int(uint32_t(to >> 32));
            const int before = __shfl_up(win, 1, 64);
            const uint64_t moved = __ballot(lane > 0 && lane < n && win != before);
            if (base + 64 >= q1) {
                if (n0 + uint32_t(lane) < n1) load_rec(T2, n0 + uint32_t(lane));
            } else if (base + 64 + uint32_t(lane) < q1) {
                load_rec(T, base + 64 + uint32_t(lane));
            }
            for (int b0 = 0; b0 < n; b0 += NS) {
                const int ns = min(NS, n - b0);
                for (int p = 0; p < ns; p += 8) {
                    const int from = b0 + p + slot;
                    const R a0 = lane_read(nu0, from), a1 = lane_read(nu1, from), a2 = lane_read(nu2, from);
                    const int pl = (lane_read(places, from) + h * 0x010101) & 0x070707;
                    R hu = creg[D], hv = creg[D], ht = SAME ? creg[D] : czreg[D];
#pragma unroll
                    for (int k = D - 1; k >= 0; --k) {
                        hu = hu * a0 + creg[k];
                        hv = hv * a1 + creg[k];
                        ht = ht * a2 + (SAME ? creg[k] : czreg[k]);
                    }
                    R* my = st + (p + slot) * Cfg::kSlot;
                    my[pl & 255] = hu;
                    my[8 + ((pl >> 8) & 255)] = hv;
                    my[16 + (pl >> 16)] = ht;
                }
                wave_sync();
                const uint64_t mv = moved >> b0;
                for (int j = 0; j < ns;) {
                    // the next records of one window: [j, end)
                    const uint64_t rest = mv >> (j + 1);
                    const int end = min(min(j + 16, ns), rest ? j + 1 + int(__builtin_ctzll(rest)) : ns);
                    const int w = __builtin_amdgcn_readlane(win, b0 + j);
                    const int wr = (w & 255) - 128, ws = ((w >> 8) & 255) - 128, wt = ((w >> 16) & 255) - 128;
                    const bool lo = ws > -4, hi = ws < kTileS - 4;       // the window's halves in v that meet the tile
                    if (w != cur) {
                        cur = w;
                        const int t = wt + (i16 >> 1), s = ws + g;
                        const bool tok = unsigned(t) < unsigned(kTileT);
                        const bool ok0 = tok && unsigned(s) < unsigned(kTileS), ok1 = tok && unsigned(s + 4) < unsigned(kTileS);
                        const R* base_c = reinterpret_cast<const R*>(cells) + (i16 & 1);
                        const int c0 = ok0 ? t * LT + s : 0, c1 = ok1 ? t * LT + s + 4 : 0;
#pragma unroll
                        for (int x = 0; x < kWin; ++x) {
                            if (unsigned(wr + x) < unsigned(kTileR)) {
                                const int row = (wr + x) * kTileS;
                                const R y0 = base_c[2 * (c0 + row)], y1 = base_c[2 * (c1 + row)];
                                b[2 * x] = ok0 ? y0 : R(0);
                                b[2 * x + 1] = ok1 ? y1 : R(0);
                            }
                        }
                    }
                    const R* row = st + min(j + i16, NS - 1) * Cfg::kSlot;
                    R wu[kWin];
#pragma unroll
                    for (int x = 0; x < kWin; ++x) wu[x] = row[x];
                    const R v0 = row[8 + g], v1 = row[12 + g];
                    typename M::V d0{R(0), R(0), R(0), R(0)}, d1{R(0), R(0), R(0), R(0)};
#pragma unroll
                    for (int x = 0; x < kWin; ++x) {
                        if (unsigned(wr + x) < unsigned(kTileR)) {
                            if (lo) d0 = M::mul(wu[x] * v0, b[2 * x], d0);
                            if (hi) d1 = M::mul(wu[x] * v1, b[2 * x + 1], d1);
                        }
                    }
                    // times the layer weights, summed over the layers: lane 2 v + c takes row v
                    R out = R(0);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
#pragma clang fp contract(off)
                        R y = (d0[v] + d1[v]) * st[min(j + M::row(lane, v), NS - 1) * Cfg::kSlot + 16 + (i16 >> 1)];
                        // in this order, without fused multiply-adds, every lane forms the same
                        // sum, bit for bit: a record's result does not depend on its row
                        y += row_ror<8>(y);
                        y += row_ror<4>(y);
                        y += row_ror<2>(y);
                        out = (i16 >> 1) == v ? y : out;
                    }
                    const int k = M::row(lane, (i16 >> 1) & 3), from = b0 + j + k;
                    const uint32_t plo = uint32_t(lane_read(to_lo, from & 63)), phi = uint32_t(lane_read(to_hi, from & 63));
                    if (i16 < 8 && j + k < end)
                        reinterpret_cast<R*>(part + (((unsigned long long)phi << 32) | plo))[i16 & 1] = out;
                    j = end;
                }
                wave_sync();
            }
        }
        if (!more) break;
        run.place += run.step;
        q0 = n0;
        q1 = n1;
        __syncthreads();
    }
}

// Gather in FP32, and in FP64 for W < 6 and W > 8: lanes over records.  The tile
// sits in LDS as complex cells, rows kLR = 17 cells and layers kLT = 16 kLR + 8
// (FP64 16 kLR + 1) cells apart (the padding cells are zero), with a zero guard of (kLR + 1)(W - 1)
// cells before and after, so that for any support start (dr, ds) in [-(W-1), 15]
// the cell address base + kLR x + y of every support offset is inside the array.
// Each lane evaluates its own record's weights, sets those of out-of-tile indices
// to zero (the cells read there are finite neighbours or zeros), clamps the layer of
// each residue and sums the W^3 products; no cross-lane reduction is needed.
template <typename R, int W>
struct GatherCfg {
    // strides of rows and layers (cells), which skew them over the LDS banks: with a
    // layer one cell off too, the starts (t + 1, u) and (t, u + 1) of one window share
    // their banks, which cost records in order of windows (a shared binning's) up to a
    // third (46,000 visibilities at 512^2, prepared: 119 -> 96 us; tracks 1 % less)
    static constexpr int kLR = kTileS + 1;
    static constexpr int kLT = kTileR * kLR + (sizeof(R) == 4 ? 8 : 1);
    static_assert(15 * (kLR + 1) < kLT, "a support's last row of the last layer ends inside the guard");
    static constexpr int kGuard = (kLR + 1) * (W - 1);
    static constexpr int kCells = kTileT * kLT;
    static constexpr int kLen = kCells + 2 * kGuard;
};

// At least two waves per SIMD: left alone, the FP64 instances hold a layer's
// cell loads in flight in 320 registers (one wave per SIMD); at two waves they
// spill a little and run 1.5x faster (FP32 is at four waves either way).
template <typename R, int W, int WZ, bool SAME>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_degrid_tiles(const Rec<R>* __restrict__ rec,
                                                      const TileRec* __restrict__ tlist,
                                                      const uint32_t* __restrict__ tpos, DevParams P,
                                                      const R* __restrict__ coef_g,
                                                      const R* __restrict__ coefz_g,
                                                      const cpx<R>* __restrict__ stack, cpx<R>* __restrict__ part,
                                                      size_t part_stride) {
    using G = GatherCfg<R, W>;
    constexpr int D = KernelDegree<R>::value;
    constexpr int WB = 64;
    __shared__ cpx<R> g[G::kLen];
    __shared__ R coef[W * (D + 1)];
    __shared__ R coefz[SAME ? 1 : WZ * (D + 1)];

    const int place = tile_of_block(P, tpos);
    if (place < 0) return;     // only occupied tiles are visited
    const TileRec& T = tlist[place];
    const int tile = int(T.tile);
    const int br = tile % P.nbr, bs = (tile / P.nbr) % P.nbs, bt = tile / (P.nbr * P.nbs);
    const int r0 = br * kTileR, s0 = bs * kTileS, t0 = bt * kTileT;
    const int nt_valid = min(kTileT, P.n_layers - t0 % (P.nbt * kTileT));   // layers of its channel
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

    for (int i = tid; i < W * (D + 1); i += 256) coef[i] = coef_g[i];
    if (!SAME)
        for (int i = tid; i < WZ * (D + 1); i += 256) coefz[i] = coefz_g[i];
    __syncthreads();
    const uint32_t total = T.total;
    if (total == 0) return;     // a tile no visibility reaches is not read at all
    const uint32_t quarter = (total + 3) / 4;
    const uint32_t q0 = min(total, quarter * uint32_t(wv)), q1 = min(total, q0 + quarter);

    // (with a w-axis design of its own, W_z = 3 would then hold 170 registers, a wave less per SIMD)
    const std::conditional_t<SAME, HeldRanges, ReadRanges> ranges(T);
    Rec<R> nxt;
    uint32_t nxt_p = 0, nxt_m = 0;
    if (q0 + uint32_t(lane) < q1) {
        nxt_p = ranges.record(q0 + uint32_t(lane), nxt_m);
        nxt = rec[nxt_p];
    }
    for (int i = tid; i < G::kLen; i += 256) {
        const int c = i - G::kGuard;
        const int tt = c / G::kLT, rem = c % G::kLT, rr = rem / G::kLR, ss = rem % G::kLR;
        if (c < 0 || tt >= nt_valid || rr >= kTileR || ss >= kTileS) g[i] = cpx<R>{R(0), R(0)};
    }
    // the tile's cells, in the order pass A stored them, one of each layer per thread
    {
        int rr, ss;
        degrid_place(tid, bs, P.classes, rr, ss);
        const cpx<R>* src = stack + tile_base(P, t0 - P.pl0, br, bs) * (kTileR * kTileS) + tid;
        const size_t layer = size_t(P.nbr) * P.nbs * (kTileR * kTileS);
        cpx<R>* dst = g + G::kGuard + rr * G::kLR + ss - s0;
#pragma unroll 4
        for (int tt = 0; tt < nt_valid; ++tt) dst[tt * G::kLT] = src[tt * layer];
    }
    __syncthreads();

    for (uint32_t base = q0; base < q1; base += WB) {
        const bool live = base + uint32_t(lane) < q1;
        const Rec<R> r = nxt;
        const uint32_t p = nxt_p, m = nxt_m;
        const uint32_t vn = base + WB + uint32_t(lane);
        if (vn < q1) {
            nxt_p = ranges.record(vn, nxt_m);
            nxt = rec[nxt_p];
        }
        if (!live) continue;

        const int dr = wrap_offset(int(r.ruv & 0xffffu), r0, P.Np);
        const int ds = wrap_offset(int(r.ruv >> 16), s0, P.Np);
        const int dt = int(r.rt) - t0;
        R wu[W], wv_[W], wt[WZ];
        record_weights<R, W, WZ, SAME>(r, coef, coefz, wu, wv_, wt);
#pragma unroll
        for (int a = 0; a < W; ++a) {
            wu[a] = unsigned(dr + a) < unsigned(kTileR) ? wu[a] : R(0);
            wv_[a] = unsigned(ds + a) < unsigned(kTileS) ? wv_[a] : R(0);
        }
#pragma unroll
        for (int a = 0; a < WZ; ++a) wt[a] = unsigned(dt + a) < unsigned(nt_valid) ? wt[a] : R(0);
        const cpx<R>* row = g + (G::kGuard + dr * G::kLR + ds);
        R sx = R(0), sy = R(0);
#pragma unroll
        for (int a = 0; a < WZ; ++a) {
            const int tt = min(max(dt + a, 0), kTileT - 1);
            const cpx<R>* pa = row + tt * G::kLT;
            R ax = R(0), ay = R(0);
#pragma unroll
            for (int x = 0; x < W; ++x) {
                R bx = R(0), by = R(0);
#pragma unroll
                for (int y = 0; y < W; ++y) {
                    const cpx<R> q = pa[x * G::kLR + y];
                    bx += q.x * wv_[y];
                    by += q.y * wv_[y];
                }
                ax += bx * wu[x];
                ay += by * wu[x];
            }
            sx += ax * wt[a];
            sy += ay * wt[a];
        }
        // this tile's part of record p, in the slot of the tile's offset from
        // the record's own bin (no two tiles share a slot)
        part[(size_t)m * part_stride + p] = cpx<R>{sx, sy};
    }
}

// Sum of each record's parts over the tiles it reaches (slot m is written by
// the tile one step forward along the axes of m, present when the record's
// touch class contains m), times the phase exp(-i 2 pi w (n0 - 1)), conjugated
// for a folded visibility, stored to its visibility.  The M - n_rec skipped
// visibilities, whose indices follow the records, are zero.
template <typename R>
__global__ void k_degrid_finish(const Rec<R>* __restrict__ rec, const uint32_t* __restrict__ n_rec,
                                const cpx<R>* __restrict__ part, size_t part_stride, size_t M, int W, int Wz,
                                cpx<R>* __restrict__ vis) {
    const size_t p = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= M) return;
    if (p >= *n_rec) {
        vis[rec[p].idx] = cpx<R>{R(0), R(0)};
        return;
    }
    const Rec<R> r = rec[p];
    const int c = class_of(int(r.rt) & (kTileT - 1), int(r.ruv & 0xffffu) & (kTileR - 1),
                           int(r.ruv >> 16) & (kTileS - 1), 17 - Wz, 17 - W);
    R sx = R(0), sy = R(0);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        if ((c & m) == m) {
            const cpx<R> q = part[(size_t)m * part_stride + p];
            sx += q.x;
            sy += q.y;
        }
    }
    R ox = sx * r.v[0] - sy * r.v[1], oy = sx * r.v[1] + sy * r.v[0];
    if (r.idx & 0x80000000u) oy = -oy;
    vis[r.idx & 0x7fffffffu] = cpx<R>{ox, oy};
}

// --------------------------------------------------------------- FFT passes --
//
// The stack is tiled: [t][u tile][v tile][16 x 16 cells], [r][s] within a tile
// in the grid direction, class by class in the degrid direction (degrid_cell).
// Pass A transforms along s and writes (reads, in the degrid direction) the
// intermediate [t][q / 16][r / 16][16 q][16 r] in segments of up to 16 consecutive
// r, pass B transforms its whole lines along r (q is the image row).  Image rows
// j <-> q and columns i <-> p.  The FFT output bin f of a line maps to image index
// (f + N/2) mod N' and is kept when below N (Algorithm 5 step 3c); the degrid
// input places image index p at bin (p - N/2) mod N' (zero padding, Algorithm 6
// step 3b).

template <typename R, int NP>
struct FftCfg {
    static constexpr int N = NP;
    static constexpr int T = N / 16;
    // lines per block for the row passes: at least ~256 threads; lengths 3 2^a
    // (T = 3 2^b) take 384 threads in FP32, so that 2048 rows fill whole rounds
    // of blocks (one 192-thread line per block left a partly empty last round;
    // FP64 at 384 threads measured 28 % slower)
    static constexpr int kNLr =
        (T >= 256) ? 1 : (N % 3 == 0 && T < 384 && sizeof(R) == 4) ? 384 / T : 256 / T;
};

// (f + N/2) mod N' for a bin f < N' (image index of FFT bin f, or the bin of
// image index f)
template <int NP>
__device__ __forceinline__ int shift_half(int f, int half) {
    const int q = f + half;
    return q >= NP ? q - NP : q;
}

// Pass A splits a line of N' = C F cells into C classes of outputs (f = C a + b
// for class b), each an F-point transform of F <= 1024 points:
//     X[C a + b] = sum_n W_F^(n a) W_N'^(n b) sum_m x[n + F m] W_C^(m b).
// A block holds kRows lines of a row of tiles at one class, a line per T = F/16
// lanes of one wave (no block barrier inside a transform), so that the lines fit
// in its registers and LDS and leave transposed, in segments of kRows
// frequencies r: no pass over the intermediate is spent on transposing it.  The
// classes of a line read the same inputs, which their blocks share in the L2: of
// the degrid direction's reads 84 % hit it at N' = 4096 and 93 % at 8192 (eight
// classes: 18 TB/s through the L2, 6.3 GB of 133 from memory).
// Bound by latency and VALU issue (vector instructions on 53-69 % of a SIMD's
// cycles, two blocks of 8 waves per CU).  Wide field (N' = 4096, 49 layers, one pass), with
// the transpose of the intermediate that a whole-line pass needs: FP32 grid
// 2.13 -> 1.56 ms, degrid 2.06 -> 1.83; FP64 4.55 -> 2.96 and 4.58 -> 3.43;
// N' = 3072 FP32 degrid 1.63 -> 0.94.  Rows are dealt to the XCDs in turn: the
// marked rows thin out towards the upper layers, and with a contiguous range of
// rows per XCD the grid direction took 2.90 ms.  At kRows = 16 (one block of
// 1024 threads per CU) FP32 took 2.99 ms.  Twiddles gathered from the table of
// N' roots instead of pass_a_table's order cost 0.65 ms.
template <typename R, int NP>
struct PassACfg {
    static constexpr int kClasses = pass_a_classes(NP);
    static constexpr int F = NP / kClasses, T = F / 16;
    // two blocks per CU: at most 512 threads of 128 registers (FP32) or 256 of 256 (FP64), 80 KB of LDS
    static constexpr int kMost = sizeof(R) == 8 ? 256 : 512;
    static constexpr int kRows = 16 * T <= kMost ? 16 : kMost / T;
    static constexpr int kHalves = kTileR / kRows;               // blocks per row of tiles and class
    static constexpr int kThreads = kRows * T;
    static constexpr int kWaves = kThreads < kMost ? 1 : sizeof(R) == 8 ? 2 : 4;     // per SIMD, as two full blocks hold
    static_assert(T <= 64 && 64 % T == 0 && (F & (F - 1)) == 0, "a line's lanes lie in one wave");
    // degrid blocks that take several layers: from N' = 2048 to 6144 (one layer each: 2.00 ->
    // 1.83 ms at wide field, FP64 3.81 -> 3.43; N' = 6144 4.23 -> 4.20 and 8.20 -> 7.87); with the
    // loop's registers N' = 8192 (8 classes) and the shorter transforms took 2-6 % longer, N' = 1024
    // 3 % (FP32; 2 % less in FP64)
    static constexpr bool kDegridLoop = F == 1024 && kClasses >= 2 && kClasses <= 6;
    // line stride in LDS: the transposed accesses of kRows lines meet distinct banks
    static constexpr int kBanks = 256 / int(sizeof(cpx<R>));
    static constexpr int LP = (LinePad<F>::size + kBanks - 1) / kBanks * kBanks + (kBanks >= kRows ? kBanks / kRows : 1);
};

// grid pass A: IFFT along s of kRows lines of a row of tiles for one class,
// image rows q kept, written to the intermediate.  The marked tiles of the row
// (about a fifth of them at wide field) are listed and only they are read; a row
// of tiles with none marked is neither transformed nor written (pass B reads it
// as zeros).  A block takes `each` layers of a tile layer, whose marks they
// share, and loads the next one's cells while it transforms (a layer per block:
// 1.76 ms at wide field, FP64 3.49; 16 cells instead of 8 in flight spill: 1.66).
// Layer t of the pass is virtual layer t + t_base; in a batched call
// (chl = the channels' layer stride, else 0) a padding layer (virtual layer mod
// chl >= n_layers) is skipped.
template <typename R, int NP>
__global__ void __launch_bounds__((PassACfg<R, NP>::kThreads)) __attribute__((amdgpu_waves_per_eu(PassACfg<R, NP>::kWaves)))
    k_grid_fft_a(const cpx<R>* __restrict__ stack, const uint32_t* __restrict__ mask, cpx<R>* __restrict__ inter,
                 const cpx<R>* __restrict__ tw, int N, int n_layers, int chl, int nbr, int t_base, int pln,
                 int each) {
    using A = PassACfg<R, NP>;
    constexpr int C = A::kClasses, F = A::F, T = A::T, RW = A::kRows, LP = A::LP, NB = NP / kTileS, TH = A::kThreads;
    constexpr int MW = mask_words(NB), PART = RW * kTileS;       // cells of a tile in the block
    // G groups of PART threads (or one of fewer, Q cells each) share out the cells n = s mod F
    // by their tile n / 16 mod G
    constexpr int G = T >= 16 ? T / 16 : 1, Q = T >= 16 ? 1 : 16 / T, EG = F / kTileS / G * C;
    constexpr PassATable TB = pass_a_table(NP);
    __shared__ cpx<R> buf[RW * LP];
    __shared__ cpx<R> tab[TB.second > 0 ? TB.second : 1];
    __shared__ uint16_t list[G * EG];
    // the tiles' twiddles, where two blocks still fit in a CU's LDS with them
    constexpr bool TURNS = sizeof(R) == 4 || G * EG <= 384;
    __shared__ cpx<R> tile_turn[TURNS ? G * EG : 1];
    __shared__ int count[G];
    __shared__ uint32_t empty[G];        // bit k: no marked tile among the parts of n / 16 = k G + group
    int lb = xcd_interleave<A::kHalves * C>(blockIdx.x, gridDim.x);
    const int b = lb % C;
    lb /= C;
    const int h = lb % A::kHalves;
    lb /= A::kHalves;
    // the block's layers, of one tile layer; padding layers of a channel (at a tile layer's end) left out
    const int rt = lb % nbr, first = lb / nbr * each;
    int end = min(pln, first + each);
    if (chl > 0) end = min(end, first + max(0, n_layers - (first + t_base) % chl));
    if (first >= end) return;
    const uint32_t* mrow = mask + size_t(((first + t_base) / kTileT) * nbr + rt) * MW;     // the row's marked tiles
    uint32_t any = 0;
#pragma unroll
    for (int i = 0; i < MW; ++i) any |= mrow[i];
    if (any == 0) return;
    const int tid = threadIdx.x, line = tid / T, j = tid % T;
    // each group's marked tiles, the parts m of one n / 16 together, the last of them flagged
    {
        constexpr int STEP = (TH < 64 ? TH : 64) / C * C;
        const int lane = tid & 63, w = tid >> 6;
        if (w < G) {
            int n = 0;
            uint32_t none = 0;
            for (int i0 = 0; i0 < EG; i0 += STEP) {
                const int i = i0 + lane, m = i % C, bs = i / C * G + w + m * (F / kTileS);
                const bool on = lane < STEP && i < EG && ((mrow[bs >> 5] >> (bs & 31)) & 1u);
                const uint64_t all = __ballot(on);
                if (on) {
                    const bool last = ((all >> lane) >> 1 & ((1ull << (C - 1 - m)) - 1ull)) == 0ull;
                    const int at = w * EG + n + __popcll(all & ((1ull << lane) - 1ull));
                    list[at] = uint16_t(bs | (last ? 0x8000 : 0));
                    if constexpr (TURNS) tile_turn[at] = tw[bs * kTileS * b % NP];
                }
                const uint64_t here = (all >> lane) & ((1ull << C) - 1ull);
                none |= lane < STEP && i < EG && m == 0 && here == 0ull ? 1u << (i / C) : 0u;
                n += __popcll(all);
            }
#pragma unroll
            for (int o = (TH < 64 ? TH : 64) / 2; o > 0; o >>= 1) none |= uint32_t(__shfl_xor(int(none), o, 64));
            if (lane == 0) {
                count[w] = n;
                empty[w] = none;
            }
        }
    }
    for (int i = tid; i < TB.second; i += TH) tab[i] = tw[NP + i];
    __syncthreads();
    const int g = G > 1 ? __builtin_amdgcn_readfirstlane(tid / PART) : 0, e0 = tid % PART;
    const int n_list = __builtin_amdgcn_readfirstlane(count[g]);
    const uint32_t none = uint32_t(__builtin_amdgcn_readfirstlane(int(empty[g])));
    constexpr int kBatch = (8 + Q - 1) / Q;
    cpx<R> turn[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) turn[q] = tw[(e0 + q * TH) % kTileS * b];
    cpx<R> x[kBatch][Q];
    auto load = [&](int t, int base) {
        const cpx<R>* src = stack + (size_t(t) * nbr + rt) * (size_t(NB) * kTileR * kTileS) + h * PART;
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (base + u < n_list) {
                const int bs = __builtin_amdgcn_readfirstlane(int(list[g * EG + base + u])) & 0x7fff;
#pragma unroll
                for (int q = 0; q < Q; ++q) x[u][q] = src[size_t(bs) * (kTileR * kTileS) + (e0 + q * TH)];
            }
    };
    load(first, 0);
    const int half = N / 2;
    for (int t = first; t < end; ++t) {
        // buf[r][n] = sum_m x[n + F m] W_N'^((n + F m) b): each cell of the marked
        // tiles is read once, kBatch tiles in flight per thread (the next layer's
        // first ones during this layer's transform); W_N'^(s b) is the tile's
        // W_N'^(16 bs b) (wave-uniform) times the cell's W_N'^((s mod 16) b).  A
        // group's threads write every n of theirs.
        if (t > first) __syncthreads();
        for (uint32_t z = none; z; z &= z - 1) {
            const int n16 = __builtin_ctz(z) * G + g;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int e = e0 + q * TH;
                buf[e / kTileS * LP + lpad(n16 * kTileS + e % kTileS)] = cpx<R>{R(0), R(0)};
            }
        }
        cpx<R> acc[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[q] = cpx<R>{R(0), R(0)};
        for (int base = 0; base < n_list; base += kBatch) {
            if (base > 0) load(t, base);
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                if (base + u < n_list) {
                    const int en = __builtin_amdgcn_readfirstlane(int(list[g * EG + base + u])), bs = en & 0x7fff;
                    const cpx<R> w = TURNS ? tile_turn[g * EG + base + u] : tw[bs * kTileS * b % NP];
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        acc[q].x += x[u][q].x * w.x - x[u][q].y * w.y;
                        acc[q].y += x[u][q].x * w.y + x[u][q].y * w.x;
                        if (en & 0x8000) {
                            const int e = e0 + q * TH, n = (bs * kTileS + e % kTileS) & (F - 1);
                            buf[e / kTileS * LP + lpad(n)] = cmul(acc[q], turn[q]);
                            acc[q] = cpx<R>{R(0), R(0)};
                        }
                    }
                }
            }
        }
        if (t + 1 < end) load(t + 1, 0);
        __syncthreads();
        cpx<R>* lbuf = buf + line * LP;
        const int pj = lpad(j);
        cpx<R> v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = lbuf[lpad_at<T>(j, pj, k)];
        fft_wave<R, F, +1>(v, lbuf, tab, tw + NP + TB.second, j);
        // class output a is bin f = C a + b, image row (f + N/2) mod N': the kept
        // ones are a < a0 (image rows from N/2) and a >= a1 (image rows below N/2)
        const int a0 = (N - half - b + C - 1) / C, a1 = (NP - half - b + C - 1) / C;
        wave_sync();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int a = j + T * k;
            if (a < a0 || a >= a1) lbuf[lpad_at<T>(j, pj, k)] = v[k];
        }
        __syncthreads();
        // lanes over r; step T classes outputs = C T image rows
        const int r = tid % RW, i0 = tid / RW;
        cpx<R>* dst = inter + (size_t(t) * inter_blocks(N) * nbr + rt) * 256 + h * RW;          // block-uniform
        auto put = [&](int a, int hi, int q0) {       // outputs a, a + T, ... < hi; a = 0 is image row q0
            const cpx<R>* from = buf + r * LP;
            if constexpr (C * T % 16 == 0 && T % 16 == 0) {
                const int q = q0 + C * a;
                uint32_t to = uint32_t(q >> 4) * uint32_t(nbr * 256) + uint32_t((q & 15) * 16 + r);
                from += lpad(a);
                for (; a < hi; a += T, to += uint32_t(C * T / 16) * uint32_t(nbr * 256), from += T + T / 16) dst[to] = *from;
            } else {
                for (; a < hi; a += T) {
                    const int q = q0 + C * a;
                    dst[uint32_t(q >> 4) * uint32_t(nbr * 256) + uint32_t((q & 15) * 16 + r)] = from[lpad(a)];
                }
            }
        };
        put(i0, min(a0, F), b + half);
        if (a1 < F) put(a1 + i0, F, b + half - NP);
    }
}

// Offset of frequency r within a row q of the intermediate.
__device__ __forceinline__ int inter_cell(int r) { return (r >> 4) * 256 + (r & 15); }

// Bit k set when frequency r = j + T k (the k-th value of thread j of a line)
// lies in a marked row of tiles of the tile layer whose marks start at `mark`.
template <int T>
__device__ __forceinline__ uint32_t live_mask(const uint8_t* __restrict__ mark, int j) {
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) m |= uint32_t(mark[(j + T * k) / kTileR] != 0) << k;
    return m;
}

// grid pass B: IFFT along r of intermediate rows [t][q][:] for every layer t,
// w-screen exp(+i 2 pi t z) and accumulation of the real part in registers
// (Algorithm 5 steps 3b-4), then the 3-D correction (step 5): dirty[q][p].
// One launch covers a segment of P.pln consecutive layers of one channel: the
// segment starts at layer seg0 of the pass's buffer and at layer tloc0 of the
// channel; `accumulate` adds to the map instead of writing it.  Where the image
// has too few rows to fill the chip, gridDim.y parts of the layers run in blocks
// of their own and leave their uncorrected sums in `partial` ([part][N][N]) for
// k_map_sum.
template <typename R, int NP>
__global__ void __launch_bounds__((FftCfg<R, NP>::kNLr * FftCfg<R, NP>::T)) __attribute__((amdgpu_waves_per_eu(2)))
    k_grid_fft_b(const cpx<R>* __restrict__ inter, const uint8_t* __restrict__ rows, const cpx<R>* __restrict__ tw,
                 const R* __restrict__ corr, R* __restrict__ dirty, R* __restrict__ partial, DevParams P, int seg0,
                 int tloc0, int accumulate) {
    using C = FftCfg<R, NP>;
    constexpr int Np = C::N, T = C::T, NL = C::kNLr, LP = LinePad<Np>::size;
    __shared__ cpx<R> buf[NL * LP];
    const int N = P.N, half = N / 2;
    const int line = threadIdx.x / T, j = threadIdx.x % T;
    const int q = xcd_remap(blockIdx.x, gridDim.x) * NL + line;
    const bool row_ok = q < N;
    const int qq = row_ok ? q : 0;
    cpx<R>* lbuf = buf + line * LP;
    double z[16];
    R acc[16];
    uint32_t in = 0;        // bit k: bin j + T k is an image column
    const double m = double(qq - half) * P.dl;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int f = j + T * k;
        const int p = shift_half<Np>(f, half);
        in |= uint32_t(row_ok && p < N) << k;
        const double l = double(min(p, N - 1) - half) * P.dl;   // bins outside the image are not used
        const double r2 = l * l + m * m;
        const double nm1 = -r2 / (1.0 + sqrt(1.0 - r2));     // n - 1
        z[k] = nm1 / P.nscale + P.zshift;                     // (n - n0) / n_scale
        acc[k] = R(0);
    }
    // bit k: frequency r = j + T k lies in a row of tiles with an occupied tile
    // in the current tile layer (the others are zero and not stored)
    uint32_t live = 0;
    int live_layer = -1;
    const int per = (P.pln + gridDim.y - 1) / gridDim.y, t1 = min(P.pln, int(blockIdx.y + 1) * per);
    for (int t = blockIdx.y * per; t < t1; ++t) {
        const cpx<R>* src = inter + ((size_t)(seg0 + t) * inter_blocks(N) + (qq >> 4)) * (P.nbr * 256) + (qq & 15) * 16;
        const int tile_layer = __builtin_amdgcn_readfirstlane((P.pl0 + seg0 + t) / kTileT);
        if (tile_layer != live_layer) {
            live_layer = tile_layer;
            live = live_mask<T>(rows + (size_t)tile_layer * P.nbr, j);
        }
        cpx<R> v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = (live >> k) & 1u ? src[inter_cell(j + T * k)] : cpx<R>{R(0), R(0)};
        // FP64 reads the twiddles again for each layer: kept in registers across the layers
        // (30 of them) they left one wave per SIMD (wide field: grid 2.15 -> 1.94 ms, degrid
        // 2.10 -> 1.69).  In FP32 they stay (read again: 0.78 -> 0.86 and 0.71 -> 0.86 ms).
        // The offset is hidden from the compiler, not the pointers, whose loads would then be
        // flat ones, which wait for the LDS.  The FP64 kernel holds 256 registers and spills
        // up to 58 words a thread (N' = 3 2^a; 40 at 4096), most of them z.
        int again = 0;
        if constexpr (sizeof(R) == 8) asm volatile("" : "+s"(again));
        const cpx<R>*root = tw + again, *tab = root + line_table_at(NP);
        fft_line<R, NP, +1>(v, lbuf, root, tab, j);
        const double tl = double(tloc0 + t + P.t_lo) + P.tphase;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if ((in >> k) & 1u) {
                R s, c;
                phase_turns(tl * z[k], &s, &c);
                acc[k] += v[k].x * c - v[k].y * s;
            }
        }
    }
    if (!row_ok) return;
    if (gridDim.y > 1) {
        R* out = partial + (size_t(blockIdx.y) * N + q) * N;
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if ((in >> k) & 1u) out[shift_half<Np>(j + T * k, half)] = acc[k];
        return;
    }
    // the channel's first layer segment writes the map, later ones add to it
#pragma unroll
    for (int k = 0; k < 16; ++k)
        if ((in >> k) & 1u) {
            const size_t o = (size_t)q * N + shift_half<Np>(j + T * k, half);
            const R d = acc[k] * corr[o];
            dirty[o] = accumulate ? dirty[o] + d : d;
        }
}

// Sum of the parts that a split pass B left, and the correction.
template <typename R>
__global__ void __launch_bounds__(256) k_map_sum(const R* __restrict__ partial, int parts, const R* __restrict__ corr,
                                                 R* __restrict__ dirty, int n, int accumulate) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    R a = R(0);
#pragma unroll 4
    for (int p = 0; p < parts; ++p) a += partial[size_t(p) * n + i];
    const R d = a * corr[i];
    dirty[i] = accumulate ? dirty[i] + d : d;
}

// degrid pass B': for each image row q and layer t: f h_x h_y h_z exp(-i 2 pi t z)
// zero-padded along p, FFT along p -> intermediate [t][q][r] (Algorithm 6 steps 2-3).
// Segments of one channel's layers as for k_grid_fft_b; gridDim.y parts of the
// layers run in blocks of their own.
template <typename R, int NP>
__global__ void __launch_bounds__((FftCfg<R, NP>::kNLr * FftCfg<R, NP>::T))
    k_degrid_fft_b(const R* __restrict__ image, const R* __restrict__ corr, const cpx<R>* __restrict__ tw,
                   const uint8_t* __restrict__ rows, cpx<R>* __restrict__ inter, DevParams P, int seg0, int tloc0) {
    using C = FftCfg<R, NP>;
    constexpr int Np = C::N, T = C::T, NL = C::kNLr, LP = LinePad<Np>::size;
    __shared__ cpx<R> buf[NL * LP];
    const int N = P.N, half = N / 2;
    const int line = threadIdx.x / T, j = threadIdx.x % T;
    const int q = xcd_remap(blockIdx.x, gridDim.x) * NL + line;
    const bool row_ok = q < N;
    const int qq = row_ok ? q : 0;
    cpx<R>* lbuf = buf + line * LP;
    double z[16];
    R g[16];
    const double m = double(qq - half) * P.dl;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int f = j + T * k;
        const int p = shift_half<Np>(f, half);
        const bool ok = row_ok && p < N;
        g[k] = ok ? image[(size_t)qq * N + p] * corr[(size_t)qq * N + p] : R(0);
        const double l = double(min(p, N - 1) - half) * P.dl;   // keeps z finite on padding bins
        const double r2 = l * l + m * m;
        const double nm1 = -r2 / (1.0 + sqrt(1.0 - r2));
        z[k] = nm1 / P.nscale + P.zshift;
    }
    uint32_t live = 0;
    int live_layer = -1;
    const int per = (P.pln + gridDim.y - 1) / gridDim.y, t1 = min(P.pln, int(blockIdx.y + 1) * per);
    for (int t = blockIdx.y * per; t < t1; ++t) {
        const double tl = double(tloc0 + t + P.t_lo) + P.tphase;
        cpx<R> v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            R s, c;
            phase_turns(-tl * z[k], &s, &c);
            v[k] = cpx<R>{g[k] * c, g[k] * s};
        }
        int again = 0;
        if constexpr (sizeof(R) == 8) asm volatile("" : "+s"(again));      // as in k_grid_fft_b
        const cpx<R>*root = tw + again, *tab = root + line_table_at(NP);
        fft_line<R, NP, -1>(v, lbuf, root, tab, j);
        if (row_ok) {
            // only frequencies r of rows of tiles with an occupied tile are used later
            const int tile_layer = __builtin_amdgcn_readfirstlane((P.pl0 + seg0 + t) / kTileT);
            if (tile_layer != live_layer) {
                live_layer = tile_layer;
                live = live_mask<T>(rows + (size_t)tile_layer * P.nbr, j);
            }
            cpx<R>* dst = inter + ((size_t)(seg0 + t) * inter_blocks(N) + (q >> 4)) * (P.nbr * 256) + (q & 15) * 16;
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if ((live >> k) & 1u) store_stream(dst + inter_cell(j + T * k), v[k]);
        }
    }
}

// degrid pass A': for each layer t and frequency r: the intermediate column
// [t][:][r] placed at its bins and zero-padded along q, FFT along q, the marked
// tiles of the stack written (the gather reads no other); class b holds the
// outputs s = C a + b, which a tile stores class by class (degrid_cell).  A row
// of tiles with none marked is skipped.  Layers and padding layers as for
// k_grid_fft_a.
template <typename R, int NP>
__global__ void __launch_bounds__((PassACfg<R, NP>::kThreads)) __attribute__((amdgpu_waves_per_eu(PassACfg<R, NP>::kWaves)))
    k_degrid_fft_a(const cpx<R>* __restrict__ inter, const uint32_t* __restrict__ mask, const cpx<R>* __restrict__ tw,
                   cpx<R>* __restrict__ stack, int N, int n_layers, int chl, int nbr, int t_base, int pln,
                   int each) {
    using A = PassACfg<R, NP>;
    constexpr int C = A::kClasses, F = A::F, T = A::T, RW = A::kRows, LP = A::LP, NB = NP / kTileS;
    constexpr int MW = mask_words(NB), TE = kTileR * kTileS;
    constexpr PassATable TB = pass_a_table(NP);
    __shared__ cpx<R> buf[RW * LP];
    __shared__ cpx<R> tab[TB.second > 0 ? TB.second : 1];
    int lb = xcd_interleave<A::kHalves * C>(blockIdx.x, gridDim.x);
    const int b = lb % C;
    lb /= C;
    const int h = lb % A::kHalves;
    lb /= A::kHalves;
    // the block's layers, as for k_grid_fft_a (or one)
    if constexpr (!A::kDegridLoop) each = 1;
    const int rt = lb % nbr, first = lb / nbr * each;
    int end = min(pln, first + each);
    if (chl > 0) end = min(end, first + max(0, n_layers - (first + t_base) % chl));
    if (first >= end) return;
    if constexpr (!A::kDegridLoop) end = first + 1;
    const uint32_t* mrow = mask + size_t(((first + t_base) / kTileT) * nbr + rt) * MW;
    uint32_t mw[MW + 1], any = 0;                              // the row's marks (block-uniform)
#pragma unroll
    for (int i = 0; i < MW; ++i) any |= mw[i] = mrow[i];
    mw[MW] = 0;
    if (any == 0) return;
    const int tid = threadIdx.x;
    for (int i = tid; i < TB.second; i += A::kThreads) tab[i] = tw[NP + i];
    // lanes over r: y[n] = W_N'^(-n b) sum_m x[n + F m] W_C^(-m b) of line r,
    // n = n0 + T k; bin f = n + F m carries image row q = (f + N/2) mod N' when
    // that is below N (f < N/2 or f >= N' - N/2)
    const int N_ = N, nbr_ = nbr, tid_ = tid;
    for (int t = first; t < end; ++t) {
        // the addresses and conditions are formed again for each layer: kept across the
        // layers they spill
        int N = N_, nbr = nbr_, tid = tid_;
        if constexpr (A::kDegridLoop) asm volatile("" : "+s"(N), "+s"(nbr), "+v"(tid));
        const int half = N / 2, r = tid % RW, n0 = tid / RW, line = tid / T, j = tid % T;
        const cpx<R>* src = inter + (size_t(t) * inter_blocks(N) * nbr + rt) * 256 + h * RW;      // block-uniform
        auto at = [&](int q) { return src[uint32_t(q >> 4) * uint32_t(nbr * 256) + uint32_t((q & 15) * 16 + r)]; };
        cpx<R> y[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) y[k] = cpx<R>{R(0), R(0)};
#pragma unroll
        for (int m = 0; m < C; ++m) {
            if (F * m >= half && F * (m + 1) <= NP - half) continue;       // padding bins only
            cpx<R> x[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int f0 = T * k + F * m;              // the T bins from f0 (block-uniform cases)
                x[k] = cpx<R>{R(0), R(0)};
                if (f0 + T <= half) {
                    x[k] = at(n0 + f0 + half);
                } else if (f0 >= NP - half) {
                    x[k] = at(n0 + f0 + half - NP);
                } else if (f0 < half || f0 + T > NP - half) {
                    const int q = shift_half<NP>(n0 + f0, half);
                    if (q < N) x[k] = at(q);
                }
            }
            const cpx<R> wm = tw[(m * b % C) * F];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                y[k].x += x[k].x * wm.x + x[k].y * wm.y;
                y[k].y += x[k].y * wm.x - x[k].x * wm.y;
            }
            __builtin_amdgcn_sched_barrier(0);     // 16 loads in flight per thread are enough, more spill
        }
        cpx<R>* lbuf = buf + line * LP;
        const int pj = lpad(j), pn = lpad(n0);
        if (t > first) __syncthreads();      // the lines of the layer before are read
        const cpx<R>* turn_b = tw + NP + TB.entries + b * F;               // W_N'^(n b)
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if (b > 0) {
                const cpx<R> w = turn_b[n0 + T * k];
                y[k] = cmul(y[k], cpx<R>{w.x, -w.y});
            }
            buf[r * LP + lpad_at<T>(n0, pn, k)] = y[k];
        }
        __syncthreads();
        cpx<R> v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = lbuf[lpad_at<T>(j, pj, k)];
        fft_wave<R, F, -1>(v, lbuf, tab, tw + NP + TB.second, j);
        cpx<R>* dst = stack + (size_t(t) * nbr + rt) * (size_t(NB) * TE);
        if constexpr (NP % 256 == 0) {
            // the values k of a thread are NP / 256 tiles apart, at one place within their tiles
            constexpr int STEP = NP / 256;
            const int s0 = C * j + b, tile0 = s0 / kTileS;
            const uint32_t cell = uint32_t(tile0 * TE + degrid_cell<C>(s0, h * RW + line));
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const uint32_t marks = uint32_t(((uint64_t(mw[STEP * k / 32 + 1]) << 32) | mw[STEP * k / 32]) >> (STEP * k % 32));
                if ((marks >> tile0) & 1u) dst[cell + uint32_t(STEP * k * TE)] = v[k];
            }
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int s = C * (j + T * k) + b, tile = s / kTileS;
                if ((mw[0] >> tile) & 1u) dst[tile * TE + degrid_cell<C>(s, h * RW + line)] = v[k];
            }
        }
    }
}

// --------------------------------------------------------------- plan tables --
//
// Correction map corr[j][i] = h(x_i) h(y_j) h_z(z_ji) (Algorithm 5 step 5): h at
// the pixel columns comes from the host, h_z is evaluated here from the
// pointwise optimality formula h(z) = int Re g dnu / int |g|^2 dnu over
// Gauss-Legendre nodes nu_j, g(z, nu) = sum_a c_a(nu) exp(i 2 pi (s_a - nu) z),
// with the w-axis design's c (width Wz); hz_one: no correction along z (the
// original W-stacking corrects in x and y only, Algorithm 3 step 5).
static __global__ void k_corr_map(const double* __restrict__ hx, const double* __restrict__ cnodes,
                           const double* __restrict__ nun, const double* __restrict__ wn, int n_nu, int Wz,
                           int hz_one, DevParams P, double* __restrict__ corr64, float* __restrict__ corr32) {
    const int N = P.N, half = N / 2;
    const int i = blockIdx.x * blockDim.x + threadIdx.x, jrow = blockIdx.y;
    if (i >= N) return;
    if (hz_one) {
        const double v = hx[i] * hx[jrow];
        corr64[(size_t)jrow * N + i] = v;
        corr32[(size_t)jrow * N + i] = float(v);
        return;
    }
    const double l = double(i - half) * P.dl, m = double(jrow - half) * P.dl;
    const double r2 = l * l + m * m;
    const double z = (-r2 / (1.0 + sqrt(1.0 - r2))) / P.nscale + P.zshift;
    const int W = Wz;
    double step_s, step_c;
    sincospi(2.0 * z, &step_s, &step_c);                         // exp(i 2 pi z)
    double num = 0.0, den = 0.0;
    for (int jn = 0; jn < n_nu; ++jn) {
        double es, ec;
        sincospi(2.0 * (-0.5 * (W - 1) - nun[jn]) * z, &es, &ec);  // a = 0 term
        double gr = 0.0, gi = 0.0;
        for (int a = 0; a < W; ++a) {
            const double c = cnodes[jn * W + a];
            gr += c * ec;
            gi += c * es;
            const double nc = ec * step_c - es * step_s, ns = ec * step_s + es * step_c;
            ec = nc;
            es = ns;
        }
        num += wn[jn] * gr;
        den += wn[jn] * (gr * gr + gi * gi);
    }
    const double v = hx[i] * hx[jrow] * (num / den);
    corr64[(size_t)jrow * N + i] = v;
    corr32[(size_t)jrow * N + i] = float(v);
}

}  // namespace wsg
