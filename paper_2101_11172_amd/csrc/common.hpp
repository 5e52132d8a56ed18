// Device-side types shared by the wsgrid kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace wsg {

template <typename R>
struct cpx {
    R x, y;
};

// Store of a complex value that is read back only by a later kernel (the FFT
// intermediates): non-temporal, so it streams through the caches.
typedef float nt_f2 __attribute__((ext_vector_type(2)));
typedef double nt_d2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_stream(cpx<float>* p, cpx<float> v) {
    __builtin_nontemporal_store(nt_f2{v.x, v.y}, reinterpret_cast<nt_f2*>(p));
}
__device__ __forceinline__ void store_stream(cpx<double>* p, cpx<double> v) {
    __builtin_nontemporal_store(nt_d2{v.x, v.y}, reinterpret_cast<nt_d2*>(p));
}

template <typename R>
__device__ __forceinline__ cpx<R> cmul(cpx<R> a, cpx<R> b) {
    return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename R>
__device__ __forceinline__ cpx<R> cadd(cpx<R> a, cpx<R> b) { return {a.x + b.x, a.y + b.y}; }
template <typename R>
__device__ __forceinline__ cpx<R> csub(cpx<R> a, cpx<R> b) { return {a.x - b.x, a.y - b.y}; }

// exp(i 2 pi f) for a phase f given in turns, reduced to [-1/2, 1/2] in float64
// first.  Float32: the hardware sine and cosine, which take their argument in
// turns (one instruction each; absolute error <= 1.2e-7, RMS 4.9e-8 and no
// bias over [-1/2, 1/2], measured against float64 on 2^24 points).
__device__ __forceinline__ void phase_turns(double f, float* s, float* c) {
    const float r = float(f - rint(f));
    *s = __builtin_amdgcn_sinf(r);
    *c = __builtin_amdgcn_cosf(r);
}
__device__ __forceinline__ void phase_turns(double f, double* s, double* c) {
    double r = f - rint(f);
    sincospi(2.0 * r, s, c);
}

// Orders this wave's LDS accesses around a hand-over between its lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One binned visibility.  ruv packs the first support index along u (low 16
// bits) and v (high 16 bits), both taken modulo N'; rt is the first support
// layer counted from t_lo.  nu are the fractional offsets in [-1/2, 1/2).
// grid:   v = V exp(+i 2 pi w (n0 - 1)), conjugated first if folded; idx unused.
// degrid: v = exp(-i 2 pi w (n0 - 1)); idx = k | (folded << 31).
template <typename R>
struct Rec {
    uint32_t ruv;
    uint32_t rt;
    R nu[3];
    R v[2];
    uint32_t idx;
};

// Scalars every kernel needs, passed by value.
struct DevParams {
    int N, Np, W, n_layers, t_lo;
    int Wz;                 // width of the w-axis gridding function (W: the same on all axes)
    int tclamp;             // original W-stacking: the last w bin is closed at wmax
    double wshift;          // w' = n_scale w + wshift (original W-stacking: -1/2)
    double tphase;          // layer t's w-screen uses t + tphase (original W-stacking: bin midpoints, 1/2)
    int nbr, nbs, nbt;      // bins (= tiles) along r (u), s (v), t (w) of one channel
    // Channels of a batched call: channel c's layers are the virtual layers
    // [c chl, c chl + n_layers) with chl = nbt kTileT (its tile layers follow
    // the previous channel's); virtual layers beyond n_layers in a channel are
    // padding that nothing reads or writes.  One channel: virtual = plain.
    int nch;
    // layer pass: virtual layers [pl0, pl0 + pln) (pl0 a multiple of kTileT)
    // sit in the stack and FFT buffers, local layer index t - pl0
    int pl0, pln;
    int classes;            // pass_a_classes(Np)
    int euv, et;            // window blocks' starts along u, v and along w by which records are ordered (1: by start)
    double umul;            // l_max / x0: u -> u'
    double nscale;          // w -> w'
    double zshift;          // (1 - n0) / n_scale: z = (n - 1) / n_scale + zshift
    double wmax;
    double dl;              // pixel size L / N
};

constexpr int kTileR = 16, kTileS = 16, kTileT = 16;

// Windows.  The matrix kernels of width W <= 8 work on windows of kWin = 8 cells
// along each axis, which hold the support of every record whose start lies in
// the window's first 9 - W cells: a class's part of an axis is cut into blocks
// of window_edge starts, and a class's records are ordered by block (layer, u,
// v), then by start, where a kernel on windows reads them, else by start alone.
constexpr int kWin = 8;
__host__ __device__ constexpr int window_edge(int W) { return W <= kWin ? kWin + 1 - W : 1; }

// Whether the scatter, and the gather, of these widths is the matrix kernel, else
// the kernel whose lanes own residues (scatter) or records (gather).  The matrix
// kernels' work hardly falls with the widths: they take windows of 8 cells per axis
// whatever the support.  Stage times in us, matrix against lanes, on Earth-rotation
// tracks (3.3M at 2048^2 and 1M at 1024^2) and 20,000 scattered visibilities:
//   scatter FP32  (W, W_z) = (2, 2): 561/419, 158/127, 23/19; (3, 3): 603/488, 160/157,
//                 23/23, 65,536 scattered 29/39; (4, 4): 639/571, 168/207, 23/35; (7, 1):
//                 742/565, 250/192, 31/28; (8, 1): 916/692, 349/232, 34/38; (7, 2):
//                 760/659, 248/244, 29/39; (7, 7): 930/1371, 268/546, 31/89
//   scatter FP64  (2, 2): 777/867, 267/253, 26/21; (7, 1): 1128/1224, 428/351, 37/24, and
//                 70/50 on 46,332 visibilities of snapshots (original W-stacking); (8, 1):
//                 1426/1914, 576/562, 40/37; (7, 2): 1164/1355, 432/391, 38/28; (7, 7):
//                 1360/1864, 452/513, 38/39
//   gather FP64   (4, 4): 1092/859, 364/234, 40/25; (5, 5): 1210/1029, 395/272, 47/30;
//                 (6, 6): 1394/1719, 482/452, 53/48; (7, 7): 1696/2912, 606/750, 58/71;
//                 (5, 1): 1491/839, 502/242, 48/26; (6, 1): 1634/3100, 597/899, 54/82; (8, 1):
//                 2325/2571, 959/743, 62/60
// Many visibilities in few bins favour the matrix scatter at every width (65,536 in
// one bin, W = 2 225/537, W = 7 450/1529) and the lanes' gather up to W = 5 (834/390).
// In FP32 the gather is better off with lanes at every width (see k_degrid_tiles_mat).
__host__ __device__ constexpr bool mat_scatter(bool f64, int W, int Wz) {
    return W <= kWin && (f64 ? W != 7 || Wz > 1 : W > 2 && Wz > 1);
}
__host__ __device__ constexpr bool mat_gather(bool f64, int W, int Wz) { return f64 && W >= 6 && W <= kWin; }

// Words of the marks of one row of nbs tiles.
__host__ __device__ constexpr int mask_words(int nbs) { return (nbs + 31) / 32; }

// Classes of outputs that FFT pass A splits a line of N' cells into (the
// transforms inside a class have at most 1024 points, without a factor 3), at
// every N'.  Against the whole-line pass and the transpose of the intermediate that
// it needs, 39 layers, grid / degrid in ms: N' = 6144 FP32 5.87 -> 3.17 / 5.72 ->
// 4.20, FP64 17.3 -> 6.1 / 20.1 -> 7.9; N' = 8192 with N = 4096 8.47 -> 5.69 / 8.86 ->
// 7.88, FP64 21.4 -> 11.9 / 24.3 -> 16.0, with N = 8192 9.98 -> 7.05 / 10.5 -> 11.7,
// FP64 29.1 -> 13.8 / 32.6 -> 23.9.  The FP32 degrid direction at N' = 8192 is the
// one place where it is slower (also three passes of 128-antenna tracks at 4096^2:
// 20.6 -> 21.8): each of the eight classes reads and multiplies the whole line.  It
// stays: the calls are not slower, and the whole-line pass wants a second
// intermediate in the workspace.
__host__ __device__ constexpr int pass_a_classes(int Np) {
    const int p2 = Np % 3 == 0 ? Np / 3 : Np;
    return (Np % 3 == 0 ? 3 : 1) * (p2 > 1024 ? p2 / 1024 : 1);
}

// Pass A's twiddle table behind the plan's Np roots of unity: for an F-point
// transform (F = Np / classes = 2^a) the twiddles W_(16 n)^(k m) of each pass in
// the order its lanes read them, [m][k < n] (n: points joined before the pass):
// 16 x 16 for the second radix-16 pass, then those of the last pass of radix
// 2, 4 or 8; then the class twiddles W_Np^(n b), [b][n < F].
__host__ __device__ constexpr int log2_floor(int n) {
    int l = 0;
    while ((2 << l) <= n) ++l;
    return l;
}
struct PassATable {
    int F, second, last_radix, last_n, entries;     // entries without the class twiddles
};
__host__ __device__ constexpr PassATable pass_a_table(int Np) {
    const int F = Np / pass_a_classes(Np), l = log2_floor(F), rem = l % 4;
    const int second = l >= 8 ? 256 : 0, radix = rem ? 1 << rem : 0, n = rem ? F / radix : 0;
    return {F, second, radix, n, second + radix * n};
}

// Pass B's twiddle table behind pass A's: for a line of Np = 2^a or 3 2^a points
// the twiddles of each pass after the first, [m][k < n], n the points joined
// before the pass: its radix-16 passes, then that of radix 2, 4 or 8 (the
// radix-3 pass reads the roots themselves).
__host__ __device__ constexpr int line_table_size(int Np) {
    const int p2 = Np % 3 == 0 ? Np / 3 : Np, l = log2_floor(p2);
    int n = 16, size = 0;
    for (int p = 1; p < l / 4; ++p, n *= 16) size += 16 * n;
    return size + (l % 4 ? (1 << (l % 4)) * n : 0);
}
__host__ __device__ constexpr int line_table_at(int Np) {        // its place in the plan's table
    return Np + pass_a_table(Np).entries + Np;
}

// Cells of one layer of a tile as the degrid direction stores them: class by
// class (cell s of a line is of class s mod C), the 16 rows of the class's cells
// of the tile each, so that a pass A block, which holds one class of the tile's
// rows, writes contiguous pieces.
// first class output a (cell s = C a + c) of v tile bs
__host__ __device__ constexpr int tile_class_first(int bs, int c, int C) { return (kTileS * bs - c + C - 1) / C; }
// cells of class c per row of v tile bs
__host__ __device__ constexpr int tile_class_cells(int bs, int c, int C) {
    return tile_class_first(bs + 1, c, C) - tile_class_first(bs, c, C);
}
// place of cell s of row r within its tile's layer
template <int C>
__device__ __forceinline__ int degrid_cell(int s, int r) {
    const int c = s % C, bs = s / kTileS;
    int before = 0;
    for (int k = 0; k < c; ++k) before += tile_class_cells(bs, k, C);
    return before * kTileR + r * tile_class_cells(bs, c, C) + s / C - tile_class_first(bs, c, C);
}
// its inverse: the row r and the cell s of place e of v tile bs
__device__ __forceinline__ void degrid_place(int e, int bs, int C, int& r, int& s) {
    int c = 0, n = tile_class_cells(bs, 0, C);
    while (e >= n * kTileR) {
        e -= n * kTileR;
        n = tile_class_cells(bs, ++c, C);
    }
    r = e / n;
    s = C * (tile_class_first(bs, c, C) + e % n) + c;
}

// The intermediate between the FFT passes: [t][q / 16][r / 16][16 q][16 r].
__host__ __device__ constexpr int inter_blocks(int N) { return (N + 15) / 16; }     // blocks of image rows q

// Index of the tile (br, bs) of layer tl of the pass among the pass's tile layers.
__device__ __forceinline__ size_t tile_base(const DevParams& P, int tl, int br, int bs) {
    return (size_t(tl) * P.nbr + br) * P.nbs + bs;
}

// One marked tile: its index and the records that reach it, at most ten ranges of
// the record array concatenated into a virtual list [0, total): range g holds
// the virtual positions from off[g] (0xffffffff past the last), position v the
// record v + delta[g]; bits 3 g .. 3 g + 2 of nbrs are the range's bin, the set
// it | ir << 1 | is << 2 of axes along which it lies one tile back.
struct __align__(128) TileRec {
    uint32_t tile, total, nbrs, pad;
    uint32_t off[10];
    uint32_t delta[10];
    uint32_t pad2[8];
};

// blockIdx -> logical block so that each XCD (blocks are dealt round-robin to
// the 8 XCDs) walks a contiguous range of logical blocks.  For uniform work
// (the FFT passes): neighbouring lines share cache lines in that XCD's L2.
__device__ __forceinline__ int xcd_remap(int b, int n) {
    int per = n >> 3, rem = n & 7;
    int x = b & 7, i = b >> 3;
    return x * per + min(x, rem) + i;
}

// blockIdx -> logical block dealing groups of G consecutive logical blocks to
// the XCDs in turn.  For the tile kernels, whose work is concentrated in the
// dense centre of the uv plane: the load spreads over all XCDs while runs of G
// neighbouring tiles (which share visibility bins) stay on one L2.  The last
// partial round keeps the identity mapping so the result is a permutation.
template <int G>
__device__ __forceinline__ int xcd_interleave(int b, int n) {
    const int full = (n / (8 * G)) * (8 * G);
    if (b >= full) return b;
    const int x = b & 7, i = b >> 3;
    return (i / G) * (8 * G) + x * G + (i % G);
}

}  // namespace wsg
