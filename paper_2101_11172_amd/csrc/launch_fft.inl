// FFT-pass launchers for one precision (included by fft_f32.hip and
// fft_f64.hip, which instantiate them).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"
#include "launch.hpp"

namespace wsg {

// One layer pass of the FFT stages.  Pass B (along u / p, with the w-screen)
// runs once per channel segment of the pass: the virtual layers of channel c
// in the pass, whose map is dirty + c N^2 (grid, written by the channel's first
// segment and added to by later ones) or image + c N^2 (degrid).
template <typename R, int NP>
void launch_fft_n(bool grid, const DevParams& P, const uint32_t* mask, const uint8_t* rows, cpx<R>* stack,
                  cpx<R>* inter, const cpx<R>* tw, const R* corr, const R* image, R* dirty, hipStream_t s) {
    using C = FftCfg<R, NP>;
    using A = PassACfg<R, NP>;
    const unsigned grid_a = unsigned(P.pln) * unsigned(P.nbr * A::kHalves * A::kClasses);     // a class of kRows lines each
    // layers of a tile layer that a block takes one after the other, as long as eight
    // rounds of blocks are left
    int each = kTileT;
    while (each > 1 && grid_a / unsigned(each) < 4096u) each /= 2;
    const unsigned blocks_a = grid_a / unsigned(P.pln) * unsigned((P.pln + each - 1) / each);
    const unsigned degrid_a = A::kDegridLoop ? blocks_a : grid_a;
    const unsigned grid_b = unsigned((P.N + C::kNLr - 1) / C::kNLr);
    const int chl = P.nbt * kTileT;
    const size_t map = size_t(P.N) * size_t(P.N);
    // Pass B walks the layers of a row in one block, about 3 us a layer however few
    // blocks there are.  Where they do not fill the chip (eight waves on a CU) the
    // layers are split, as far as the blocks still run at the same time: beyond
    // that each more part repeats the row's set-up (1024^2 FP32, 512 blocks in two
    // parts: 88 -> 93 us).  FP64 at 192 x 192: 51 -> 13 us, FP32 at 512 x 512 37 -> 15.
    constexpr int kFill = 256 * std::max(1, 512 / (C::kNLr * C::T));
    auto parts = [&](int layers) { return std::max(1, std::min(layers, kFill / int(grid_b))); };
    auto segments = [&](auto&& fn) {
        for (int c = P.pl0 / chl; c < P.nch && c * chl < P.pl0 + P.pln; ++c) {
            const int lo = std::max(P.pl0, c * chl), hi = std::min(P.pl0 + P.pln, c * chl + P.n_layers);
            if (hi > lo) fn(c, lo, hi);
        }
    };
    if (grid) {
        {
            StageMark mark(s, 2);
            hipLaunchKernelGGL((k_grid_fft_a<R, NP>), dim3(blocks_a), dim3(A::kThreads), 0, s, (const cpx<R>*)stack, mask, inter, tw, P.N, P.n_layers,
                               P.nch > 1 ? chl : 0, P.nbr, P.pl0, P.pln, each);
        }
        StageMark mark(s, 3);
        segments([&](int c, int lo, int hi) {
            DevParams Q = P;
            Q.pln = hi - lo;
            const int S = parts(Q.pln), acc = lo > c * chl ? 1 : 0;
            R* partial = reinterpret_cast<R*>(stack);        // pass A has read it
            hipLaunchKernelGGL((k_grid_fft_b<R, NP>), dim3(grid_b, S), dim3(C::kNLr * C::T), 0, s,
                               (const cpx<R>*)inter, rows, tw, corr, dirty + size_t(c) * map, partial, Q, lo - P.pl0,
                               lo - c * chl, acc);
            if (S > 1)
                hipLaunchKernelGGL(k_map_sum<R>, dim3(unsigned((map + 255) / 256)), dim3(256), 0, s,
                                   (const R*)partial, S, corr, dirty + size_t(c) * map, int(map), acc);
        });
    } else {
        {
            StageMark mark(s, 5);
            segments([&](int c, int lo, int hi) {
                DevParams Q = P;
                Q.pln = hi - lo;
                hipLaunchKernelGGL((k_degrid_fft_b<R, NP>), dim3(grid_b, parts(Q.pln)), dim3(C::kNLr * C::T), 0, s,
                                   image + size_t(c) * map, corr, tw, rows, inter, Q, lo - P.pl0, lo - c * chl);
            });
        }
        StageMark mark(s, 6);
        hipLaunchKernelGGL((k_degrid_fft_a<R, NP>), dim3(degrid_a), dim3(A::kThreads), 0, s, (const cpx<R>*)inter,
                           mask, tw, stack, P.N, P.n_layers, P.nch > 1 ? chl : 0, P.nbr, P.pl0, P.pln, each);
    }
}

#define WSG_FFT_SIZES(X) \
    X(64) X(96) X(128) X(192) X(256) X(384) X(512) X(768) X(1024) X(1536) X(2048) X(3072) X(4096) X(6144) X(8192)

template <typename R>
bool launch_fft(bool grid, const DevParams& P, const uint32_t* mask, const uint8_t* rows, cpx<R>* stack,
                cpx<R>* inter, const cpx<R>* tw, const R* corr, const R* image, R* dirty, hipStream_t s) {
    switch (P.Np) {
#define WSG_N(n) \
    case n: launch_fft_n<R, n>(grid, P, mask, rows, stack, inter, tw, corr, image, dirty, s); return true;
        WSG_FFT_SIZES(WSG_N)
#undef WSG_N
        default: return false;
    }
}

}  // namespace wsg
