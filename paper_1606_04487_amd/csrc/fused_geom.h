// Geometry of the fused convolution kernels (implicit.hip, whole_patch.hip): what a plan holds and which input pixels a
// column tile needs.  Not part of the C ABI.
#pragma once

#include <type_traits>

#include "common.h"
#include "mma_epilogue.h"

namespace omni {
namespace fused {

constexpr int CH = 32;           // channels per reduction chunk
constexpr int NG = CH / 8;       // 16-byte packs per pixel and chunk
constexpr int MAX_SLOTS = 8;     // images a column tile may touch
constexpr uint32_t NO_PIX = 0xffffu;

struct Geom {
    int32_t N, C, H, W;      // input  [N][C][H][W]
    int32_t F, Ho, Wo;       // output [N][F][Ho][Wo],  Ho = H + 2*ph - kh + 1
    int32_t kh, kw, ph, pw;  // window, zero padding
    int32_t Wp;              // row pitch of the patch: at least W + 2*pw, the width of a padded row
    int32_t HW, HoWo, M, KK;
    uint32_t sn, sc;         // elements from an input image to the next and from a channel's plane to the next
    int32_t n_chunks;        // C / CH
    int32_t Fp;              // F rounded up to the row tile
    int32_t tiles_f, tiles_m, n_items, per_xcd;
    int32_t splits, chunks_per_split;  // the reduction's chunks cut into `splits` ranges (1: not split)
    int32_t whole;           // the larger tiles' reduction is not split, and then no tile's is: sums that a ReLU mask can follow
    int32_t bn;              // columns per workgroup: BN_SMALL, BN_NARROW, BN_MID or BN_WIDE
    int32_t bm;              // filter rows per workgroup: 128, 64 (with BN_SMALL), or 96 (with BN_WIDE) for layers of few filters
    int32_t config;          // >= 0: the product runs on this tile of whole_patch.hip, bm x bn
    int32_t plane;           // its patch pixels per channel pack
    int32_t piece;           // elements a loader task takes of each of its planes: 8, or 7 (whole_patch.hip)
    int32_t cols_fastest;    // its work items in order of columns within rows
    FastDiv div_tiles;       // tiles_m if cols_fastest, else tiles_f
    FastDiv div_HoWo, div_Wo, div_W;
};

// What a column tile [col0, m_last] needs of image n: padded rows [ra, ra + nrows) of which the real
// input rows are [ya, ya + len / W).
struct SlotSpan { int ra, nrows, ya, len; };
__host__ __device__ inline SlotSpan slot_span(const Geom &g, int col0, int m_last, int n)
{
    int base = n * g.HoWo;
    int qa = col0 > base ? col0 - base : 0;
    int qb = m_last - base < g.HoWo - 1 ? m_last - base : g.HoWo - 1;
    int oya = (int)g.div_Wo.div((uint32_t)qa), oyb = (int)g.div_Wo.div((uint32_t)qb);
    SlotSpan s;
    s.ra = oya;
    s.nrows = oyb - oya + g.kh;
    int ya = s.ra - g.ph, yb = s.ra + s.nrows - g.ph;
    if (ya < 0) ya = 0;
    if (yb > g.H) yb = g.H;
    s.ya = ya;
    s.len = yb > ya ? (yb - ya) * g.W : 0;
    return s;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t lo16(uint32_t a, uint32_t b) { return (a & 0xffffu) | (b << 16); }
__device__ __forceinline__ uint32_t hi16(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); }

// Compile-time loop: the body receives std::integral_constant<int, I>.
template <int I, int N, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// whole_patch.hip: tiles of the kernel that holds a column tile's pixels of all channels in LDS at once.
struct WholeTile { int bm, bn, waves; size_t lds; };  // lds: what adding the wavefronts' sums takes
constexpr int WHOLE_CONFIGS = 4;
WholeTile whole_tile(int config);
constexpr size_t WHOLE_LDS = 158 * 1024;  // of the 160 KB that a workgroup can have; the kernel has no other LDS
void launch_whole_patch(const Geom &g, bool rows_in, const bf16_t *X, const bf16_t *wt, const FwdEpilogue<bf16_t> &epi, hipStream_t s);

}  // namespace fused
}  // namespace omni
