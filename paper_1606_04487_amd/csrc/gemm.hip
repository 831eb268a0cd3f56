// MFMA GEMM for the three matrix products of a lowered convolution layer (gfx950).
//
// One kernel template serves the paper's "multiply phase" (App. C, "Convolution by Lowering and
// GEMM") in its three uses:
//   forward : Y-hat [F x M] = K-hat   [F x K] * D-hat  [K x M]      epilogue: +bias, ReLU, lifting
//   dgrad   : dD-hat[K x M] = K-hat^T [K x F] * dY-hat [F x M]      epilogue: plain row-major store
//   wgrad   : dK-hat[F x K] = dY-hat  [F x M] * D-hat^T[M x K]      split along M, fp32 partials
// In every use the "row operand" (index i of the result) is contiguous along the reduction index,
// and the "column operand" (index j, the contiguous index of the result) is either contiguous
// along j (forward, dgrad: D-hat and dY-hat have M as their fastest index) or along the reduction
// (wgrad).
//
// Tiling: a workgroup of 4 or 8 wavefronts of 64 lanes owns a tile of the result, 32 x 128 to 256 x 256 (kTiles); each
// wavefront owns a grid of 32 x 32 MFMA tiles, accumulated in fp32.  The reduction is walked in steps of 128 bytes per row
// (64 bf16 or 32 fp32).  Both operands are staged in LDS as [pack][row] arrays of 16-byte packs, a pack being 8 (bf16) or 4
// (fp32) consecutive reduction indices of one row, so that an MFMA fragment is one 16-byte LDS read per lane and 32
// consecutive lanes read 512 consecutive bytes.  A column operand that is contiguous along j is transposed in registers
// on its way into LDS.  Global loads of the next step are issued under the MFMAs of the current one and land in the other
// LDS buffer.
//
// Two kernels share this: gemm_stream_kernel runs the products on lowered matrices, on fully connected layers' tensors and
// on dY in place; gemm_kernel the model gradients whose column operand comes from X (DirectLoader, Phase3Loader) and
// products whose operands take 4 GB or more.
//
// fp32 uses v_mfma_f32_32x32x2_f32 four times per pack: within one instruction lane-half h
// supplies reduction index 4*(2s+h)+e for both operands, which is a permutation of the slab's 8
// indices -- a sum does not care about the order of its terms.  bf16 uses
// v_mfma_f32_32x32x16_bf16, one instruction per pair of packs.
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "common.h"
#include "mma_epilogue.h"

namespace omni {

constexpr int NPACK = 8;  // 16-byte packs along the reduction per LDS tile (128 bytes of every row)

template <typename T> struct Pack;
template <> struct Pack<float> { static constexpr int KP = 4; };
template <> struct Pack<bf16_t> { static constexpr int KP = 8; };

template <typename T> constexpr int dtype_of() { return sizeof(T) == 2 ? OMNI_BF16 : OMNI_F32; }

int gemm_red_tile(int dtype) { return dtype == OMNI_BF16 ? NPACK * 8 : NPACK * 4; }

// ------------------------------------------------------------------------------------------------
// Operand loaders: global memory -> registers (issue()), registers -> LDS (commit()).
// An LDS tile of R rows is uint4[NPACK][R + 1]: pack g of row r at g*(R+1) + r.  The extra pack of
// padding per group spreads the 8 packs of one row over the banks when they are written together.
// ------------------------------------------------------------------------------------------------

// Operand stored [rows][ld] with the reduction index contiguous.  Element (r, k) is valid for
// r < rows and k < red; ld and red are multiples of the pack size and the base is 16-byte aligned.
template <typename T, int TILE_ROWS, int NT> struct RedContigLoader {
    static constexpr int KP = Pack<T>::KP;
    static constexpr int TASKS = TILE_ROWS * NPACK;
    static constexpr int PER_THREAD = (TASKS + NT - 1) / NT;
    static constexpr bool RAGGED = TASKS % NT != 0;  // the last round of tasks covers only part of the threads
    uint4 regs[PER_THREAD];

    __device__ __forceinline__ void issue(const T *base, int64_t ld, int rows, int64_t red, int row0,
                                          int64_t k0, int tid)
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            int t = tid + q * NT;
            int g = t % NPACK, r = t / NPACK;
            int64_t k = k0 + (int64_t)g * KP;
            uint4 v = make_uint4(0, 0, 0, 0);
            if ((!RAGGED || t < TASKS) && row0 + r < rows && k < red)
                v = *reinterpret_cast<const uint4 *>(base + (int64_t)(row0 + r) * ld + k);
            regs[q] = v;
        }
    }
    __device__ __forceinline__ void commit(uint4 *lds, int tid) const
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            int t = tid + q * NT;
            int g = t % NPACK, r = t / NPACK;
            if (!RAGGED || t < TASKS) lds[g * (TILE_ROWS + 1) + r] = regs[q];
        }
    }
};

// Operand stored [red][ld] with the result's column index j contiguous.  Element (k, j) is valid
// for k < red and j < cols; ld and cols are multiples of 8 and the base is 16-byte aligned.
// One task = one pack group g (KP reduction rows) x 4 consecutive columns, transposed in registers.
template <typename T, int TILE_COLS, int NT> struct OuterContigLoader;

template <int TILE_COLS, int NT> struct OuterContigLoader<float, TILE_COLS, NT> {
    static constexpr int CHUNKS = TILE_COLS / 4;
    static constexpr int PER_THREAD = NPACK * CHUNKS / NT;
    static_assert(NPACK * CHUNKS % NT == 0, "tile must divide over the threads");
    uint4 regs[PER_THREAD][4];
    __device__ __forceinline__ void issue(const float *base, int64_t ld, int64_t red, int cols,
                                          int64_t k0, int col0, int tid)
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            int t = tid + q * NT;
            int jc = t % CHUNKS, g = t / CHUNKS;
            int j = col0 + jc * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int64_t k = k0 + g * 4 + e;
                uint4 v = make_uint4(0, 0, 0, 0);
                if (k < red && j < cols) v = *reinterpret_cast<const uint4 *>(base + k * ld + j);
                regs[q][e] = v;
            }
        }
    }
    __device__ __forceinline__ void commit(uint4 *lds, int tid) const
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            int t = tid + q * NT;
            int jc = t % CHUNKS, g = t / CHUNKS;
            uint4 *dst = lds + g * (TILE_COLS + 1) + jc * 4;
            const uint4 *r = regs[q];
            dst[0] = make_uint4(r[0].x, r[1].x, r[2].x, r[3].x);
            dst[1] = make_uint4(r[0].y, r[1].y, r[2].y, r[3].y);
            dst[2] = make_uint4(r[0].z, r[1].z, r[2].z, r[3].z);
            dst[3] = make_uint4(r[0].w, r[1].w, r[2].w, r[3].w);
        }
    }
};

template <int TILE_COLS, int NT> struct OuterContigLoader<bf16_t, TILE_COLS, NT> {
    static constexpr int CHUNKS = TILE_COLS / 4;
    static constexpr int PER_THREAD = NPACK * CHUNKS / NT;
    static_assert(NPACK * CHUNKS % NT == 0, "tile must divide over the threads");
    uint2 regs[PER_THREAD][8];
    __device__ __forceinline__ void issue(const bf16_t *base, int64_t ld, int64_t red, int cols,
                                          int64_t k0, int col0, int tid)
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            int t = tid + q * NT;
            int jc = t % CHUNKS, g = t / CHUNKS;
            int j = col0 + jc * 4;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                int64_t k = k0 + g * 8 + e;
                uint2 v = make_uint2(0, 0);
                if (k < red && j < cols) v = *reinterpret_cast<const uint2 *>(base + k * ld + j);
                regs[q][e] = v;
            }
        }
    }
    static __device__ __forceinline__ uint32_t lo(uint32_t a, uint32_t b) { return (a & 0xffffu) | (b << 16); }
    static __device__ __forceinline__ uint32_t hi(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); }
    __device__ __forceinline__ void commit(uint4 *lds, int tid) const
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            int t = tid + q * NT;
            int jc = t % CHUNKS, g = t / CHUNKS;
            uint4 *dst = lds + g * (TILE_COLS + 1) + jc * 4;
            const uint2 *r = regs[q];
            // column j = 2d + h of the 8 x 4 block becomes one pack: 8 reduction indices of column j
            dst[0] = make_uint4(lo(r[0].x, r[1].x), lo(r[2].x, r[3].x), lo(r[4].x, r[5].x), lo(r[6].x, r[7].x));
            dst[1] = make_uint4(hi(r[0].x, r[1].x), hi(r[2].x, r[3].x), hi(r[4].x, r[5].x), hi(r[6].x, r[7].x));
            dst[2] = make_uint4(lo(r[0].y, r[1].y), lo(r[2].y, r[3].y), lo(r[4].y, r[5].y), lo(r[6].y, r[7].y));
            dst[3] = make_uint4(hi(r[0].y, r[1].y), hi(r[2].y, r[3].y), hi(r[4].y, r[5].y), hi(r[6].y, r[7].y));
        }
    }
};

// ------------------------------------------------------------------------------------------------
// The lowered matrix read straight from the input tensor (stride-1 layers, bf16), for the model gradient.
// The reduction runs over padded columns.  Row mode: column ((n*Ho + oy) * P8 + i) * 8 + e stands for output
// position (n, oy, 8i + e), P8 = ceil(Wo / 8); plane mode (further down): only whole image planes are
// padded.  dY-hat is packed the same way with zeros in the padding (a sum does not care about the order or
// about zero terms).  A pack of 8 columns of row k = (c, ky, kx) of D-hat is then 8 consecutive input
// pixels: one 16-byte load at element granularity plus a mask for pixels in the zero padding or outside
// the image.  The same input bytes serve the kh*kw
// window taps of a channel, so nearly all of these loads hit in L1/L2; D-hat is never written or read.
// ------------------------------------------------------------------------------------------------
struct DirectSrc {
    const bf16_t *X;
    int32_t C, H, W, HW, K, ph, pw;
    int32_t rows;   // padded units in the batch: N * Ho output rows, or N image planes
    int32_t total;  // elements of X (< 2^31)
    FastDiv div_p8, div_Ho, div_khkw, div_kw;
    int32_t HoWo, KK;  // plane mode: output positions per image, window taps
    FastDiv div_W;
    int32_t sh;        // row mode: vertical stride (input rows per output row)
    int32_t F, Wo;     // DIRECT_ROWS_ONES: dY is [N][F][Ho][Wo], read by DyLoader
};

// Plane mode.  When the output is as wide as the input (stride 1, 2*pw = kw - 1), output position q of an
// image and window tap (ky, kx) meet input element q + (ky - ph) * W + (kx - pw) of the channel's plane,
// also where q wraps from one output row to the next.  So only each image's whole plane is padded to a
// multiple of 8 positions (not every row), a pack is still one 16-byte load, and which of its 8 elements
// are real pixels depends on (pack within the plane, tap) alone: a table in LDS, one byte per element,
// built when the workgroup starts.  Row (pack j, tap KK) of the table is zero: result columns beyond K.
constexpr int DIRECT_TAB = 2560;  // table entries (8 bytes each) a workgroup can hold beside its tiles
enum { DIRECT_ROWS = 1, DIRECT_ROWS_FIXED = 2, DIRECT_PLANES = 3, DIRECT_ROWS_ONES = 4, DIRECT_PHASE3 = 5 };
// DIRECT_ROWS_ONES: row mode in which (a) row K of the operand -- the first result column beyond the gradient
// -- is all ones, so that result column K is the sum of dY over every position: the bias gradient, from the
// same MFMAs; and (b) the row operand is read from dY as it lies in memory (DyLoader), not from a packed copy.

__device__ __forceinline__ void build_plane_table(const DirectSrc &d, uint2 *tab, int tid, int nt)
{
    const int p8 = (int)d.div_p8.d, kw = (int)d.div_kw.d;
    for (int idx = tid; idx < p8 * (d.KK + 1); idx += nt) {
        const int j = idx / (d.KK + 1), tap = idx - j * (d.KK + 1);
        uint32_t ky, kx;
        d.div_kw.divmod((uint32_t)(tap < d.KK ? tap : 0), ky, kx);
        uint32_t w[2] = {0u, 0u};
        for (int e = 0; e < 8; ++e) {
            const int q = 8 * j + e;
            uint32_t oy, ox;
            d.div_W.divmod((uint32_t)q, oy, ox);
            const bool ok = tap < d.KK && q < d.HoWo && (unsigned)((int)oy + (int)ky - d.ph) < (unsigned)d.H &&
                            (unsigned)((int)ox + (int)kx - d.pw) < (unsigned)d.W;
            if (ok) w[e / 4] |= 0xffu << (8 * (e % 4));
        }
        tab[idx] = make_uint2(w[0], w[1]);
    }
    (void)kw;
}

// MODE DIRECT_ROWS_FIXED: the row-padded rows are 1, 2, 4 or 8 packs long, so a reduction step (8 packs)
// moves every thread by whole output rows and the pack's place in its row -- hence which of its 8 elements
// fall beside the image for a given window column -- is the same in every step: those masks are built once.
template <int TILE_ROWS, int NT, int MODE> struct DirectLoader {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    static constexpr bool FIXED = MODE == DIRECT_ROWS_FIXED, PLANES = MODE == DIRECT_PLANES, ONES = MODE == DIRECT_ROWS_ONES;
    static constexpr int PER_THREAD = TILE_ROWS * NPACK / NT;
    static_assert(TILE_ROWS * NPACK % NT == 0 && NT % NPACK == 0, "tile must divide over the threads");
    u32x4 v[PER_THREAD];
    uint32_t ones[ONES ? PER_THREAD : 1];   // 0x3f803f80 (two bf16 ones) for the row of ones, else 0
    // rows: bits 0..7: which elements are real pixels (FIXED: bit 0: the input row exists).
    // bits 8..11: signed element shift (non-zero only where the 16 bytes had to be moved to stay inside
    // the tensor: first and last row of X)
    uint32_t masks[PER_THREAD];
    int kbase[PER_THREAD];
    int dky[PLANES ? 1 : PER_THREAD], dkx[FIXED || PLANES ? 1 : PER_THREAD];
    u32x4 colmask[FIXED ? PER_THREAD : 1];
    int tap[PLANES ? PER_THREAD : 1];       // planes: column of the mask table
    uint2 emask[PLANES ? PER_THREAD : 1];   // planes: this step's table entries

    static __device__ __forceinline__ uint32_t spread(uint32_t m, int bit)  // two mask bits -> two 16-bit fields
    {
        uint32_t lo = (uint32_t)((int32_t)(m << (31 - bit)) >> 31), hi = (uint32_t)((int32_t)(m << (30 - bit)) >> 31);
        return (lo & 0xffffu) | (hi & 0xffff0000u);
    }
    __device__ __forceinline__ void init(const DirectSrc &d, int col0, int tid)
    {
        uint32_t row_unused, i;
        d.div_p8.divmod((uint32_t)(tid % NPACK), row_unused, i);  // FIXED: this thread's pack within its row
        const int ox0 = 8 * (int)i;
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            int k = col0 + (tid + q * NT) / NPACK;
            uint32_t c, rem, ky, kx;
            d.div_khkw.divmod((uint32_t)(k < d.K ? k : 0), c, rem);
            d.div_kw.divmod(rem, ky, kx);
            const int dx = (int)kx - d.pw;
            kbase[q] = (int)c * d.HW + ((int)ky - d.ph) * d.W + dx;
            if constexpr (PLANES) {
                tap[q] = k < d.K ? (int)rem : d.KK;
            } else {
                if constexpr (ONES) ones[q] = k == d.K ? 0x3f803f80u : 0u;
                dky[q] = k < d.K ? (int)ky - d.ph : -(1 << 24);  // rows beyond K: no input row is ever valid
                if constexpr (FIXED) {
                    const int ix = ox0 + dx;
                    const int lo = ix < 0 ? -ix : 0, hi = d.W - ix < 8 ? d.W - ix : 8;
                    const uint32_t m = hi > lo ? (1u << hi) - (1u << lo) : 0u;
                    if (m == 0u) dky[q] = -(1 << 24);
#pragma unroll
                    for (int w = 0; w < 4; ++w) colmask[q][w] = spread(m, 2 * w);
                } else {
                    dkx[q] = dx;
                }
            }
        }
    }
    // m0: first padded column of this thread's packs -- the same for all of them, NT being a multiple of
    // NPACK.  tab: the plane mode's mask table.
    __device__ __forceinline__ void issue(const DirectSrc &d, int m0, const uint2 *tab)
    {
        const int top = d.total - 8;
        const char *xb = reinterpret_cast<const char *>(d.X);
        if constexpr (PLANES) {
            uint32_t n, j;
            d.div_p8.divmod((uint32_t)m0 >> 3, n, j);
            const bool live = (int)n < d.rows;
            const int base = (live ? (int)n : 0) * d.C * d.HW + 8 * (int)j;
            const int trow = (int)j * (d.KK + 1);
#pragma unroll
            for (int p = 0; p < PER_THREAD; ++p) {
                // element offset of the load, moved inside [0, total - 8] where it sticks out (by at most 7
                // elements if any element of the pack is a real pixel; else the mask is zero anyway)
                const int e = base + kbase[p];
                const int c = e < 0 ? 0 : (e > top ? top : e);
                __builtin_memcpy(&v[p], xb + 2u * (uint32_t)c, 16);
                masks[p] = (uint32_t)(e - c) & 15u;
                emask[p] = tab[live ? trow + tap[p] : d.KK];
            }
        } else {
            uint32_t row, i, n, oy;
            d.div_p8.divmod((uint32_t)m0 >> 3, row, i);
            const bool live = (int)row < d.rows;
            d.div_Ho.divmod(live ? row : 0u, n, oy);
            const int ox0 = 8 * (int)i;
            const int iy = (int)oy * d.sh;
            const int base = (int)n * d.C * d.HW + iy * d.W + ox0;
#pragma unroll
            for (int p = 0; p < PER_THREAD; ++p) {
                bool ok = live && (unsigned)(iy + dky[p]) < (unsigned)d.H;
                uint32_t m = 1u;
                if constexpr (!FIXED) {
                    const int ix = ox0 + dkx[p];
                    const int lo = ix < 0 ? -ix : 0, hi = d.W - ix < 8 ? d.W - ix : 8;
                    ok = ok && hi > lo;
                    m = (1u << hi) - (1u << lo);
                }
                // element offset of the load, moved inside [0, total - 8] where it sticks out
                const int e = base + kbase[p];
                const int c = ok ? (e < 0 ? 0 : (e > top ? top : e)) : 0;
                const uint32_t sft = ok ? (uint32_t)(e - c) & 15u : 0u;
                __builtin_memcpy(&v[p], xb + 2u * (uint32_t)c, 16);
                masks[p] = (ok ? m : 0u) | (sft << 8);
            }
        }
    }
    // element j of the result = element j + s of x (s = 4-bit two's complement, |s| <= 7 where it matters)
    static __device__ __forceinline__ u32x4 shifted(u32x4 x4, uint32_t s4)
    {
        unsigned __int128 x = ((unsigned __int128)(((uint64_t)x4[3] << 32) | x4[2]) << 64) | (((uint64_t)x4[1] << 32) | x4[0]);
        const int up = 16 - (int)s4 > 7 ? 7 : 16 - (int)s4;
        x = (s4 & 8u) ? x << (16 * up) : x >> (16 * (int)s4);
        uint64_t lo = (uint64_t)x, hi = (uint64_t)(x >> 64);
        return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
    }
    __device__ __forceinline__ void commit(uint4 *lds, int tid) const
    {
#pragma unroll
        for (int p = 0; p < PER_THREAD; ++p) {
            int t = tid + p * NT;
            int g = t % NPACK, r = t / NPACK;
            u32x4 a = v[p];
            u32x4 o;
            if constexpr (PLANES) {
                if (masks[p]) a = shifted(a, masks[p]);  // first or last few elements of the tensor only
                // one mask byte per element -> 16 bits per element (both operands the same word: either
                // half of the selector range picks from it)
                o[0] = a[0] & __builtin_amdgcn_perm(emask[p].x, emask[p].x, 0x01010000u);
                o[1] = a[1] & __builtin_amdgcn_perm(emask[p].x, emask[p].x, 0x03030202u);
                o[2] = a[2] & __builtin_amdgcn_perm(emask[p].y, emask[p].y, 0x01010000u);
                o[3] = a[3] & __builtin_amdgcn_perm(emask[p].y, emask[p].y, 0x03030202u);
            } else {
                if (masks[p] >> 8) a = shifted(a, (masks[p] >> 8) & 15u);
                if constexpr (FIXED) {
                    const uint32_t row_ok = 0u - (masks[p] & 1u);
#pragma unroll
                    for (int w = 0; w < 4; ++w) o[w] = a[w] & colmask[p][w] & row_ok;
                } else {
#pragma unroll
                    for (int w = 0; w < 4; ++w) o[w] = a[w] & spread(masks[p], 2 * w);
                    if constexpr (ONES) {
#pragma unroll
                        for (int w = 0; w < 4; ++w) o[w] |= ones[p];  // the masks of a row beyond K are zero
                    }
                }
            }
            reinterpret_cast<u32x4 *>(lds)[g * (TILE_ROWS + 1) + r] = o;
        }
    }
};

// DIRECT_PHASE3: the lowered operand of the phase-split stride-4 model gradient (launch_gemm_wgrad_phase) when a
// window row has three groups (kw = 9 .. 12).  Rows 3t, 3t + 1, 3t + 2 of the operand are then the same ten
// consecutive elements of phase image (c', ky) shifted by 0, 1 and 2: one 16-byte load and one 4-byte load
// (both aligned: X4's rows are 16-byte multiples and a pack starts at a multiple of 8) serve three packs, and
// only the K' / 3 real triples are loaded.  Nothing needs a mask: every address is inside X4 (8 * P8 + 2 <= WP),
// columns beyond the batch meet zeros of the other operand, rows beyond K' + 1 are never written (their
// results are columns the epilogue does not store), and row K' is the row of ones.
template <int TILE_ROWS, int NT> struct Phase3Loader {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    static constexpr int ROUNDS = (TILE_ROWS / 3 + NT / NPACK - 1) / (NT / NPACK);  // triples per thread
    u32x4 w[ROUNDS];
    uint32_t x[ROUNDS];
    int kbase[ROUNDS];  // element offset of the triple's input row from the pack's base; -1: no such triple

    __device__ __forceinline__ void init(const DirectSrc &d, int, int tid)
    {
        const int kh = (int)d.div_khkw.d / 3;
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            const int tr = tid / NPACK + q * (NT / NPACK);
            const int c = tr / kh, ky = tr - c * kh;
            kbase[q] = 3 * tr < d.K ? c * d.HW + ky * d.W : -1;
        }
    }
    __device__ __forceinline__ void issue(const DirectSrc &d, int m0, const uint2 *)
    {
        uint32_t row, i, n, oy;
        d.div_p8.divmod((uint32_t)m0 >> 3, row, i);
        const bool live = (int)row < d.rows;
        d.div_Ho.divmod(live ? row : 0u, n, oy);
        const int base = (int)n * d.C * d.HW + (int)oy * d.sh * d.W + 8 * (int)i;
        const char *xb = reinterpret_cast<const char *>(d.X);
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            const int e = live && kbase[q] >= 0 ? base + kbase[q] : 0;
            __builtin_memcpy(&w[q], xb + 2u * (uint32_t)e, 16);
            __builtin_memcpy(&x[q], xb + 2u * (uint32_t)e + 16, 4);
        }
    }
    __device__ __forceinline__ void commit(uint4 *lds, int tid) const
    {
        u32x4 *dst = reinterpret_cast<u32x4 *>(lds) + (tid % NPACK) * (TILE_ROWS + 1);
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            const int tr = tid / NPACK + q * (NT / NPACK);
            if (kbase[q] >= 0) {
                const u32x4 a = w[q];
                dst[3 * tr] = a;
                dst[3 * tr + 1] = u32x4{__builtin_amdgcn_alignbit(a[1], a[0], 16), __builtin_amdgcn_alignbit(a[2], a[1], 16),
                                        __builtin_amdgcn_alignbit(a[3], a[2], 16), __builtin_amdgcn_alignbit(x[q], a[3], 16)};
                dst[3 * tr + 2] = u32x4{a[1], a[2], a[3], x[q]};
            }
        }
    }
    // the row of ones (row K of the operand), rewritten with every tile by the first NPACK threads
    __device__ __forceinline__ void commit_ones(uint4 *lds, int tid, int K) const
    {
        if (tid < NPACK) reinterpret_cast<u32x4 *>(lds)[tid * (TILE_ROWS + 1) + K] = u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    }
};

// The row operand of the model gradient read from dY [N][F][Ho][Wo] itself: row f, padded column
// ((n * Ho + oy) * P8 + i) * 8 + e is dY(n, f, oy, 8 i + e), zero for 8 i + e >= Wo and for columns beyond the
// batch.  The 16 bytes of a row's ragged last pack are read so that they END at the row's end (always inside
// the tensor, Wo >= 8) and are shifted down, which also zeroes the padding.
template <int TILE_ROWS, int NT> struct DyLoader {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    static constexpr int TASKS = TILE_ROWS * NPACK;
    static constexpr int PER_THREAD = (TASKS + NT - 1) / NT;
    static constexpr bool RAGGED = TASKS % NT != 0;
    u32x4 regs[PER_THREAD];
    uint32_t okbits;
    int back;  // elements the loads were moved back by

    // m0: first padded column of this thread's packs (the same for all of them)
    __device__ __forceinline__ void issue(const bf16_t *dY, const DirectSrc &d, int row0, int m0, int tid)
    {
        uint32_t row, i, n, oy;
        d.div_p8.divmod((uint32_t)m0 >> 3, row, i);
        const bool live = (int)row < d.rows;
        d.div_Ho.divmod(live ? row : 0u, n, oy);
        const int valid = d.Wo - 8 * (int)i < 8 ? d.Wo - 8 * (int)i : 8;
        back = 8 - valid;
        const int base = (int)n * d.F * d.HoWo + (int)oy * d.Wo + 8 * (int)i - back;
        okbits = 0u;
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            const int t = tid + q * NT;
            const int f = row0 + t / NPACK;
            const bool ok = live && f < d.F && (!RAGGED || t < TASKS);
            const int e = ok ? base + f * d.HoWo : 0;
            __builtin_memcpy(&regs[q], reinterpret_cast<const char *>(dY) + 2u * (uint32_t)e, 16);
            okbits |= (ok ? 1u : 0u) << q;
        }
    }
    __device__ __forceinline__ void commit(uint4 *lds, int tid) const
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            const int t = tid + q * NT;
            const int g = t % NPACK, r = t / NPACK;
            u32x4 v = regs[q];
            if (back) {
                unsigned __int128 x = ((unsigned __int128)(((uint64_t)v[3] << 32) | v[2]) << 64) | (((uint64_t)v[1] << 32) | v[0]);
                x >>= 16 * back;
                const uint64_t lo = (uint64_t)x, hi = (uint64_t)(x >> 64);
                v = u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
            }
            const uint32_t keep = 0u - ((okbits >> q) & 1u);
#pragma unroll
            for (int w = 0; w < 4; ++w) v[w] &= keep;
            if (!RAGGED || t < TASKS) reinterpret_cast<u32x4 *>(lds)[g * (TILE_ROWS + 1) + r] = v;
        }
    }
};

// ------------------------------------------------------------------------------------------------
// The kernel
// ------------------------------------------------------------------------------------------------
struct GemmShape {
    int rows;         // extent of i
    int cols;         // extent of j (valid columns of the column operand)
    int64_t red;      // extent of the reduction index (what the loaders may touch)
    int64_t chunk;    // reduction extent handled by one split (multiple of the LDS tile)
    int tiles_i, tiles_j;
    int n_blocks;     // tiles_i * tiles_j
    int n_items;      // n_blocks * splits: work items of the launch
    int per_xcd;      // ceil(n_items / 8); the launch has 8 * per_xcd workgroups
    int fast_store;   // the result is below 4 GB: 32-bit store offsets
};

// Tile configuration: BM x BN result tile, WM x WN wavefronts, PF reduction steps of global loads in
// flight (register staging sets).
template <int BM_, int BN_, int WM_, int WN_, int PF_> struct Tile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, PF = PF_;
    static constexpr int NT = 64 * WM * WN;
    static constexpr int TI = BM / WM / 32, TJ = BN / WN / 32;  // 32 x 32 MFMA tiles per wavefront
    static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0, "wavefront tiles are multiples of 32");
};

template <typename T, typename Cfg, bool COL_OUTER, typename Epi, int DIRECT = 0>  // DIRECT_ROWS ... DIRECT_PLANES
__global__ __launch_bounds__(Cfg::NT) void gemm_kernel(const T *__restrict__ A, int64_t lda,
                                                       const T *__restrict__ B, int64_t ldb,
                                                       GemmShape sh, Epi epi, DirectSrc direct)
{
    static_assert(!DIRECT || (!COL_OUTER && std::is_same<T, bf16_t>::value), "direct operand: bf16 model gradient only");
    constexpr int KP = Pack<T>::KP;
    constexpr int BK = NPACK * KP;
    constexpr int BM = Cfg::BM, BN = Cfg::BN, NT = Cfg::NT, TI = Cfg::TI, TJ = Cfg::TJ, PF = Cfg::PF;
    constexpr int LA = BM + 1, LB = BN + 1;
    __shared__ uint4 lds_all[2 * NPACK * (LA + LB)];  // A buffers 0, 1 then B buffers 0, 1
    __shared__ float lds_add[Epi::HAS_ROW_ADD ? BM : 1];
    auto lds_a = [&](int buf) { return lds_all + buf * (NPACK * LA); };
    auto lds_b = [&](int buf) { return lds_all + 2 * NPACK * LA + buf * (NPACK * LB); };

    // Workgroups are handed to the 8 XCDs round-robin; give each XCD a contiguous range of the work
    // items (tile, split), tiles fastest: neighbouring tiles share operand panels and each XCD has its
    // own L2.  The launch is one-dimensional and padded to a multiple of 8.
    int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    int item = xcd * sh.per_xcd + slot;
    if (item >= sh.n_items) return;
    int z = item / sh.n_blocks, tile = item - z * sh.n_blocks;
    int ti = tile % sh.tiles_i, tj = tile / sh.tiles_i;  // row tiles fastest: they share the big column panel
    int row0 = ti * BM, col0 = tj * BN;
    int64_t k_begin = (int64_t)z * sh.chunk;
    int64_t k_end = k_begin + sh.chunk < sh.red ? k_begin + sh.chunk : sh.red;
    int steps = k_end > k_begin ? (int)((k_end - k_begin + BK - 1) / BK) : 0;

    int tid = threadIdx.x;
    int lane = tid % 64, wave = tid / 64;
    int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
    int li = lane % 32, h = lane / 32;
    if constexpr (Epi::HAS_ROW_ADD)  // read back after the main loop's barriers
        for (int i = tid; i < BM; i += NT) lds_add[i] = epi.row_add(row0 + i);

    f32x16 acc[TI][TJ];
#pragma unroll
    for (int t = 0; t < TI; ++t)
#pragma unroll
        for (int u = 0; u < TJ; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][u][v] = 0.f;

    constexpr bool DY_DIRECT = DIRECT == DIRECT_ROWS_ONES || DIRECT == DIRECT_PHASE3;  // the row operand comes from dY as it is
    typename std::conditional<DY_DIRECT, DyLoader<BM, NT>, RedContigLoader<T, BM, NT>>::type la[PF];
    struct Unused {};  // only the column loader in use is instantiated: not every tile suits every loader
    typename std::conditional<!COL_OUTER && !DIRECT, RedContigLoader<T, BN, NT>, Unused>::type lb_red[PF];
    typename std::conditional<COL_OUTER, OuterContigLoader<T, BN, NT>, Unused>::type lb_out[PF];
    typename std::conditional<DIRECT == DIRECT_PHASE3, Phase3Loader<BN, NT>, DirectLoader<BN, NT, DIRECT>>::type lb_dir[DIRECT ? PF : 1];
    __shared__ uint2 plane_tab[DIRECT == DIRECT_PLANES ? DIRECT_TAB : 1];
    if constexpr (DIRECT != 0) {
#pragma unroll
        for (int p = 0; p < PF; ++p) lb_dir[p].init(direct, col0, tid);
        if constexpr (DIRECT == DIRECT_PLANES) {
            build_plane_table(direct, plane_tab, tid, NT);
            __syncthreads();
        }
    }

    auto issue = [&](int set, int64_t k0) {
        if constexpr (DY_DIRECT)
            la[set].issue(A, direct, row0, (int)k0 + (tid % NPACK) * 8, tid);
        else
            la[set].issue(A, lda, sh.rows, sh.red, row0, k0, tid);
        if constexpr (DIRECT)
            lb_dir[set].issue(direct, (int)k0 + (tid % NPACK) * 8, plane_tab);
        else if constexpr (COL_OUTER)
            lb_out[set].issue(B, ldb, sh.red, sh.cols, k0, col0, tid);
        else
            lb_red[set].issue(B, ldb, sh.cols, sh.red, col0, k0, tid);
    };
    auto commit = [&](int set, int buf) {
        la[set].commit(lds_a(buf), tid);
        if constexpr (DIRECT) {
            lb_dir[set].commit(lds_b(buf), tid);
            if constexpr (DIRECT == DIRECT_PHASE3) lb_dir[set].commit_ones(lds_b(buf), tid, direct.K);
        } else if constexpr (COL_OUTER)
            lb_out[set].commit(lds_b(buf), tid);
        else
            lb_red[set].commit(lds_b(buf), tid);
    };
    auto compute = [&](int buf, auto s0c, auto s1c) {
        constexpr int S0 = decltype(s0c)::value, S1 = decltype(s1c)::value;
        const uint4 *pa = lds_a(buf) + wm * (BM / Cfg::WM) + li;
        const uint4 *pb = lds_b(buf) + wn * (BN / Cfg::WN) + li;
#pragma unroll
        for (int slab = S0; slab < S1; ++slab) {
            int g = slab * 2 + h;
            uint4 a[TI], b[TJ];
#pragma unroll
            for (int t = 0; t < TI; ++t) a[t] = pa[g * LA + 32 * t];
#pragma unroll
            for (int u = 0; u < TJ; ++u) b[u] = pb[g * LB + 32 * u];
#pragma unroll
            for (int t = 0; t < TI; ++t)
#pragma unroll
                for (int u = 0; u < TJ; ++u) Mma<T>::run(a[t], b[u], acc[t][u]);
        }
    };

    // Step s computes tile s from LDS buffer s&1.  Global loads of tile s+PF are issued at the start
    // of step s into register set s%PF; the set holding tile s+1 is written to the other LDS buffer during
    // step s.  The loop is unrolled by PF so that set indices are compile-time constants.
#pragma unroll
    for (int p = 0; p < PF; ++p)
        if (p < steps) issue(p, k_begin + (int64_t)p * BK);
    if (steps > 0) commit(0, 0);
    __syncthreads();

    for (int s0 = 0; s0 < steps; s0 += PF) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            int s = s0 + p;
            if (s < steps) {
                if (s + PF < steps) issue(p, k_begin + (int64_t)(s + PF) * BK);
                // The next tile goes to LDS after the first of the step's four slabs (it lands in the other
                // buffer, which every wavefront left before the last barrier): the loads have had a slab's
                // MFMAs to arrive, and the stores and their address and mask arithmetic run under the
                // remaining three slabs of the other wavefronts (measured over the CaffeNet model gradients:
                // after 1 / 2 / 3 / 4 slabs 699 / 708 / 712 / 740 us in total).
                typedef std::integral_constant<int, 0> I0;
                typedef std::integral_constant<int, 1> I1;
                typedef std::integral_constant<int, NPACK / 2> I2;
                compute(s & 1, I0{}, I1{});
                if (s + 1 < steps) commit((p + 1) % PF, (s + 1) & 1);
                compute(s & 1, I1{}, I2{});
                __syncthreads();
            }
        }
    }

    if (sh.fast_store) {
        if constexpr (std::is_same<Epi, PartialEpilogue>::value) {
            store_tile32<TI, TJ>(acc, row0 + wm * (BM / Cfg::WM), col0 + wn * (BN / Cfg::WN), li, h, z, epi);
        } else {
            __syncthreads();  // every wavefront is done with the operand tiles (and with none, if steps == 0)
            constexpr int STRIP = 16 * staged_pitch(TJ);
            static_assert((NT / 64) * STRIP <= (int)sizeof(lds_all), "staging strips fit in the operand buffers");
            store_tile_staged<TI, TJ, 16>(acc, row0 + wm * (BM / Cfg::WM), col0 + wn * (BN / Cfg::WN), lane, z, epi,
                                          reinterpret_cast<char *>(lds_all) + wave * STRIP, lds_add, row0);
        }
        return;
    }
    // 64-bit addressing for results beyond 4 GB
#pragma unroll
    for (int u = 0; u < TJ; ++u) {
        int j = col0 + wn * (BN / Cfg::WN) + u * 32 + li;
        typename Epi::Col col = epi.column(j);
#pragma unroll
        for (int t = 0; t < TI; ++t) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int i = row0 + wm * (BM / Cfg::WM) + t * 32 + 8 * (v / 4) + 4 * h + (v % 4);
                epi.store(i, col, acc[t][u][v], epi.row_add(i), z);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The same product with an instruction stream that keeps the matrix cores fed ("stream" kernel), for operands below
// 4 GB.
//
// What the kernel above loses is not bandwidth: in fp32 its matrix cores are busy 0.80 of the time whatever the tile,
// because at every slab both wavefronts of a SIMD wait for the same LDS reads, and at every step for predicated loads,
// the transposing stores and the barrier in a row.  Here
//   - loads are unpredicated buffer loads: 32-bit offsets that only need an addition per step, reads beyond the
//     operand return zero;
//   - a slab's fragments are read one slab ahead into a second register set, across the step's end too: the barrier
//     stands before the step's LAST slab, whose fragments are in registers by then, and the next step's first
//     fragments are read behind it, under that slab's MFMAs;
//   - the next tile goes to the other LDS buffer in the middle of the third slab, so its loads have two and a half
//     slabs to arrive and its stores run under MFMAs.
// Measured (TFLOP/s, plain -> this): fp32 256 x 186624 x 2400 123 -> 131 (matrix cores busy 0.80 -> 0.86), model gradient
// 384 x 3456 x 43264 122 -> 130; bf16 with the lowered matrix in memory 633 -> 727 and 567 -> 663; what is left in fp32 is
// the last round of tiles and the clock (2.06 GHz under this load).
// ------------------------------------------------------------------------------------------------
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}

// [rows][ld], reduction index contiguous; rows beyond the operand repeat the last one (their results are not stored).
// AHEAD: steps whose loads are in flight, i.e. loaders that take turns
template <typename T, int TILE_ROWS, int NT, int AHEAD> struct RedStream {
    static constexpr int KP = Pack<T>::KP;
    static constexpr int TASKS = TILE_ROWS * NPACK;
    static constexpr int PER_THREAD = (TASKS + NT - 1) / NT;
    static_assert(TASKS % NT == 0, "tile must divide over the threads");
    u32x4_t regs[PER_THREAD];
    uint32_t off[PER_THREAD];
    __device__ __forceinline__ void init(int64_t ld, int rows, int row0, int64_t k0, int tid)
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            const int t = tid + q * NT;
            int r = row0 + t / NPACK;
            r = r < rows ? r : rows - 1;
            off[q] = (uint32_t)(((int64_t)r * ld + k0 + (t % NPACK) * KP) * (int64_t)sizeof(T));
        }
    }
    // the packs of the next tile that begin at or behind `left` reduction indices read as zero
    __device__ __forceinline__ void cut(int left, int tid)
    {
        if ((tid % NPACK) * KP >= left)
#pragma unroll
            for (int q = 0; q < PER_THREAD; ++q) off[q] = 0xfffffff0u;  // beyond any operand
    }
    __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t src, uint32_t)
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            regs[q] = __builtin_amdgcn_raw_buffer_load_b128(src, off[q], 0, 0);
            off[q] += AHEAD * NPACK * 16;
        }
    }
    __device__ __forceinline__ void commit(uint4 *lds, int tid) const
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            const int t = tid + q * NT;
            reinterpret_cast<u32x4_t *>(lds)[(t % NPACK) * (TILE_ROWS + 1) + t / NPACK] = regs[q];
        }
    }
};

// [red][ld], the result's column index contiguous: a task is one pack group x 4 columns, transposed in registers.  In LDS
// the columns of a block of 32 change places, so that the transposing stores of neighbouring lanes, which hold columns 4
// apart, do not meet on a bank (in plain order four lanes share one, and the stores take four times their cycles): lane l of
// a fragment then holds column outer_column(l), which the epilogues are told.
__device__ __forceinline__ int outer_column(int place) { return 4 * (place % 8) + place / 8; }
template <typename T, int TILE_COLS, int NT, int AHEAD> struct OuterStream {
    static constexpr int KP = Pack<T>::KP;
    static constexpr int CHUNKS = TILE_COLS / 4;
    static constexpr int TASKS = NPACK * CHUNKS;
    static constexpr int PER_THREAD = (TASKS + NT - 1) / NT;
    static_assert(TASKS % NT == 0 || TASKS < NT, "tile must divide over the threads");
    typedef typename std::conditional<sizeof(T) == 4, u32x4_t, uint2>::type Piece;
    Piece regs[PER_THREAD][KP];
    uint32_t off[PER_THREAD];
    __device__ __forceinline__ void init(int64_t ld, int col0, int64_t k0, int tid)
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            const int t = tid + q * NT;
            off[q] = (uint32_t)(((k0 + (t / CHUNKS % NPACK) * KP) * ld + col0 + (t % CHUNKS) * 4) * (int64_t)sizeof(T));
        }
    }
    // row_bytes: ld * sizeof(T)
    __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t src, uint32_t row_bytes)
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
#pragma unroll
            for (int e = 0; e < KP; ++e) {
                if constexpr (sizeof(T) == 4)
                    regs[q][e] = __builtin_amdgcn_raw_buffer_load_b128(src, off[q] + e * row_bytes, 0, 0);
                else
                    regs[q][e] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(src, off[q] + e * row_bytes, 0, 0));
            }
            off[q] += AHEAD * NPACK * KP * row_bytes;
        }
    }
    static __device__ __forceinline__ uint32_t lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
    static __device__ __forceinline__ uint32_t hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
    __device__ __forceinline__ void commit(uint4 *lds, int tid) const
    {
#pragma unroll
        for (int q = 0; q < PER_THREAD; ++q) {
            const int t = tid + q * NT;
            if (TASKS < NT && t >= TASKS) return;  // fewer tasks than threads: the others loaded a copy for nothing
            // column 4c + j of a block of 32 lies at place 8j + c (outer_column): neighbouring lanes store side by side
            u32x4_t *dst = reinterpret_cast<u32x4_t *>(lds) + (t / CHUNKS) * (TILE_COLS + 1) + (t % CHUNKS) / 8 * 32 + (t % CHUNKS) % 8;
            const Piece *r = regs[q];
            if constexpr (sizeof(T) == 4) {
#pragma unroll
                for (int j = 0; j < 4; ++j) dst[8 * j] = u32x4_t{r[0][j], r[1][j], r[2][j], r[3][j]};
            } else {
                dst[0] = u32x4_t{lo(r[0].x, r[1].x), lo(r[2].x, r[3].x), lo(r[4].x, r[5].x), lo(r[6].x, r[7].x)};
                dst[8] = u32x4_t{hi(r[0].x, r[1].x), hi(r[2].x, r[3].x), hi(r[4].x, r[5].x), hi(r[6].x, r[7].x)};
                dst[16] = u32x4_t{lo(r[0].y, r[1].y), lo(r[2].y, r[3].y), lo(r[4].y, r[5].y), lo(r[6].y, r[7].y)};
                dst[24] = u32x4_t{hi(r[0].y, r[1].y), hi(r[2].y, r[3].y), hi(r[4].y, r[5].y), hi(r[6].y, r[7].y)};
            }
        }
    }
};

// fp32: the column operand of a stride-1 layer's data gradient read from dY [N][F][H][W]: element (k, j), k = (tap, f), is
// the entry of filter f's plane that tap (ky, kx) joins to input pixel j = (n, iy, ix), zero beyond the border, for f >= F
// and behind the last tap.  A reduction step is 32 filters of one tap (filters padded to whole steps).  A thread keeps one
// column for the whole product and fetches PER packs of 4 consecutive filters, the same for all lanes of a wavefront: where
// the tap falls is worked out once per step (which taps miss the image is a bit mask per column), an entry costs an
// addition, an or and a 4-byte load whose 64 lanes are neighbours, and a pack goes to LDS as it is.  The kernel puts one
// load behind each matrix instruction, which hides it; fetched together at the start of a step they cost a third of the rate.
struct ConvSrc {
    int32_t H, W, kh, kw, ph, pw;  // of dY's planes; the window and padding of the layer
    uint32_t plane, image;         // elements of a plane and of an image of dY
    int32_t F, f_steps;            // filters, steps per tap
    int32_t M;
    FastDiv div_out, div_W;        // input plane, its width
    // column j -> its output position at tap (0, 0); bit t of the result: tap t joins no entry of dY to it (at most 31 taps;
    // the bits behind the last tap are set)
    __device__ __forceinline__ uint32_t column(int j, uint32_t &n, int &y0, int &x0) const
    {
        uint32_t q, iy, ix;
        div_out.divmod((uint32_t)(j < M ? j : 0), n, q);
        div_W.divmod(q, iy, ix);
        y0 = (int)iy + ph, x0 = (int)ix + pw;
        uint32_t miss = 0u;
        int t = 0;
        for (int ky = 0; ky < kh; ++ky)
            for (int kx = 0; kx < kw; ++kx, ++t)
                if ((uint32_t)(y0 - ky) >= (uint32_t)H || (uint32_t)(x0 - kx) >= (uint32_t)W) miss |= 1u << t;
        return j < M ? miss | (0xffffffffu << t) : 0xffffffffu;  // a column that does not exist meets nothing
    }
};
template <int TILE_COLS, int NT> struct ConvStream {
    static constexpr int PER = NPACK * TILE_COLS / NT;
    static constexpr int PIXELS = PER * 4;  // of a thread and step
    static_assert(PER * NT == NPACK * TILE_COLS && TILE_COLS % 64 == 0, "a wavefront's lanes share their packs");
    uint32_t regs[PER][4];
    uint32_t base;           // bytes to the entry of filter 0 at tap (0, 0) (modulo 2^32)
    uint32_t miss;           // bit t: tap t is outside
    uint32_t at, out;        // of this step: bytes to filter 0's entry; all ones (times 4) where the tap is outside
    uint32_t tap, kx, step;  // wave-uniform: tap and step of the next fetch
    uint32_t up, f0, f;      // bytes back to the tap's entry; this wavefront's first filter in a step; of the next fetch
    __device__ __forceinline__ void init(const ConvSrc &c, int col0, int tid)
    {
        uint32_t n;
        int y0, x0;
        miss = c.column(col0 + tid % TILE_COLS, n, y0, x0);
        base = (n * c.image + (uint32_t)y0 * (uint32_t)c.W + (uint32_t)x0) * 4u;
        f0 = (uint32_t)__builtin_amdgcn_readfirstlane(tid / TILE_COLS) * PIXELS;
        tap = kx = step = up = 0u;
    }
    __device__ __forceinline__ void start(const ConvSrc &)  // of a step
    {
        at = base - up;
        out = (uint32_t)((int32_t)(miss << (31u - tap)) >> 31) & 0xfffffffcu;  // beyond any tensor: reads as zero
        f = f0 + step * (NPACK * 4);
    }
    __device__ __forceinline__ void fetch(__amdgpu_buffer_rsrc_t src, const ConvSrc &c, int e)  // e = 0 ... PIXELS - 1 in turn
    {
        const uint32_t none = f + e < (uint32_t)c.F ? 0u : 0xfffffffcu;
        regs[e / 4][e % 4] = __builtin_amdgcn_raw_buffer_load_b32(src, (at + (f + e) * c.plane * 4u) | out | none, 0, 0);
    }
    __device__ __forceinline__ void end(const ConvSrc &c)
    {
        if (++step == (uint32_t)c.f_steps) {
            step = 0u, ++tap, up += 4u;
            if (++kx == (uint32_t)c.kw) kx = 0u, up += (uint32_t)(c.W - c.kw) * 4u;
        }
    }
    __device__ __forceinline__ void commit(uint4 *lds, int tid) const
    {
        u32x4_t *dst = reinterpret_cast<u32x4_t *>(lds) + (tid / TILE_COLS * PER) * (TILE_COLS + 1) + tid % TILE_COLS;
#pragma unroll
        for (int q = 0; q < PER; ++q) dst[q * (TILE_COLS + 1)] = u32x4_t{regs[q][0], regs[q][1], regs[q][2], regs[q][3]};
    }
};

// What the column operand is in memory: contiguous along the reduction, along the result's columns, or dY as it lies
enum { COLS_RED = 0, COLS_OUTER = 1, COLS_CONV = 2 };

// wavefronts per SIMD that COLS_CONV's registers have to leave room for: as many workgroups as LDS lets reside
template <typename Cfg> constexpr int conv_waves()
{
    const int n = 160 * 1024 / (2 * NPACK * (Cfg::BM + Cfg::BN + 2) * 16 + Cfg::BM * 4);
    return n < 4 ? n : 4;
}

// Steps whose loads are in flight.  Two for column operands contiguous along the columns, except on the largest tile, whose
// accumulators leave no room for a second set of registers, and over few steps, where the longer prologue and code only cost.
// Operands contiguous along the reduction gain nothing: with 16 bytes a load their loads are few.  dY in place spreads its
// loads over the step.  (One -> two: fp32 32 x 32768 x 800 on 32 x 128 tiles 25.8 -> 21.0 us, 384 x 676 x 2304 on 64 x 64 60 ->
// 49; bf16 256 x 23328 x 2400 on 128 x 128 58.9 -> 54.0, the stores' order included.  Three steps, fp32 32 x 131072 x 75: 17.4
// -> 18.5; one step, bf16 75 x 102400 x 32: 12.2 -> 13.4.)
constexpr int FEW_STEPS = 5;
template <typename Cfg, int COL, bool FEW> constexpr int stream_ahead() { return COL != COLS_OUTER || FEW || Cfg::BM * Cfg::BN >= 256 * 256 ? 1 : 2; }

// CUT: the row operand is not padded with zeros to whole reduction steps, and what stands behind its last one (the next
// row's first elements) may be infinite, which the column operand's zeros would not cancel: it reads as zero
template <typename T, typename Cfg, int COL, typename Epi, bool CUT = false, bool FEW = false>
__global__ __launch_bounds__(Cfg::NT, COL == COLS_CONV ? conv_waves<Cfg>() : 1) void gemm_stream_kernel(const T *__restrict__ A, int64_t lda, uint32_t a_bytes,
                                                              const T *__restrict__ B, int64_t ldb, uint32_t b_bytes,
                                                              GemmShape sh, Epi epi, ConvSrc conv)
{
    constexpr int KP = Pack<T>::KP;
    constexpr int BK = NPACK * KP;
    constexpr int BM = Cfg::BM, BN = Cfg::BN, NT = Cfg::NT, TI = Cfg::TI, TJ = Cfg::TJ;
    constexpr int LA = BM + 1, LB = BN + 1;
    constexpr int SLABS = NPACK / 2;
    __shared__ uint4 lds_all[2 * NPACK * (LA + LB)];  // A buffers 0, 1 then B buffers 0, 1
    __shared__ float lds_add[Epi::HAS_ROW_ADD ? BM : 1];
    auto lds_a = [&](int buf) { return lds_all + buf * (NPACK * LA); };
    auto lds_b = [&](int buf) { return lds_all + 2 * NPACK * LA + buf * (NPACK * LB); };

    const int item = (blockIdx.x % 8) * sh.per_xcd + blockIdx.x / 8;  // contiguous ranges of (tile, split) per XCD
    if (item >= sh.n_items) return;
    const int z = item / sh.n_blocks, tile = item - z * sh.n_blocks;
    const int ti = tile % sh.tiles_i, tj = tile / sh.tiles_i;
    const int row0 = ti * BM, col0 = tj * BN;
    const int64_t k_begin = (int64_t)z * sh.chunk;
    const int64_t k_end = k_begin + sh.chunk < sh.red ? k_begin + sh.chunk : sh.red;
    const int steps = k_end > k_begin ? (int)((k_end - k_begin + BK - 1) / BK) : 0;

    const int tid = threadIdx.x;
    const int lane = tid % 64, wave = tid / 64;
    const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
    const int li = lane % 32, h = lane / 32;
    if constexpr (Epi::HAS_ROW_ADD)  // read back after the main loop's barriers
        for (int i = tid; i < BM; i += NT) lds_add[i] = epi.row_add(row0 + i);

    f32x16 acc[TI][TJ];
#pragma unroll
    for (int t = 0; t < TI; ++t)
#pragma unroll
        for (int u = 0; u < TJ; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][u][v] = 0.f;

    const __amdgpu_buffer_rsrc_t ra = buffer_of(A, a_bytes), rb = buffer_of(B, b_bytes);
    constexpr int AHEAD = stream_ahead<Cfg, COL, FEW>();
    RedStream<T, BM, NT, AHEAD> loader_a[AHEAD];
    typename std::conditional<COL == COLS_CONV, ConvStream<BN, NT>,
                              typename std::conditional<COL == COLS_OUTER, OuterStream<T, BN, NT, AHEAD>, RedStream<T, BN, NT, AHEAD>>::type>::type loader_b[AHEAD];
    auto &la = loader_a[0];
    auto &lb = loader_b[0];
    const uint32_t b_row = (uint32_t)(ldb * (int64_t)sizeof(T));
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
        loader_a[i].init(lda, sh.rows, row0, k_begin + i * BK, tid);
        if constexpr (COL == COLS_CONV) loader_b[i].init(conv, col0, tid);
        else if constexpr (COL == COLS_OUTER) loader_b[i].init(ldb, col0, k_begin + i * BK, tid);
        else loader_b[i].init(ldb, sh.cols, col0, k_begin + i * BK, tid);
    }
    auto issue_b = [&]() {  // of the first tile
        if constexpr (COL == COLS_CONV) {
            lb.start(conv);
#pragma unroll
            for (int e = 0; e < lb.PIXELS; ++e) lb.fetch(rb, conv, e);
            lb.end(conv);
        } else {
            lb.issue(rb, b_row);
        }
    };
    // COLS_CONV: a tap's sum over the filters is complete after conv.f_steps steps; the taps' sums are added to a second set of
    // accumulators in ascending order.  These are the sums, and this is the order, of the route over dD-hat and col2im: the
    // two give the same bits, so that which of them a batch's size selects shows in no result.
    // A tap that joins nothing to a column is left out there, not added as zero: an infinite or NaN weight would make NaN of
    // the zeros it was multiplied with.
    f32x16 total[COL == COLS_CONV ? TI : 1][COL == COLS_CONV ? TJ : 1];
    [[maybe_unused]] uint32_t miss[COL == COLS_CONV ? TJ : 1];
    auto flush = [&]([[maybe_unused]] uint32_t tap) {
        if constexpr (COL == COLS_CONV) {
#pragma unroll
            for (int u = 0; u < TJ; ++u) {
                if ((miss[u] >> tap & 1u) == 0u) {
#pragma unroll
                    for (int t = 0; t < TI; ++t)
#pragma unroll
                        for (int v = 0; v < 16; ++v) total[t][u][v] += acc[t][u][v];
                }
#pragma unroll
                for (int t = 0; t < TI; ++t)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[t][u][v] = 0.f;
            }
        }
    };
    if constexpr (COL == COLS_CONV) {
#pragma unroll
        for (int u = 0; u < TJ; ++u) {
            uint32_t n;
            int y0, x0;
            miss[u] = conv.column(col0 + wn * (BN / Cfg::WN) + 32 * u + li, n, y0, x0);
#pragma unroll
            for (int t = 0; t < TI; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) total[t][u][v] = 0.f;
        }
    }

    uint4 fa[2][TI], fb[2][TJ];
    auto read_frag = [&](auto set, int buf, int slab) {
        constexpr int S = decltype(set)::value;
        const uint4 *pa = lds_a(buf) + (slab * 2 + h) * LA + wm * (BM / Cfg::WM) + li;
        const uint4 *pb = lds_b(buf) + (slab * 2 + h) * LB + wn * (BN / Cfg::WN) + li;
#pragma unroll
        for (int t = 0; t < TI; ++t) fa[S][t] = pa[32 * t];
#pragma unroll
        for (int u = 0; u < TJ; ++u) fb[S][u] = pb[32 * u];
    };
    auto mma_cols = [&](auto set, int u0, int u1) {
        constexpr int S = decltype(set)::value;
#pragma unroll
        for (int u = 0; u < TJ; ++u)
            if (u >= u0 && u < u1)
#pragma unroll
                for (int t = 0; t < TI; ++t) Mma<T>::run(fa[S][t], fb[S][u], acc[t][u]);
    };
    // A slab's matrix instructions one at a time, `EACH` of the next tile's pixels (from the E0-th on) behind each.
    auto mma_fetch = [&](auto set, auto e0, auto each) {
        if constexpr (COL == COLS_CONV) {
            constexpr int S = decltype(set)::value, E0 = decltype(e0)::value, EACH = decltype(each)::value;
            int e = E0;
#pragma unroll
            for (int u = 0; u < TJ; ++u)
#pragma unroll
                for (int t = 0; t < TI; ++t)
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const uint32_t av = x == 0 ? fa[S][t].x : x == 1 ? fa[S][t].y : x == 2 ? fa[S][t].z : fa[S][t].w;
                        const uint32_t bv = x == 0 ? fb[S][u].x : x == 1 ? fb[S][u].y : x == 2 ? fb[S][u].z : fb[S][u].w;
                        acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(av), __uint_as_float(bv), acc[t][u], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int i = 0; i < EACH; ++i, ++e)
                            if (e < lb.PIXELS) lb.fetch(rb, conv, e);
                        __builtin_amdgcn_sched_barrier(0);
                    }
        }
    };
    typedef std::integral_constant<int, 0> S0;
    typedef std::integral_constant<int, 1> S1;
    static_assert(SLABS == 4, "the schedule below");
    // one entry of dY per matrix instruction, over the first two slabs where one slab has too few for all pixels; two where two have
    constexpr int MMAS = 4 * TI * TJ, CONV_PIXELS = NPACK * BN / NT * 4, EACH = CONV_PIXELS > 2 * MMAS ? 2 : 1;
    static_assert(COL != COLS_CONV || 2 * MMAS * EACH >= CONV_PIXELS, "all of a tile's pixels fit behind two slabs");

    [[maybe_unused]] const int cut_step = k_end == sh.red ? steps - 1 : -1, cut_left = (int)(sh.red % BK);
    if constexpr (AHEAD == 2) {
        // A step of a small tile takes less than a memory latency, and waited for its successor's loads every time: the loads of
        // two steps are in flight, in two sets of registers that take turns.
        auto issue = [&](auto set, int st) {
            constexpr int P = decltype(set)::value;
            if constexpr (CUT)
                if (st == cut_step) loader_a[P].cut(cut_left, tid);
            loader_a[P].issue(ra, 0);
            loader_b[P].issue(rb, b_row);
        };
        auto commit = [&](auto set, int buf) {
            constexpr int P = decltype(set)::value;
            loader_a[P].commit(lds_a(buf), tid);
            loader_b[P].commit(lds_b(buf), tid);
        };
        // Step s, whose tile lies in buffer P = s mod 2; the next one's loads are in flight in the other set of registers.
        auto step = [&](auto set, int s, bool load, bool more) {
            constexpr int P = decltype(set)::value;
            typedef std::integral_constant<int, P ^ 1> Other;
            if (load) issue(set, s + 2);
            read_frag(S1{}, P, 1);
            __builtin_amdgcn_sched_barrier(0);
            mma_cols(S0{}, 0, TJ);
            __builtin_amdgcn_sched_barrier(0);
            read_frag(S0{}, P, 2);
            __builtin_amdgcn_sched_barrier(0);
            mma_cols(S1{}, 0, TJ);
            __builtin_amdgcn_sched_barrier(0);
            read_frag(S1{}, P, 3);
            __builtin_amdgcn_sched_barrier(0);
            mma_cols(S0{}, 0, TJ / 2);
            __builtin_amdgcn_sched_barrier(0);
            if (more) commit(Other{}, P ^ 1);
            __builtin_amdgcn_sched_barrier(0);
            mma_cols(S0{}, TJ / 2, TJ);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            if (more) read_frag(S0{}, P ^ 1, 0);
            __builtin_amdgcn_sched_barrier(0);
            mma_cols(S1{}, 0, TJ);
            __builtin_amdgcn_sched_barrier(0);
        };
        if (steps > 1) {
            issue(S0{}, 0);
            issue(S1{}, 1);
            commit(S0{}, 0);
        } else if (steps > 0) {
            issue(S0{}, 0);
            commit(S0{}, 0);
        }
        __syncthreads();
        if (steps > 0) read_frag(S0{}, 0, 0);
        int s = 0;
        // unconditional loads: those in flight can be told apart only where no condition decides on them
        for (; s + 3 < steps; s += 2) {
            step(S0{}, s, true, true);
            step(S1{}, s + 1, true, true);
        }
        if (s < steps) step(S0{}, s, s + 2 < steps, s + 1 < steps);
        if (s + 1 < steps) step(S1{}, s + 1, false, s + 2 < steps);
        if (s + 2 < steps) step(S0{}, s + 2, false, false);
    } else {
    if (steps > 0) {
        if constexpr (CUT)
            if (cut_step == 0) la.cut(cut_left, tid);
        la.issue(ra, 0);
        issue_b();
        la.commit(lds_a(0), tid);
        lb.commit(lds_b(0), tid);
    }
    __syncthreads();
    if (steps > 0) read_frag(S0{}, 0, 0);
    [[maybe_unused]] int until_flush = conv.f_steps, tap = 0;
    for (int s = 0; s < steps; ++s) {
        const int buf = s & 1;
        // COLS_CONV also fetches the tile behind the last one, which reads as zero: its loads in flight could not be told
        // from those of an earlier step if they depended on a condition, and every fetch would wait for the one before it
        const bool more = COL == COLS_CONV || s + 1 < steps;
        if (more) {
            if constexpr (CUT)
                if (s + 1 == cut_step) la.cut(cut_left, tid);
            la.issue(ra, 0);
            if constexpr (COL == COLS_CONV) lb.start(conv);
            else lb.issue(rb, b_row);
        }
        read_frag(S1{}, buf, 1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (COL == COLS_CONV) mma_fetch(S0{}, std::integral_constant<int, 0>{}, std::integral_constant<int, EACH>{});
        else mma_cols(S0{}, 0, TJ);
        __builtin_amdgcn_sched_barrier(0);
        read_frag(S0{}, buf, 2);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (COL == COLS_CONV && MMAS * EACH < CONV_PIXELS)
            mma_fetch(S1{}, std::integral_constant<int, MMAS * EACH>{}, std::integral_constant<int, EACH>{});
        else
            mma_cols(S1{}, 0, TJ);
        if constexpr (COL == COLS_CONV) lb.end(conv);
        __builtin_amdgcn_sched_barrier(0);
        read_frag(S1{}, buf, 3);
        __builtin_amdgcn_sched_barrier(0);
        mma_cols(S0{}, 0, TJ / 2);
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            la.commit(lds_a(buf ^ 1), tid);
            lb.commit(lds_b(buf ^ 1), tid);
        }
        __builtin_amdgcn_sched_barrier(0);
        mma_cols(S0{}, TJ / 2, TJ);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        if (more) read_frag(S0{}, buf ^ 1, 0);
        __builtin_amdgcn_sched_barrier(0);
        mma_cols(S1{}, 0, TJ);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (COL == COLS_CONV) {
            if (--until_flush == 0) flush(tap), ++tap, until_flush = conv.f_steps;
        }
    }
    }
    if constexpr (COL == COLS_CONV) {
#pragma unroll
        for (int t = 0; t < TI; ++t)
#pragma unroll
            for (int u = 0; u < TJ; ++u) acc[t][u] = total[t][u];
    }

    const int lane_col = COL == COLS_OUTER ? outer_column(li) : li;
    if constexpr (std::is_same<Epi, PartialEpilogue>::value) {
        store_tile32<TI, TJ>(acc, row0 + wm * (BM / Cfg::WM), col0 + wn * (BN / Cfg::WN), lane_col, h, z, epi);
    } else {
        __syncthreads();  // every wavefront has read its last fragments
        constexpr int STRIP = 16 * staged_pitch(TJ);
        static_assert((NT / 64) * STRIP <= (int)sizeof(lds_all), "staging strips fit in the operand buffers");
        store_tile_staged<TI, TJ, 16>(acc, row0 + wm * (BM / Cfg::WM), col0 + wn * (BN / Cfg::WN), lane, z, epi,
                                      reinterpret_cast<char *>(lds_all) + wave * STRIP, lds_add, row0, nullptr, 1, 0, lane_col);
    }
}

// Sum the per-split partial results into the final fp32 tensor, in a fixed order (deterministic): a
// workgroup takes 64 consecutive elements; wavefront l adds splits l, l+4, l+8, ... in that order, four
// loads in flight, and the four sums are then added as (s0 + s1) + (s2 + s3).
// The launch may carry extra workgroups (blockIdx >= main_blocks) that finish the bias gradient: one
// wavefront per filter adds that filter's per-block sums left by the dY packing kernel (strided per lane in
// block order, then a fixed tree) -- the same arithmetic as bias_reduce_kernel, without a launch of its own.
// PHASED: the partial results are [F][K' + 1] in the phase-split order of a stride-4 layer (see
// launch_gemm_wgrad_phase), K' index ((c * 4 + ph) * kh + ky) * kwq + kq standing for window column
// kx = 4 kq + ph; entries with kx >= kw are padding and are dropped, the others go to [F][C][kh][kw];
// column K' is the bias gradient.
struct PhaseMap { int32_t C, kh, kw; FastDiv div_Kp, div_khkwq, div_kwq; };

template <bool PHASED>
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float *__restrict__ partials, int splits,
                                                              int64_t count, float *__restrict__ out, unsigned main_blocks,
                                                              const float *__restrict__ bias_partials, int bias_blocks,
                                                              int F, float *__restrict__ dbias, PhaseMap pm)
{
    __shared__ float part[4][64];
    const int c = threadIdx.x % 64, l = threadIdx.x / 64;
    if (blockIdx.x >= main_blocks) {
        const int f = (int)(blockIdx.x - main_blocks) * 4 + l;
        if (f < F) {
            float acc = 0.f;
            for (int b = c; b < bias_blocks; b += 64) acc += bias_partials[(int64_t)f * bias_blocks + b];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
            if (c == 0) dbias[f] = acc;
        }
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * 64 + c;
    float acc = 0.f;
    if (i < count) {
        const float *p = partials + i;
        int z = l;
        for (; z + 12 < splits; z += 16) {
            float a0 = p[(int64_t)z * count], a1 = p[(int64_t)(z + 4) * count];
            float a2 = p[(int64_t)(z + 8) * count], a3 = p[(int64_t)(z + 12) * count];
            acc += a0, acc += a1, acc += a2, acc += a3;
        }
        for (; z < splits; z += 4) acc += p[(int64_t)z * count];
    }
    part[l][c] = acc;
    __syncthreads();
    if (l == 0 && i < count) {
        const float sum = (part[0][c] + part[1][c]) + (part[2][c] + part[3][c]);
        if constexpr (PHASED) {
            uint32_t f, kp, cp, rem, ky, kq;
            pm.div_Kp.divmod((uint32_t)i, f, kp);  // columns per row: K' + 1, the last one the bias gradient
            pm.div_khkwq.divmod(kp, cp, rem);
            pm.div_kwq.divmod(rem, ky, kq);
            const int kx = 4 * (int)kq + (int)(cp % 4u);
            if (kp + 1u == pm.div_Kp.d) {
                if (dbias != nullptr) dbias[f] = sum;
            } else if (kx < pm.kw) {
                out[(((int64_t)f * pm.C + cp / 4u) * pm.kh + ky) * pm.kw + kx] = sum;
            }
        } else {
            out[i] = sum;
        }
    }
}

// The same ordered sum for element counts that are a multiple of 4: a thread owns four consecutive elements and adds
// the splits in ascending order, eight 16-byte loads in flight (the 4-byte loads of the kernel above keep too few
// bytes in flight to reach the memory system's rate).  Extra workgroups finish the bias gradient as above.
__global__ __launch_bounds__(256) void reduce_partials_vec_kernel(const float4 *__restrict__ partials, int splits, int64_t count4,
                                                                  float4 *__restrict__ out, unsigned main_blocks,
                                                                  const float *__restrict__ bias_partials, int bias_blocks,
                                                                  int F, float *__restrict__ dbias)
{
    if (blockIdx.x >= main_blocks) {
        const int c = threadIdx.x % 64, f = (int)(blockIdx.x - main_blocks) * 4 + threadIdx.x / 64;
        if (f < F) {
            float acc = 0.f;
            for (int b = c; b < bias_blocks; b += 64) acc += bias_partials[(int64_t)f * bias_blocks + b];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
            if (c == 0) dbias[f] = acc;
        }
        return;
    }
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count4) return;
    const float4 *p = partials + i;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int z = 0;
    for (; z + 8 <= splits; z += 8) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(int64_t)(z + u) * count4];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc.x += v[u].x, acc.y += v[u].y, acc.z += v[u].z, acc.w += v[u].w;
    }
    for (; z < splits; ++z) {
        const float4 v = p[(int64_t)z * count4];
        acc.x += v.x, acc.y += v.y, acc.z += v.z, acc.w += v.w;
    }
    out[i] = acc;
}

// The same for a gradient of few elements over many splits (first layers: 32 x 75 elements, 512 splits): sixteen lanes
// share an element's splits (lane l takes l, l + 16, ...) and their sums are added in a fixed tree, so that the launch
// has sixteen times the threads (32 x 75 x 512: 27 -> 5 us).
__global__ __launch_bounds__(256) void reduce_partials_deep_kernel(const float4 *__restrict__ partials, int splits, int64_t count4,
                                                                   float4 *__restrict__ out, unsigned main_blocks,
                                                                   const float *__restrict__ bias_partials, int bias_blocks,
                                                                   int F, float *__restrict__ dbias)
{
    if (blockIdx.x >= main_blocks) {
        const int c = threadIdx.x % 64, f = (int)(blockIdx.x - main_blocks) * 4 + threadIdx.x / 64;
        if (f < F) {
            float acc = 0.f;
            for (int b = c; b < bias_blocks; b += 64) acc += bias_partials[(int64_t)f * bias_blocks + b];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
            if (c == 0) dbias[f] = acc;
        }
        return;
    }
    __shared__ float4 part[16][16];
    const int c = threadIdx.x % 16, l = threadIdx.x / 16;
    const int64_t i = (int64_t)blockIdx.x * 16 + c;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < count4) {
        const float4 *p = partials + i;
        int z = l;
        for (; z + 112 < splits; z += 128) {
            float4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p[(int64_t)(z + 16 * u) * count4];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc.x += v[u].x, acc.y += v[u].y, acc.z += v[u].z, acc.w += v[u].w;
        }
        for (; z < splits; z += 16) {
            const float4 v = p[(int64_t)z * count4];
            acc.x += v.x, acc.y += v.y, acc.z += v.z, acc.w += v.w;
        }
    }
    part[l][c] = acc;
    for (int half = 8; half > 0; half >>= 1) {
        __syncthreads();
        if (l < half) {
            const float4 v = part[l + half][c];
            acc.x += v.x, acc.y += v.y, acc.z += v.z, acc.w += v.w;
            part[l][c] = acc;
        }
    }
    if (l == 0 && i < count4) out[i] = acc;
}

static GemmShape make_shape(int rows, int cols, int64_t red, int64_t chunk, int bm, int bn, int splits)
{
    GemmShape s;
    s.rows = rows;
    s.cols = cols;
    s.red = red;
    s.chunk = chunk;
    s.tiles_i = (rows + bm - 1) / bm;
    s.tiles_j = (cols + bn - 1) / bn;
    s.n_blocks = s.tiles_i * s.tiles_j;
    s.n_items = s.n_blocks * splits;
    s.per_xcd = (s.n_items + 7) / 8;
    s.fast_store = 0;
    return s;
}

// Tile configurations compiled in.  Index = the tuning override (omni_tuning_set, for sweeps) or the choice of
// pick_tile() / gemm_split_plan().  The direct model gradient only has tiles 1 and 2.
typedef Tile<128, 128, 2, 2, 1> Tile0;
typedef Tile<256, 256, 4, 2, 1> Tile1;
typedef Tile<384, 128, 4, 2, 1> Tile2;  // model gradient only
typedef Tile<96, 128, 1, 4, 1> Tile3;
typedef Tile<64, 128, 2, 2, 1> Tile4;
typedef Tile<64, 64, 2, 2, 1> Tile5;
typedef Tile<32, 128, 1, 4, 1> Tile6;
typedef Tile<192, 256, 2, 4, 1> Tile7;
constexpr int N_TILES = 8;
static const struct {
    int bm, bn;
    int resident;        // workgroups per compute unit (LDS)
    double eff_f32;      // share of the 256 x 256 tile's rate on a large fp32 product
} kTiles[N_TILES] = {{128, 128, 2, 0.93}, {256, 256, 1, 1.0}, {384, 128, 1, 0.98}, {96, 128, 2, 0.91},
                     {64, 128, 3, 0.9},   {64, 64, 4, 0.87},  {32, 128, 3, 0.8},   {192, 256, 1, 0.98}};

static int g_tile_override = -1;  // omni_tuning_set(OMNI_TUNE_GEMM_TILE, ...): sweeps and tests only
void set_gemm_tile_override(int v) { g_tile_override = (v >= 0 && v < N_TILES) ? v : -1; }
static int tile_override() { return g_tile_override; }

// Tile of a product whose reduction is not split: the one with the least estimated time per reduction step.  m is the
// matrix cores' time for one workgroup's step (BM BN / 4 cycles in fp32, / 32 in bf16, at 2.1 GHz).  A step also has a
// serial part (loads to registers to LDS, a barrier) that only other workgroups on the compute unit can fill: a
// workgroup alone takes m + 0.4 us per fp32 step and m + 1.0 us per bf16 step, measured with 16 ... 256 workgroups.
//   fp32: with r workgroups per compute unit in all the matrix cores bound it, r m / eff, unless r is so small that
//         the serial part shows.  (256 x 43264 x 3456: 169 tiles of 256 x 256 take 836 us, 676 of 128 x 128 677;
//         384 x 1352 x 2304: 168 us with 33 tiles of 128 x 128, 64 us with 132 of 64 x 64; 32 x 32768 x 800: 65 us with
//         128 rows, 28 us with 32.)
//   bf16: m is so short that the serial part always counts; resident workgroups overlap theirs, with some loss to each
//         other (15 % per neighbour).  (With one step of loads in flight, 256 x 23328 x 2400: 78 us with 92 tiles of
//         256 x 256, 57 with 366 of 128 x 128; 256 x 186624 x 2400 316 and 400 us.)
// `wavefronts4`: only the tiles of four wavefronts.  *us: the estimated time of a step.
static int estimate_tile(int rows, int cols, int dtype, bool wavefronts4, double *us)
{
    int best = 0;
    double least = 0.0;
    for (int t = 0; t < N_TILES; ++t) {
        if (t == 2 || (wavefronts4 && kTiles[t].resident == 1)) continue;
        const double area = (double)kTiles[t].bm * kTiles[t].bn;
        const int64_t tiles = (int64_t)((rows + kTiles[t].bm - 1) / kTiles[t].bm) * ((cols + kTiles[t].bn - 1) / kTiles[t].bn);
        const int64_t r = (tiles + 255) / 256, resident = r < kTiles[t].resident ? r : kTiles[t].resident;
        const double rounds = (double)((r + resident - 1) / resident);
        double cost;
        if (dtype == OMNI_BF16) {
            const double m = area / 32.0 / 2100.0;
            cost = rounds * (m + 1.0) * (1.0 + 0.15 * (double)(resident - 1));
        } else {
            const double m = area / 4.0 / 2100.0, bound = (double)r * m / kTiles[t].eff_f32;
            cost = rounds * (m + 0.4) > bound ? rounds * (m + 0.4) : bound;
        }
        if (t == 0 || cost < least) best = t, least = cost;
    }
    *us = least;
    return best;
}
static int pick_tile(int rows, int cols, int dtype)
{
    const int o = tile_override();
    double us;
    return o >= 0 ? o : estimate_tile(rows, cols, dtype, false, &us);
}

// The large tile that a result fills about as well as 128 x 128: 256 x 256, or (tall) 384 x 128 for results of 384 rows;
// 0: neither.
static int pick_large_tile(int64_t rows, int64_t cols, bool tall)
{
    auto fill = [](int64_t n, int64_t t) { return (double)n / (double)(((n + t - 1) / t) * t); };
    const double u256 = fill(rows, 256) * fill(cols, 256), u128 = fill(rows, 128) * fill(cols, 128);
    const double u384 = fill(rows, 384) * fill(cols, 128);
    if (tall && u384 > u256 && u384 >= 0.9 * u128) return 2;
    return u256 >= 0.9 * u128 ? 1 : 0;
}

// The direct model gradient (column operand from X) has the two large tiles only.
static int pick_direct_tile(int rows, int cols) { return pick_large_tile(rows, cols, true); }

// Whether the model gradient of this layer takes its column operand straight from X.  Assembling a pack
// costs vector ALU work that is shared by the rows of the result tile, so this pays only with the
// 256 x 256 tile (measured: with 128-row tiles lowering first and streaming D-hat is faster).
bool wgrad_direct_supported(const ConvGeom &g, int dtype)
{
    return dtype == OMNI_BF16 && g.sh == 1 && g.sw == 1 && g.pw < 24 && pick_direct_tile(g.F, g.K) != 0 &&
           (int64_t)g.N * g.C * g.H * g.W < 0x7fffffffll - 16 && (int64_t)g.N * g.C * g.H * g.W >= 8;
}

// Whether the direct model gradient pads whole image planes (see DIRECT_PLANES) rather than output rows.
bool wgrad_direct_planes(const ConvGeom &g)
{
    return g.sh == 1 && g.sw == 1 && g.Wo == g.W &&
           (int64_t)((g.Ho * g.Wo + 7) / 8) * (g.kh * g.kw + 1) <= DIRECT_TAB;
}

int64_t gemm_large_tiles(int64_t rows, int64_t cols, bool outer, bool *small)
{
    const int t = pick_large_tile(rows, cols, !outer);
    *small = t == 0;
    return ((rows + kTiles[t].bm - 1) / kTiles[t].bm) * ((cols + kTiles[t].bn - 1) / kTiles[t].bn);
}

// Estimated time of a product whose reduction is split, in microseconds (a constant part left out), and of adding its sums:
//   compute: of every round of workgroups (as many per compute unit as reside there) each reduction step takes lat + k m per
//            workgroup on the unit, m being the matrix cores' time for one (BM BN / 4 cycles in fp32, / 32 in bf16, at
//            2.1 GHz); lat, the step's serial part, grows with the columns staged.  A round also has a fixed part, and the
//            last of several takes as long as a full one (640 x 19200 x 2825 fp32 on 750 workgroups of 128 x 128: 680 us; on
//            3 000 of 64 x 64, 548).
//   memory:  the operands once, at `once` MB per us, and again for every further row and column of tiles, at `again`.
//   The two overlap partly: the root of the sum of their squares.
//   sums:    written and added at `sums` us per MB, and a launch for it.
// The constants are least-squares fits to 245 000 measured times: 8 770 products of 1 to 1 200 rows, 32 to 24 000 columns
// and reductions of 256 to 770 000, every tile, 1 to 500 ranges, operands of the outer form cold.  Mean deviation 4 % in fp32,
// 6 to 9 % in bf16; the tile and ranges it picks are 1 to 2 % (outer bf16 3 %) slower than the best measured ones on average
// and 0.69 to 0.90 times as long as one round of 256 x 256 tiles or two workgroups per unit of 128 x 128, at most 1.11 times.
struct SplitModel { double lat, lat_cols, k, round, sums, add, once, again; };
static const SplitModel kSplitModel[2][2] = {
    // reduction contiguous (model gradient): fp32, bf16
    {{0.151, 0.140, 0.924, 0.21, 0.333, 7.1, 9.13, 1e9}, {0.448, 0.045, 1.017, 2.71, 0.259, 5.7, 5.64, 96.0}},
    // columns contiguous (forward, data gradient)
    {{0.281, 0.083, 0.929, 1.37, 0.332, 0.3, 9.33, 1e9}, {0.685, 0.064, 1.138, 1.35, 0.296, 4.5, 6.53, 31.8}}};

static double split_us(int t, int64_t rows, int64_t cols, int64_t red, int dtype, bool outer, int64_t splits)
{
    const SplitModel &c = kSplitModel[outer][dtype == OMNI_BF16];
    const double bm = kTiles[t].bm, bn = kTiles[t].bn, e = dtype == OMNI_BF16 ? 2e-6 : 4e-6;
    const int64_t ti = (rows + kTiles[t].bm - 1) / kTiles[t].bm, tj = (cols + kTiles[t].bn - 1) / kTiles[t].bn, bk = gemm_red_tile(dtype);
    const int64_t steps = ((red + splits - 1) / splits + bk - 1) / bk, r = (ti * tj * splits + 255) / 256, resident = kTiles[t].resident;
    const int64_t full = r / resident, rest = r - full * resident;
    const double m = bm * bn / (dtype == OMNI_BF16 ? 32.0 : 4.0) / 2100.0, lat = c.lat + c.lat_cols * bn / 128.0;
    const double step = (double)full * (lat + (double)resident * m * c.k) + (rest > 0 ? lat + (double)(full > 0 ? resident : rest) * m * c.k : 0.0);
    const double compute = (double)steps * step + c.round * (double)(full + (rest > 0 ? 1 : 0));
    const double memory = (double)red * e * ((double)(rows + cols) / c.once + ((double)rows * (double)(tj - 1) + (double)cols * (double)(ti - 1)) / c.again);
    const double sums = splits > 1 ? c.add + c.sums * (double)splits * (double)rows * (double)cols * 4e-6 : 0.0;
    return sqrt(compute * compute + memory * memory) + sums;
}

int64_t gemm_split_most(int64_t rows, int64_t cols, bool outer)
{
    int64_t most = 1;
    for (int t = 0; t < N_TILES; ++t) {
        const int64_t tiles = ((rows + kTiles[t].bm - 1) / kTiles[t].bm) * ((cols + kTiles[t].bn - 1) / kTiles[t].bn);
        if (!(t == 2 && outer) && 256 * kTiles[t].resident / tiles > most) most = 256 * kTiles[t].resident / tiles;
    }
    return most;
}

// Operands below 4 GB, as launch_stream() asks (the result is far smaller)
bool gemm_streams(int64_t rows, int64_t cols, int64_t red, int dtype, bool outer)
{
    const double e = dtype == OMNI_BF16 ? 2.0 : 4.0, reach = (double)red + (outer ? 2.0 * gemm_red_tile(dtype) : 0.0);
    return (double)rows * reach * e < 4.0e9 && (double)cols * reach * e < 4.0e9;
}

// Every tile (384 x 128 only where it is the large tile of a model gradient) with the ranges that give each compute unit one
// workgroup, two, ... as many as reside there, and with `least`.
SplitPlan gemm_split_plan(int64_t rows, int64_t cols, int64_t red, int dtype, bool outer, int64_t least, int64_t most, double room)
{
    SplitPlan best{0, least};
    if (!gemm_streams(rows, cols, red, dtype, outer)) return best;  // the plain kernel's own tile: `least` is made for it
    double least_us = 0.0;
    bool found = false;
    const int o = outer ? -1 : tile_override();
    const bool tall = !outer && pick_large_tile(rows, cols, true) == 2;
    const double slice = (double)rows * (double)cols * 4.0;
    for (int t = 0; t < N_TILES; ++t) {
        if (o >= 0 ? t != o : t == 2 && !tall) continue;
        const int64_t tiles = ((rows + kTiles[t].bm - 1) / kTiles[t].bm) * ((cols + kTiles[t].bn - 1) / kTiles[t].bn);
        int64_t last = 0;
        for (int r = 0; r <= kTiles[t].resident; ++r) {
            int64_t n = r == 0 ? least : 256 * r / tiles;
            n = n < most ? n : most;
            if (n < least || n == last || (n > least && (double)n * slice > room)) continue;
            last = n;
            const double us = split_us(t, rows, cols, red, dtype, outer, n);
            if (!found || us < least_us) best = SplitPlan{t, n}, least_us = us, found = true;
        }
    }
    return best;
}

template <typename T, typename Cfg, bool OUTER, typename Epi>
static bool launch_stream(const T *A, int64_t lda, const T *B, int64_t ldb, int rows, int cols, int64_t red,
                          int64_t chunk, int splits, const Epi &epi, hipStream_t s)
{
    constexpr int BK = NPACK * Pack<T>::KP;
    const double a_bytes = (double)rows * lda * sizeof(T), b_bytes = (double)(OUTER ? red : cols) * ldb * sizeof(T);
    const double b_reach = b_bytes + (OUTER ? (double)(2 * BK) * ldb * sizeof(T) : 0.0);  // last step's rows beyond `red`
    if (!epi.fits32() || a_bytes >= 4.0e9 || b_reach >= 4.0e9 || lda % Pack<T>::KP != 0 || (!OUTER && ldb % BK != 0)) return false;
    GemmShape sh = make_shape(rows, cols, red, chunk, Cfg::BM, Cfg::BN, splits);
    const bool few = (chunk < red ? chunk : red) <= FEW_STEPS * BK;
    auto launch = [&](auto cut, auto short_red) {
        hipLaunchKernelGGL((gemm_stream_kernel<T, Cfg, OUTER ? COLS_OUTER : COLS_RED, Epi, decltype(cut)::value, decltype(short_red)::value>),
                           dim3(sh.per_xcd * 8), dim3(Cfg::NT), 0, s, A, lda, (uint32_t)a_bytes, B, ldb, (uint32_t)b_bytes, sh, epi, ConvSrc{});
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    constexpr bool two = stream_ahead<Cfg, OUTER ? COLS_OUTER : COLS_RED, false>() == 2;  // else there is one variant
    if constexpr (OUTER && !std::is_same<Epi, FwdEpilogue<T>>::value)
        if (lda % BK != 0) {  // dY of a fully connected layer (4096 x 4096 x 1000 bf16: 39 us, on the 128 x 128 plain kernel 61)
            if constexpr (two) {
                if (few) launch(yes, yes);
                else launch(yes, no);
            } else {
                launch(yes, no);
            }
            return true;
        }
    if (lda % BK != 0) return false;
    if constexpr (two) {
        if (few) launch(no, yes);
        else launch(no, no);
    } else {
        launch(no, no);
    }
    return true;
}

// Model gradient with the column operand read from X (see DirectLoader), in the mode the geometry allows.
template <typename Cfg>
static void launch_direct(const bf16_t *A, int64_t lda, const DirectSrc &d, int rows, int cols, int64_t red,
                          int64_t chunk, int splits, const PartialEpilogue &epi, hipStream_t s)
{
    GemmShape sh = make_shape(rows, cols, red, chunk, Cfg::BM, Cfg::BN, splits);
    sh.fast_store = epi.fits32() ? 1 : 0;
    dim3 grid(sh.per_xcd * 8, 1, 1);
    const int p8 = (int)d.div_p8.d;
    if (d.KK > 0)
        hipLaunchKernelGGL((gemm_kernel<bf16_t, Cfg, false, PartialEpilogue, DIRECT_PLANES>), grid, dim3(Cfg::NT), 0, s, A,
                           lda, (const bf16_t *)nullptr, (int64_t)0, sh, epi, d);
    else if (p8 == 1 || p8 == 2 || p8 == 4 || p8 == 8)
        hipLaunchKernelGGL((gemm_kernel<bf16_t, Cfg, false, PartialEpilogue, DIRECT_ROWS_FIXED>), grid, dim3(Cfg::NT), 0, s,
                           A, lda, (const bf16_t *)nullptr, (int64_t)0, sh, epi, d);
    else
        hipLaunchKernelGGL((gemm_kernel<bf16_t, Cfg, false, PartialEpilogue, DIRECT_ROWS>), grid, dim3(Cfg::NT), 0, s, A, lda,
                           (const bf16_t *)nullptr, (int64_t)0, sh, epi, d);
}

template <typename T, typename Cfg, bool COL_OUTER, typename Epi>
static void launch_plain(const T *A, int64_t lda, const T *B, int64_t ldb, int rows, int cols, int64_t red, int64_t chunk, int splits,
                         const Epi &epi, hipStream_t s)
{
    GemmShape sh = make_shape(rows, cols, red, chunk, Cfg::BM, Cfg::BN, splits);
    sh.fast_store = epi.fits32() ? 1 : 0;
    hipLaunchKernelGGL((gemm_kernel<T, Cfg, COL_OUTER, Epi>), dim3(sh.per_xcd * 8), dim3(Cfg::NT), 0, s, A, lda, B, ldb, sh, epi,
                       DirectSrc{});
}

template <typename T, bool COL_OUTER, typename Epi>
static void launch_any(int tile, const T *A, int64_t lda, const T *B, int64_t ldb, int rows, int cols, int64_t red,
                       int64_t chunk, int splits, const Epi &epi, hipStream_t s)
{
    bool done = false;
    switch (tile) {
    case 1: done = launch_stream<T, Tile1, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s); break;
    case 2:
        if constexpr (!COL_OUTER) {  // too few columns for the column-contiguous loader's tasks
            done = launch_stream<T, Tile2, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s);
            break;
        }
        [[fallthrough]];
    case 3: done = launch_stream<T, Tile3, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s); break;
    case 4: done = launch_stream<T, Tile4, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s); break;
    case 5: done = launch_stream<T, Tile5, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s); break;
    case 6: done = launch_stream<T, Tile6, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s); break;
    case 7: done = launch_stream<T, Tile7, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s); break;
    default: done = launch_stream<T, Tile0, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s); break;
    }
    if (done) return;
    // operands or a result of 4 GB and more: 256 x 256 (model gradients also 384 x 128) where the result fills it about as
    // well as 128 x 128 (2400 x 1548800 x 96 bf16: 6.6 ms so, 7.7 on 128 x 128)
    const int plain = COL_OUTER ? pick_large_tile(rows, cols, false) : pick_large_tile(rows, cols, true);
    if (plain == 1) {
        launch_plain<T, Tile1, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s);
        return;
    }
    if constexpr (!COL_OUTER)
        if (plain == 2) {
            launch_plain<T, Tile2, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s);
            return;
        }
    launch_plain<T, Tile0, COL_OUTER, Epi>(A, lda, B, ldb, rows, cols, red, chunk, splits, epi, s);
}

template <typename T, typename Epi>
static void launch_split(int tile, const T *A, int64_t lda, const T *B, int64_t ldb, int rows, int cols, int64_t red, int64_t chunk,
                         int splits, float *partials, const Epi &epi, hipStream_t s)
{
    PartialEpilogue pe{partials, rows, cols};
    launch_any<T, true, PartialEpilogue>(tile, A, lda, B, ldb, rows, cols, red, chunk, splits, pe, s);
    launch_reduce_store(partials, splits, rows, cols, epi, s);
}

template <typename T>
static int run_forward(const ConvGeom &g, const GemmFwdArgs &a, hipStream_t s)
{
    constexpr int BK = NPACK * Pack<T>::KP;
    // K-hat is zero-padded along K to a multiple of the pack size; rows of D-hat beyond K read as zero.
    FwdEpilogue<T> epi{(T *)a.Y, a.bias, g.F, g.M, g.HoWo, g.div_HoWo, a.relu};
    ProfScope prof(KID_GEMM_FWD, s, 2.0 * g.M * (double)g.K * g.F,
                   ((double)g.F * g.K + (double)g.K * g.M + (double)g.F * g.M) * sizeof(T));
    if (a.splits > 1)
        launch_split<T>(a.tile, (const T *)a.Khat, a.ldk, (const T *)a.Dhat, a.ldd, g.F, (int)a.ldd, g.K, a.chunk, a.splits, a.partials,
                        epi, s);
    else
        launch_any<T, true, FwdEpilogue<T>>(pick_tile(g.F, (int)a.ldd, dtype_of<T>()), (const T *)a.Khat, a.ldk, (const T *)a.Dhat, a.ldd,
                                            g.F, (int)a.ldd, g.K, round_up(g.K, BK), 1, epi, s);
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

int launch_gemm_forward(const ConvGeom &g, int dtype, const GemmFwdArgs &a, hipStream_t s)
{
    return dtype == OMNI_BF16 ? run_forward<bf16_t>(g, a, s) : run_forward<float>(g, a, s);
}

template <typename T>
static int run_dgrad(const ConvGeom &g, const GemmDgradArgs &a, hipStream_t s)
{
    constexpr int BK = NPACK * Pack<T>::KP;
    RowMajorEpilogue<T> epi{(T *)a.dDhat, a.ldd, g.K, (int)a.ldd};
    ProfScope prof(KID_GEMM_DGRAD, s, 2.0 * g.M * (double)g.K * g.F,
                   ((double)g.F * g.K + (double)g.K * g.M + (double)g.F * g.M) * sizeof(T));
    if (a.splits > 1)
        launch_split<T>(a.tile, (const T *)a.KhatT, a.ldk, (const T *)a.dYhat, a.ldd, g.K, (int)a.ldd, g.F, a.chunk, a.splits,
                        a.partials, epi, s);
    else
        launch_any<T, true, RowMajorEpilogue<T>>(pick_tile(g.K, (int)a.ldd, dtype_of<T>()), (const T *)a.KhatT, a.ldk, (const T *)a.dYhat,
                                                 a.ldd, g.K, (int)a.ldd, g.F, round_up(g.F, BK), 1, epi, s);
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

int launch_gemm_dgrad(const ConvGeom &g, int dtype, const GemmDgradArgs &a, hipStream_t s)
{
    return dtype == OMNI_BF16 ? run_dgrad<bf16_t>(g, a, s) : run_dgrad<float>(g, a, s);
}

// ------------------------------------------------------------------------------------------------
// fp32 data gradient of a stride-1 layer as one product: dX [C x N H W] = K-hat^T [C x kh kw F] * the lowered dY, whose
// entries the product reads from dY as it lies (ConvStream).  The route over dD-hat packs dY, writes a matrix kh kw times
// the size of dX and adds its entries up again (col2im); here only the reordered weights exist.  The matrix cores do the
// same work, unless few channels leave a tile's rows empty or few tiles the chip.
// 96 channels, 256 filters, 27 x 27, window 5, 256 images: 2 390 us for packing, product and col2im, 1 920 here.
// ------------------------------------------------------------------------------------------------
static int64_t dgrad_conv_lda(const ConvGeom &g) { return round_up(g.F, NPACK * 4) * g.kh * g.kw; }

static int g_dgrad_conv = 0;  // omni_tuning_set(OMNI_TUNE_DGRAD_CONV, ...): sweeps and tests only
static const int kDgradConvTiles[] = {0, 3, 4, 5, 6};  // the tiles of four wavefronts
int set_dgrad_conv_override(int v)
{
    bool known = v == 0 || v == 1;
    for (int t : kDgradConvTiles) known = known || v == 2 + t;
    if (!known) return OMNI_INVALID_ARGUMENT;
    g_dgrad_conv = v;
    return OMNI_OK;
}
static int dgrad_conv_tile(const ConvGeom &g, double *us)
{
    const int t = estimate_tile(g.C, g.N * g.H * g.W, OMNI_F32, true, us);
    return g_dgrad_conv >= 2 ? g_dgrad_conv - 2 : t;
}

// Where it runs: the estimated times of both routes, per step of 32 terms as pick_tile() has them; this one takes 1.12 times
// that (its loads and the second accumulators), the route over dD-hat also moves dY twice and dD-hat twice at about
// 4.5 TB/s and takes a launch more.  (8 x 3 x 32 x 32, 32 filters, window 5: 30 us here for a tile of 3 rows in 32, 15
// there; 64 x 64 x 56 x 56, 64 filters, window 3: 145 here, 383 there.  Over 17 layers at 1 to 256 images the route chosen
// is at most 9 % behind the other one.)  A forced tile keeps the lowered route.
bool dgrad_conv_supported(const ConvGeom &g, int dtype)
{
    if (dtype != OMNI_F32 || g.sh != 1 || g.sw != 1 || g.kh * g.kw > 31 || g.kh - 1 < g.ph || g.kw - 1 < g.pw) return false;
    const int64_t cols = (int64_t)g.N * g.H * g.W, lda = dgrad_conv_lda(g);
    if (cols > 0x7fffffffll - 4096 || (double)g.C * lda >= 1.0e9 || (double)cols * g.C * 4.0 >= 4.0e9 || (double)g.M * g.F * 4.0 >= 4.0e9)
        return false;
    if (g_dgrad_conv != 0) return g_dgrad_conv >= 2;
    if (tile_override() >= 0) return false;
    double here, there;
    dgrad_conv_tile(g, &here);
    estimate_tile(g.K, (int)dhat_ld(g), dtype, false, &there);
    const double moved = 8.0 * ((double)g.F + g.K) * g.M;  // bytes
    return 1.12 * here * (double)(lda / 32) < there * (double)round_up(g.F, 32) / 32.0 + moved / 4.5e6 + 3.0;
}

template <typename Cfg>
static void launch_conv_product(const float *A, int64_t lda, const float *dY, uint32_t dy_bytes, int rows, int cols, const ConvSrc &cs,
                                const FwdEpilogue<float> &epi, hipStream_t s)
{
    GemmShape sh = make_shape(rows, cols, lda, lda, Cfg::BM, Cfg::BN, 1);
    hipLaunchKernelGGL((gemm_stream_kernel<float, Cfg, COLS_CONV, FwdEpilogue<float>>), dim3(sh.per_xcd * 8), dim3(Cfg::NT), 0, s, A,
                       lda, (uint32_t)((double)rows * lda * 4.0), dY, (int64_t)0, dy_bytes, sh, epi, cs);
}

// Wf: scratch for K-hat^T with F rounded up to 32 (the lowered route's, rounded up to 64, takes at least as much)
int launch_dgrad_conv(const ConvGeom &g, const void *dY, const void *W, void *dX, void *Wf, hipStream_t s)
{
    const int64_t lda = dgrad_conv_lda(g);
    const int cols = g.N * g.H * g.W, Fp = (int)round_up(g.F, NPACK * 4);
    int st = launch_pack_khat_t(g, OMNI_F32, W, Wf, g.K, Fp, s);
    if (st != OMNI_OK) return st;
    ConvSrc cs{g.Ho, g.Wo, g.kh, g.kw, g.ph, g.pw, (uint32_t)g.HoWo, (uint32_t)g.F * (uint32_t)g.HoWo, g.F, Fp / (NPACK * 4), cols,
               g.div_HW, g.div_W};
    FwdEpilogue<float> epi{(float *)dX, nullptr, g.C, cols, g.H * g.W, g.div_HW, 0};
    ProfScope prof(KID_GEMM_DGRAD, s, 2.0 * g.M * (double)g.K * g.F, 4.0 * ((double)g.F * g.K + (double)g.F * g.M + (double)g.C * cols));
    const float *A = (const float *)Wf, *B = (const float *)dY;
    const uint32_t bytes = (uint32_t)((double)g.M * g.F * 4.0);
    double us;
    switch (dgrad_conv_tile(g, &us)) {
    case 3: launch_conv_product<Tile3>(A, lda, B, bytes, g.C, cols, cs, epi, s); break;
    case 4: launch_conv_product<Tile4>(A, lda, B, bytes, g.C, cols, cs, epi, s); break;
    case 5: launch_conv_product<Tile5>(A, lda, B, bytes, g.C, cols, cs, epi, s); break;
    case 6: launch_conv_product<Tile6>(A, lda, B, bytes, g.C, cols, cs, epi, s); break;
    default: launch_conv_product<Tile0>(A, lda, B, bytes, g.C, cols, cs, epi, s); break;
    }
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

// Data gradient of a layer whose window is the whole, unpadded image (a fully connected layer, Sec. II-C):
// dX [N][K] = dY [N][F] * W [F][K] with all three tensors in their natural layouts -- dY's rows run along the
// reduction, W's rows along the result's columns -- so nothing is packed, transposed or scattered back.
bool dgrad_dense_supported(const ConvGeom &g)
{
    return g.Ho == 1 && g.Wo == 1 && g.ph == 0 && g.pw == 0 && g.kh == g.H && g.kw == g.W && g.F % 8 == 0 && g.K % 8 == 0;
}

template <typename T>
static int run_dgrad_dense(const ConvGeom &g, const void *dY, const void *W, void *dX, float *partials, int splits,
                           int64_t chunk, int tile, hipStream_t s)
{
    constexpr int BK = NPACK * Pack<T>::KP;
    RowMajorEpilogue<T> epi{(T *)dX, (int64_t)g.K, g.N, g.K};
    ProfScope prof(KID_GEMM_DGRAD, s, 2.0 * g.N * (double)g.K * g.F,
                   ((double)g.F * g.K + (double)g.K * g.N + (double)g.F * g.N) * sizeof(T));
    if (splits > 1)
        launch_split<T>(tile, (const T *)dY, (int64_t)g.F, (const T *)W, (int64_t)g.K, g.N, g.K, g.F, chunk, splits, partials, epi, s);
    else
        launch_any<T, true, RowMajorEpilogue<T>>(pick_tile(g.N, g.K, dtype_of<T>()), (const T *)dY, (int64_t)g.F, (const T *)W, (int64_t)g.K,
                                                 g.N, g.K, g.F, round_up(g.F, BK), 1, epi, s);
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

int launch_gemm_dgrad_dense(const ConvGeom &g, int dtype, const void *dY, const void *W, void *dX, float *partials,
                            int splits, int64_t chunk, int tile, hipStream_t s)
{
    return dtype == OMNI_BF16 ? run_dgrad_dense<bf16_t>(g, dY, W, dX, partials, splits, chunk, tile, s)
                              : run_dgrad_dense<float>(g, dY, W, dX, partials, splits, chunk, tile, s);
}

template <typename T>
static int run_wgrad(const ConvGeom &g, const GemmWgradArgs &a, hipStream_t s)
{
    float *target = a.splits == 1 ? a.dW : a.partials;
    PartialEpilogue epi{target, g.F, g.K};
    {
        ProfScope prof(KID_GEMM_WGRAD, s, 2.0 * g.M * (double)g.K * g.F,
                       ((double)g.K * g.M + (double)g.F * g.M) * sizeof(T) + 4.0 * g.F * g.K * a.splits);
        if (a.X_direct != nullptr) {
            if constexpr (std::is_same<T, bf16_t>::value) {
                const bool planes = wgrad_direct_planes(g);
                const int unit = planes ? g.Ho * g.Wo : g.Wo;  // what is padded to a multiple of 8 positions
                DirectSrc d{(const bf16_t *)a.X_direct, g.C, g.H, g.W, g.H * g.W, g.K, g.ph, g.pw,
                            planes ? g.N : g.N * g.Ho, (int32_t)((int64_t)g.N * g.C * g.H * g.W),
                            FastDiv((uint32_t)((unit + 7) / 8)), FastDiv((uint32_t)g.Ho), g.div_khkw, g.div_kw,
                            g.Ho * g.Wo, planes ? g.kh * g.kw : 0, FastDiv((uint32_t)g.W), 1, g.F, g.Wo};
                if (pick_direct_tile(g.F, g.K) == 2)
                    launch_direct<Tile2>((const bf16_t *)a.dYhat, a.ldd, d, g.F, g.K, a.ldd, a.chunk, a.splits, epi, s);
                else
                    launch_direct<Tile1>((const bf16_t *)a.dYhat, a.ldd, d, g.F, g.K, a.ldd, a.chunk, a.splits, epi, s);
            }
        } else {
            launch_any<T, false, PartialEpilogue>(a.tile, (const T *)a.dYhat, a.ldd, (const T *)a.Dhat,
                                                  a.ldd, g.F, g.K, a.ldd, a.chunk, a.splits, epi, s);
        }
    }
    OMNI_LAUNCH_CHECK();
    if (a.splits > 1) return launch_wgrad_reduce(g, a.partials, a.splits, a.dW, a.bias_partials, a.bias_blocks, a.dbias, s);
    return OMNI_OK;
}

int launch_wgrad_reduce(const ConvGeom &g, const float *partials, int splits, float *dW, const float *bias_partials,
                        int bias_blocks, float *dbias, hipStream_t s)
{
    int64_t count = (int64_t)g.F * g.K;
    const unsigned bias_wgs = dbias != nullptr ? (unsigned)((g.F + 3) / 4) : 0u;
    ProfScope prof(KID_REDUCE_PARTIALS, s, 0.0, 4.0 * count * (splits + 1));
    if (count % 4 == 0) {
        const unsigned vec_blocks = (unsigned)((count / 4 + 255) / 256);
        // sixteen lanes per element where one lane each would leave most of the chip idle on a long chain of loads
        if (splits >= 32 && vec_blocks < 128) {
            const unsigned blocks = (unsigned)((count / 4 + 15) / 16);
            hipLaunchKernelGGL(reduce_partials_deep_kernel, dim3(blocks + bias_wgs), dim3(256), 0, s, (const float4 *)partials, splits,
                               count / 4, (float4 *)dW, blocks, bias_partials, bias_blocks, g.F, dbias);
            OMNI_LAUNCH_CHECK();
            return OMNI_OK;
        }
        hipLaunchKernelGGL(reduce_partials_vec_kernel, dim3(vec_blocks + bias_wgs), dim3(256), 0, s, (const float4 *)partials, splits,
                           count / 4, (float4 *)dW, vec_blocks, bias_partials, bias_blocks, g.F, dbias);
        OMNI_LAUNCH_CHECK();
        return OMNI_OK;
    }
    const unsigned main_blocks = (unsigned)((count + 63) / 64);
    hipLaunchKernelGGL(reduce_partials_kernel<false>, dim3(main_blocks + bias_wgs), dim3(256), 0, s, partials, splits, count, dW,
                       main_blocks, bias_partials, bias_blocks, g.F, dbias, PhaseMap{});
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

// ------------------------------------------------------------------------------------------------
// Model gradient of a layer with horizontal stride 4 and no padding (CaffeNet's conv1) without D-hat.
// The input is first split by x mod 4 into four phase images, X4 [N][C * 4][H][WP] with
// X4(n, 4c + ph, y, xq) = X(n, c, y, 4 xq + ph) (zero where that column does not exist).  Window column
// kx = 4 kq + ph of output column ox then meets phase image ph at xq = ox + kq: the layer is a convolution
// of X4 with horizontal stride 1, 4C channels and a window of kh x ceil(kw / 4), which the row mode of
// DirectLoader reads as it stands (8 consecutive output columns = 8 consecutive xq).  The result is
// [F][K'] in that order, K' = 4C * kh * ceil(kw / 4), window columns beyond kw being padding; the ordered
// reduction of the split partial results puts it back into [F][C][kh][kw].
// One 96 x 512 result tile (8 wavefronts, 96 x 64 each) holds the whole gradient, so the launch is one
// workgroup per split of the reduction.  Few images give few splits, and then a workgroup's own chain (first loads,
// its steps, 96 rows of partial results through the LDS strips) is the whole time: 32 rows per workgroup cut the
// MFMAs and the results of that chain to a third.
// ------------------------------------------------------------------------------------------------
typedef Tile<96, 512, 1, 8, 1> TilePhase;
typedef Tile<32, 512, 1, 8, 1> TilePhaseFew;  // few splits, or up to 32 filters

static int phase_kwq(const ConvGeom &g) { return (g.kw + 3) / 4; }
int wgrad_phase_kp(const ConvGeom &g) { return 4 * g.C * g.kh * phase_kwq(g); }
int wgrad_phase_wp(const ConvGeom &g) { return (int)round_up((g.W + 3) / 4, 8); }

bool wgrad_phase_supported(const ConvGeom &g, int dtype)
{
    if (dtype != OMNI_BF16 || g.sw != 4 || g.ph != 0 || g.pw != 0 || g.F > TilePhase::BM || g.Wo < 8) return false;
    if (wgrad_phase_kp(g) + 1 > TilePhase::BN) return false;  // + 1: the column of the bias gradient
    int64_t total4 = (int64_t)g.N * g.C * 4 * g.H * wgrad_phase_wp(g);
    return total4 < 0x7fffffffll - 16 && total4 >= 8 && (int64_t)g.N * g.C * g.H * g.W < 0x7fffffffll - 64 &&
           (int64_t)g.N * g.F * g.HoWo < 0x7fffffffll - 16;
}

// partials: [splits][F][K' + 1] floats; `ld` = the padded reduction extent (dyhat_rows_ld)
int launch_gemm_wgrad_phase(const ConvGeom &g, const void *X4, const void *dY, int64_t ld, float *partials, int splits,
                            int64_t chunk, float *dW, float *dbias, hipStream_t s)
{
    const int kwq = phase_kwq(g), Kp = wgrad_phase_kp(g), WP = wgrad_phase_wp(g);
    PartialEpilogue epi{partials, g.F, Kp + 1};
    {
        ProfScope prof(KID_GEMM_WGRAD, s, 2.0 * g.M * (double)g.K * g.F,
                       ((double)g.N * g.C * 4 * g.H * WP + (double)g.F * g.M) * 2.0 + 4.0 * g.F * (Kp + 1) * splits);
        DirectSrc d{(const bf16_t *)X4, 4 * g.C, g.H, WP, g.H * WP, Kp, 0, 0, g.N * g.Ho,
                    (int32_t)((int64_t)g.N * g.C * 4 * g.H * WP), FastDiv((uint32_t)((g.Wo + 7) / 8)), FastDiv((uint32_t)g.Ho),
                    FastDiv((uint32_t)(g.kh * kwq)), FastDiv((uint32_t)kwq), g.Ho * g.Wo, 0, FastDiv((uint32_t)WP), g.sh,
                    g.F, g.Wo};
        // three groups per window row and every pack's ten elements inside its row of X4: one load per three rows
        const bool triples = kwq == 3 && 8 * ((g.Wo + 7) / 8) + 2 <= WP;
        auto launch = [&](auto tile) {
            typedef decltype(tile) Cfg;
            GemmShape sh = make_shape(g.F, Kp + 1, ld, chunk, Cfg::BM, Cfg::BN, splits);
            sh.fast_store = epi.fits32() ? 1 : 0;
            if (triples)
                hipLaunchKernelGGL((gemm_kernel<bf16_t, Cfg, false, PartialEpilogue, DIRECT_PHASE3>), dim3(sh.per_xcd * 8),
                                   dim3(Cfg::NT), 0, s, (const bf16_t *)dY, (int64_t)0, (const bf16_t *)nullptr, (int64_t)0, sh, epi, d);
            else
                hipLaunchKernelGGL((gemm_kernel<bf16_t, Cfg, false, PartialEpilogue, DIRECT_ROWS_ONES>), dim3(sh.per_xcd * 8),
                                   dim3(Cfg::NT), 0, s, (const bf16_t *)dY, (int64_t)0, (const bf16_t *)nullptr, (int64_t)0, sh, epi, d);
        };
        // 32 rows where all those workgroups run at once (one per compute unit; beyond it they would load the column
        // panel three times in turn).  With the reduction's launch, 3 x 227 x 227 -> 96, 11 x 11: 1 image 22.3 -> 16.8 us,
        // 4 images 25.0 -> 19.7; 3 x 224 x 224 -> 32, 4 x 4, 64 images: 53.0 -> 46.3.  The same sums either way.
        if (splits * ((g.F + 31) / 32) <= 256)
            launch(TilePhaseFew{});
        else
            launch(TilePhase{});
    }
    OMNI_LAUNCH_CHECK();
    const int64_t count = (int64_t)g.F * (Kp + 1);
    ProfScope prof(KID_REDUCE_PARTIALS, s, 0.0, 4.0 * count * (splits + 1));
    const unsigned main_blocks = (unsigned)((count + 63) / 64);
    PhaseMap pm{g.C, g.kh, g.kw, FastDiv((uint32_t)(Kp + 1)), FastDiv((uint32_t)(g.kh * kwq)), FastDiv((uint32_t)kwq)};
    hipLaunchKernelGGL(reduce_partials_kernel<true>, dim3(main_blocks), dim3(256), 0, s, partials, splits, count, dW,
                       main_blocks, (const float *)nullptr, 0, g.F, dbias, pm);
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

int launch_gemm_wgrad(const ConvGeom &g, int dtype, const GemmWgradArgs &a, hipStream_t s)
{
    return dtype == OMNI_BF16 ? run_wgrad<bf16_t>(g, a, s) : run_wgrad<float>(g, a, s);
}

}  // namespace omni
