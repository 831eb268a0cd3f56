// Data-movement kernels of the lowered convolution (gfx950): batched lowering X -> D-hat, its
// transpose col2im dD-hat -> dX, the reshaping of the model into K-hat / K-hat^T, and the packing
// of an output-shaped gradient into the matrix dY-hat (with the bias gradient as a by-product).
//
// All of them are bound by HBM traffic, so the rules are: every thread writes 16 bytes, lanes of a
// wavefront touch consecutive addresses, indices are decoded once per thread with multiply-high
// divisions, and nothing is reduced with floating point atomics.
#include <cmath>
#include <type_traits>

#include "common.h"

namespace omni {

// ------------------------------------------------------------------------------------------------
// Batched lowering (App. C, lowering phase; Sec. III-B: all N images before any GEMM)
//   D-hat[(c,ky,kx)][(n,oy,ox)] = X[n,c,oy*sh-ph+ky,ox*sw-pw+kx]   or 0 in the padding
// U is an unsigned integer of the element's width: lowering copies bit patterns.
// Each thread produces VEC consecutive columns of one row; columns in [M, ld) are written as zero.
// ------------------------------------------------------------------------------------------------
template <typename U, int VEC> struct alignas(sizeof(U) * VEC) VecOf { U v[VEC]; };

template <typename U, int VEC>
__global__ __launch_bounds__(256) void lower_kernel(ConvGeom g, const U *__restrict__ X, U *__restrict__ D,
                                                    int64_t ld, int64_t vecs_per_row)
{
    int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= vecs_per_row) return;
    uint32_t m0 = (uint32_t)(v * VEC);
    uint32_t n, rem, oy, ox;
    g.div_HoWo.divmod(m0 < (uint32_t)g.M ? m0 : 0u, n, rem);
    g.div_Wo.divmod(rem, oy, ox);

    for (int k = blockIdx.y; k < g.K; k += gridDim.y) {
        uint32_t c, r2, ky, kx;
        g.div_khkw.divmod((uint32_t)k, c, r2);
        g.div_kw.divmod(r2, ky, kx);
        VecOf<U, VEC> out;
        uint32_t nn = n, yy = oy, xx = ox;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            U val = 0;
            if (m0 + e < (uint32_t)g.M) {
                int iy = (int)yy * g.sh - g.ph + (int)ky;
                int ix = (int)xx * g.sw - g.pw + (int)kx;
                if (iy >= 0 && iy < g.H && ix >= 0 && ix < g.W)
                    val = X[(((int64_t)nn * g.C + c) * g.H + iy) * g.W + ix];
            }
            out.v[e] = val;
            if (++xx == (uint32_t)g.Wo) {
                xx = 0;
                if (++yy == (uint32_t)g.Ho) {
                    yy = 0;
                    ++nn;
                }
            }
        }
        *reinterpret_cast<VecOf<U, VEC> *>(D + (int64_t)k * ld + m0) = out;
    }
}

// ------------------------------------------------------------------------------------------------
// K-hat: the model as a matrix (App. C: "the kernel does not require any replication").
// W [F][K] -> K-hat [Fp][Kp] zero padded;  K-hat^T [Kp][Fp] zero padded.  Eight consecutive results per thread.  The job
// is small, and every pass needs another kernel that does not depend on it, so it rides on that one's launch as extra
// workgroups (a launch of its own takes 2 to 5 us whatever its size).
// ------------------------------------------------------------------------------------------------
template <typename U> struct KhatJob {
    const U *W;
    U *out;
    int F, K;
    int64_t rows, cols;  // of the result; cols is a multiple of 8
    int transpose;
    __host__ __device__ int64_t blocks() const { return (rows * (cols / 8) + 255) / 256; }
    double bytes() const { return out != nullptr ? 2.0 * F * (double)K * sizeof(U) : 0.0; }
};
template <typename U> __device__ __forceinline__ void khat_body(const KhatJob<U> &j, int64_t block)
{
    const int64_t t = block * 256 + threadIdx.x, c8 = j.cols / 8;
    if (t >= j.rows * c8) return;
    // transposed: neighbouring threads take neighbouring rows k, so that their loads W[f * K + k] are consecutive
    const int64_t r = j.transpose ? t % j.rows : t / c8, c = (j.transpose ? t / j.rows : t - r * c8) * 8;
    VecOf<U, 16 / sizeof(U)> o[8 * sizeof(U) / 16];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int64_t f = j.transpose ? c + e : r, k = j.transpose ? r : c + e;
        o[e * sizeof(U) / 16].v[e % (16 / sizeof(U))] = (f < j.F && k < j.K) ? j.W[f * j.K + k] : (U)0;
    }
#pragma unroll
    for (int q = 0; q < (int)(8 * sizeof(U) / 16); ++q)
        *reinterpret_cast<VecOf<U, 16 / sizeof(U)> *>(j.out + r * j.cols + c + q * (16 / sizeof(U))) = o[q];
}
template <typename U> __global__ __launch_bounds__(256) void pack_khat_kernel(KhatJob<U> j) { khat_body(j, blockIdx.x); }

// LDS-staged variant.  A workgroup takes one input channel c of a group of images (small planes) or
// of a band of output rows of one image (large planes), copies the zero-padded patch it needs into
// LDS once with coalesced reads, and then writes all kh*kw rows of D-hat that stem from that patch:
// for each row the columns of the group are one contiguous range, written 16 bytes per lane.  Columns
// at the ragged ends of the range (ranges need not start on a 16-byte boundary) are stored one by one.
// X is read from HBM once; every store instruction of a wavefront covers 1 KiB of consecutive bytes.
struct LowerPlan {
    int nb;        // images per workgroup (1 in banded mode)
    int br;        // output rows per band (Ho when nb > 1)
    int bands;     // bands per image
    int groups;    // image groups
    int rows_in;   // input rows held per image: (br-1)*sh + kh
    int wp;        // padded row pitch: W + 2*pw
    int ky_per;    // window rows per workgroup (blockIdx.z takes the next ones)
    FastDiv div_wp, div_rows_in;
};

template <typename U, int VEC, int KW>  // KW > 0: window width known at compile time (inner loop unrolled)
__device__ __forceinline__ void lower_body(const ConvGeom &g, const LowerPlan &p, const U *__restrict__ X, U *__restrict__ D,
                                           int64_t ld, int bx, int c, int bz)
{
    extern __shared__ __align__(16) unsigned char lower_smem[];
    U *tile = reinterpret_cast<U *>(lower_smem);
    const int tid = threadIdx.x;
    const int band = bx % p.bands, grp = bx / p.bands;
    const int n0 = grp * p.nb;
    const int nb = g.N - n0 < p.nb ? g.N - n0 : p.nb;
    const int oy0 = band * p.br;
    const int br = g.Ho - oy0 < p.br ? g.Ho - oy0 : p.br;
    const int rows_used = (br - 1) * g.sh + g.kh;
    const int kw = KW > 0 ? KW : g.kw;
    const int ky0 = bz * p.ky_per, ky1 = ky0 + p.ky_per < g.kh ? ky0 + p.ky_per : g.kh;
    constexpr int VECL = 16 / sizeof(U);  // elements per 16-byte global load

    // patch -> LDS.  The padding is zeroed first; then the pixels, which for one image are one
    // contiguous run of whole input rows, are fetched 16 bytes per lane (the run need not be 16-byte
    // aligned) and dropped into the padded layout one element at a time.
    {
        const int patch16 = (nb * p.rows_in * p.wp * (int)sizeof(U) + 15) / 16;
        uint4 *t16 = reinterpret_cast<uint4 *>(lower_smem);
        for (int i = tid; i < patch16; i += 256) t16[i] = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    {
        int iy_lo = oy0 * g.sh - g.ph, iy_hi = iy_lo + rows_used;  // input rows the patch covers
        const int ry0 = iy_lo < 0 ? -iy_lo : 0;                     // first patch row that lies in the image
        if (iy_lo < 0) iy_lo = 0;
        if (iy_hi > g.H) iy_hi = g.H;
        const int run = (iy_hi - iy_lo) * g.W;                      // elements per image
        const int chunks = (run + VECL - 1) / VECL;
        for (int t = tid; t < nb * chunks; t += 256) {
            int inb = t / chunks, ch = t - inb * chunks;
            const U *src = X + (((int64_t)(n0 + inb) * g.C + c) * g.H + iy_lo) * g.W + ch * VECL;
            U vals[VECL];
            if ((ch + 1) * VECL <= run) {
                __builtin_memcpy(vals, src, sizeof(vals));
            } else {
#pragma unroll
                for (int e = 0; e < VECL; ++e) vals[e] = ch * VECL + e < run ? src[e] : (U)0;
            }
            uint32_t ry, ix;
            g.div_W.divmod((uint32_t)(ch * VECL), ry, ix);
            U *drow = tile + (inb * p.rows_in + ry0 + (int)ry) * p.wp + g.pw;
#pragma unroll
            for (int e = 0; e < VECL; ++e) {
                if (ch * VECL + e < run) drow[ix] = vals[e];
                if (++ix == (uint32_t)g.W) {
                    ix = 0;
                    drow += p.wp;
                }
            }
        }
    }
    __syncthreads();

    // the contiguous column range of this workgroup
    const int seg = p.nb > 1 ? g.HoWo : br * g.Wo;  // columns per image
    const int64_t m_lo = (int64_t)n0 * g.HoWo + (int64_t)oy0 * g.Wo;
    const int64_t m_hi = m_lo + (int64_t)(p.nb > 1 ? nb : 1) * seg;
    const int64_t v_lo = (m_lo + VEC - 1) / VEC, v_hi = m_hi / VEC;  // slots that lie entirely inside the range
    const int khkw = g.kh * kw;
    auto locate = [&](int64_t m) -> int {  // LDS index of the window origin of column m
        uint32_t t = (uint32_t)(m - m_lo), inb = 0, rem = t, oy, ox;
        if (p.nb > 1) g.div_HoWo.divmod(t, inb, rem);
        g.div_Wo.divmod(rem, oy, ox);
        return ((int)inb * p.rows_in + (int)oy * g.sh) * p.wp + (int)ox * g.sw;
    };

    for (int64_t v = v_lo + tid; v < v_hi; v += 256) {
        int a[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) a[e] = locate(v * VEC + e);
        U *dst = D + ((int64_t)c * khkw + ky0 * kw) * ld + v * VEC;
        for (int ky = ky0; ky < ky1; ++ky) {
            const U *src[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) src[e] = tile + a[e] + ky * p.wp;
            if constexpr (KW > 0) {
#pragma unroll
                for (int kx = 0; kx < KW; ++kx) {
                    VecOf<U, VEC> out;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) out.v[e] = src[e][kx];
                    *reinterpret_cast<VecOf<U, VEC> *>(dst) = out;
                    dst += ld;
                }
            } else {
                for (int kx = 0; kx < kw; ++kx) {
                    VecOf<U, VEC> out;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) out.v[e] = src[e][kx];
                    *reinterpret_cast<VecOf<U, VEC> *>(dst) = out;
                    dst += ld;
                }
            }
        }
    }
    // ragged ends: the columns before the first and after the last whole slot, one (row, column) per thread
    const int head = (int)(v_lo * VEC - m_lo < m_hi - m_lo ? v_lo * VEC - m_lo : m_hi - m_lo);
    const int tail = v_hi >= v_lo ? (int)(m_hi - v_hi * VEC) : 0;
    const int edge = head + tail, r0 = ky0 * kw, nr = (ky1 - ky0) * kw;
    for (int idx = tid; idx < edge * nr; idx += 256) {
        int r = idx / edge, j = idx - r * edge;
        r += r0;
        int64_t m = j < head ? m_lo + j : v_hi * VEC + (j - head);
        int ky = r / kw, kx = r - ky * kw;
        D[((int64_t)c * khkw + r) * ld + m] = tile[locate(m) + ky * p.wp + kx];
    }
    // columns in [M, ld) of this channel's rows are zero; the workgroup that owns the last column writes them
    if (m_hi == g.M && ld > g.M) {
        const int padc = (int)(ld - g.M);
        for (int idx = tid; idx < nr * padc; idx += 256) {
            int r = idx / padc, cc = idx - r * padc;
            D[((int64_t)c * khkw + r0 + r) * ld + g.M + cc] = 0;
        }
    }
}

// `khat` (optional, out != null): workgroups beyond the channels (blockIdx.y >= C) pack the model
template <typename U, int VEC, int KW>
__global__ __launch_bounds__(256) void lower_lds_kernel(ConvGeom g, LowerPlan p, const U *__restrict__ X, U *__restrict__ D,
                                                        int64_t ld, KhatJob<U> khat)
{
    if ((int)blockIdx.y < g.C)
        lower_body<U, VEC, KW>(g, p, X, D, ld, blockIdx.x, blockIdx.y, blockIdx.z);
    else
        khat_body(khat, ((int64_t)(blockIdx.y - g.C) * gridDim.z + blockIdx.z) * gridDim.x + blockIdx.x);
}

// Stride 1 and an output as wide as the input: column (n, q) of row (c, ky, kx) of D-hat is element q + (ky - ph) W + (kx - pw)
// of plane (n, c) of X, also across a row's end, or a zero of the padding.  So the KW rows of a window row are, 16 bytes of
// columns at a time, KW shifts of one run of 16 bytes and KW - 1 elements of X: a thread reads that run straight from memory
// (the taps of a window read it again and again, from the caches), shifts it in registers, blanks the padding and stores.  No
// LDS, no barrier, no element-wise staging, so that the stores alone bound it.  A D-hat that the 256 MB of last-level cache
// hold is stored into it, for the product that reads it next; a larger one past the caches, which it would only sweep.  (70
// random layers of both types, against D-hat staged in LDS: 205 to 230 MB, forward, lowering and col2im in turn, model gradient 0.95,
// 0.82 and 1.00 into the caches, 0.98, 0.90 and 1.01 past; 260 to 300 MB 0.85, 0.78, 0.98 and 0.81, 0.74, 0.95; 300 to 420 MB 0.89, 0.90, 0.98
// and 0.81, 0.74, 0.92; the sides cross between 230 and 260.)  A piece that runs from one image into the next
// takes its later columns from a second run.  bf16 runs start at the multiple of 4 bytes at or before their first element:
// 16-byte loads at 2-byte boundaries take three times as long.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <typename U, int KW> struct FlatRun {  // KW - 1 + V elements from element `at` of X on
    static constexpr int V = 16 / (int)sizeof(U), ODD = sizeof(U) == 2 ? 1 : 0;
    static constexpr int WORDS = ((V + KW - 1) * (int)sizeof(U) + 3) / 4;  // 32-bit words once shifted
    static constexpr int REACH = (WORDS + ODD) * 4 / (int)sizeof(U);       // elements from the first loaded one on
    uint32_t w[WORDS];
    // X has `total` elements; what lies outside it reads as zero
    __device__ __forceinline__ void load(const U *__restrict__ X, int64_t at, int64_t total)
    {
        const int64_t first = ODD ? at & ~(int64_t)1 : at;
        uint32_t r[WORDS + ODD];
        if (first >= 0 && first + REACH <= total) {
            __builtin_memcpy(r, __builtin_assume_aligned(X + first, 4), sizeof r);
        } else {
            U v[REACH];
#pragma unroll
            for (int i = 0; i < REACH; ++i) v[i] = first + i >= 0 && first + i < total ? X[first + i] : (U)0;
            __builtin_memcpy(r, v, sizeof r);
        }
        const uint32_t shift = ODD ? (uint32_t)(at & 1) * 16u : 0u;
#pragma unroll
        for (int i = 0; i < WORDS; ++i) w[i] = ODD ? __builtin_amdgcn_alignbit(r[i + ODD], r[i], shift) : r[i];
    }
    template <int KX> __device__ __forceinline__ uint32_t word(int i) const  // of the V elements from element KX on
    {
        if constexpr (sizeof(U) == 4) return w[KX + i];
        else if constexpr (KX % 2 == 0) return w[KX / 2 + i];
        else return __builtin_amdgcn_alignbit(w[KX / 2 + i + 1], w[KX / 2 + i], 16);
    }
};

template <int I, int N, typename F> __device__ __forceinline__ void flat_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        flat_for<I + 1, N>(f);
    }
}

// Which of V consecutive pixels of a plane W wide, the first in column x, have what; as bits, and as masks over their 16 bytes.
// W is at least V + 2, so that at most one row ends among them.
template <typename U> struct FlatCols {
    static constexpr int V = 16 / (int)sizeof(U), ALL = (1 << V) - 1;
    uint32_t wrap, at;  // pixels before the next row's first, pixels since the own row's first; neither above 24
    __device__ __forceinline__ FlatCols(int x, int W) : wrap(W - x < 24 ? W - x : 24), at(x < 24 ? x : 24) {}
    __device__ __forceinline__ uint32_t own_row() const { return ((1u << wrap) - 1u) & ALL; }
    // the ones with a column d to the left (d < 0: -d to the right) in the row
    template <int D> __device__ __forceinline__ uint32_t inside() const
    {
        constexpr uint32_t N = (1u << (D < 0 ? -D : D)) - 1u;
        if constexpr (D >= 0) return ~((N >> at) | (N << wrap)) & ALL;
        else return ~((N << wrap) >> -D) & ALL;
    }
    static __device__ __forceinline__ void mask(uint32_t bits, uint32_t (&m)[4])
    {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if constexpr (sizeof(U) == 4) m[w] = (uint32_t)__builtin_amdgcn_sbfe((int)bits, (unsigned)w, 1u);
            else m[w] = __builtin_amdgcn_perm((uint32_t)__builtin_amdgcn_sbfe((int)bits, 2u * w + 1u, 1u),
                                              (uint32_t)__builtin_amdgcn_sbfe((int)bits, 2u * w, 1u), 0x05040100u);
        }
    }
};

template <typename U, int KW, bool PAST>
__device__ __forceinline__ void lower_flat_body(const ConvGeom &g, int ky_per, const U *__restrict__ X, U *__restrict__ D,
                                                int64_t ld, int64_t m0, int c, int bz)
{
    typedef FlatRun<U, KW> Run;
    constexpr int V = Run::V;
    const int ky0 = bz * ky_per, ky1 = ky0 + ky_per < g.kh ? ky0 + ky_per : g.kh, hw = g.H * g.W;
    uint32_t n, q, oy, ox;
    g.div_HoWo.divmod((uint32_t)m0, n, q);
    g.div_Wo.divmod(q, oy, ox);
    U *out = D + ((int64_t)c * g.kh + ky0) * KW * ld + m0;
    const int own = g.HoWo - (int)q < V ? g.HoWo - (int)q : V;  // columns of image n; the others are image n + 1's
    const bool second = own < V && m0 + own < g.M;
    const int64_t at_a = ((int64_t)n * g.C + c) * hw + (int)q - g.ph * g.W - g.pw, at_b = ((int64_t)(n + 1) * g.C + c) * hw - own - g.ph * g.W - g.pw;
    const int64_t total = (int64_t)g.N * g.C * hw;
    // the columns whose window column lies in the image, the columns of image n
    const FlatCols<U> cols((int)ox, g.W);
    const uint32_t live = g.M - m0 >= V ? (uint32_t)FlatCols<U>::ALL : g.M > m0 ? (1u << (g.M - m0)) - 1u : 0u, row = cols.own_row();
    const int y0 = (int)oy - g.ph, y1 = ((int)oy + 1 == g.Ho ? 0 : (int)oy + 1) - g.ph;  // input row of window row 0, own and next row
    uint32_t mx[KW][4], sel[4];
    flat_for<0, KW>([&](auto tap) {
        constexpr int KX = decltype(tap)::value;
        FlatCols<U>::mask(cols.template inside<KW / 2 - KX>() & live, mx[KX]);
    });
    FlatCols<U>::mask((1u << own) - 1u, sel);
    for (int ky = ky0; ky < ky1; ++ky) {
        Run a, b;
        a.load(X, at_a + (int64_t)ky * g.W, total);
        if (second) b.load(X, at_b + (int64_t)ky * g.W, total);
        uint32_t my[4];
        FlatCols<U>::mask(((unsigned)(y0 + ky) < (unsigned)g.H ? row : 0u) | ((unsigned)(y1 + ky) < (unsigned)g.H ? ~row : 0u), my);
        flat_for<0, KW>([&](auto tap) {
            constexpr int KX = decltype(tap)::value;
            uint32_t t[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) t[w] = a.template word<KX>(w);
            if (second)
#pragma unroll
                for (int w = 0; w < 4; ++w) t[w] = (t[w] & sel[w]) | (b.template word<KX>(w) & ~sel[w]);
            const u32x4 v = {t[0] & mx[KX][0] & my[0], t[1] & mx[KX][1] & my[1], t[2] & mx[KX][2] & my[2], t[3] & mx[KX][3] & my[3]};
            if constexpr (PAST) __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(out));
            else *reinterpret_cast<u32x4 *>(out) = v;
            out += ld;
        });
    }
}

// Which thread takes which 16 bytes of columns, which channel and which window rows: in order of columns, window rows,
// channels, the columns either all of them or, where the caches hold the matrix, an eighth per XCD, the eighth that the XCD
// will read: the products give every XCD a contiguous range of column tiles, col2im_flat_kernel one of images.  Rows dealt to
// the XCDs in turn meet, as they are stored, lines that other XCDs' caches still hold from the last reader, and are fetched
// by the next from another XCD's.  (24 x 32 x 13 x 13, window 5, fp32, 64 filters: forward 30.1 us with rows in turn, 26.1 with
// eighths, 30.8 staged in LDS, model gradient 25.8, 21.2 and 22.4; 8 x 31 x 45 x 44, window 3, fp32, 20 filters: forward 21.1, 16.3 and
// 18.2; 100 x 32 x 16 x 16, window 5, bf16, 32 filters: 26.8, 20.2 and 32.6.)  Eighths are whole cache lines, and of at least
// a wavefront: a matrix of fewer than 512 such columns is not cut.
// What else is packed in the same launch comes first: few workgroups, each with a serial chain, which behind the lowering's
// would start when those are done (206 x 256 x 13 x 13, window 3, fp32, 32 filters, model gradient: 159 us behind, 144 first).
// Their number is a multiple of 8, so that the others' XCDs do not depend on it.
// Past the caches every row that a thread stores in turn is one more stream to memory for as many wavefronts as are resident,
// and too many of them halve its rate.  So windows of 5 take a window row per thread, and fp32 windows of 3 four workgroups
// per compute unit (256 x 384 x 13 x 13, fp32, lowering and col2im in turn: 291 us with eight, 260 with five, 258 with four,
// 276 with two, 295 staged in LDS; forward 1007, 980, 974, 993 and 1003.  96 x 27 x 27, window 5, 64 images, fp32: forward 548
// with all window rows, 537 with one, 547 staged; bf16, 256 images: 459 and 447.  bf16 windows of 3 gain nothing from fewer
// workgroups: 256 x 384 x 13 x 13 model gradient 244 with eight, 255 with four.)
struct FlatPlan {
    unsigned blocks;
    int32_t columns, own;          // 16-byte columns of the matrix, and of one XCD, or (past) in whole workgroups
    int32_t rows;                  // channels times groups of window rows
    int ky_per;                    // window rows per thread
    int past;                      // store past the caches
    unsigned lds;                  // bytes that a workgroup claims and does not use
    FastDiv div_own, div_gz;
};

constexpr int64_t MOST_WORKGROUPS = 0xffffffffll / 256;  // of 256 threads: a grid dimension holds less than 2^32 threads
constexpr double CACHED_BYTES = 230e6;                   // of a lowered matrix: see lower_flat_body
static unsigned packing_blocks(int64_t n) { return (unsigned)round_up(n, 8); }

// Which layers: see lower_flat_body.  Window rows over threads of their own where the launch has few.  `packing`: the
// workgroups that pack something else in the same launch.
static bool make_flat_plan(const ConvGeom &g, size_t elem, int64_t ld, int64_t packing, FlatPlan *p)
{
    const int V = (int)(16 / elem);
    if (g.sh != 1 || g.sw != 1 || g.Wo != g.W || (g.kw != 1 && g.kw != 3 && g.kw != 5)) return false;
    if (ld % V != 0 || ld > 0x7fffffffll - 4096 || g.W < V + 2 || 2 * g.pw != g.kw - 1) return false;
    p->past = (double)g.K * (double)ld * (double)elem > CACHED_BYTES ? 1 : 0;
    p->columns = (int32_t)(ld / V);
    const bool cut = !p->past && p->columns >= 512;
    p->own = cut ? (p->columns + 63) / 64 * 8 : p->past ? (int32_t)round_up(p->columns, 256) : p->columns;
    const int64_t pieces = (int64_t)p->columns * g.C, least = 1024 * 256;
    const int kz = pieces >= least ? 1 : (int)((least - 1) / pieces) + 1;
    p->ky_per = kz >= g.kh || (p->past && g.kw == 5) ? 1 : (g.kh + kz - 1) / kz;
    p->lds = p->past && g.kw == 3 && elem == 4 ? 38 * 1024 : 0;  // four workgroups per compute unit
    const int gz = (g.kh + p->ky_per - 1) / p->ky_per;
    const int64_t rows = (int64_t)g.C * gz, threads = p->own * rows, blocks = (threads + 255) / 256 * (cut ? 8 : 1);
    if (threads > 0x7fffffffll - 4096 || blocks + round_up(packing, 8) > MOST_WORKGROUPS) return false;
    p->blocks = (unsigned)blocks, p->rows = (int32_t)rows;
    p->div_own = FastDiv((uint32_t)p->own), p->div_gz = FastDiv((uint32_t)gz);
    return true;
}

template <typename U, int KW>
__device__ __forceinline__ void lower_flat_block(const ConvGeom &g, const FlatPlan &p, const U *__restrict__ X, U *__restrict__ D,
                                                 int64_t ld, unsigned block)
{
    const bool cut = p.own < p.columns;  // an XCD has its own columns
    uint32_t row, at, c, bz;
    p.div_own.divmod((cut ? block / 8 : block) * 256u + threadIdx.x, row, at);
    const uint32_t column = at + (cut ? block % 8 * (uint32_t)p.own : 0u);
    if (row >= (uint32_t)p.rows || column >= (uint32_t)p.columns) return;
    p.div_gz.divmod(row, c, bz);
    const int64_t m0 = (int64_t)column * FlatRun<U, KW>::V;
    if (p.past) lower_flat_body<U, KW, true>(g, p.ky_per, X, D, ld, m0, (int)c, (int)bz);
    else lower_flat_body<U, KW, false>(g, p.ky_per, X, D, ld, m0, (int)c, (int)bz);
}

template <typename U, int KW>
__global__ __launch_bounds__(256) void lower_flat_kernel(ConvGeom g, FlatPlan p, const U *__restrict__ X, U *__restrict__ D, int64_t ld,
                                                         KhatJob<U> khat)
{
    const unsigned packing = gridDim.x - p.blocks;
    if (blockIdx.x < packing)
        khat_body(khat, (int64_t)blockIdx.x);
    else
        lower_flat_block<U, KW>(g, p, X, D, ld, blockIdx.x - packing);
}

// Estimated time of a staged lowering in microseconds: a workgroup stages its patch (LDS cleared, then one pixel at a time),
// stores a 16-byte piece per thread and row of D-hat, and the ragged ends element by element; 3.3 workgroups per compute
// unit overlap, fewer where LDS holds fewer; beside that the bytes.  Fitted to 44 000 times of 8 800 lowerings (1 to 600
// channels, planes of 5 x 5 to 120 x 120, windows of 1 to 11, strides 1, 2, 4, both types) under five rules for the groups;
// mean deviation 11 %.
static double lower_us(const ConvGeom &g, size_t elem, const LowerPlan &p)
{
    // (host time of every small call: no 64-bit divisions)
    const int log_vec = elem == 2 ? 3 : 2, parts = (g.kh + p.ky_per - 1) / p.ky_per;
    const int64_t vec = (int64_t)1 << log_vec, images = p.nb, rows_in = (int64_t)(p.br - 1) * g.sh + g.kh, cols = images * p.br * g.Wo;
    const int64_t wgs = (int64_t)((g.N + p.nb - 1) / p.nb) * p.bands * g.C * parts;
    auto per_thread = [](int64_t n) { return (double)((uint64_t)(n + 255) >> 8); };
    const int64_t pixels = (rows_in < g.H ? rows_in : g.H) * g.W, lds = images * rows_in * p.wp * (int64_t)elem, rows = (int64_t)p.ky_per * g.kw;
    const bool ragged = ((p.bands == 1 ? images * g.HoWo : (int64_t)p.br * g.Wo) & (vec - 1)) != 0;
    const double wg = 0.122 * per_thread(images * ((pixels + vec - 1) >> log_vec)) * (double)vec + 0.0235 * per_thread((lds >> 4) + 1) +
                      0.0502 * per_thread((cols + vec - 1) >> log_vec) * (double)rows + (ragged ? 0.288 * per_thread(vec * rows) : 0.0);
    const double fit = 163840.0 / (double)(lds > 16384 ? lds : 16384), overlap = fit < 3.32 ? (fit > 1.0 ? floor(fit) : 1.0) : 3.32;
    const double rounds = (double)((uint64_t)(wgs + 255) >> 8) / overlap, compute = wg * (rounds > 1.0 ? rounds : 1.0);
    const double memory = ((double)g.N * g.C * g.H * g.W + (double)g.K * g.M) * (double)elem / 4.87e6;
    return 2.8 + sqrt(compute * compute + memory * memory);
}

// Few channels and images (first layers, small batches) leave a launch with few workgroups, which then lasts as long as one
// workgroup's work: smaller groups, then bands, and the window rows of a patch over workgroups of their own, where the
// estimate says that saves a tenth.  (8 x 3 x 32 x 32, window 5, fp32, which lower_flat_kernel takes now: 14 -> 3.7 us; not 6 x 512 x 41 x 41, window 11, bf16,
// where 1024 workgroups instead of 512 take 338 us instead of 250.)  5 850 random lowerings: 0.8 times as long as without
// on average, 40 of them longer than 6 us and more than 1.05 times as long; launches of 4 us are up to 0.7 us longer.
static void spread_lower_plan(const ConvGeom &g, size_t elem, LowerPlan *p)
{
    p->ky_per = g.kh;
    int64_t wgs = (int64_t)((g.N + p->nb - 1) / p->nb) * p->bands * g.C;
    if (wgs >= 1024) return;
    LowerPlan best = *p, q = *p;
    double least = 0.9 * lower_us(g, elem, q);
    for (;;) {
        const int kz = (int)(1023 / (int)wgs) + 1;
        q.ky_per = kz >= g.kh ? 1 : (g.kh + kz - 1) / kz;
        const double us = lower_us(g, elem, q);
        if (us < least) best = q, least = us;
        if (wgs >= 1024) break;
        if (q.nb > 1) {
            q.nb = (q.nb + 1) / 2;
        } else if (q.br > 16 || (q.bands > 1 && q.br > 4)) {
            q.br = (q.br + 1) / 2;
            q.bands = (g.Ho + q.br - 1) / q.br;
        } else {
            break;
        }
        wgs = (int64_t)((g.N + q.nb - 1) / q.nb) * q.bands * g.C;
    }
    best.rows_in = (best.br - 1) * g.sh + g.kh;
    *p = best;
}

// Choose the staging plan; returns false when not even one output row's patch fits in LDS.
static bool make_lower_plan(const ConvGeom &g, size_t elem, LowerPlan *p, size_t *lds_bytes)
{
    const size_t small_budget = 32 * 1024, band_budget = 40 * 1024;
    p->wp = g.W + 2 * g.pw;
    int rows_full = (g.Ho - 1) * g.sh + g.kh;
    size_t plane = (size_t)rows_full * p->wp * elem;
    if (2 * plane <= small_budget) {
        int nb = (int)(small_budget / plane);
        if (nb > 32) nb = 32;
        if (nb > g.N) nb = g.N;
        p->nb = nb;
        p->br = g.Ho;
        p->bands = 1;
        p->rows_in = rows_full;
    } else {
        size_t row_bytes = (size_t)p->wp * elem;
        if ((size_t)g.kh * row_bytes > 64 * 1024) return false;
        int64_t rows_fit = (int64_t)(band_budget / row_bytes);
        int br = rows_fit >= g.kh ? (int)((rows_fit - g.kh) / g.sh + 1) : 1;
        if (br > g.Ho) br = g.Ho;
        p->nb = 1;
        p->br = br;
        p->bands = (g.Ho + br - 1) / br;
        p->rows_in = (br - 1) * g.sh + g.kh;
    }
    spread_lower_plan(g, elem, p);
    p->groups = (g.N + p->nb - 1) / p->nb;
    p->div_wp = FastDiv((uint32_t)p->wp);
    p->div_rows_in = FastDiv((uint32_t)p->rows_in);
    *lds_bytes = (size_t)p->nb * p->rows_in * p->wp * elem;
    if ((int64_t)p->bands * p->groups > 0x7fffffffll || g.C > 65535) return false;
    return true;
}

// Transpose of a matrix [rows][cols] into [cols][ld] (columns from `rows` to ld zero): the lowering of a layer whose
// window is the whole unpadded image (a fully connected layer: D-hat is X [N][K] transposed) and the packing of a
// gradient with one output position per image (dY [N][F]).  A workgroup takes TR_C source columns; per round it has
// 256 source rows in flight as 16-byte loads, turns them in LDS and stores 16-byte pieces along the destination's rows.
// With `sums` it runs over all rows itself (gridDim.y == 1) and leaves every column's fp32 sum there.
// Why: the general kernels give such layers one workgroup per channel with one pixel per image, which wrote 32-byte
// pieces: X of 256 x 4096 bf16 41 us and dY of 256 x 4096 12 us, here 5 and 5.
constexpr int TR_C = 32, TR_R = 256;
template <typename T, typename U, bool PACK_DY>  // PACK_DY: the packing of a gradient (else a lowering): may leave sums
__global__ __launch_bounds__(256) void transpose_kernel(const U *__restrict__ src, int rows, int cols, U *__restrict__ dst,
                                                        int64_t ld, float *__restrict__ sums, float *__restrict__ sums2)
{
    constexpr int VEC = 16 / (int)sizeof(U);
    constexpr int SEG = TR_C / VEC;               // 16-byte pieces per source row of the tile
    constexpr int RP = TR_R / VEC;                // 16-byte pieces per destination row of the tile
    constexpr int PT = TR_R * SEG / 256;          // pieces per thread, both ways
    constexpr int PITCH = TR_R + VEC;             // elements; a multiple of 16 bytes
    static_assert(RP == 32 || RP == 64, "a column's pieces are half a wavefront or one");
    __shared__ __align__(16) U tile[TR_C * PITCH];
    const int tid = threadIdx.x, c0 = blockIdx.x * TR_C;
    float sum[PT];
#pragma unroll
    for (int i = 0; i < PT; ++i) sum[i] = 0.f;
    for (int64_t r0 = (int64_t)blockIdx.y * TR_R; r0 < ld; r0 += (int64_t)gridDim.y * TR_R) {
        VecOf<U, VEC> v[PT];
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int t = tid + 256 * i, c = c0 + t % SEG * VEC;
            const int64_t r = r0 + t / SEG;
            if (r < rows && c + VEC <= cols) {
                __builtin_memcpy(&v[i], src + r * cols + c, 16);
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) v[i].v[e] = r < rows && c + e < cols ? src[r * cols + c + e] : (U)0;
            }
        }
        __syncthreads();  // the previous round has been read
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int t = tid + 256 * i;
#pragma unroll
            for (int e = 0; e < VEC; ++e) tile[(t % SEG * VEC + e) * PITCH + t / SEG] = v[i].v[e];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int t = tid + 256 * i, c = t / RP;
            const VecOf<U, VEC> o = *reinterpret_cast<const VecOf<U, VEC> *>(tile + c * PITCH + t % RP * VEC);
            const int64_t m = r0 + t % RP * VEC;
            if (c0 + c < cols && m < ld) {  // ld is a multiple of the piece
                *reinterpret_cast<VecOf<U, VEC> *>(dst + (int64_t)(c0 + c) * ld + m) = o;
                if constexpr (PACK_DY)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        T x;
                        __builtin_memcpy(&x, &o.v[e], sizeof(T));
                        sum[i] += Elem<T>::to_f32(x);
                    }
            }
        }
    }
    if (PACK_DY && sums != nullptr) {
#pragma unroll
        for (int i = 0; i < PT; ++i) {  // a column's pieces lie in RP neighbouring lanes: a fixed tree over them
            float a = sum[i];
#pragma unroll
            for (int off = RP / 2; off > 0; off >>= 1) a += __shfl_down(a, off, RP);
            const int t = tid + 256 * i, c = c0 + t / RP;
            if (t % RP == 0 && c < cols) {
                sums[c] = a;
                if (sums2 != nullptr) sums2[c] = a;
            }
        }
    }
}

static bool lower_is_transpose(const ConvGeom &g)
{
    return g.HoWo == 1 && g.ph == 0 && g.pw == 0 && g.kh == g.H && g.kw == g.W;
}

template <typename T, typename U, bool PACK_DY>
static void run_transpose(const void *src, int rows, int cols, void *dst, int64_t ld, float *sums, float *sums2, hipStream_t s)
{
    const unsigned gy = sums != nullptr ? 1u : (unsigned)((ld + TR_R - 1) / TR_R < 65535 ? (ld + TR_R - 1) / TR_R : 65535);
    hipLaunchKernelGGL((transpose_kernel<T, U, PACK_DY>), dim3((unsigned)((cols + TR_C - 1) / TR_C), gy), dim3(256), 0, s,
                       (const U *)src, rows, cols, (U *)dst, ld, sums, sums2);
}

template <typename U> static void run_khat(const KhatJob<U> &j, hipStream_t s)
{
    ProfScope prof(KID_PACK_KHAT, s, 0.0, j.bytes());
    hipLaunchKernelGGL(pack_khat_kernel<U>, dim3((unsigned)j.blocks()), dim3(256), 0, s, j);
}

int launch_pack_khat_t(const ConvGeom &g, int dtype, const void *W, void *KhatT, int64_t Kp, int64_t Fp, hipStream_t s)
{
    if (dtype == OMNI_BF16) run_khat(KhatJob<uint16_t>{(const uint16_t *)W, (uint16_t *)KhatT, g.F, g.K, Kp, Fp, 1}, s);
    else run_khat(KhatJob<uint32_t>{(const uint32_t *)W, (uint32_t *)KhatT, g.F, g.K, Kp, Fp, 1}, s);
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

// khat.out != null: K-hat is packed as well
template <typename U>
static int run_lower(const ConvGeom &g, const U *X, U *D, int64_t ld, KhatJob<U> khat, hipStream_t s)
{
    constexpr int VEC = 16 / sizeof(U);
    LowerPlan plan;
    size_t lds = 0;
    const bool transpose = lower_is_transpose(g) && ld % VEC == 0;
    FlatPlan flat;
    const int64_t packing = khat.out != nullptr ? khat.blocks() : 0;
    if (!transpose && make_flat_plan(g, sizeof(U), ld, packing, &flat)) {
        ProfScope prof(KID_LOWER, s, 0.0, ((double)g.N * g.C * g.H * g.W + (double)g.K * g.M) * sizeof(U) + khat.bytes());
        const dim3 grid(flat.blocks + packing_blocks(packing));
        if (g.kw == 1) hipLaunchKernelGGL((lower_flat_kernel<U, 1>), grid, dim3(256), flat.lds, s, g, flat, X, D, ld, khat);
        else if (g.kw == 3) hipLaunchKernelGGL((lower_flat_kernel<U, 3>), grid, dim3(256), flat.lds, s, g, flat, X, D, ld, khat);
        else hipLaunchKernelGGL((lower_flat_kernel<U, 5>), grid, dim3(256), flat.lds, s, g, flat, X, D, ld, khat);
        OMNI_LAUNCH_CHECK();
        return OMNI_OK;
    }
    if (!transpose && make_lower_plan(g, sizeof(U), &plan, &lds)) {
        const unsigned gx = (unsigned)(plan.bands * plan.groups), gz = (unsigned)((g.kh + plan.ky_per - 1) / plan.ky_per);
        int64_t extra = (packing + (int64_t)gx * gz - 1) / ((int64_t)gx * gz);
        if (g.C + extra > 65535) {
            run_khat(khat, s);
            khat.out = nullptr, extra = 0;
        }
        ProfScope prof(KID_LOWER, s, 0.0, ((double)g.N * g.C * g.H * g.W + (double)g.K * g.M) * sizeof(U) + khat.bytes());
        dim3 grid(gx, (unsigned)(g.C + extra), gz);
        const int vec = ld % VEC != 0 ? 1 : VEC;
#define OMNI_LOWER_CASE(V, KWT) hipLaunchKernelGGL((lower_lds_kernel<U, V, KWT>), grid, dim3(256), lds, s, g, plan, X, D, ld, khat)
#define OMNI_LOWER_KW(V)                                  \
    do {                                                  \
        if (g.kw == 3) OMNI_LOWER_CASE(V, 3);             \
        else if (g.kw == 5) OMNI_LOWER_CASE(V, 5);        \
        else if (g.kw == 11) OMNI_LOWER_CASE(V, 11);      \
        else OMNI_LOWER_CASE(V, 0);                       \
    } while (0)
        if (vec == 1) OMNI_LOWER_CASE(1, 0);
        else OMNI_LOWER_KW(VEC);
#undef OMNI_LOWER_KW
#undef OMNI_LOWER_CASE
        OMNI_LAUNCH_CHECK();
        return OMNI_OK;
    }
    if (khat.out != nullptr) run_khat(khat, s);
    ProfScope prof(KID_LOWER, s, 0.0, ((double)g.N * g.C * g.H * g.W + (double)g.K * g.M) * sizeof(U));
    if (transpose) {
        typedef typename std::conditional<sizeof(U) == 2, bf16_t, float>::type T;
        run_transpose<T, U, false>(X, g.N, g.K, D, ld, nullptr, nullptr, s);
        OMNI_LAUNCH_CHECK();
        return OMNI_OK;
    }
    unsigned gy = (unsigned)(g.K < 65535 ? g.K : 65535);
    if (ld % VEC == 0) {
        int64_t vpr = ld / VEC;
        dim3 grid((unsigned)((vpr + 255) / 256), gy, 1);
        hipLaunchKernelGGL((lower_kernel<U, VEC>), grid, dim3(256), 0, s, g, X, D, ld, vpr);
    } else {
        dim3 grid((unsigned)((ld + 255) / 256), gy, 1);
        hipLaunchKernelGGL((lower_kernel<U, 1>), grid, dim3(256), 0, s, g, X, D, ld, ld);
    }
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

int launch_lower(const ConvGeom &g, int dtype, const void *X, void *Dhat, int64_t ld, hipStream_t s)
{
    return launch_lower_khat(g, dtype, X, Dhat, ld, nullptr, nullptr, 0, 0, s);
}

int launch_lower_khat(const ConvGeom &g, int dtype, const void *X, void *Dhat, int64_t ld, const void *W, void *Khat, int64_t Fp,
                      int64_t Kp, hipStream_t s)
{
    if (dtype == OMNI_BF16)
        return run_lower<uint16_t>(g, (const uint16_t *)X, (uint16_t *)Dhat, ld,
                                   KhatJob<uint16_t>{(const uint16_t *)W, (uint16_t *)Khat, g.F, g.K, Fp, Kp, 0}, s);
    return run_lower<uint32_t>(g, (const uint32_t *)X, (uint32_t *)Dhat, ld,
                               KhatJob<uint32_t>{(const uint32_t *)W, (uint32_t *)Khat, g.F, g.K, Fp, Kp, 0}, s);
}

// ------------------------------------------------------------------------------------------------
// col2im (transpose of the lowering map), gather form: one thread per input pixel sums the entries
// of dD-hat that were copies of that pixel, in ascending (ky, kx) order, in fp32.  No atomics.
// ------------------------------------------------------------------------------------------------
// The window positions that cover input coordinate i along one axis: k = first, first+s, ... <= last,
// with output coordinate o(first) = (i + pad - first)/s decreasing by one per step.  No per-tap division.
struct TapRange { int first, last, o_first; };
__device__ __forceinline__ TapRange tap_range(int i, int pad, int k, int s, int out, const FastDiv &div_s)
{
    TapRange t;
    int top = i + pad;                       // k = top gives o = 0
    int lo = top - (out - 1) * s;            // smallest k with o <= out-1
    if (lo < 0) lo = 0;
    uint32_t q, r;
    div_s.divmod((uint32_t)(top - lo), q, r);  // top - lo >= 0 whenever the range is non-empty
    t.first = lo + (int)r;                   // same residue as top modulo s
    t.o_first = (int)q;
    t.last = top < k - 1 ? top : k - 1;
    if (top < lo) t.last = -1;               // empty
    return t;
}

template <typename T>
__global__ __launch_bounds__(256) void col2im_kernel(ConvGeom g, const T *__restrict__ D, int64_t ld,
                                                     T *__restrict__ dX, uint32_t plane0, uint32_t count)
{
    // One launch covers `count` < 2^31 pixels starting at plane (n*C + c) = plane0.
    uint32_t local = blockIdx.x * 256u + threadIdx.x;
    if (local >= count) return;
    uint32_t pl, pix, iy, ix;
    g.div_HW.divmod(local, pl, pix);
    g.div_W.divmod(pix, iy, ix);
    uint32_t plane = plane0 + pl;
    uint32_t n = plane / (uint32_t)g.C, c = plane - n * (uint32_t)g.C;

    float acc = 0.f;
    const TapRange ry = tap_range((int)iy, g.ph, g.kh, g.sh, g.Ho, g.div_sh);
    const TapRange rx = tap_range((int)ix, g.pw, g.kw, g.sw, g.Wo, g.div_sw);
    for (int ky = ry.first, oy = ry.o_first; ky <= ry.last; ky += g.sh, --oy)
        for (int kx = rx.first, ox = rx.o_first; kx <= rx.last; kx += g.sw, --ox) {
            int64_t row = ((int64_t)c * g.kh + ky) * g.kw + kx;
            int64_t col = ((int64_t)n * g.Ho + oy) * g.Wo + ox;
            acc += Elem<T>::to_f32(D[row * ld + col]);
        }
    dX[(int64_t)plane * g.H * g.W + pix] = Elem<T>::from_f32(acc);
}

// Strided layers whose segments do not fit in LDS (CaffeNet's conv1: 11 x 11 window, stride 4).  With stride S an
// input pixel meets only the taps of its own residue class, kx = (ix + pw) mod S + S*j, and for one such tap the
// pixels ix, ix + S, ix + 2S, ... of a row read consecutive columns of one row of dD-hat.  So a thread takes the S
// consecutive pixels S*b .. S*b + S - 1 of an input row and neighbouring lanes take neighbouring b: every load
// instruction of a wavefront then reads one run of consecutive elements (the per-pixel form above reads S runs with
// gaps, and fetched three times the matrix on conv1), and every thread stores S consecutive pixels at once.
// At most JY x JX taps per pixel (ceil(kh / S), ceil(kw / S)), all issued together with the absent ones masked;
// each pixel's terms are added in ascending (ky, kx), as above.
template <typename T, int S, int JY, int JX>
__global__ __launch_bounds__(256) void col2im_strided_kernel(ConvGeom g, const T *__restrict__ D, int64_t ld,
                                                             T *__restrict__ dX, uint32_t plane0, uint32_t count,
                                                             FastDiv div_rows, FastDiv div_bw)
{
    // One launch covers `count` < 2^31 (plane, row, group of S pixels) triples starting at plane plane0.
    const uint32_t local = blockIdx.x * 256u + threadIdx.x;
    if (local >= count) return;
    uint32_t pl, rest, iy, b;
    div_rows.divmod(local, pl, rest);  // rows of groups per plane: H * ceil(W / S)
    div_bw.divmod(rest, iy, b);
    const uint32_t plane = plane0 + pl;
    const uint32_t n = plane / (uint32_t)g.C, c = plane - n * (uint32_t)g.C;
    const TapRange ry = tap_range((int)iy, g.ph, g.kh, S, g.Ho, g.div_sh);
    TapRange rx[S];
#pragma unroll
    for (int px = 0; px < S; ++px) {
        const int ix = S * (int)b + px;
        rx[px] = tap_range(ix < g.W ? ix : g.W - 1, g.pw, g.kw, S, g.Wo, g.div_sw);
        if (ix >= g.W) rx[px].last = -1;
    }
    float v[JY][S][JX];
    bool ok[JY][S][JX];
#pragma unroll
    for (int jy = 0; jy < JY; ++jy) {
        const int ky = ry.first + jy * S, oy = ry.o_first - jy;
        const bool vy = ky <= ry.last;
        const int64_t col0 = ((int64_t)n * g.Ho + oy) * g.Wo;
#pragma unroll
        for (int px = 0; px < S; ++px)
#pragma unroll
            for (int jx = 0; jx < JX; ++jx) {
                const int kx = rx[px].first + jx * S, ox = rx[px].o_first - jx;
                ok[jy][px][jx] = vy && kx <= rx[px].last;
                const int64_t at = ok[jy][px][jx] ? (((int64_t)c * g.kh + ky) * g.kw + kx) * ld + col0 + ox : 0;
                v[jy][px][jx] = Elem<T>::to_f32(D[at]);
            }
    }
    T res[S];
#pragma unroll
    for (int px = 0; px < S; ++px) {
        float acc = 0.f;
#pragma unroll
        for (int jy = 0; jy < JY; ++jy)
#pragma unroll
            for (int jx = 0; jx < JX; ++jx) acc += ok[jy][px][jx] ? v[jy][px][jx] : 0.f;
        res[px] = Elem<T>::from_f32(acc);
    }
    T *out = dX + ((int64_t)plane * g.H + iy) * g.W + S * (int64_t)b;
    if (S * (int)b + S <= g.W) {
        __builtin_memcpy(out, res, sizeof(res));  // element-aligned store of S pixels
    } else {
#pragma unroll
        for (int px = 0; px < S; ++px)
            if (S * (int)b + px < g.W) out[px] = res[px];
    }
}

// LDS-staged variant.  A workgroup takes channel c of a group of nb images.  Step 1 copies, for each of
// the kh*kw rows of that channel, the column range of the group from dD-hat into LDS with 16-byte loads
// (all loads are in flight together).  Step 2 is the same gather as above, served from LDS: one thread
// per input pixel, ascending (ky, kx), fp32.  dD-hat is read from HBM exactly once, in full vectors.
struct Col2imPlan {
    int nb;      // images per workgroup
    int groups;  // image groups
    int pitch;   // LDS elements per row segment (multiple of the vector width)
};

// KH, KW > 0: stride 1 and a window known at compile time.  Pixel (iy, ix) then receives tap (ky, kx) from output
// position (iy + ph - ky, ix + pw - kx), i.e. from LDS element  base - ky * Wo - kx  of row ky * KW + kx: one
// address per pixel, constant offsets per tap, and the taps that fall outside the output are masked instead of
// being skipped by loops with data-dependent bounds (the vector ALU, not memory, is what bounded this kernel).
template <typename T, int KH, int KW>
__global__ __launch_bounds__(256) void col2im_lds_kernel(ConvGeom g, Col2imPlan p, const T *__restrict__ D,
                                                         int64_t ld, T *__restrict__ dX)
{
    constexpr int VEC = 16 / sizeof(T);
    extern __shared__ __align__(16) unsigned char col2im_smem[];
    T *seg = reinterpret_cast<T *>(col2im_smem);
    const int tid = threadIdx.x;
    const int c = blockIdx.y;
    const int n0 = blockIdx.x * p.nb;
    const int nb = g.N - n0 < p.nb ? g.N - n0 : p.nb;
    const int khkw = g.kh * g.kw;
    const int64_t m_lo = (int64_t)n0 * g.HoWo, m_hi = m_lo + (int64_t)nb * g.HoWo;
    const int64_t v_lo = m_lo / VEC, v_hi = (m_hi + VEC - 1) / VEC;  // 16-byte slots covering the range
    const int slots = (int)(v_hi - v_lo);
    const int skew = (int)(m_lo - v_lo * VEC);                        // position of column m_lo inside its slot

    const uint4 *src = reinterpret_cast<const uint4 *>(D + (int64_t)c * khkw * ld) + v_lo;
    const int64_t row_slots = ld / VEC;
    uint4 *dst = reinterpret_cast<uint4 *>(col2im_smem);
    const int pitch_slots = p.pitch / VEC;
    {
        // batches of loads into registers, then into LDS: a plain copy loop waits for each load before it
        // issues the next one, and a workgroup's whole segment is only about ten loads per thread
        constexpr int BATCH = 12;
        const int total = khkw * slots;
        for (int i0 = tid; i0 < total; i0 += 256 * BATCH) {
            uint4 regs[BATCH];
            int where[BATCH];
            // branch-free: indices past the end repeat the last slot (the same bytes land in the same place twice)
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                int i = i0 + 256 * u;
                i = i < total ? i : total - 1;
                const int r = i / slots, v = i - r * slots;
                regs[u] = src[r * row_slots + v];
                where[u] = r * pitch_slots + v;
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) dst[where[u]] = regs[u];
        }
    }
    __syncthreads();

    const int hw = g.H * g.W;
    for (int px = tid; px < nb * hw; px += 256) {
        uint32_t inb, pix, iy, ix;
        g.div_HW.divmod((uint32_t)px, inb, pix);
        g.div_W.divmod(pix, iy, ix);
        float acc = 0.f;
        if constexpr (KH > 0) {
            const int oy0 = (int)iy + g.ph, ox0 = (int)ix + g.pw;     // output position of tap (0, 0)
            const int base = skew + (int)inb * g.HoWo + oy0 * g.Wo + ox0;
            bool vx[KW];
#pragma unroll
            for (int kx = 0; kx < KW; ++kx) vx[kx] = (unsigned)(ox0 - kx) < (unsigned)g.Wo;
#pragma unroll
            for (int ky = 0; ky < KH; ++ky) {
                const bool vy = (unsigned)(oy0 - ky) < (unsigned)g.Ho;
#pragma unroll
                for (int kx = 0; kx < KW; ++kx) {
                    const bool ok = vy && vx[kx];
                    const int idx = ok ? (ky * KW + kx) * p.pitch + base - ky * g.Wo - kx : 0;
                    const float v = Elem<T>::to_f32(seg[idx]);
                    acc += ok ? v : 0.f;
                }
            }
        } else {
            const T *base = seg + skew + (int)inb * g.HoWo;
            const TapRange ry = tap_range((int)iy, g.ph, g.kh, g.sh, g.Ho, g.div_sh);
            const TapRange rx = tap_range((int)ix, g.pw, g.kw, g.sw, g.Wo, g.div_sw);
            for (int ky = ry.first, oy = ry.o_first; ky <= ry.last; ky += g.sh, --oy) {
                const T *row = base + ky * g.kw * p.pitch + oy * g.Wo;
                for (int kx = rx.first, ox = rx.o_first; kx <= rx.last; kx += g.sw, --ox)
                    acc += Elem<T>::to_f32(row[kx * p.pitch + ox]);
            }
        }
        dX[((int64_t)(n0 + inb) * g.C + c) * hw + pix] = Elem<T>::from_f32(acc);
    }
}

// Stride 1 and an output as wide as the input: pixel q of a plane receives tap (ky, kx) from output position
// q + (ph - ky) W + (pw - kx) of the same image, also across a row's end, unless that leaves the image.  So the terms of 16
// bytes of consecutive pixels are, tap by tap, 16 consecutive bytes of a row of dD-hat: a thread reads them straight from
// memory, blanks what the window joins to positions outside the image, and adds them in fp32 in ascending (ky, kx).  Every
// entry of dD-hat is one term of one pixel, so there is nothing that staging in LDS could save: the copy, its barrier and 16-bit
// reads per term only cost (384 channels, 13 x 13, window 3, 256 images, bf16: 98 us; 299 MB are read).  bf16 loads start at the
// multiple of 4 bytes at or before the first term and are shifted: 16 bytes at a 2-byte boundary take three times as long.
// A matrix that the caches hold is read where it was written (FlatPlan): every XCD takes `own` of the N * groups 16-byte columns
// of pixels, all channels (100 x 32 x 16 x 16, window 5, bf16, data gradient 33.6 -> 28.6 us; lowering and col2im in
// turn 24.9 -> 19.1, staged in LDS 34.5).  A larger one (own == 0), and one of few columns, in order of channels, then images.
template <typename T, int KH, int KW>
__global__ __launch_bounds__(256) void col2im_flat_kernel(ConvGeom g, const T *__restrict__ D, int64_t ld, T *__restrict__ dX,
                                                          uint32_t plane0, uint32_t count, uint32_t own, FastDiv div_groups, FastDiv div_inner)
{
    constexpr int V = 16 / sizeof(T);
    uint32_t j, c, n, at;
    if (own != 0u) {
        div_inner.divmod(blockIdx.x / 8u * 256u + threadIdx.x, c, at);
        at += blockIdx.x % 8u * own;
        if (c >= (uint32_t)g.C || at >= count) return;
        div_groups.divmod(at, n, j);
    } else {
        at = blockIdx.x * 256u + threadIdx.x;
        if (at >= count) return;
        uint32_t pl;
        div_groups.divmod(at, pl, j);
        div_inner.divmod(plane0 + pl, c, n);  // planes in order of channels, then images: neighbours in dD-hat's rows
    }
    const int hw = g.H * g.W, q0 = (int)j * V;
    uint32_t iy, ix;
    g.div_W.divmod((uint32_t)q0, iy, ix);
    const int64_t at0 = (int64_t)c * (KH * KW) * ld + (int64_t)n * g.HoWo + q0 + g.ph * g.W + g.pw;  // of tap (0, 0)
    const int64_t at_last = at0 + (int64_t)(KH * KW - 1) * ld - (KH - 1) * g.W - (KW - 1), total = (int64_t)(g.K - 1) * ld + g.M;
    T *out = dX + ((int64_t)n * g.C + c) * hw + q0;

    // which terms exist, as masks over the 16 bytes (bits and words, the latter for 16-bit elements in pairs)
    const FlatCols<T> cols((int)ix, g.W);
    const uint32_t row = cols.own_row();
    uint32_t mx[KW][4], my[KH][4];
    flat_for<0, KW>([&](auto tap) {
        constexpr int KX = decltype(tap)::value;
        FlatCols<T>::mask(cols.template inside<KX - KW / 2>(), mx[KX]);
    });
#pragma unroll
    for (int ky = 0; ky < KH; ++ky)
        FlatCols<T>::mask(((unsigned)((int)iy + g.ph - ky) < (unsigned)g.Ho ? row : 0u) | ((unsigned)((int)iy + 1 + g.ph - ky) < (unsigned)g.Ho ? ~row : 0u), my[ky]);
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    if (at_last + V + 2 <= total) {
#pragma unroll
        for (int ky = 0; ky < KH; ++ky) {
            uint4 v[KW];
            uint32_t next[KW];
#pragma unroll
            for (int kx = 0; kx < KW; ++kx) {
                const int64_t at = at0 + (int64_t)(ky * KW + kx) * ld - ky * g.W - kx;
                if constexpr (sizeof(T) == 4) {
                    __builtin_memcpy(&v[kx], D + at, 16);
                    next[kx] = 0u;
                } else {
                    const T *p = D + (at & ~(int64_t)1);
                    __builtin_memcpy(&v[kx], __builtin_assume_aligned(p, 4), 16);
                    __builtin_memcpy(&next[kx], __builtin_assume_aligned(p + 8, 4), 4);
                }
            }
#pragma unroll
            for (int kx = 0; kx < KW; ++kx) {
                uint32_t u[4] = {v[kx].x, v[kx].y, v[kx].z, v[kx].w};
                if constexpr (sizeof(T) == 2) {
                    const uint32_t shift = (uint32_t)((at0 + (int64_t)(ky * KW + kx) * ld - ky * g.W - kx) & 1) * 16u;
                    u[0] = __builtin_amdgcn_alignbit(v[kx].y, v[kx].x, shift), u[1] = __builtin_amdgcn_alignbit(v[kx].z, v[kx].y, shift);
                    u[2] = __builtin_amdgcn_alignbit(v[kx].w, v[kx].z, shift), u[3] = __builtin_amdgcn_alignbit(next[kx], v[kx].w, shift);
                }
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const uint32_t t = u[w] & mx[kx][w] & my[ky][w];
                    if constexpr (sizeof(T) == 4) acc[w] += __uint_as_float(t);
                    else acc[2 * w] += __uint_as_float(t << 16), acc[2 * w + 1] += __uint_as_float(t & 0xffff0000u);
                }
            }
        }
    } else {  // the 16 bytes of a last term would leave the matrix: one term at a time
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
            for (int ky = 0; ky < KH; ++ky)
#pragma unroll
                for (int kx = 0; kx < KW; ++kx) {
                    const uint32_t bits = sizeof(T) == 4 ? 0xffffffffu : (e % 2 ? 0xffff0000u : 0x0000ffffu);
                    const int w = sizeof(T) == 4 ? e : e / 2;
                    if (q0 + e < hw && (mx[kx][w] & my[ky][w] & bits) != 0u)
                        acc[e] += Elem<T>::to_f32(D[at0 + e + (int64_t)(ky * KW + kx) * ld - ky * g.W - kx]);
                }
    }
    T res[V];
#pragma unroll
    for (int e = 0; e < V; ++e) res[e] = Elem<T>::from_f32(acc[e]);
    if (q0 + V <= hw) {
        __builtin_memcpy(out, res, 16);  // element-aligned
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (q0 + e < hw) out[e] = res[e];
    }
}

static bool make_col2im_plan(const ConvGeom &g, size_t elem, int64_t ld, Col2imPlan *p, size_t *lds_bytes)
{
    const int vec = (int)(16 / elem);
    if (ld % vec != 0 || g.C > 65535) return false;
    const size_t budget = 40 * 1024, hard_limit = 80 * 1024;  // two workgroups per compute unit at the limit
    const int khkw = g.kh * g.kw;
    size_t per_image = (size_t)khkw * g.HoWo * elem;
    int nb = (int)(budget / per_image);
    if (nb < 1) nb = 1;
    if (nb > 32) nb = 32;
    if (nb > g.N) nb = g.N;
    p->nb = nb;
    p->groups = (g.N + nb - 1) / nb;
    p->pitch = (int)round_up((int64_t)nb * g.HoWo + vec, vec) + vec;  // room for the skew at both ends
    *lds_bytes = (size_t)khkw * p->pitch * elem;
    return *lds_bytes <= hard_limit;
}

int launch_col2im(const ConvGeom &g, int dtype, const void *dDhat, int64_t ld, void *dX, hipStream_t s)
{
    int64_t planes = (int64_t)g.N * g.C, hw = (int64_t)g.H * g.W;
    ProfScope prof(KID_COL2IM, s, 0.0, ((double)planes * hw + (double)g.K * g.M) * elem_size(dtype));
    const int V = 16 / (int)elem_size(dtype);
    Col2imPlan plan;
    size_t lds = 0;
    const bool staged = make_col2im_plan(g, elem_size(dtype), ld, &plan, &lds);
    // Staged in LDS, a bf16 window of 5 x 5 is as fast as its one round: a pixel per thread and about a workgroup per compute
    // unit, as in small layers of one image.  There the 25 loads of a thread's chain here cost more (1 x 128 x 13 x 13: 4.2 us
    // staged, 5.2 here, its data gradient 11.3 and 13.0; 1 x 268 x 7 x 10, 13.1 and 13.8; 1 x 384 x 13 x 13 alone 5.2 and 5.2; two
    // pixels per thread, 2 x 128 x 13 x 13, 6.1 and 5.1).
    const bool one_round = staged && dtype == OMNI_BF16 && g.kh == 5 && plan.nb * hw <= 256 && (int64_t)plan.groups * g.C <= 384;
    if (!one_round && g.sh == 1 && g.sw == 1 && g.Wo == g.W && g.W >= V + 2 && g.kh == g.kw && (g.kh == 3 || g.kh == 5)) {
        const int64_t groups = (hw + V - 1) / V, per_launch = (0x7fffffffll - 4096) / groups;
        const bool cut = (double)g.K * (double)ld * (double)elem_size(dtype) <= CACHED_BYTES && g.N * groups >= 512;
        const uint32_t own = cut ? (uint32_t)((g.N * groups + 63) / 64 * 8) : 0u;
        const FastDiv div_groups((uint32_t)groups), div_inner(cut ? own : (uint32_t)g.N);
        for (int64_t p0 = 0; p0 < planes; p0 += per_launch) {  // (one launch where it is cut)
            const int64_t np = planes - p0 < per_launch ? planes - p0 : per_launch;
            const uint32_t count = (uint32_t)(cut ? g.N * groups : np * groups);  // of 16-byte columns, of pieces
            const uint32_t blocks = cut ? (uint32_t)(((int64_t)own * g.C + 255) / 256 * 8) : (count + 255u) / 256u;
#define OMNI_COL2IM_FLAT(T_, K_)                                                                                             \
    hipLaunchKernelGGL((col2im_flat_kernel<T_, K_, K_>), dim3(blocks), dim3(256), 0, s, g, (const T_ *)dDhat, ld, (T_ *)dX, \
                       (uint32_t)p0, count, own, div_groups, div_inner)
            if (dtype == OMNI_BF16 && g.kh == 3) OMNI_COL2IM_FLAT(bf16_t, 3);
            else if (dtype == OMNI_BF16) OMNI_COL2IM_FLAT(bf16_t, 5);
            else if (g.kh == 3) OMNI_COL2IM_FLAT(float, 3);
            else OMNI_COL2IM_FLAT(float, 5);
#undef OMNI_COL2IM_FLAT
            OMNI_LAUNCH_CHECK();
        }
        return OMNI_OK;
    }
    if (staged) {
        dim3 grid((unsigned)plan.groups, (unsigned)g.C, 1);
        const bool unit = g.sh == 1 && g.sw == 1;
#define OMNI_COL2IM_CASE(KH, KW)                                                                                              \
    do {                                                                                                                      \
        if (dtype == OMNI_BF16)                                                                                               \
            hipLaunchKernelGGL((col2im_lds_kernel<bf16_t, KH, KW>), grid, dim3(256), lds, s, g, plan, (const bf16_t *)dDhat,   \
                               ld, (bf16_t *)dX);                                                                              \
        else                                                                                                                  \
            hipLaunchKernelGGL((col2im_lds_kernel<float, KH, KW>), grid, dim3(256), lds, s, g, plan, (const float *)dDhat, ld, \
                               (float *)dX);                                                                                   \
    } while (0)
        if (unit && g.kh == 3 && g.kw == 3) OMNI_COL2IM_CASE(3, 3);
        else if (unit && g.kh == 5 && g.kw == 5) OMNI_COL2IM_CASE(5, 5);
        else OMNI_COL2IM_CASE(0, 0);
#undef OMNI_COL2IM_CASE
        OMNI_LAUNCH_CHECK();
        return OMNI_OK;
    }
    // strided layers: the form whose loads are contiguous per wavefront, when the window has at most 3 x 3 taps per pixel
    const int S = g.sh;
    if (g.sh == g.sw && (S == 2 || S == 4) && (g.kh + S - 1) / S <= 3 && (g.kw + S - 1) / S <= 3) {
        const int64_t bw = (g.W + S - 1) / S, rows = (int64_t)g.H * bw;
        const int64_t per_launch = (0x7fffffffll - 4096) / rows;
        const FastDiv div_rows((uint32_t)rows), div_bw((uint32_t)bw);
        for (int64_t p0 = 0; p0 < planes; p0 += per_launch) {
            const int64_t np = planes - p0 < per_launch ? planes - p0 : per_launch;
            const uint32_t count = (uint32_t)(np * rows);
            dim3 grid((count + 255u) / 256u);
#define OMNI_COL2IM_STRIDED(T_, S_)                                                                                       \
    hipLaunchKernelGGL((col2im_strided_kernel<T_, S_, 3, 3>), grid, dim3(256), 0, s, g, (const T_ *)dDhat, ld, (T_ *)dX,   \
                       (uint32_t)p0, count, div_rows, div_bw)
            if (dtype == OMNI_BF16 && S == 4) OMNI_COL2IM_STRIDED(bf16_t, 4);
            else if (dtype == OMNI_BF16) OMNI_COL2IM_STRIDED(bf16_t, 2);
            else if (S == 4) OMNI_COL2IM_STRIDED(float, 4);
            else OMNI_COL2IM_STRIDED(float, 2);
#undef OMNI_COL2IM_STRIDED
            OMNI_LAUNCH_CHECK();
        }
        return OMNI_OK;
    }
    int64_t planes_per_launch = (0x7fffffffll - 4096) / hw;
    for (int64_t p0 = 0; p0 < planes; p0 += planes_per_launch) {
        int64_t np = planes - p0 < planes_per_launch ? planes - p0 : planes_per_launch;
        uint32_t count = (uint32_t)(np * hw);
        dim3 grid((count + 255u) / 256u);
        if (dtype == OMNI_BF16)
            hipLaunchKernelGGL(col2im_kernel<bf16_t>, grid, dim3(256), 0, s, g, (const bf16_t *)dDhat, ld, (bf16_t *)dX, (uint32_t)p0, count);
        else
            hipLaunchKernelGGL(col2im_kernel<float>, grid, dim3(256), 0, s, g, (const float *)dDhat, ld, (float *)dX, (uint32_t)p0, count);
        OMNI_LAUNCH_CHECK();
    }
    return OMNI_OK;
}

// ------------------------------------------------------------------------------------------------
// dY [N][F][Ho][Wo] -> dY-hat [F][ld] (the inverse of lifting), columns in [M, ld) zero.
// Each block covers PACK_COLS columns of one row f; with bias_partials != null it also leaves the
// fp32 sum of its columns in bias_partials[f][block], reduced in block order by the second kernel.
// ------------------------------------------------------------------------------------------------
constexpr int PACK_VEC = 8;
constexpr int PACK_UNR = 4;                          // packs per thread
constexpr int PACK_COLS = 256 * PACK_VEC * PACK_UNR;  // columns per workgroup

template <typename T, typename U>
__device__ __forceinline__ void pack_dyhat_body(const ConvGeom &g, const T *__restrict__ dY, U *__restrict__ out, int64_t ld,
                                                float *__restrict__ bias_partials, int block, int blocks, int f)
{
    // PACK_UNR packs per thread, 256 packs apart.  Their loads are issued together and unconditionally: a
    // pack that cannot be read with one load (it straddles two images or the end of the matrix) reads the
    // first bytes of dY instead and is then assembled element by element.
    const bool can_vec = (int64_t)g.N * g.F * g.HoWo >= PACK_VEC;
    float sum = 0.f;
    int64_t m0[PACK_UNR];
    uint32_t n[PACK_UNR], r[PACK_UNR];
    bool fast[PACK_UNR];
    VecOf<U, PACK_VEC> o[PACK_UNR];
#pragma unroll
    for (int u = 0; u < PACK_UNR; ++u) {
        m0[u] = (((int64_t)block * PACK_UNR + u) * 256 + threadIdx.x) * PACK_VEC;
        g.div_HoWo.divmod(m0[u] < g.M ? (uint32_t)m0[u] : 0u, n[u], r[u]);
        fast[u] = can_vec && m0[u] + PACK_VEC <= g.M && r[u] + PACK_VEC <= (uint32_t)g.HoWo;
        const T *src = fast[u] ? dY + ((int64_t)n[u] * g.F + f) * g.HoWo + r[u] : dY;
        if (can_vec) __builtin_memcpy(&o[u], src, sizeof(o[u]));
    }
#pragma unroll
    for (int u = 0; u < PACK_UNR; ++u) {
        if (m0[u] >= ld) continue;
        if (fast[u]) {
#pragma unroll
            for (int e = 0; e < PACK_VEC; ++e) {
                T v;
                __builtin_memcpy(&v, &o[u].v[e], sizeof(T));
                sum += Elem<T>::to_f32(v);
            }
        } else {
            uint32_t nn = n[u], rr = r[u];
#pragma unroll
            for (int e = 0; e < PACK_VEC; ++e) {
                U bits = 0;
                if (m0[u] + e < g.M) {
                    const T *src = dY + ((int64_t)nn * g.F + f) * g.HoWo + rr;
                    bits = *reinterpret_cast<const U *>(src);
                    sum += Elem<T>::to_f32(*src);
                }
                o[u].v[e] = bits;
                if (++rr == (uint32_t)g.HoWo) {
                    rr = 0;
                    ++nn;
                }
            }
        }
        // 8 x 4 bytes does not fit one 16-byte store: write two halves for fp32
        if constexpr (sizeof(U) == 2) {
            *reinterpret_cast<VecOf<U, 8> *>(out + (int64_t)f * ld + m0[u]) = o[u];
        } else {
            VecOf<U, 4> a, b;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a.v[e] = o[u].v[e];
                b.v[e] = o[u].v[4 + e];
            }
            *reinterpret_cast<VecOf<U, 4> *>(out + (int64_t)f * ld + m0[u]) = a;
            *reinterpret_cast<VecOf<U, 4> *>(out + (int64_t)f * ld + m0[u] + 4) = b;
        }
    }
    if (bias_partials != nullptr) {
        // fixed-shape tree: lanes, then the four wavefronts in order
        __shared__ float wave_sum[4];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
        if ((threadIdx.x & 63) == 0) wave_sum[threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0)
            bias_partials[(int64_t)f * blocks + block] = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
    }
}

// khat.out != null: workgroups beyond the filters (blockIdx.y >= F) pack the model (transposed, for the data gradient)
template <typename T, typename U>
__global__ __launch_bounds__(256) void pack_dyhat_kernel(ConvGeom g, const T *__restrict__ dY, U *__restrict__ out, int64_t ld,
                                                         float *__restrict__ bias_partials, KhatJob<U> khat)
{
    if ((int)blockIdx.y < g.F)
        pack_dyhat_body<T, U>(g, dY, out, ld, bias_partials, blockIdx.x, gridDim.x, blockIdx.y);
    else
        khat_body(khat, (int64_t)(blockIdx.y - g.F) * gridDim.x + blockIdx.x);
}

// The model gradient's two preparations in one launch: lowering of X and packing of dY
template <typename T, typename U, int VEC, int KW>
__global__ __launch_bounds__(256) void lower_dyhat_kernel(ConvGeom g, LowerPlan p, const U *__restrict__ X, U *__restrict__ D,
                                                          const T *__restrict__ dY, U *__restrict__ out, int64_t ld,
                                                          float *__restrict__ bias_partials, int blocks)
{
    if ((int)blockIdx.y < g.C) {
        lower_body<U, VEC, KW>(g, p, X, D, ld, blockIdx.x, blockIdx.y, blockIdx.z);
    } else {
        const int64_t b = ((int64_t)(blockIdx.y - g.C) * gridDim.z + blockIdx.z) * gridDim.x + blockIdx.x;
        const int f = (int)(b / blocks);
        if (f < g.F) pack_dyhat_body<T, U>(g, dY, out, ld, bias_partials, (int)(b - (int64_t)f * blocks), blocks, f);
    }
}

template <typename T, typename U, int KW>
__global__ __launch_bounds__(256) void lower_flat_dyhat_kernel(ConvGeom g, FlatPlan p, const U *__restrict__ X, U *__restrict__ D,
                                                               const T *__restrict__ dY, U *__restrict__ out, int64_t ld,
                                                               float *__restrict__ bias_partials, int blocks)
{
    const unsigned packing = gridDim.x - p.blocks;
    if (blockIdx.x < packing) {
        const int f = (int)(blockIdx.x / (unsigned)blocks);
        if (f < g.F) pack_dyhat_body<T, U>(g, dY, out, ld, bias_partials, (int)(blockIdx.x - (unsigned)f * (unsigned)blocks), blocks, f);
    } else {
        lower_flat_block<U, KW>(g, p, X, D, ld, blockIdx.x - packing);
    }
}

__global__ __launch_bounds__(64) void bias_reduce_kernel(const float *__restrict__ partials, int blocks, float *__restrict__ dbias)
{
    // one wavefront per filter: strided partial sums per lane (fixed order), then a fixed tree
    int f = blockIdx.x;
    float acc = 0.f;
    for (int b = threadIdx.x; b < blocks; b += 64) acc += partials[(int64_t)f * blocks + b];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if (threadIdx.x == 0) dbias[f] = acc;
}

static int run_bias_reduce(const ConvGeom &g, const float *bias_partials, int blocks, float *dbias, hipStream_t s)
{
    ProfScope prof(KID_BIAS_REDUCE, s, 0.0, 4.0 * g.F * (blocks + 1));
    hipLaunchKernelGGL(bias_reduce_kernel, dim3((unsigned)g.F), dim3(64), 0, s, bias_partials, blocks, dbias);
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

// The same matrix with every output row padded with zeros to a multiple of 8 columns:
// column ((n*Ho + oy) * P8 + i) * 8 + e holds dY[n][f][oy][8i + e], P8 = ceil(Wo / 8).  A pack of 8 columns
// then never leaves its output row, which is what lets the model-gradient product read the matching
// entries of D-hat straight from X with one load per pack.  One thread per pack; bias partial sums as above.
__global__ __launch_bounds__(256) void pack_dyhat_rows_kernel(ConvGeom g, FastDiv div_p8, FastDiv div_Ho,
                                                              const bf16_t *__restrict__ dY, uint16_t *__restrict__ out,
                                                              int64_t ld, float *__restrict__ bias_partials)
{
    const int f = blockIdx.y;
    const bool can_vec = (int64_t)g.N * g.F * g.Ho * g.Wo >= 8;
    float sum = 0.f;
    int64_t pack[PACK_UNR];
    uint32_t i[PACK_UNR];
    const bf16_t *src[PACK_UNR];
    bool live[PACK_UNR], fast[PACK_UNR];
    int back[PACK_UNR];
    VecOf<uint16_t, 8> o[PACK_UNR];
#pragma unroll
    for (int u = 0; u < PACK_UNR; ++u) {
        pack[u] = ((int64_t)blockIdx.x * PACK_UNR + u) * 256 + threadIdx.x;
        uint32_t row, n, oy;
        div_p8.divmod((uint32_t)(pack[u] * 8 < ld ? pack[u] : 0), row, i[u]);
        div_Ho.divmod(row, n, oy);
        live[u] = pack[u] * 8 < ld && (int)n < g.N;
        src[u] = dY + (((int64_t)(live[u] ? n : 0) * g.F + f) * g.Ho + oy) * g.Wo + 8 * i[u];
        // a row's ragged last pack is read so that the 16 bytes END at the row's end (inside the tensor) and
        // shifted down afterwards, which zeroes its padding
        const int valid = g.Wo - 8 * (int)i[u];
        back[u] = valid < 8 ? 8 - valid : 0;
        fast[u] = can_vec && live[u] && (back[u] == 0 || g.Wo >= 8);
        if (can_vec) __builtin_memcpy(&o[u], fast[u] ? src[u] - back[u] : dY, 16);  // element-aligned 16-byte loads, issued together
    }
#pragma unroll
    for (int u = 0; u < PACK_UNR; ++u) {
        if (pack[u] * 8 >= ld) continue;
        if (fast[u]) {
            if (back[u]) {
                unsigned __int128 x;
                __builtin_memcpy(&x, &o[u], 16);
                x >>= 16 * back[u];
                __builtin_memcpy(&o[u], &x, 16);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) sum += bf16_to_f32(o[u].v[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                uint16_t bits = 0;
                if (live[u] && 8 * (int)i[u] + e < g.Wo) {
                    bits = src[u][e];
                    sum += bf16_to_f32(bits);
                }
                o[u].v[e] = bits;
            }
        }
        *reinterpret_cast<VecOf<uint16_t, 8> *>(out + (int64_t)f * ld + pack[u] * 8) = o[u];
    }
    if (bias_partials != nullptr) {
        __shared__ float wave_sum[4];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
        if ((threadIdx.x & 63) == 0) wave_sum[threadIdx.x >> 6] = sum;
        __syncthreads();
        if (threadIdx.x == 0)
            bias_partials[(int64_t)f * gridDim.x + blockIdx.x] = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
    }
}

// The padded unit is the output row, or the whole plane of an image where the direct model gradient
// works on planes: a plane is then handled as one long row.
static ConvGeom padded_unit_view(const ConvGeom &g)
{
    ConvGeom v = g;
    if (wgrad_direct_planes(g)) v.Wo = g.Ho * g.Wo, v.Ho = 1;
    return v;
}

int64_t dyhat_rows_ld(const ConvGeom &g)
{
    ConvGeom v = padded_unit_view(g);
    return round_up((int64_t)v.N * v.Ho * ((v.Wo + 7) / 8) * 8, 64);
}
int pack_dyhat_rows_blocks(const ConvGeom &g) { return (int)((dyhat_rows_ld(g) + PACK_COLS - 1) / PACK_COLS); }

int launch_pack_dyhat_rows(const ConvGeom &geom, const void *dY, void *dYhat, int64_t ld, float *bias_partials,
                           int bias_blocks, float *dbias, hipStream_t s)
{
    const ConvGeom g = padded_unit_view(geom);
    int blocks = (int)((ld + PACK_COLS - 1) / PACK_COLS);
    if (bias_partials != nullptr && bias_blocks != blocks) return OMNI_INVALID_ARGUMENT;
    dim3 grid((unsigned)blocks, (unsigned)g.F, 1);
    {
        ProfScope prof(KID_PACK_DYHAT, s, 0.0, 2.0 * g.F * (double)g.M * 2.0);
        hipLaunchKernelGGL(pack_dyhat_rows_kernel, grid, dim3(256), 0, s, g, FastDiv((uint32_t)((g.Wo + 7) / 8)),
                           FastDiv((uint32_t)g.Ho), (const bf16_t *)dY, (uint16_t *)dYhat, ld, bias_partials);
    }
    OMNI_LAUNCH_CHECK();
    return bias_partials != nullptr && dbias != nullptr ? run_bias_reduce(g, bias_partials, blocks, dbias, s) : OMNI_OK;
}

int pack_dyhat_blocks(const ConvGeom &g) { return (int)((dhat_ld(g) + PACK_COLS - 1) / PACK_COLS); }

template <typename T, typename U>
static int run_pack_dyhat(const ConvGeom &g, const void *dY, void *dYhat, int64_t ld, float *bias_partials, int blocks, float *dbias,
                          const void *W, void *KhatT, int64_t Kp, int64_t Fp, hipStream_t s)
{
    KhatJob<U> khat{(const U *)W, (U *)KhatT, g.F, g.K, Kp, Fp, 1};
    const double bytes = 2.0 * g.F * (double)g.M * sizeof(U);
    if (g.HoWo == 1 && (blocks == 1 || bias_partials == nullptr)) {
        // one output position per image: dY [N][F] transposed; one workgroup sees all images, so its sums are the
        // bias gradient already
        if (KhatT != nullptr) run_khat(khat, s);
        ProfScope prof(KID_PACK_DYHAT, s, 0.0, bytes);
        run_transpose<T, U, true>(dY, g.N, g.F, dYhat, ld, bias_partials, dbias, s);
        OMNI_LAUNCH_CHECK();
        return OMNI_OK;
    }
    const int64_t extra = KhatT != nullptr ? (khat.blocks() + blocks - 1) / blocks : 0;
    const bool ride = g.F + extra <= 65535;
    if (!ride) {
        run_khat(khat, s);
        khat.out = nullptr;
    }
    {
        ProfScope prof(KID_PACK_DYHAT, s, 0.0, bytes + khat.bytes());
        hipLaunchKernelGGL((pack_dyhat_kernel<T, U>), dim3((unsigned)blocks, (unsigned)(g.F + (ride ? extra : 0)), 1), dim3(256), 0, s, g,
                           (const T *)dY, (U *)dYhat, ld, bias_partials, khat);
    }
    OMNI_LAUNCH_CHECK();
    return bias_partials != nullptr && dbias != nullptr ? run_bias_reduce(g, bias_partials, blocks, dbias, s) : OMNI_OK;
}

int launch_pack_dyhat(const ConvGeom &g, int dtype, const void *dY, void *dYhat, int64_t ld, float *bias_partials,
                      int bias_blocks, float *dbias, hipStream_t s, const void *W, void *KhatT, int64_t Kp, int64_t Fp)
{
    int blocks = (int)((ld + PACK_COLS - 1) / PACK_COLS);
    if (bias_partials != nullptr && bias_blocks != blocks) return OMNI_INVALID_ARGUMENT;
    return dtype == OMNI_BF16 ? run_pack_dyhat<bf16_t, uint16_t>(g, dY, dYhat, ld, bias_partials, blocks, dbias, W, KhatT, Kp, Fp, s)
                              : run_pack_dyhat<float, uint32_t>(g, dY, dYhat, ld, bias_partials, blocks, dbias, W, KhatT, Kp, Fp, s);
}

template <typename T, typename U>
static int run_lower_dyhat(const ConvGeom &g, int dtype, const void *X, void *Dhat, const void *dY, void *dYhat, int64_t ld,
                           float *bias_partials, int blocks, float *dbias, hipStream_t s)
{
    constexpr int VEC = 16 / sizeof(U);
    LowerPlan plan;
    FlatPlan flat;
    size_t lds = 0;
    const int64_t packing = (int64_t)blocks * g.F;
    const bool is_flat = g.HoWo != 1 && make_flat_plan(g, sizeof(U), ld, packing, &flat);
    const bool together = is_flat || (g.HoWo != 1 && ld % VEC == 0 && make_lower_plan(g, sizeof(U), &plan, &lds));
    const unsigned gx = !together || is_flat ? 1u : (unsigned)(plan.bands * plan.groups);
    const unsigned gz = !together || is_flat ? 1u : (unsigned)((g.kh + plan.ky_per - 1) / plan.ky_per);
    const int64_t extra = is_flat ? 0 : (packing + (int64_t)gx * gz - 1) / ((int64_t)gx * gz);
    if (!together || (!is_flat && g.C + extra > 65535)) {
        // (dY first: it is usually fresh in the last-level cache, which D-hat would flush)
        int st = launch_pack_dyhat(g, dtype, dY, dYhat, ld, bias_partials, blocks, dbias, s);
        return st != OMNI_OK ? st : launch_lower(g, dtype, X, Dhat, ld, s);
    }
    ProfScope prof(KID_LOWER, s, 0.0, ((double)g.N * g.C * g.H * g.W + (double)g.K * g.M + 2.0 * g.F * (double)g.M) * sizeof(U));
    if (is_flat) {
        const dim3 grid(flat.blocks + packing_blocks(packing));
#define OMNI_CASE(KWT)                                                                                                           \
    hipLaunchKernelGGL((lower_flat_dyhat_kernel<T, U, KWT>), grid, dim3(256), flat.lds, s, g, flat, (const U *)X, (U *)Dhat,            \
                       (const T *)dY, (U *)dYhat, ld, bias_partials, blocks)
        if (g.kw == 1) OMNI_CASE(1);
        else if (g.kw == 3) OMNI_CASE(3);
        else OMNI_CASE(5);
#undef OMNI_CASE
    } else {
        const dim3 grid(gx, (unsigned)(g.C + extra), gz);
#define OMNI_CASE(KWT)                                                                                                           \
    hipLaunchKernelGGL((lower_dyhat_kernel<T, U, VEC, KWT>), grid, dim3(256), lds, s, g, plan, (const U *)X, (U *)Dhat,           \
                       (const T *)dY, (U *)dYhat, ld, bias_partials, blocks)
        if (g.kw == 3) OMNI_CASE(3);
        else if (g.kw == 5) OMNI_CASE(5);
        else if (g.kw == 11) OMNI_CASE(11);
        else OMNI_CASE(0);
#undef OMNI_CASE
    }
    OMNI_LAUNCH_CHECK();
    return bias_partials != nullptr && dbias != nullptr ? run_bias_reduce(g, bias_partials, blocks, dbias, s) : OMNI_OK;
}

int launch_lower_dyhat(const ConvGeom &g, int dtype, const void *X, void *Dhat, const void *dY, void *dYhat, int64_t ld,
                       float *bias_partials, int bias_blocks, float *dbias, hipStream_t s)
{
    int blocks = (int)((ld + PACK_COLS - 1) / PACK_COLS);
    if (bias_partials != nullptr && bias_blocks != blocks) return OMNI_INVALID_ARGUMENT;
    return dtype == OMNI_BF16 ? run_lower_dyhat<bf16_t, uint16_t>(g, dtype, X, Dhat, dY, dYhat, ld, bias_partials, blocks, dbias, s)
                              : run_lower_dyhat<float, uint32_t>(g, dtype, X, Dhat, dY, dYhat, ld, bias_partials, blocks, dbias, s);
}

}  // namespace omni
