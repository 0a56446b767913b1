// The stem layer of a quaternion network on gfx950: the Poincare mapping of
// RGB pixels to quaternions (Section III-A, eq. 4) feeding the first
// quaternion convolution (Section III-B, eqs. 5/6), whose one input channel
// makes it a short contraction: K = 4 components x k_h*k_w taps (36 for a
// 3x3 stem) against a few dozen output reals per pixel.  The implicit-GEMM
// kernel would stage 16 input channels per step with 15 of them zero; this
// kernel builds each MFMA's K = 16 slice (two taps x four components) of
// one output pixel per lane from the colour planes, with the map of eq. 4
// evaluated in fp32 and rounded once to bf16.  The layer is bound by writing
// its output (4 * c_out reals per pixel against 3 inputs).
//
// A work-group takes bands of consecutive output rows of one image.  It maps
// the band's input rows once per pixel into LDS (8 bytes a quaternion, zeros
// outside the image), where every tap of every output pixel then finds them:
// the map costs a load of three planes and a division per input pixel, which
// per tap was 2.25 (stride 2) to 9 times as much.  A band whose input rows do
// not fit (wide or strongly dilated layers) maps per tap from memory.
//
// Per wave: 32 consecutive output pixels at a time, D = W^T X^T with
//   A (32 output reals x 16 k): the signed Hamilton block weight of eq. 6,
//       row r = p * c_out + c (component p, channel c), k = 4 * tap + q,
//       entry sign(p, q) * W_{p xor q}[c][tap]; built once per work-group in
//       LDS as NBLK blocks of 32 rows x KM slices of 16 k (one 1 KB MFMA
//       fragment each);
//   B (16 k x 32 pixels): lane l holds pixel l % 32, k = 16m + 8(l/32) + e,
//       i.e. taps 4m + 2(l/32) and 4m + 2(l/32) + 1, all four components;
//   D: lane l holds rows 8j + 4(l/32) + i (i, j < 4) of its pixel.  The wave
//       parks 64 of them at a time in LDS (rows padded by 8 bytes, so the 32
//       pixels' 8-byte pieces fall on different banks) and stores 16 bytes a
//       lane, whole lines, where 8-byte stores from D touched 32 lines each.
// 64 x 224 x 224 RGB, 3x3 stride 2 to 16 channels: 53.6 -> 32.0 us (122 MB; a
// device copy of as much takes 24).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gfx950_dma.h"
#include "quan_launch.h"

namespace quan {
namespace {

typedef __bf16 stem_bf16x8 __attribute__((ext_vector_type(8)));
typedef float stem_f32x16 __attribute__((ext_vector_type(16)));

constexpr int kStemThreads = 256;
constexpr int kStemWaves = kStemThreads / 64;
constexpr int kStemMaxFrags = 32;  // NBLK x KM weight fragments held in LDS (1 KB each)
constexpr int kStemMaxBand = 32;   // output rows of a band at most
// LDS of a work-group: three fit a compute unit (160 KB), and no launch needs
// more than the 64 KB that a kernel gets without asking.
constexpr size_t kStemLds = 52 * 1024, kStemMaxLds = 64 * 1024;

struct StemArgs {
    const __bf16 *rgb;   // [n][3][h][w]
    const __bf16 *wpack; // packed weights: W_m[o][tap] at ((tap * 4 + m) * cout_pad + o) * pk
    const __bf16 *bias;  // [4][c_out] or NULL
    __bf16 *out;         // [n][h_out][w_out][4][c_out]
    int h, w, c_out, k_h, k_w, s_h, s_w, p_h, p_w, d_h, d_w, h_out, w_out;
    int cout_pad, pk;
    int km;              // K slices of 16: ceil(taps / 4)
    int band;            // output rows of a band
    int img_bands;       // bands per image
    int bands;           // of all images
    int patch_w;         // staged columns: input columns -p_w .. patch_w - p_w - 1
    int patch;           // staged pixels of a band (the zero pixel follows); 0: not staged
    FastDiv by_c_out, by_w_out, by_patch_w, by_last;  // by_last: pieces of the last parked slice of a pixel
};

// The quaternion of an RGB pixel (eq. 4) in bf16.
__device__ __forceinline__ uint2 stem_quaternion(const __bf16 *px, int hw)
{
    const float r = float(px[0]), g = float(px[hw]), bl = float(px[2 * hw]);
    const float n2 = r * r + g * g + bl * bl;
    const float inv = 1.0f / (1.0f + n2);
    const __bf16 q[4] = {__bf16((1.0f - n2) * inv), __bf16((2.0f * r) * inv), __bf16((2.0f * g) * inv),
                         __bf16((2.0f * bl) * inv)};
    uint2 v;
    __builtin_memcpy(&v, q, 8);
    return v;
}

// Bytes of one parked pixel (a slice of up to two blocks of 32 reals), and of
// a work-group's LDS.
__host__ __device__ constexpr int stem_park_row(int nblk)
{
    return 64 * (nblk < 2 ? nblk : 2) + 8;
}
__host__ __device__ constexpr size_t stem_lds_bytes(int nblk, int km, int patch)
{
    return size_t(nblk) * km * 1024 + size_t(32) * nblk * 4 + size_t(kStemWaves) * 32 * stem_park_row(nblk) +
           size_t(4 * km) * 4 + (patch > 0 ? (size_t(patch) + 1) * 8 : 0);
}
static_assert(stem_lds_bytes(8, kStemMaxFrags / 8, 0) <= kStemLds && stem_lds_bytes(1, kStemMaxFrags, 0) <= kStemLds,
              "every kernel fits without a patch");

template <int NBLK, bool STAGED>
__global__ __launch_bounds__(kStemThreads) void qconv2d_stem(StemArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    // A fragments of the signed block weight, fragment (b, m) for lane l:
    // rows 32b + l%32, k = 16m + 8(l/32) .. +7; the bias of every row; the
    // waves' parked output; each tap's offset in the patch; the patch
    stem_bf16x8(*const wtab)[64] = reinterpret_cast<stem_bf16x8(*)[64]>(lds);
    float *const btab = reinterpret_cast<float *>(lds + size_t(NBLK) * a.km * 1024);
    unsigned char *const parks = reinterpret_cast<unsigned char *>(btab + 32 * NBLK);
    constexpr int prow = stem_park_row(NBLK);
    uint2 *const patch = reinterpret_cast<uint2 *>(parks + kStemWaves * 32 * prow);
    int *const taps_at = reinterpret_cast<int *>(patch + (STAGED ? a.patch + 1 : 0));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, l32 = lane & 31;
    const int taps = a.k_h * a.k_w;
    const int rows = 4 * a.c_out;
    static_assert(32 * NBLK <= kStemThreads, "one row's bias per thread");
    float bias = 0.0f;
    if (a.bias != nullptr && int(threadIdx.x) < rows)
        bias = float(a.bias[threadIdx.x]);
    // The kernels' own values first, four loads in flight per thread, where the
    // parked output will lie: every work-group reads the same few lines (two
    // bytes of each 32), and a table built straight from memory read each value
    // sixteen times.
    __bf16 *const vals = reinterpret_cast<__bf16 *>(parks);
    const int n_vals = 4 * taps * a.c_out;
    static_assert(4 * (4 * kStemMaxFrags / NBLK) * 8 * NBLK * 2 <= kStemWaves * 32 * prow, "the values fit the parks");
    for (int i = threadIdx.x; i < n_vals; i += 4 * kStemThreads) {
        __bf16 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int at = i + u * kStemThreads < n_vals ? i + u * kStemThreads : i;
            const int tm = fast_div(at, a.by_c_out);
            v[u] = a.wpack[(size_t(tm) * a.cout_pad + (at - tm * a.c_out)) * a.pk];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * kStemThreads < n_vals)
                vals[i + u * kStemThreads] = v[u];
    }
    if (threadIdx.x < 32 * NBLK)
        btab[threadIdx.x] = bias;
    __syncthreads();
    for (int idx = threadIdx.x; idx < NBLK * a.km * 64; idx += kStemThreads) {
        const int fl = idx & 63, fm = (idx >> 6) % a.km, fb = (idx >> 6) / a.km;
        const int r = 32 * fb + (fl & 31);
        const int p = r < rows ? fast_div(r, a.by_c_out) : 0, c = r < rows ? r - p * a.c_out : 0;
        stem_bf16x8 f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = 16 * fm + 8 * (fl >> 5) + e, tap = k >> 2, q = k & 3;
            float v = 0.0f;
            if (r < rows && tap < taps) {
                v = float(vals[(tap * 4 + (p ^ q)) * a.c_out + c]);
                if ((kHamiltonNeg >> (4 * p + q)) & 1u)
                    v = -v;
            }
            f[e] = __bf16(v);
        }
        wtab[fb * a.km + fm][fl] = f;
    }
    if constexpr (STAGED) {
        // taps past the kernel (zero weights) read the zero pixel; -1 marks
        // them, as their address does not move with the output pixel
        for (int t = threadIdx.x; t < 4 * a.km; t += kStemThreads)
            taps_at[t] = t < taps ? t / a.k_w * a.d_h * a.patch_w + t % a.k_w * a.d_w : -1;
        if (threadIdx.x == 0)
            patch[a.patch] = uint2{0u, 0u};
    }

    const int hw = a.h * a.w;
    unsigned char *const park = parks + wave * 32 * prow;
    for (int bd = blockIdx.x; bd < a.bands; bd += gridDim.x) {
        const int img = bd / a.img_bands, y0 = (bd - img * a.img_bands) * a.band;
        const int nrows = a.h_out - y0 < a.band ? a.h_out - y0 : a.band;
        const __bf16 *plane = a.rgb + size_t(img) * 3 * hw;
        const int iy0 = y0 * a.s_h - a.p_h;
        if constexpr (STAGED) {
            __syncthreads();  // the previous band's patch is read
            const int need = ((nrows - 1) * a.s_h + (a.k_h - 1) * a.d_h + 1) * a.patch_w;
            // four pixels' loads in flight per thread
            for (int i = threadIdx.x; i < need; i += 4 * kStemThreads) {
                const __bf16 *px[4];
                bool in[4];
                uint2 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = i + u * kStemThreads;
                    const int yy = fast_div(j, a.by_patch_w);
                    const int iy = iy0 + yy, ix = j - yy * a.patch_w - a.p_w;
                    in[u] = j < need && (unsigned)iy < (unsigned)a.h && (unsigned)ix < (unsigned)a.w;
                    px[u] = plane + (in[u] ? iy * a.w + ix : 0);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    v[u] = stem_quaternion(px[u], hw);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (i + u * kStemThreads < need)
                        patch[i + u * kStemThreads] = in[u] ? v[u] : uint2{0u, 0u};
            }
        }
        __syncthreads();
        const int pixels = nrows * a.w_out;
        __bf16 *const oband = a.out + (size_t(img) * a.h_out + y0) * a.w_out * rows;
        for (int p0 = 32 * wave; p0 < pixels; p0 += 32 * kStemWaves) {
            const int n_live = pixels - p0 < 32 ? pixels - p0 : 32;
            // (pixels past the band repeat its last one and are not stored)
            const int pix = p0 + (l32 < n_live ? l32 : n_live - 1);
            const int oy = fast_div(pix, a.by_w_out), ox = pix - oy * a.w_out;
            // accumulators start at the bias of the lane's rows 32b + 8j + 4*half + i
            stem_f32x16 acc[NBLK];
#pragma unroll
            for (int b = 0; b < NBLK; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    acc[b][i] = btab[32 * b + 8 * (i >> 2) + 4 * half + (i & 3)];
            const int at = oy * a.s_h * a.patch_w + ox * a.s_w;
            for (int m = 0; m < a.km; ++m) {
                // the pixel's quaternions at taps 4m + 2*half and 4m + 2*half + 1
                uint2 q[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int tap = 4 * m + 2 * half + u;
                    if constexpr (STAGED) {
                        const int t = taps_at[tap];
                        q[u] = patch[t >= 0 ? at + t : a.patch];
                    } else {
                        q[u] = uint2{0u, 0u};
                        const int ky = tap / a.k_w, kx = tap - ky * a.k_w;
                        const int iy = iy0 + oy * a.s_h + ky * a.d_h, ix = ox * a.s_w - a.p_w + kx * a.d_w;
                        if (tap < taps && (unsigned)iy < (unsigned)a.h && (unsigned)ix < (unsigned)a.w)
                            q[u] = stem_quaternion(plane + iy * a.w + ix, hw);
                    }
                }
                stem_bf16x8 xq;
                __builtin_memcpy(&xq, q, 16);
#pragma unroll
                for (int b = 0; b < NBLK; ++b)
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wtab[b * a.km + m][lane], xq, acc[b], 0, 0, 0);
            }
            __bf16 *const orun = oband + size_t(p0) * rows;
            constexpr int SB = NBLK < 2 ? NBLK : 2;  // blocks of a slice
            const bool direct = (a.c_out & 1) != 0;  // 8-byte pieces only
#pragma unroll
            for (int b0 = 0; b0 < NBLK; b0 += SB) {
#pragma unroll
                for (int b = b0; b < b0 + SB; ++b)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int r0 = 32 * b + 8 * j + 4 * half;
                        if (r0 < rows) {
                            __bf16 v[4];
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                v[i] = __bf16(acc[b][4 * j + i]);
                            uint2 bits;
                            __builtin_memcpy(&bits, v, 8);
                            if (!direct)
                                *reinterpret_cast<uint2 *>(park + l32 * prow + 2 * (r0 - 32 * b0)) = bits;
                            else if (l32 < n_live)
                                *reinterpret_cast<uint2 *>(orun + l32 * rows + r0) = bits;
                        }
                    }
                const int left = rows - 32 * b0;
                if (!direct && left > 0) {
                    // (a wave's LDS accesses are in order: no barrier)
                    __builtin_amdgcn_wave_barrier();
                    const bool whole = left >= 32 * SB;
                    const int chunks = whole ? 4 * SB : left / 8;
                    for (int i = lane; i < n_live * chunks; i += 64) {
                        const int pl = whole ? i / (4 * SB) : fast_div(i, a.by_last), c = i - pl * chunks;
                        const unsigned char *src = park + pl * prow + 16 * c;
                        const uint2 lo = *reinterpret_cast<const uint2 *>(src);
                        const uint2 hi = *reinterpret_cast<const uint2 *>(src + 8);
                        *reinterpret_cast<uint4 *>(orun + pl * rows + 32 * b0 + 8 * c) =
                            uint4{lo.x, lo.y, hi.x, hi.y};
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
    }
}

template <int NBLK>
hipError_t launch_stem(StemArgs a, int64_t n, hipStream_t stream)
{
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int64_t span_h = int64_t(a.k_h - 1) * a.d_h + 1, span_w = int64_t(a.k_w - 1) * a.d_w + 1;
    const int64_t cols = int64_t(a.w_out - 1) * a.s_w + span_w;
    auto patch_of = [&](int band) { return (int64_t(band - 1) * a.s_h + span_h) * cols; };
    a.band = 1;
    const size_t fixed = stem_lds_bytes(NBLK, a.km, 0);
    auto fits = [&](int band, size_t lds) {
        const int64_t px = patch_of(band);
        return px < int64_t(lds / 8) && fixed + size_t(px + 1) * 8 <= lds;
    };
    const bool staged = fits(1, kStemMaxLds);
    // The band: even parts of an image that take the least time by a model: a
    // work-group alone needs 1 us per round of its four waves' pixels and a
    // band's staging (0.5 + 0.4 per round of loads), those of a compute unit
    // share its stores, and each builds the table.  A row of a narrow image
    // fills few of the four waves' lanes, and a work-group a row leaves its
    // table's cost to few pixels: in bands of one row, rows of 14 to 86 pixels
    // and 36 or 64 channels took up to 2.9 times as long as pixels dealt without
    // regard to rows (64 x 37 x 37, 1x1 stride 2 to 64: 10.1 us so, 29.6, now
    // 10.2).  One image of wide rows is left 0.3 to 2.4 us slower than that: a row
    // of 138 pixels is two rounds, the second nearly empty.
    auto rounds_of = [&](int64_t rows) { return (rows * a.w_out + 32 * kStemWaves - 1) / (32 * kStemWaves); };
    double best = 0.0, costs[kStemMaxBand + 1] = {};
    int64_t caps[kStemMaxBand + 1] = {};  // work-groups
    for (int band = 1; band <= a.h_out && band <= kStemMaxBand; ++band) {
        const int parts = (a.h_out + band - 1) / band;
        if ((a.h_out + parts - 1) / parts != band)
            continue;  // (not even)
        if (band > 1 && staged && !fits(band, kStemMaxLds))
            break;
        // (two resident work-groups by registers or LDS, else three)
        const int64_t slots = int64_t(NBLK == 8 || (staged && !fits(band, kStemLds)) ? 2 : 3) * cus;
        const int64_t bands = n * parts, wgs = std::min(bands, slots);
        const double stage = staged ? 0.5 + 0.4 * double((patch_of(band) + 1023) / 1024) : 0.2;
        const double alone = stage + double(rounds_of(band));
        const double shared = (slots < 3 * cus ? 1.15 : 1.0) * (0.35 * NBLK * double(rounds_of(band)) + 0.4 * stage);
        // one band each of `groups` work-groups
        auto turn = [&](int64_t groups) { return std::max(alone, double((groups + cus - 1) / cus) * shared); };
        const double cost = double(bands / wgs) * turn(wgs) + (bands % wgs ? turn(bands % wgs) : 0.0) +
                            0.1 * NBLK * a.km * std::max(1.0, double(wgs) / cus);
        costs[band] = cost;
        caps[band] = slots;
        best = band == 1 ? cost : std::min(best, cost);
    }
    // (the least band within 4 %: more bands even out better)
    while (costs[a.band] == 0.0 || costs[a.band] > 1.04 * best)
        ++a.band;
    const int64_t cap = caps[a.band];
    a.img_bands = (a.h_out + a.band - 1) / a.band;
    a.bands = int(n * a.img_bands);
    a.patch_w = staged ? int(cols) : 1;
    a.patch = staged ? int(patch_of(a.band)) : 0;
    a.by_c_out = FastDiv(a.c_out);
    a.by_w_out = FastDiv(a.w_out);
    a.by_patch_w = FastDiv(a.patch_w);
    const int last = 4 * a.c_out % (NBLK < 2 ? 32 : 64) / 8;
    a.by_last = FastDiv(last > 0 ? last : 1);
    const size_t lds = stem_lds_bytes(NBLK, a.km, a.patch);
    const dim3 wgs(unsigned(a.bands < cap ? a.bands : cap));
    if (staged)
        hipLaunchKernelGGL((qconv2d_stem<NBLK, true>), wgs, dim3(kStemThreads), lds, stream, a);
    else
        hipLaunchKernelGGL((qconv2d_stem<NBLK, false>), wgs, dim3(kStemThreads), lds, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t qconv2d_stem_run(const PackGeom &pg, const ConvGeom &g, DType dt, const void *rgb, const void *wpack,
                            const void *bias, void *out, hipStream_t stream)
{
    const int taps = g.k_h * g.k_w;
    const int km = (taps + 3) / 4;
    const int nblk = (4 * g.c_out + 31) / 32;
    // the kernel's block count (a power of two) sizes its weight table
    const int nblk_t = nblk <= 1 ? 1 : nblk <= 2 ? 2 : nblk <= 4 ? 4 : 8;
    if (dt != DType::BF16 || g.c_in != 1 || nblk > 8 || nblk_t * km > kStemMaxFrags)
        return hipErrorNotSupported;
    StemArgs a;
    a.rgb = static_cast<const __bf16 *>(rgb);
    a.wpack = static_cast<const __bf16 *>(wpack);
    a.bias = static_cast<const __bf16 *>(bias);
    a.out = static_cast<__bf16 *>(out);
    a.h = g.h;
    a.w = g.w;
    a.c_out = g.c_out;
    a.k_h = g.k_h;
    a.k_w = g.k_w;
    a.s_h = g.s_h;
    a.s_w = g.s_w;
    a.p_h = g.p_h;
    a.p_w = g.p_w;
    a.d_h = g.d_h;
    a.d_w = g.d_w;
    a.h_out = g.h_out;
    a.w_out = g.w_out;
    a.cout_pad = pg.cout_pad;
    a.pk = pg.pk;
    a.km = km;
    if (nblk == 1)
        return launch_stem<1>(a, g.n, stream);
    if (nblk == 2)
        return launch_stem<2>(a, g.n, stream);
    if (nblk <= 4)
        return launch_stem<4>(a, g.n, stream);
    return launch_stem<8>(a, g.n, stream);
}

}  // namespace quan
