// Weight gradients by output rows: several taps of a kernel row per
// work-group (gfx950).
//
// The gradient of one tap is G = dY^T X over the output pixels, X shifted by
// the tap.  The one-tap-per-work-group kernel (qconv2d_wgrad) stages dY and X
// anew for each tap; a layer whose channels are few then spends its time
// on staging and barriers, not on the matrix cores.  Here a work-group takes
// up to three neighbouring taps (ky, kx0..kx0+2) of one kernel row: a chunk
// of dY and the window of X that the three taps cover are staged once, and
// every dY fragment feeds the MFMAs of all three.
//
// A chunk is RH output rows x one column segment of 4*U pixels (the segment
// is the work-group's for the whole launch, so every address but the rows'
// own is fixed).  Pixels go to the MFMA's K dimension four at a time (the
// transposing LDS read takes four pixels of 16 channels), so only the last
// quad of a segment carries padding: 56, 28, 80 or 160 columns carry none.
// In LDS a pixel's staged reals are one row; tap t reads t rows further on:
// at stride and dilation 1 the taps share one window, else every pixel's taps
// are staged side by side.  A lane whose pixel lies past the segment or the
// chunk reads zero rows (never 0 * Inf).  All of a lane's row addresses are
// fixed for the launch and kept in registers, the tap an immediate offset:
// computing them per K step made the kernel VALU-bound (cifar-shaped layer,
// 128 x 32 x 32 x 16 channels: 32 us against 24).
//
// The 4*C reals of a pixel are one row of the product (dense): G holds all
// sixteen component pairs, the same useful work as adding them into four dW_m
// by component, without padding each component to a tile.  For a layer whose
// rows fit one tile the signed sum over p that makes dW_m is taken from LDS, in
// fp64, and its partials written as such.  The rows are multiples of 8 bytes (bf16) or
// 16 (fp32) whatever C is, so odd channel counts load in whole pieces too.
//
// The WK waves that share a block split the chunk's K steps and are added
// at the end in wave order; slices of the rows write partials (fp32, fp64 once
// summed over p) which the reduction adds in slice order in fp64: deterministic.
//
// Bound by staging: each tensor is read k_h times from L2, once from memory.
// A form with four components per row and four dW_m accumulators per tap
// (192 registers, one wave per SIMD) was measured at half the rate of
// qconv2d_wgrad on layers of 24 to 256 channels, every wait exposed; those
// layers stay there.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "qconv2d_wgrad.h"

namespace quan {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr unsigned kOutside = 0x80000000u;  // a byte offset past every buffer

struct RArgs {
    const void *x, *dy;
    float *part;
    int c_in, h, w, c_out;  // reals of a pixel row: 4 * C
    int k_h, k_w, s_h, s_w, p_h, p_w, d_h, d_w, h_out, w_out;
    int rows;        // output rows: n * h_out
    int segs, u4;    // column segments of u4 = 4 * U pixels
    int rh;          // output rows per chunk
    int ksteps;      // MFMA K steps per chunk (16 pixels in bf16, 2 in fp32)
    int x_pos;       // window positions per row
    int step;        // positions from one pixel to the next: 1 (shared window) or the taps of a group
    unsigned magic;  // ceil(2^20 / u4), for quotients of pixel indices
    unsigned magic_x, magic_c, magic_s;  // ceil(2^20 / x_pos), .. / q_in, .. / step
    int chunks;      // chunks of all rows
    int per_split;   // chunks of one slice
    int kx_groups, o_tiles, c_tiles;
    int groups;      // slices x segments
    unsigned x_img_bytes, x_row_bytes, dy_row_bytes;
    int fold;        // one tile: write dW_m partials
    int sep;
    int q_out, q_in; // quaternion channels
};

template <typename T>
struct Frag;
template <>
struct Frag<__bf16> {
    typedef bf16x8 type;
};
template <>
struct Frag<float> {
    typedef float type;
};

// LDS bytes from one staged pixel row to the next: bf16 rows 64 bytes apart
// modulo 256, so that the four pixels x 64 bytes of a transposing read meet
// in no bank; fp32 rows 128 apart, two pixels per read.
template <typename T>
constexpr int row_pitch(int reals)
{
    const int bytes = reals * int(sizeof(T));
    if (sizeof(T) == 2)
        return bytes + ((bytes % 256 == 64 || bytes % 256 == 192) ? 0 : 64);
    return bytes + (bytes % 256 == 128 ? 0 : 128);
}

template <typename T, int WO, int WC>
struct Geo {
    static constexpr int TO = 32 * WO, TC = 32 * WC;
    static constexpr int pitch_y = row_pitch<T>(TO), pitch_x = row_pitch<T>(TC);
    // pixels of a chunk and LDS bytes: three work-groups share a CU
    static constexpr int max_pix = 128 / (int(sizeof(T)) / 2);
    static constexpr int lds_bytes = 52 * 1024;
    static constexpr int epc = 16 / int(sizeof(T));
    static constexpr int cpr_y = TO / epc, cpr_x = TC / epc;
    // 16-byte pieces per thread and chunk
    static constexpr int items_y = (max_pix * cpr_y + kThreads - 1) / kThreads;
    static constexpr int max_pos = max_pix * 2;  // window positions of a chunk (all rows)
    static constexpr int items_x = (max_pos * cpr_x + kThreads - 1) / kThreads;
    static constexpr int items_x1 = (max_pix * 5 / 4 * cpr_x + kThreads - 1) / kThreads;  // enough for most
    static constexpr int ppk = sizeof(T) == 2 ? 16 : 2;  // pixels per K step
    static constexpr int wk = 4 / (WO * WC);
    static constexpr int max_ks = max_pix / ppk / wk;  // K steps of one wave
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
}

// v / d for 0 <= v < 2^10 and d <= 2^9 given magic = ceil(2^20 / d).
__device__ __forceinline__ int quot(int v, unsigned magic)
{
    return int(__umul24(unsigned(v), magic) >> 20);
}

// PIECE8: 16 bytes as two 8-byte loads (rows that are multiples of 8 bytes
// only, so a piece can straddle the end of the buffer).
template <bool PIECE8>
__device__ __forceinline__ u32x4 load_piece(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    if constexpr (PIECE8) {
        const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
        const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off + 8u, 0, 0));
        return u32x4{a[0], a[1], b[0], b[1]};
    } else {
        return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    }
}

// KW: taps of a work-group (at most).  WO x WC blocks of 32 x 32 of G, WK
// waves to a block.
template <typename T, int WO, int WC, int KW, bool PIECE8>
__global__ __launch_bounds__(kThreads, 2) void qconv2d_wgrad_rows(RArgs a)
{
    constexpr int WK = 4 / (WO * WC);
    static_assert(WO * WC * WK == 4, "four waves");
    static_assert(!PIECE8 || sizeof(T) == 2, "fp32 rows are whole 16-byte pieces");
    using G = Geo<T, WO, WC>;
    constexpr int ES = int(sizeof(T));
    constexpr int EPC = G::epc;
    constexpr int PPK = ES == 2 ? 16 : 2;  // pixels per K step
    typedef typename Frag<T>::type F;
    __shared__ __attribute__((aligned(16))) unsigned char lds[G::lds_bytes];
    __shared__ unsigned row_off[2][64][2];  // per chunk row: byte offset of its dY row and its X row

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // work-group b (on XCD b % 8) takes tap group and tile (b / 8) % inner of
    // group b % 8 + 8 * (b / 8 / inner): the re-reads of one slice share an L2
    const int inner = a.k_h * a.kx_groups * a.o_tiles * a.c_tiles;
    const int xs = int(blockIdx.x) >> 3;
    int in = xs % inner;
    const int grp = (int(blockIdx.x) & 7) + 8 * (xs / inner);
    if (grp >= a.groups)
        return;
    const int ct = in % a.c_tiles;
    in /= a.c_tiles;
    const int ot = in % a.o_tiles;
    in /= a.o_tiles;
    const int kx0 = (in % a.kx_groups) * KW, ky = in / a.kx_groups;
    const int kn = a.k_w - kx0 < KW ? a.k_w - kx0 : KW;
    const int seg = grp % a.segs, split = grp / a.segs;
    const int o0 = ot * G::TO, c0 = ct * G::TC;
    const int col0 = seg * a.u4;
    const int w_seg = a.w_out - col0 < a.u4 ? a.w_out - col0 : a.u4;  // real columns
    const int chunk0 = split * a.per_split;
    const int chunk1 = chunk0 + a.per_split < a.chunks ? chunk0 + a.per_split : a.chunks;
    const int row0 = chunk0 * a.rh;
    const int img0 = row0 / a.h_out;

    const int pix = a.rh * a.u4;           // pixels of a chunk
    const int pix_pad = a.ksteps * PPK;    // rounded up to whole K steps
    const int pos = a.rh * a.x_pos;        // staged X rows of a chunk
    unsigned char *const y_lds = lds;
    unsigned char *const x_lds = lds + pix_pad * G::pitch_y;
    const unsigned zero_row = unsigned(pos * G::pitch_x);  // within x_lds

    // dY from the slice's first row on, X from its first image on
    const unsigned char *const dy_s = static_cast<const unsigned char *>(a.dy) + size_t(row0) * a.dy_row_bytes;
    const unsigned char *const x_s = static_cast<const unsigned char *>(a.x) + size_t(img0) * a.x_img_bytes;
    const int row1 = chunk1 * a.rh < a.rows ? chunk1 * a.rh : a.rows;
    const unsigned dy_bytes = unsigned(row1 - row0) * a.dy_row_bytes;
    const unsigned x_bytes = unsigned((row1 - 1) / a.h_out + 1 - img0) * a.x_img_bytes;
    const __amdgpu_buffer_rsrc_t dy_r = rsrc_of(dy_s, dy_bytes);
    const __amdgpu_buffer_rsrc_t x_r = rsrc_of(x_s, x_bytes);

    // ---- staging plan: piece i of this thread, fixed for the launch.
    // LDS offset (high 16 bits: in 16-byte units) and chunk row (low 8 bits);
    // byte offset within the image row, kOutside where nothing is loaded.
    unsigned y_at[G::items_y], y_col[G::items_y], x_at[G::items_x], x_col[G::items_x];
    const int n_y = pix * G::cpr_y, n_x = pos * G::cpr_x;
#pragma unroll
    for (int i = 0; i < G::items_y; ++i) {
        const int id = tid + i * kThreads;
        const int cc = id % G::cpr_y, p = id / G::cpr_y;
        const int r = quot(p, a.magic), c = p - r * a.u4;
        y_at[i] = (unsigned(p * G::pitch_y + cc * EPC * ES) >> 4 << 16) | unsigned(r & 0xff);
        const bool ok = id < n_y && c < w_seg && o0 + cc * EPC < a.c_out;
        y_col[i] = ok ? unsigned(((col0 + c) * a.c_out + o0 + cc * EPC) * ES) : kOutside;
    }
#pragma unroll
    for (int i = 0; i < G::items_x; ++i) {
        const int id = tid + i * kThreads;
        const int cc = id % G::cpr_x, p = id / G::cpr_x;
        const int r = quot(p, a.magic_x), c = p - r * a.x_pos;
        x_at[i] = (unsigned(p * G::pitch_x + cc * EPC * ES) >> 4 << 16) | unsigned(r & 0xff);
        const int cs = quot(c, a.magic_s), kx = c - cs * a.step;  // (shared window: kx = 0)
        const int ix = (col0 + cs) * a.s_w - a.p_w + (kx0 + kx) * a.d_w;
        const bool ok = id < n_x && kx < kn && unsigned(ix) < unsigned(a.w) && c0 + cc * EPC < a.c_in;
        x_col[i] = ok ? unsigned((ix * a.c_in + c0 + cc * EPC) * ES) : kOutside;
    }
    // Byte offsets of a chunk's rows (kOutside: no such row), by the threads
    // of the first wave.
    auto fill_rows = [&](int k, int buf) {
        if (tid < a.rh) {
            const int row = k * a.rh + tid;
            unsigned yo = kOutside, xo = kOutside;
            if (row < row1) {
                const int img = row / a.h_out, oy = row - img * a.h_out;
                const int iy = oy * a.s_h - a.p_h + ky * a.d_h;
                yo = unsigned(row - row0) * a.dy_row_bytes;
                if (unsigned(iy) < unsigned(a.h))
                    xo = unsigned(img - img0) * a.x_img_bytes + unsigned(iy) * a.x_row_bytes;
            }
            row_off[buf][tid][0] = yo;
            row_off[buf][tid][1] = xo;
        }
    };
    u32x4 st_y[G::items_y], st_x[G::items_x];
    // (every row offset is read before the first load goes out, and all loads
    // issue, those of no piece past the buffer's end: no branch or wait
    // between them)
    auto fetch = [&](int buf) {
        unsigned ry[G::items_y], rx[G::items_x];
#pragma unroll
        for (int i = 0; i < G::items_y; ++i)
            ry[i] = row_off[buf][y_at[i] & 63u][0];
#pragma unroll
        for (int i = 0; i < G::items_x; ++i)
            rx[i] = row_off[buf][x_at[i] & 63u][1];
#pragma unroll
        for (int i = 0; i < G::items_y; ++i)
            st_y[i] = load_piece<PIECE8>(dy_r, (ry[i] | y_col[i]) & kOutside ? kOutside : ry[i] + y_col[i]);
#pragma unroll
        for (int i = 0; i < G::items_x1; ++i)
            st_x[i] = load_piece<PIECE8>(x_r, (rx[i] | x_col[i]) & kOutside ? kOutside : rx[i] + x_col[i]);
        if (n_x > G::items_x1 * kThreads) {
#pragma unroll
            for (int i = G::items_x1; i < G::items_x; ++i)
                st_x[i] = load_piece<PIECE8>(x_r, (rx[i] | x_col[i]) & kOutside ? kOutside : rx[i] + x_col[i]);
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int i = 0; i < G::items_y; ++i) {
            if (i * kThreads >= n_y)
                break;
            if (tid + i * kThreads < n_y)
                *reinterpret_cast<u32x4 *>(y_lds + ((y_at[i] >> 16) << 4)) = st_y[i];
        }
#pragma unroll
        for (int i = 0; i < G::items_x; ++i) {
            if (i * kThreads >= n_x)
                break;
            if (tid + i * kThreads < n_x)
                *reinterpret_cast<u32x4 *>(x_lds + ((x_at[i] >> 16) << 4)) = st_x[i];
        }
    };

    // ---- compute: wave (wo, wc, wk)
    const int wk = wave % WK, wc = (wave / WK) % WC, wo = wave / (WK * WC);
    const int ob = wo * 32, cb = wc * 32;
    f32x16 acc[KW];
#pragma unroll
    for (int t = 0; t < KW; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            acc[t][e] = 0.0f;

    // bf16: lane l reads pixels 16ks + 8(l/32) + j (+ 4), j = (l%16)/4, of
    // channels 16((l/16)%2) + 4(l%4).. ; fp32: pixel 2ks + l/32, channel l%32
    const int g = lane >> 4;
    const int lane_pix = ES == 2 ? 8 * (g >> 1) + ((lane & 15) >> 2) : lane >> 5;
    const int lane_col = (ES == 2 ? 16 * (g & 1) + 4 * (lane & 3) : lane & 31) * ES;
    const unsigned char *const y_lane = y_lds + lane_pix * G::pitch_y + ob * ES + lane_col;
    const unsigned char *const x_lane = x_lds + cb * ES + lane_col;
    // LDS pointer of pixel p's X row at the group's first tap
    auto x_row = [&](int p) {
        const int r = quot(p, a.magic);
        const int c = p - r * a.u4;
        const bool ok = c < w_seg && r < a.rh;
        return x_lane + (ok ? unsigned((r * a.x_pos + c * a.step) * G::pitch_x) : zero_row);
    };
    constexpr int KS = G::max_ks;
    const unsigned char *x_lo[KS], *x_hi[ES == 2 ? KS : 1];
#pragma unroll
    for (int i = 0; i < KS; ++i) {
        x_lo[i] = x_row((wk + i * WK) * PPK + lane_pix);
        if constexpr (ES == 2)
            x_hi[i] = x_row((wk + i * WK) * PPK + lane_pix + 4);
    }
    const int my_ks = a.ksteps > wk ? (a.ksteps - wk + WK - 1) / WK : 0;
    auto tr_pair = [&](const unsigned char *lo, const unsigned char *hi) {
        const s16x4 a0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(lo));
        const s16x4 a1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(hi));
        s16x4 both[2] = {a0, a1};
        bf16x8 f;
        __builtin_memcpy(&f, both, 16);
        return f;
    };
    auto mfma = [&](f32x16 &d, F y, F x) {
        if constexpr (ES == 2)
            d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(y, x, d, 0, 0, 0);
        else
            d = __builtin_amdgcn_mfma_f32_32x32x2f32(y, x, d, 0, 0, 0);
    };
    // The wave's K steps of a chunk for N taps, the next step's fragments
    // read while one runs.
    const unsigned char *const y_wave = y_lane + wk * PPK * G::pitch_y;
    auto compute = [&](auto taps_c) {
        constexpr int N = decltype(taps_c)::value;
        F fy[2], fx[2][N];
        auto read = [&](int i) {
            const unsigned char *const p = y_wave + i * WK * PPK * G::pitch_y;
            if constexpr (ES == 2) {
                fy[i & 1] = tr_pair(p, p + 4 * G::pitch_y);
#pragma unroll
                for (int t = 0; t < N; ++t)
                    fx[i & 1][t] = tr_pair(x_lo[i] + t * G::pitch_x, x_hi[i] + t * G::pitch_x);
            } else {
                fy[i & 1] = *reinterpret_cast<const float *>(p);
#pragma unroll
                for (int t = 0; t < N; ++t)
                    fx[i & 1][t] = *reinterpret_cast<const float *>(x_lo[i] + t * G::pitch_x);
            }
        };
        if (my_ks == 0)
            return;
        read(0);
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            if (i >= my_ks)
                break;
            if (i + 1 < KS && i + 1 < my_ks)
                read(i + 1);
#pragma unroll
            for (int t = 0; t < N; ++t)
                mfma(acc[t], fy[i & 1], fx[i & 1][t]);
        }
    };
    using N1 = std::integral_constant<int, 1>;
    using N2 = std::integral_constant<int, KW < 2 ? KW : 2>;
    using N3 = std::integral_constant<int, KW>;

    // zero rows (one per tap), and the padding pixels of the last K step, once
    for (int i = tid; i * 16 < KW * G::pitch_x; i += kThreads)
        *reinterpret_cast<u32x4 *>(x_lds + zero_row + i * 16) = u32x4{0u, 0u, 0u, 0u};
    for (int i = tid; i * 16 < (pix_pad - pix) * G::pitch_y; i += kThreads)
        *reinterpret_cast<u32x4 *>(y_lds + pix * G::pitch_y + i * 16) = u32x4{0u, 0u, 0u, 0u};

    // Chunk k + 1's loads are in flight (in registers) while chunk k, in LDS,
    // is computed.
    if (chunk0 < chunk1) {
        fill_rows(chunk0, 0);
        __syncthreads();
        fetch(0);
        for (int k = chunk0; k < chunk1; ++k) {
            const int nb = (k + 1 - chunk0) & 1;
            store();
            if (k + 1 < chunk1)
                fill_rows(k + 1, nb);
            __syncthreads();
            if (k + 1 < chunk1)
                fetch(nb);
            if (kn == 1)
                compute(N1{});
            else if (kn == 2)
                compute(N2{});
            else
                compute(N3{});
            __syncthreads();
        }
    }

    // ---- the WK waves of a block added in wave order (through LDS)
    if constexpr (WK > 1) {
        float *const red = reinterpret_cast<float *>(lds);  // [wave][register][lane]
#pragma unroll
        for (int t = 0; t < KW; ++t) {
            if (wk > 0) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    red[(wave * 16 + e) * 64 + lane] = acc[t][e];
            }
            __syncthreads();
            if (wk == 0) {
#pragma unroll
                for (int k = 1; k < WK; ++k)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        acc[t][e] += red[((wave + k) * 16 + e) * 64 + lane];
            }
            __syncthreads();
        }
    }
    const int taps = a.k_h * a.k_w, tap0 = ky * a.k_w + kx0;
    const bool mine = wk == 0;
    if (a.fold) {
        // one tile holds the whole G: dW_m[o][c] = sum over p of sign *
        // G[(p, o)][(q, c)], q = p xor m (the separable form: q = m)
        constexpr int LD = G::TC + 1;
        static_assert(G::TO * LD * 4 <= G::lds_bytes, "G fits the LDS");
        float *const gt = reinterpret_cast<float *>(lds);
#pragma unroll
        for (int t = 0; t < KW; ++t) {
            if (t >= kn)
                break;
            if (mine) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    gt[(ob + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * LD + cb + (lane & 31)] = acc[t][r];
            }
            __syncthreads();
            const int oc = a.q_out * a.q_in;
            double *dst = reinterpret_cast<double *>(a.part) + (size_t(grp) * taps + tap0 + t) * 4 * oc;
            if (tid < oc) {  // at most 16 x 16
                const int oo = quot(tid, a.magic_c), c = tid - oo * a.q_in;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    double s = 0.0;
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int q = a.sep ? m : p ^ m;
                        const double v = double(gt[(p * a.q_out + oo) * LD + q * a.q_in + c]);
                        s = (((a.sep ? kWgradSepNeg : kWgradNeg) >> (4 * p + q)) & 1u) ? s - v : s + v;
                    }
                    dst[m * oc + tid] = s;
                }
            }
            __syncthreads();
        }
        return;
    }
    if (!mine)
        return;
    // register 4g + e of lane l is (o, c) = (ob + 8g + 4(l/32) + e, cb + l%32)
    const int c = c0 + cb + (lane & 31);
#pragma unroll
    for (int t = 0; t < KW; ++t) {
        if (t >= kn)
            break;
        float *dst = a.part + (size_t(grp) * taps + tap0 + t) * a.c_out * a.c_in;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = o0 + ob + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (o < a.c_out && c < a.c_in)
                dst[size_t(o) * a.c_in + c] = acc[t][r];
        }
    }
}

int ceil_div(int64_t a, int64_t b)
{
    return int((a + b - 1) / b);
}

// LDS and pixel limits of a (wo, wc) kernel.
template <typename T>
void limits(int wo, int wc, int *max_pix, int *max_pos, int *lds, int *py, int *px)
{
    auto set = [&](auto g) {
        using G = decltype(g);
        *max_pix = G::max_pix;
        *max_pos = G::max_pos;
        *lds = G::lds_bytes;
        *py = G::pitch_y;
        *px = G::pitch_x;
    };
    if (wo == 1)
        wc == 1 ? set(Geo<T, 1, 1>{}) : set(Geo<T, 1, 2>{});
    else
        wc == 1 ? set(Geo<T, 2, 1>{}) : set(Geo<T, 2, 2>{});
}

template <typename T, int KW, bool PIECE8>
void launch_tile(const WgradRows &p, unsigned blocks, const RArgs &a, hipStream_t stream)
{
    auto tile = [&](auto wo, auto wc) {
        hipLaunchKernelGGL((qconv2d_wgrad_rows<T, decltype(wo)::value, decltype(wc)::value, KW, PIECE8>), dim3(blocks),
                           dim3(kThreads), 0, stream, a);
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    if (p.wo == 1)
        p.wc == 1 ? tile(One{}, One{}) : tile(One{}, Two{});
    else
        p.wc == 1 ? tile(Two{}, One{}) : tile(Two{}, Two{});
}

}  // namespace

WgradRows qconv2d_wgrad_rows_plan(const ConvGeom &g, DType dt)
{
    WgradRows p{};
    const int es = dt == DType::BF16 ? 2 : 4;
    const int ppk = dt == DType::BF16 ? 16 : 2;
    const int o = 4 * g.c_out, c = 4 * g.c_in;
    p.wo = o <= 32 ? 1 : 2;
    p.wc = c <= 32 ? 1 : 2;
    p.o_tiles = ceil_div(o, 32 * p.wo);
    p.c_tiles = ceil_div(c, 32 * p.wc);
    p.fold = p.o_tiles == 1 && p.c_tiles == 1;
    // Which layers.  Against the four-component kernel (qconv2d_wgrad) the
    // MFMAs cover the padded rows instead of sixteen padded component pairs,
    // at a lower rate.  Measured, this kernel / the other, us:
    //  - rows of one tile (16 channels or fewer), always: bf16 128 x 32 x 32,
    //    16 -> 16: 27.5 / 72.7 (37.7 + 21.3 as it was); 16 x 80 x 80, 8 -> 16:
    //    21.9 / 39.9; fp32 8 -> 16: 51 / 272.
    //  - bf16 channel counts that are no multiple of 8, where the other
    //    loads single elements, up to 25 tiles of G: 12 -> 20 on 8 x 75 x 77:
    //    30 / 80; 69 -> 56: 32 / 50; 77 -> 77: 60 / 164; 99 -> 99 (49 tiles):
    //    124 / 114.  Multiples of 8: 24 -> 24: 32 / 23, 16 -> 32: 31 / 29.
    //  - fp32 at half the padded work: 12 -> 20: 88 / 130, 8 -> 64: 138 / 250,
    //    16 -> 64: 249 / 251; counts that are no multiple of 4 at nine tenths:
    //    77 -> 77: 227 / 320, 18 -> 18 (as much work): 249 / 220.
    auto pad32 = [](int v) { return int64_t(v + 31) / 32 * 32; };
    const int64_t rows_work = int64_t(p.o_tiles) * p.c_tiles * (32 * p.wo) * (32 * p.wc);
    const int64_t other_work = 16 * pad32(g.c_out) * pad32(g.c_in);
    const bool whole = g.c_in % (16 / es) == 0 && g.c_out % (16 / es) == 0;
    const bool few = int64_t(p.o_tiles) * p.c_tiles <= 25;
    const bool f32 = dt == DType::F32;
    //  - kernel widths that are no multiple of three leave a tap group part
    //    empty: fp32 then at half the work only (66 -> 40, 5x5 on 10 x 24 x 24:
    //    849 / 563; 70 -> 70: 1288 / 1016), and bf16 with more than 9 taps from
    //    1024 pixels on (70 -> 70, 5x5, 640 pixels: 62 / 55).
    const bool filled = g.k_w % 3 == 0 || g.k_w == 1;
    const bool odd = !whole && few &&
                     (f32 ? filled && 10 * rows_work <= 9 * other_work : g.k_h * g.k_w <= 9 || g.m() >= 1024);
    if (!(p.fold || odd || (f32 && 2 * rows_work <= other_work)))
        return p;
    p.kw = g.k_w == 1 ? 1 : 3;
    p.kx_groups = ceil_div(g.k_w, p.kw);
    const int kn = g.k_w < p.kw ? g.k_w : p.kw;
    int max_pix = 0, max_pos = 0, lds = 0, py = 0, px = 0;
    if (dt == DType::BF16)
        limits<__bf16>(p.wo, p.wc, &max_pix, &max_pos, &lds, &py, &px);
    else
        limits<float>(p.wo, p.wc, &max_pix, &max_pos, &lds, &py, &px);
    // Column segments and rows per chunk: the least staged and multiplied
    // pixels per real one, a chunk's barriers and row set-up counted as 16
    // pixels' work.
    double best = 0.0;
    for (int segs = 1; segs <= g.w_out && segs <= 4096; ++segs) {
        const int u4 = ceil_div(ceil_div(g.w_out, segs), 4) * 4;
        if (int64_t(u4) * (segs - 1) >= g.w_out)
            continue;  // the last segment would be empty
        if (u4 > max_pix)
            continue;
        const int step = g.s_w > 1 || g.d_w > 1 ? kn : 1;
        const int x_pos = step > 1 ? kn * u4 : u4 + kn - 1;
        for (int rh = 1; rh * u4 <= max_pix && rh <= 32; ++rh) {
            const int ks = ceil_div(rh * u4, ppk);
            const int64_t bytes = int64_t(ks) * ppk * py + (int64_t(rh) * x_pos + p.kw) * px;
            if (bytes > lds || rh * x_pos > max_pos)
                break;
            const double work = (ks * ppk + 0.25 * rh * x_pos + 16.0) * segs / (double(rh) * g.w_out);
            if (!p.takes || work < best) {
                p.takes = true;
                best = work;
                p.segs = segs;
                p.u4 = u4;
                p.rh = rh;
                p.ksteps = ks;
                p.x_pos = x_pos;
                p.step = step;
            }
        }
        if (p.takes && u4 <= 16)
            break;  // narrower segments only add padding
    }
    if (!p.takes)
        return p;
    const int64_t rows = int64_t(g.n) * g.h_out;
    p.chunks = ceil_div(rows, p.rh);
    // two work-groups per compute unit, each a few chunks long
    const int want = 512;  // (384, 768 and 1024 were 5-20% slower on most narrow layers)
    const int inner = g.k_h * p.kx_groups * p.o_tiles * p.c_tiles * p.segs;
    int splits = want / inner;
    const int most = (p.chunks + 1) / 2;
    splits = splits > most ? most : splits;
    splits = splits < 1 ? 1 : splits;
    p.most_splits = splits;  // (grows with the chunks, where the rounded p.splits may not)
    p.per_split = ceil_div(p.chunks, splits);
    p.splits = ceil_div(p.chunks, p.per_split);
    // 32-bit offsets within a slice
    const int64_t slice_rows = int64_t(p.per_split) * p.rh;
    const int64_t dy_span = slice_rows * g.w_out * 4 * g.c_out * es;
    const int64_t x_span = (slice_rows / g.h_out + 2) * g.h * g.w * 4 * g.c_in * es;
    p.takes = dy_span < 0x7fffffffLL && x_span < 0x7fffffffLL;
    return p;
}

hipError_t qconv2d_wgrad_rows_run(const WgradRows &p, const ConvGeom &g, DType dt, const void *x, const void *dy,
                                  float *part, hipStream_t stream, bool sep)
{
    if (!p.takes)
        return hipErrorNotSupported;
    const int es = dt == DType::BF16 ? 2 : 4;
    RArgs a;
    a.x = x;
    a.dy = dy;
    a.part = part;
    a.c_in = 4 * g.c_in;
    a.c_out = 4 * g.c_out;
    a.h = g.h;
    a.w = g.w;
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
    a.rows = g.n * g.h_out;
    a.segs = p.segs;
    a.u4 = p.u4;
    a.rh = p.rh;
    a.ksteps = p.ksteps;
    a.x_pos = p.x_pos;
    a.step = p.step;
    a.magic = unsigned(((1 << 20) + p.u4 - 1) / p.u4);
    a.magic_x = unsigned(((1 << 20) + p.x_pos - 1) / p.x_pos);
    a.magic_s = unsigned(((1 << 20) + p.step - 1) / p.step);
    a.magic_c = unsigned(((1 << 20) + g.c_in - 1) / g.c_in);
    a.chunks = p.chunks;
    a.per_split = p.per_split;
    a.kx_groups = p.kx_groups;
    a.o_tiles = p.o_tiles;
    a.c_tiles = p.c_tiles;
    a.groups = p.splits * p.segs;
    a.x_row_bytes = unsigned(g.w) * 4u * g.c_in * es;
    a.x_img_bytes = a.x_row_bytes * unsigned(g.h);
    a.dy_row_bytes = unsigned(g.w_out) * 4u * g.c_out * es;
    a.fold = p.fold ? 1 : 0;
    a.sep = sep ? 1 : 0;
    a.q_out = g.c_out;
    a.q_in = g.c_in;
    const int inner = g.k_h * p.kx_groups * p.o_tiles * p.c_tiles;
    const unsigned blocks = unsigned(8 * inner * ceil_div(a.groups, 8));
    if (dt == DType::F32)
        p.kw == 1 ? launch_tile<float, 1, false>(p, blocks, a, stream)
                  : launch_tile<float, 3, false>(p, blocks, a, stream);
    else if (g.c_in % 2 != 0 || g.c_out % 2 != 0)
        p.kw == 1 ? launch_tile<__bf16, 1, true>(p, blocks, a, stream)
                  : launch_tile<__bf16, 3, true>(p, blocks, a, stream);
    else
        p.kw == 1 ? launch_tile<__bf16, 1, false>(p, blocks, a, stream)
                  : launch_tile<__bf16, 3, false>(p, blocks, a, stream);
    return hipGetLastError();
}

}  // namespace quan
