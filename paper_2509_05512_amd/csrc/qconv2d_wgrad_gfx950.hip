// Weight and bias gradients of the Hamilton convolution (the backward pass of
// Section III-B's eq. 5/6 with respect to W and the bias) for gfx950.
//
// With Y_p = sum_q s(p, q) W_{p xor q} (x) X_q per tap (eq. 6's sign s and
// component index), the gradient of kernel component m at tap (ky, kx) is
//
//   dW_m[o][c] = sum_p s(p, p xor m) sum_pix dY[pix][p][o] X[pix + tap][p xor m][c],
//
// a GEMM whose reduction dimension is the output pixels (N * Ho * Wo), over
// both operands stored channels-last.  One work-group takes one tap, a tile of
// 32 or 64 output by 32 or 64 input channels and a contiguous slice of the
// pixels; it stages chunks of 32 pixels (64 on the 32 x 32 bf16 tile) of dY (all
// four components) and of the tap-shifted X (zero outside the image) in LDS,
// bank-conflict free (see row_elems) and double-buffered, with the global loads
// (16-byte buffer loads at 32-bit offsets, zeros past the end, each thread's
// pixel coordinates advanced incrementally; element by element where channels
// fill no whole 16-byte chunks) issued two chunks ahead; its four waves each
// accumulate the four dW_m of one 32 x 32 (o, c) block, on the smaller tiles a
// share of a chunk's K steps, reading the next k-step's fragments while the
// MFMAs of the current one run, a sign flip being one XOR per fragment dword.  The taps of one (slice, tile) are placed
// on one XCD (work-group b runs on XCD b % 8), so the nine reads of a slice
// of dY and its shifted copies of X share that XCD's L2.  MFMA operands need
// eight consecutive pixels per lane: bf16 fragments come from the pixel-major
// rows with two transposing LDS reads (ds_read_b64_tr_b16), fp32 fragments
// (one pixel per lane) with plain reads.  Slices write fp32 partial sums; a
// second kernel adds them in slice order in fp64 (deterministic) into dW.
// Layers of at most 16 channels, and others that it is the faster for, go to
// the row kernel (qconv2d_wgrad_rows), which leaves either such sums or the
// dense products of all sixteen component pairs, from which the reduction forms
// dW.  The bias gradient is the column sum of dY.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "qconv2d_wgrad.h"

namespace quan {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kChunk = 32;   // pixels per staged chunk (64 where four waves split the K steps)
// LDS rows of a staged chunk: bf16 rows of 64 channels (128 bytes) have the
// 16-byte chunks of rows 2..3 mod 4 XOR-swizzled by 4, so that neither the
// row-wise 16-byte stores nor the transposing 8-byte reads (four rows of
// one 64-byte column group per 16 lanes) meet in a bank; rows of 32 channels
// (64 bytes) need no swizzle; fp32 rows are padded by 16 elements.
template <typename T>
constexpr int row_elems(int tile)
{
    return sizeof(T) == 2 ? tile : tile + 16;
}
template <int TILE>
__device__ __forceinline__ int chunk_swz(int row)
{
    return TILE == 64 ? 4 * ((row >> 1) & 1) : 0;
}

struct WArgs {
    const void *x, *dy;
    float *part;  // [splits][taps][4][c_out][c_in]
    int n, c_in, h, w, c_out, k_h, k_w, s_h, s_w, p_h, p_w, d_h, d_w, h_out, w_out;
    int64_t pixels;       // n * h_out * w_out
    int64_t per_split;    // pixels of one slice
    int o_tiles, c_tiles, taps;
    int groups;  // slices x tiles
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

// 16-byte chunk of one (component, pixel) row: channels ch0 .. ch0+EPC-1 of
// a row of `len` channels starting at src, zeros where `valid` is false or
// past len.  Branch-free: an invalid lane loads from `safe` (the tensor's
// first element) and selects zero, so every load of a chunk stays in flight
// together.
template <typename T>
__device__ __forceinline__ u32x4 load_chunk(const T *src, bool valid, int ch0, int len, const T *safe)
{
    constexpr int EPC = 16 / int(sizeof(T));
    T e[EPC];
#pragma unroll
    for (int i = 0; i < EPC; ++i) {
        const bool ok = valid && ch0 + i < len;
        const T u = *(ok ? src + ch0 + i : safe);
        e[i] = ok ? u : T(0);
    }
    u32x4 v;
    __builtin_memcpy(&v, e, 16);
    return v;
}

// 16 bytes at byte offset off of the buffer [base, base + bytes); offsets
// past the end read as zeros.
__device__ __forceinline__ u32x4 load16(const void *base, unsigned bytes, unsigned off)
{
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// SEP: the separable form's gradients (eqs. 8-10), dW_q = sum_p
// S[p][q] dY_p X_q: the same sixteen component pairs, each added into the
// accumulator of its input component q with eq. 7's sign.
// WO x WC x WK: waves over (output, input) channel blocks of 32 and over the
// K steps of a chunk.
template <typename T, bool VEC, bool SEP, int WO, int WC, int WK>
__global__ __launch_bounds__(kThreads) void qconv2d_wgrad(WArgs a)
{
    static_assert(WO * WC * WK == 4, "four waves");
    constexpr int NC = 4;                      // components per pixel row
    constexpr int NM = 4;                      // accumulator sets: dW_m
    constexpr int ES = int(sizeof(T));
    constexpr int EPC = 16 / ES;               // elements per 16-byte chunk
    constexpr int CH = WK == 4 && ES == 2 ? 2 * kChunk : kChunk;  // pixels per chunk
    constexpr int TW[2] = {32 * WO, 32 * WC};  // channels of the tile: dY, X
    constexpr int CPR[2] = {TW[0] / EPC, TW[1] / EPC};  // chunks per (component, pixel) row
    constexpr int ROW[2] = {row_elems<T>(TW[0]), row_elems<T>(TW[1])};
    constexpr int COMP[2] = {CH * ROW[0], CH * ROW[1]};  // elements per component block in LDS
    constexpr int XOFF = NC * COMP[0];         // X behind dY
    constexpr int BUF = XOFF + NC * COMP[1];
    // The 256 threads move PXT pixel rows of QT components at a time.
    constexpr int PXT[2] = {kThreads / CPR[0] < CH ? kThreads / CPR[0] : CH, kThreads / CPR[1] < CH ? kThreads / CPR[1] : CH};
    constexpr int QT[2] = {kThreads / (CPR[0] * PXT[0]), kThreads / (CPR[1] * PXT[1])};
    constexpr int PASSES[2] = {CH / PXT[0], CH / PXT[1]};
    constexpr int NQ[2] = {NC / QT[0], NC / QT[1]};
    static_assert(PXT[0] * PASSES[0] == CH && PXT[1] * PASSES[1] == CH && QT[0] <= NC && QT[1] <= NC, "tile geometry");
    __shared__ __attribute__((aligned(16))) T lds[2 * BUF];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // work-group b on XCD b % 8 takes tap (b / 8) % taps of group
    // b % 8 + 8 * (b / 8 / taps)
    const int xs = int(blockIdx.x) >> 3;
    const int tap = xs % a.taps;
    int b = (int(blockIdx.x) & 7) + 8 * (xs / a.taps);
    if (b >= a.groups)
        return;  // padding of the last round of groups: nothing to do
    const int ot = b % a.o_tiles;
    b /= a.o_tiles;
    const int ct = b % a.c_tiles;
    const int split = b / a.c_tiles;
    const int ky = tap / a.k_w, kx = tap - (tap / a.k_w) * a.k_w;
    const int o0 = ot * TW[0], c0 = ct * TW[1];
    const int64_t pix0 = int64_t(split) * a.per_split;
    int64_t pix1 = pix0 + a.per_split;
    if (pix1 > a.pixels)
        pix1 = a.pixels;
    const int chunks = pix0 < pix1 ? int((pix1 - pix0 + CH - 1) / CH) : 0;
    const T *dy = static_cast<const T *>(a.dy);
    const T *x = static_cast<const T *>(a.x);
    const int hw_out = a.h_out * a.w_out;

    // ---- staging: of each tensor thread t moves chunk t % CPR of pixel row
    // t / CPR % PXT (+ PXT per pass), components t / CPR / PXT + QT * i
    const int cy = tid % CPR[0], py = tid / CPR[0] % PXT[0], qy = tid / CPR[0] / PXT[0];
    const int cx = tid % CPR[1], px = tid / CPR[1] % PXT[1], qx = tid / CPR[1] / PXT[1];
    struct Staged {
        u32x4 y[PASSES[0]][NQ[0]], x[PASSES[1]][NQ[1]];
    };
    // VEC: 16-byte buffer loads at 32-bit offsets from the slice's first
    // pixel (dY) and first image (X), zeros past a buffer's end; each pass
    // keeps its pixel's (image, row, column), advanced by one chunk per
    // fetch, so chunks are fetched in order.
    const int span = int(pix1 - pix0 > 0 ? pix1 - pix0 : 0);
    const int64_t img0 = pix0 / hw_out;
    const T *const dy_s = dy + pix0 * NC * a.c_out;
    const T *const x_s = x + img0 * int64_t(a.h) * a.w * NC * a.c_in;
    const unsigned dy_bytes = unsigned(int64_t(span) * NC * a.c_out * ES);
    const int64_t x_left = (int64_t(a.n) - img0) * a.h * a.w * NC * a.c_in * ES;
    const unsigned x_bytes = unsigned(x_left < 0x7fffffffLL ? x_left : 0x7fffffffLL);
    const bool o_in = o0 + cy * EPC < a.c_out, c_in_ok = c0 + cx * EPC < a.c_in;
    int cur_img[PASSES[1]], cur_oy[PASSES[1]], cur_ox[PASSES[1]];
#pragma unroll
    for (int i = 0; i < PASSES[1]; ++i) {
        const int64_t pix = pix0 + px + PXT[1] * i;
        const int64_t img = pix / hw_out;
        const int rr = int(pix - img * hw_out);
        cur_img[i] = int(img - img0);
        cur_oy[i] = rr / a.w_out;
        cur_ox[i] = rr - cur_oy[i] * a.w_out;
    }
    auto fetch = [&](int k, Staged &st) {
#pragma unroll
        for (int i = 0; i < PASSES[0]; ++i) {
            const int rel = k * CH + py + PXT[0] * i;  // pixel - pix0
            const bool yok = rel < span;
            if constexpr (VEC) {
                const unsigned yoff = yok && o_in ? unsigned((rel * NC * a.c_out + o0 + cy * EPC) * ES) : 0x80000000u;
#pragma unroll
                for (int q = 0; q < NQ[0]; ++q)
                    st.y[i][q] = load16(dy_s, dy_bytes, yoff + unsigned((qy + QT[0] * q) * a.c_out * ES));
            } else {
                const T *yrow = dy_s + int64_t(yok ? rel : 0) * NC * a.c_out;
#pragma unroll
                for (int q = 0; q < NQ[0]; ++q)
                    st.y[i][q] = load_chunk<T>(yrow + (qy + QT[0] * q) * a.c_out + o0, yok, cy * EPC, a.c_out - o0, dy);
            }
        }
#pragma unroll
        for (int i = 0; i < PASSES[1]; ++i) {
            const int rel = k * CH + px + PXT[1] * i;
            const bool in = rel < span;
            const int iy = cur_oy[i] * a.s_h - a.p_h + ky * a.d_h, ix = cur_ox[i] * a.s_w - a.p_w + kx * a.d_w;
            const bool xok = in && unsigned(iy) < unsigned(a.h) && unsigned(ix) < unsigned(a.w);
            if constexpr (VEC) {
                const unsigned xoff =
                    xok && c_in_ok
                        ? unsigned((((cur_img[i] * a.h + iy) * a.w + ix) * NC * a.c_in + c0 + cx * EPC) * ES)
                        : 0x80000000u;
#pragma unroll
                for (int q = 0; q < NQ[1]; ++q)
                    st.x[i][q] = load16(x_s, x_bytes, xoff + unsigned((qx + QT[1] * q) * a.c_in * ES));
            } else {
                const T *xrow = x_s + ((int64_t(cur_img[i]) * a.h + (xok ? iy : 0)) * a.w + (xok ? ix : 0)) * NC * a.c_in;
#pragma unroll
                for (int q = 0; q < NQ[1]; ++q)
                    st.x[i][q] = load_chunk<T>(xrow + (qx + QT[1] * q) * a.c_in + c0, xok, cx * EPC, a.c_in - c0, x);
            }
            // next chunk: CH pixels on
            int ox = cur_ox[i] + CH, oy = cur_oy[i], im = cur_img[i];
            while (ox >= a.w_out) {
                ox -= a.w_out;
                if (++oy == a.h_out) {
                    oy = 0;
                    ++im;
                }
            }
            cur_ox[i] = ox;
            cur_oy[i] = oy;
            cur_img[i] = im;
        }
    };
    auto store = [&](int buf, const Staged &st) {
        T *base = lds + buf * BUF;
#pragma unroll
        for (int i = 0; i < PASSES[0]; ++i)
#pragma unroll
            for (int q = 0; q < NQ[0]; ++q) {
                const int row = py + PXT[0] * i;
                *reinterpret_cast<u32x4 *>(base + (qy + QT[0] * q) * COMP[0] + row * ROW[0] +
                                           (ES == 2 ? (cy ^ chunk_swz<TW[0]>(row)) : cy) * EPC) = st.y[i][q];
            }
#pragma unroll
        for (int i = 0; i < PASSES[1]; ++i)
#pragma unroll
            for (int q = 0; q < NQ[1]; ++q) {
                const int row = px + PXT[1] * i;
                *reinterpret_cast<u32x4 *>(base + XOFF + (qx + QT[1] * q) * COMP[1] + row * ROW[1] +
                                           (ES == 2 ? (cx ^ chunk_swz<TW[1]>(row)) : cx) * EPC) = st.x[i][q];
            }
    };

    // ---- compute: wave (wo, wc) owns an o-block and a c-block, K steps wk, wk + WK, ..
    const int wk = wave % WK, ob = wave / (WK * WC) * 32, cb = wave / WK % WC * 32;
    f32x16 acc[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            acc[m][e] = 0.0f;

    // Fragment of component block `comp` of tensor t (0 dY, 1 X), channel
    // block col0, k-step ks: lane l gets channel col0 + l%32 at the pixels
    // the MFMA's operand layout assigns it.
    auto frag = [&](auto tile, const T *base, int comp, int col0, int ks) {
        constexpr int TILE = decltype(tile)::value, R = row_elems<T>(TILE);
        typename Frag<T>::type f;
        if constexpr (ES == 2) {
            // two transposing reads of rows 16ks + 8(g/2) + 4r + j, columns
            // col0 + 16(g%2) + 4a (g = l/16, a = l%4, j = (l%16)/4)
            const int g = lane >> 4, aa = lane & 3, j = (lane & 15) >> 2;
            const int row = 16 * ks + 8 * (g >> 1) + j, col = col0 + 16 * (g & 1) + 4 * aa;
            // rows row and row + 4 share the swizzle
            const T *p0 = base + comp * CH * R + row * R + (((col >> 3) ^ chunk_swz<TILE>(row)) << 3) + (col & 7);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) s16x4 *)(p0));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) s16x4 *)(p0 + 4 * R));
            s16x4 both[2] = {lo, hi};
            __builtin_memcpy(&f, both, 16);
        } else {
            // one pixel per lane: row 2ks + l/32, column col0 + l%32
            f = base[comp * CH * R + (2 * ks + (lane >> 5)) * R + col0 + (lane & 31)];
        }
        return f;
    };
    constexpr int KSTEPS = (ES == 2 ? CH / 16 : CH / 2) / WK;  // of one wave
    typedef typename Frag<T>::type F;
    struct KFrags {
        F fy[NC], fx[NC];
    };
    auto read_k = [&](int buf, int ks, KFrags &f) {
        const T *yb = lds + buf * BUF, *xb = yb + XOFF;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            f.fy[q] = frag(std::integral_constant<int, TW[0]>{}, yb, q, ob, ks * WK + wk);
            f.fx[q] = frag(std::integral_constant<int, TW[1]>{}, xb, q, cb, ks * WK + wk);
        }
    };
    // sign flip of a fragment: the sign bit of every element
    auto negate = [&](F v) {
        if constexpr (ES == 2) {
            u32x4 u = __builtin_bit_cast(u32x4, v);
            u ^= 0x80008000u;
            return __builtin_bit_cast(F, u);
        } else {
            return __builtin_bit_cast(F, __builtin_bit_cast(unsigned, v) ^ 0x80000000u);
        }
    };
    auto mfmas = [&](const KFrags &f) {
#pragma unroll
        for (int p = 0; p < NC; ++p) {
            const F pos = f.fy[p], neg = negate(f.fy[p]);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int q = p ^ m;
                const int d = SEP ? q : m;  // the gradient this pair adds into
                const bool minus = ((SEP ? kWgradSepNeg : kWgradNeg) >> (4 * p + q)) & 1u;
                if constexpr (ES == 2)
                    acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(minus ? neg : pos, f.fx[q], acc[d], 0, 0, 0);
                else
                    acc[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(minus ? neg : pos, f.fx[q], acc[d], 0, 0, 0);
            }
        }
    };
    // The k-steps of one chunk, reading k-step ks + 1 while ks runs: the
    // sign flips first, then each MFMA followed by one fragment read.
    constexpr int NRD = ES == 2 ? 16 : 8;  // LDS reads of one k-step
    auto sched = [&]() {
        __builtin_amdgcn_sched_group_barrier(0x002, ES == 2 ? 16 : 4, 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (i < NRD)
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };
    auto compute = [&](int buf) {
        KFrags fa, fb;
        read_k(buf, 0, fa);
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ks += 2) {
            __builtin_amdgcn_sched_barrier(0);
            if (ks + 1 < KSTEPS)
                read_k(buf, ks + 1, fb);
            mfmas(fa);
            if (ks + 1 < KSTEPS)
                sched();
            __builtin_amdgcn_sched_barrier(0);
            if (ks + 2 < KSTEPS)
                read_k(buf, ks + 2, fa);
            if (ks + 1 < KSTEPS)
                mfmas(fb);
            if (ks + 2 < KSTEPS)
                sched();
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Chunk k is computed from LDS buffer k % 2 while chunk k + 1 waits in
    // registers (loaded an iteration earlier) and chunk k + 2 is loaded; after
    // the computation chunk k + 1 goes to the other buffer, which the previous
    // barrier freed.  Two register sets alternate, so the loop is unrolled by
    // two.
    Staged sa, sb;
    auto iteration = [&](int k, Staged &next, Staged &after) {
        if (k + 2 < chunks)
            fetch(k + 2, after);
        compute(k & 1);
        if (k + 1 < chunks)
            store((k + 1) & 1, next);
        __syncthreads();
    };
    if (chunks > 0) {
        fetch(0, sa);
        if (chunks > 1)
            fetch(1, sb);
        store(0, sa);
        __syncthreads();
        int k = 0;
        for (; k + 1 < chunks; k += 2) {
            iteration(k, sb, sa);
            iteration(k + 1, sa, sb);
        }
        if (k < chunks)
            iteration(k, sb, sa);
    }

    // ---- the WK waves of a block added in wave order (through LDS)
    if constexpr (WK > 1) {
        float *const red = reinterpret_cast<float *>(lds);  // [wave][register][lane]
        static_assert(sizeof(lds) >= 4 * 16 * 64 * sizeof(float), "the sums fit the LDS");
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            if (wk > 0) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    red[(wave * 16 + e) * 64 + lane] = acc[m][e];
            }
            __syncthreads();
            if (wk == 0) {
#pragma unroll
                for (int k = 1; k < WK; ++k)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        acc[m][e] += red[((wave + k) * 16 + e) * 64 + lane];
            }
            __syncthreads();
        }
        if (wk > 0)
            return;
    }
    // ---- partial sums: register 4g + e of lane l is (o, c) = (ob + 8g +
    // 4(l/32) + e, cb + l%32) of the wave's block
    const int c = c0 + cb + (lane & 31);
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        float *dst = a.part + ((int64_t(split) * a.taps + tap) * NM + m) * a.c_out * a.c_in;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = o0 + ob + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            if (o < a.c_out && c < a.c_in)
                dst[int64_t(o) * a.c_in + c] = acc[m][r];
        }
    }
}

// dW_m[o][c][ky][kx] = sum over slices of the partials in fp64.  A slice is
// one run of [tap][m][o][c]; SG threads share four consecutive outputs, thread
// s taking slices s, s + SG, ... in order (U 16-byte loads in flight), and are
// added in order through LDS: deterministic.  Blocks go through the run m by m
// (`seg` blocks to a tap of one m), so that the stores of an m's taps, which lie
// side by side, meet in the caches: 25 taps of 120 -> 144 channels in 4 slices
// 30.0 us in the run's order, 13.7 so.
// Bound by reading the partials.  One thread per output walking every slice
// (the former form) kept too few loads in flight: 33.6 MB of partials (64 x
// 64 channels, 9 taps, 57 slices) took 17.4 us, now 7.5; 57 slices of a
// 16-channel layer 21.3, now 4.2.  Four-byte loads of a run of outputs of one tap
// and m instead: 13.2 and 11.1.
template <typename P, int SG, int U>
__global__ __launch_bounds__(kThreads) void qconv2d_wgrad_reduce(const P *__restrict__ part, int slices, int taps,
                                                                 int oc_n, int seg, float *__restrict__ dw0,
                                                                 float *__restrict__ dw1, float *__restrict__ dw2,
                                                                 float *__restrict__ dw3)
{
    constexpr int QUADS = kThreads / SG;  // output quads per block
    struct alignas(16) Quad {
        P e[4];
    };
    __shared__ double red[SG > 1 ? SG : 1][QUADS * 4];
    const int ql = threadIdx.x % QUADS, sg = threadIdx.x / QUADS;
    const int64_t n = int64_t(4) * taps * oc_n;  // a multiple of 4
    const int mt0 = int(blockIdx.x) / seg;  // segment (m, tap) of the order, at tap * 4 + m of the run
    const int64_t blk = int64_t(mt0 % taps * 4 + mt0 / taps) * seg + int(blockIdx.x) % seg;
    const int64_t f0 = (blk * QUADS + ql) * 4;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (f0 < n) {
        for (int sp = sg; sp < slices; sp += SG * U) {
            Quad v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int at = sp + u * SG;
                v[u] = *reinterpret_cast<const Quad *>(part + int64_t(at < slices ? at : sp) * n + f0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (sp + u * SG < slices) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        s[e] += double(v[u].e[e]);
                }
        }
    }
    if constexpr (SG > 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            red[sg][ql * 4 + e] = s[e];
        __syncthreads();
        for (int j = threadIdx.x; j < QUADS * 4; j += kThreads) {
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < SG; ++k)
                t += red[k][j];
            const int64_t f = blk * QUADS * 4 + j;
            if (f < n) {
                const int mt = int(f / oc_n), m = mt & 3, tap = mt >> 2;
                float *dw = m == 0 ? dw0 : m == 1 ? dw1 : m == 2 ? dw2 : dw3;
                dw[(f - int64_t(mt) * oc_n) * taps + tap] = float(t);
            }
        }
    } else if (f0 < n) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t f = f0 + e;
            const int mt = int(f / oc_n), m = mt & 3, tap = mt >> 2;
            float *dw = m == 0 ? dw0 : m == 1 ? dw1 : m == 2 ? dw2 : dw3;
            dw[(f - int64_t(mt) * oc_n) * taps + tap] = float(s[e]);
        }
    }
}

// Dense partials G[(p,o)][(q,c)] per slice and tap ([slices][taps][4*c_out]
// [4*c_in]): dW_m[o][c][tap] = sum over slices and p of s(p, p xor m)
// G[(p,o)][(p xor m, c)] (eq. 6's signs), in fp64; with sep (the separable
// form) of S[p][m] G[(p,o)][(m,c)] (eq. 7's signs).  SG threads share an
// output, as above.
template <int SG>
__global__ __launch_bounds__(kThreads) void qconv2d_wgrad_reduce_dense(const float *__restrict__ part, int slices,
                                                                       int taps, int c_out, int c_in, int sep,
                                                                       float *__restrict__ dw0,
                                                                       float *__restrict__ dw1,
                                                                       float *__restrict__ dw2,
                                                                       float *__restrict__ dw3)
{
    constexpr int OUTS = kThreads / SG;
    __shared__ double red[SG][OUTS];
    const int ol = threadIdx.x % OUTS, sg = threadIdx.x / OUTS;
    const int64_t oc_n = int64_t(c_out) * c_in;
    const int64_t idx = int64_t(blockIdx.x) * OUTS + ol;  // over [tap][m][o][c]
    const bool live = idx < 4 * taps * oc_n;
    const int64_t at = live ? idx : 0;
    const int64_t oc = at % oc_n;
    const int o = int(oc / c_in), c = int(oc - int64_t(o) * c_in);
    const int mt = int(at / oc_n);
    const int m = mt & 3, tap = mt >> 2;
    const int64_t g_n = int64_t(4 * c_out) * (4 * c_in);  // one slice's G of one tap
    double s = 0.0;
#pragma unroll 2
    for (int sp = sg; sp < slices; sp += SG) {
        const float *g = part + (int64_t(sp) * taps + tap) * g_n;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int q = sep ? m : p ^ m;
            const double v = double(g[int64_t(p * c_out + o) * (4 * c_in) + q * c_in + c]);
            s += (((sep ? kWgradSepNeg : kWgradNeg) >> (4 * p + q)) & 1u) ? -v : v;
        }
    }
    red[sg][ol] = s;
    __syncthreads();
    if (threadIdx.x < OUTS && live) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < SG; ++k)
            t += red[k][ol];
        float *dw = m == 0 ? dw0 : m == 1 ? dw1 : m == 2 ? dw2 : dw3;
        dw[oc * taps + tap] = float(t);
    }
}

// Bias gradient: column sums of the [pixels][cols = 4 * c_out] rows of dY.
// Thread t of a block sums the VW-element column chunk t % CG over rows
// t / CG + RPI * i of the block's row range (four rows in flight), the
// threads sharing a chunk add in a fixed order through LDS, and each block
// writes one partial per column; colsum_final adds the blocks in order in
// fp64.
template <typename T, int VW>
__global__ __launch_bounds__(kThreads) void colsum_partial(const T *__restrict__ dy, int64_t pixels, int cols,
                                                           int64_t rows_per_block, float *__restrict__ part)
{
    __shared__ float red[kThreads][VW];
    const int chunks = cols / VW;
    const int cg = chunks < kThreads ? chunks : kThreads;
    const int rpi = kThreads / cg;
    const int tid = threadIdx.x, cl = tid % cg, rl = tid / cg;
    const int chunk = blockIdx.y * cg + cl;
    const bool active = rl < rpi && chunk < chunks;
    const int64_t r0 = int64_t(blockIdx.x) * rows_per_block;
    int64_t r1 = r0 + rows_per_block;
    if (r1 > pixels)
        r1 = pixels;
    struct alignas(sizeof(T) * VW) V {
        T e[VW];
    };
    float acc[VW];
#pragma unroll
    for (int e = 0; e < VW; ++e)
        acc[e] = 0.0f;
    if (active) {
        const T *base = dy + chunk * VW;
        int64_t r = r0 + rl;
        for (; r + 3 * rpi < r1; r += 4 * rpi) {
            V v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                v[u] = *reinterpret_cast<const V *>(base + (r + u * rpi) * cols);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < VW; ++e)
                    acc[e] += float(v[u].e[e]);
        }
        for (; r < r1; r += rpi) {
            const V v = *reinterpret_cast<const V *>(base + r * cols);
#pragma unroll
            for (int e = 0; e < VW; ++e)
                acc[e] += float(v.e[e]);
        }
    }
#pragma unroll
    for (int e = 0; e < VW; ++e)
        red[tid][e] = acc[e];
    __syncthreads();
    if (rl == 0 && chunk < chunks) {
        float t[VW];
#pragma unroll
        for (int e = 0; e < VW; ++e)
            t[e] = 0.0f;
        for (int j = 0; j < rpi; ++j)
#pragma unroll
            for (int e = 0; e < VW; ++e)
                t[e] += red[j * cg + cl][e];
#pragma unroll
        for (int e = 0; e < VW; ++e)
            part[int64_t(blockIdx.x) * cols + chunk * VW + e] = t[e];
    }
}

// One wave per column: lane i adds blocks i, i+64, ... (eight loads in
// flight), then a fixed butterfly adds the lanes in fp64.
__global__ __launch_bounds__(kThreads) void colsum_final(const float *__restrict__ part, int blocks, int cols,
                                                         float *__restrict__ db)
{
    constexpr int U = 8;
    const int lane = threadIdx.x & 63;
    const int col = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (col >= cols)
        return;
    double s = 0.0;
    for (int b0 = lane; b0 < blocks; b0 += 64 * U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = b0 + 64 * u;
            v[u] = part[int64_t(b < blocks ? b : blocks - 1) * cols + col];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (b0 + 64 * u < blocks)
                s += double(v[u]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
        s += __shfl_xor(s, off);
    if (lane == 0)
        db[col] = float(s);
}

constexpr int kBiasBlocks = 512;

struct WPlan {
    int wo, wc;  // channel blocks of 32 per tile
    int o_tiles, c_tiles, taps, splits;
    int64_t most_splits;  // of this layer with this many images or fewer
    int64_t per_split;
};

WPlan wgrad_plan(const ConvGeom &g, DType dt)
{
    WPlan p;
    // A tile of 64 channels a side, or 32 where 64 would leave a block idle
    // (two or four waves then split a chunk's K steps): 32 -> 64 channels on
    // 16 x 160 x 160, stride 2: 108.8 -> 65 us with half the MFMAs of the
    // 64-wide tile gone; 32 -> 32 in fp32 on 16 x 28 x 28: 138 -> 39 us.
    // In bf16 three tiles of 32 stage more than two of 64 for their MFMAs: 87 -> 92
    // on 16 x 16 x 16 70.1 us with 64, 99.8 with 32; 96 -> 96, 5x5 stride 3 on 10 x 24
    // x 24 19.2 / 22.3 (fp32, bound by its MFMAs: 125 / 86).
    auto narrow = [&](int c) { return c <= 32 || (dt == DType::F32 && c > 64 && c <= 96); };
    p.wo = narrow(g.c_out) ? 1 : 2;
    p.wc = narrow(g.c_in) ? 1 : 2;
    p.o_tiles = (g.c_out + 32 * p.wo - 1) / (32 * p.wo);
    p.c_tiles = (g.c_in + 32 * p.wc - 1) / (32 * p.wc);
    p.taps = g.k_h * g.k_w;
    const int64_t pixels = g.m();
    const int64_t per_split_pass = int64_t(p.o_tiles) * p.c_tiles * p.taps;
    // about two work-groups per compute unit, each at least a few chunks long
    int64_t splits = (512 + per_split_pass - 1) / per_split_pass;
    // (two chunks at least; eight, where the partials of more would pass
    // kPartBytes and the loads need no hiding: 64 -> 96, 3x3 on 2 x 28 x 28, 17
    // slices of 0.9 MB 22.0 us, 7 slices 17.3; 40 -> 24, 0.14 MB: 11.2 and 13.8;
    // 87 -> 92, element loads: 40 and 56)
    constexpr int64_t kPartBytes = int64_t(8) << 20;
    const int64_t dw_bytes = int64_t(p.taps) * 4 * g.c_out * g.c_in * int64_t(sizeof(float));
    const bool whole = g.c_in % 8 == 0 && g.c_out % 8 == 0;
    auto slices_of = [&](int chunks) { return (pixels + chunks * kChunk - 1) / (chunks * kChunk); };
    int64_t max_splits = slices_of(2);
    if (dt == DType::BF16 && whole)
        max_splits = std::min(max_splits, std::max(slices_of(8), kPartBytes / dw_bytes));
    if (splits > max_splits)
        splits = max_splits;
    if (splits < 1)
        splits = 1;
    p.most_splits = splits;  // (grows with the pixels, where the rounded p.splits may not)
    p.per_split = (pixels + splits - 1) / splits;
    const int chunk = p.wo * p.wc == 1 ? 2 * kChunk : kChunk;
    p.per_split = (p.per_split + chunk - 1) / chunk * chunk;
    p.splits = int((pixels + p.per_split - 1) / p.per_split);
    return p;
}

}  // namespace

size_t qconv2d_wgrad_work_bytes(const ConvGeom &g, DType dt)
{
    // Enough for every smaller batch of the layer too, so that one that has run
    // can be captured with fewer images: a row plan's room also where only its
    // 32-bit spans refused it, and the tiles' where fewer pixels go to them.
    const WgradRows r = qconv2d_wgrad_rows_plan(g, dt);
    const size_t dw = size_t(g.k_h) * g.k_w * g.c_out * g.c_in * sizeof(float);
    const size_t rows = size_t(r.most_splits) * r.segs * (r.fold ? 4 * 2 : 16) * dw;  // (fp64 with fold)
    const size_t tiles = size_t(wgrad_plan(g, dt).most_splits) * 4 * dw;
    const size_t b_part = size_t(kBiasBlocks) * 4 * g.c_out * sizeof(float);
    return std::max(std::max(rows, tiles), b_part);
}

hipError_t qconv2d_backward_weight_run(const ConvGeom &g, DType dt, const void *x, const void *dy, float *dw_r,
                                       float *dw_i, float *dw_j, float *dw_k, float *db, void *work,
                                       hipStream_t stream, bool sep)
{
    float *const part = static_cast<float *>(work);
    const int taps = g.k_h * g.k_w;
    const WgradRows r = qconv2d_wgrad_rows_plan(g, dt);
    int slices = r.splits * r.segs;
    hipError_t e;
    if (r.takes) {
        e = qconv2d_wgrad_rows_run(r, g, dt, x, dy, part, stream, sep);
    } else {
        const WPlan p = wgrad_plan(g, dt);
        slices = p.splits;
        WArgs a;
        a.x = x;
        a.dy = dy;
        a.part = part;
        a.n = g.n;
        a.c_in = g.c_in;
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
        a.pixels = g.m();
        a.per_split = p.per_split;
        a.o_tiles = p.o_tiles;
        a.c_tiles = p.c_tiles;
        a.taps = p.taps;
        a.groups = p.splits * p.c_tiles * p.o_tiles;
        const unsigned blocks = unsigned(int64_t(8) * p.taps * ((a.groups + 7) / 8));
        const int epc = dt == DType::BF16 ? 8 : 4, es = dt == DType::BF16 ? 2 : 4;
        // the 16-byte buffer loads take 32-bit offsets within a slice's pixels
        // of dY and the images of X it touches
        const int64_t hw_out = int64_t(g.h_out) * g.w_out;
        const int64_t dy_span = p.per_split * 4 * g.c_out * es;
        const int64_t x_span = ((p.per_split + hw_out - 1) / hw_out + 1) * g.h * g.w * 4 * g.c_in * es;
        const bool vec = a.c_in % epc == 0 && a.c_out % epc == 0 && dy_span < 0x7fffffffLL && x_span < 0x7fffffffLL;
        auto launch = [&](auto t, auto v, auto sp) {
            auto tile = [&](auto wo, auto wc) {
                constexpr int WO = decltype(wo)::value, WC = decltype(wc)::value;
                hipLaunchKernelGGL((qconv2d_wgrad<decltype(t), decltype(v)::value, decltype(sp)::value, WO, WC,
                                                  4 / (WO * WC)>),
                                   dim3(blocks), dim3(kThreads), 0, stream, a);
            };
            using One = std::integral_constant<int, 1>;
            using Two = std::integral_constant<int, 2>;
            if (p.wo == 1)
                p.wc == 1 ? tile(One{}, One{}) : tile(One{}, Two{});
            else
                p.wc == 1 ? tile(Two{}, One{}) : tile(Two{}, Two{});
        };
        using Yes = std::true_type;
        using No = std::false_type;
        auto form = [&](auto t, auto v) { sep ? launch(t, v, Yes{}) : launch(t, v, No{}); };
        if (dt == DType::BF16)
            vec ? form(__bf16{}, Yes{}) : form(__bf16{}, No{});
        else
            vec ? form(float{}, Yes{}) : form(float{}, No{});
        e = hipGetLastError();
    }
    if (e != hipSuccess)
        return e;
    // as many threads to an output as its slices keep busy (70 -> 70, 25 taps, dense
    // in 2 slices, whole call: 74.3 us with sixteen, 62.7 with one)
    const int64_t outs = int64_t(4) * g.c_out * g.c_in * taps;
    using One = std::integral_constant<int, 1>;
    using Four = std::integral_constant<int, 4>;
    using Sixteen = std::integral_constant<int, 16>;
    if (r.takes && !r.fold) {
        auto reduce = [&](auto sgc) {
            constexpr int SG = decltype(sgc)::value, per_block = kThreads / SG;
            hipLaunchKernelGGL((qconv2d_wgrad_reduce_dense<SG>), dim3(unsigned((outs + per_block - 1) / per_block)),
                               dim3(kThreads), 0, stream, (const float *)part, slices, taps, g.c_out, g.c_in,
                               sep ? 1 : 0, dw_r, dw_i, dw_j, dw_k);
        };
        if (slices >= 12)
            reduce(Sixteen{});
        else if (slices >= 3)
            reduce(Four{});
        else
            reduce(One{});
    } else {
        auto launch = [&](auto of, auto sgc, auto uc) {
            using P = decltype(of);
            constexpr int SG = decltype(sgc)::value, U = decltype(uc)::value;
            const int64_t blocks = (outs + kThreads / SG * 4 - 1) / (kThreads / SG * 4);
            const int seg = int((blocks + 4 * taps - 1) / (4 * taps));
            hipLaunchKernelGGL((qconv2d_wgrad_reduce<P, SG, U>), dim3(unsigned(4 * taps) * unsigned(seg)),
                               dim3(kThreads), 0, stream, reinterpret_cast<const P *>(part), slices, taps,
                               g.c_out * g.c_in, seg, dw_r, dw_i, dw_j, dw_k);
        };
        auto reduce = [&](auto sgc, auto uc) { r.takes ? launch(double{}, sgc, uc) : launch(float{}, sgc, uc); };
        if (slices >= 64)
            reduce(Sixteen{}, std::integral_constant<int, 8>{});
        else if (slices >= 12)
            reduce(Sixteen{}, Four{});
        else if (slices >= 3)
            reduce(Four{}, std::integral_constant<int, 3>{});
        else
            reduce(One{}, Four{});
    }
    e = hipGetLastError();
    if (e != hipSuccess || db == nullptr)
        return e;
    // the partials of dW are consumed: reuse the workspace for the bias
    const int cols = 4 * g.c_out;
    const int64_t pixels = g.m();
    const int64_t rpb = (pixels + kBiasBlocks - 1) / kBiasBlocks;
    const int nb = int((pixels + rpb - 1) / rpb);
    const int vw = cols % (dt == DType::BF16 ? 8 : 4) == 0 ? (dt == DType::BF16 ? 8 : 4) : 1;
    const int chunks = cols / vw;
    const int cg = chunks < kThreads ? chunks : kThreads;
    const dim3 grid(nb, (chunks + cg - 1) / cg);
    if (dt == DType::BF16) {
        if (vw == 8)
            hipLaunchKernelGGL((colsum_partial<__bf16, 8>), grid, dim3(kThreads), 0, stream, (const __bf16 *)dy,
                               pixels, cols, rpb, part);
        else
            hipLaunchKernelGGL((colsum_partial<__bf16, 1>), grid, dim3(kThreads), 0, stream, (const __bf16 *)dy,
                               pixels, cols, rpb, part);
    } else {
        if (vw == 4)
            hipLaunchKernelGGL((colsum_partial<float, 4>), grid, dim3(kThreads), 0, stream, (const float *)dy,
                               pixels, cols, rpb, part);
        else
            hipLaunchKernelGGL((colsum_partial<float, 1>), grid, dim3(kThreads), 0, stream, (const float *)dy,
                               pixels, cols, rpb, part);
    }
    hipLaunchKernelGGL(colsum_final, dim3((cols + kThreads / 64 - 1) / (kThreads / 64)), dim3(kThreads), 0, stream,
                       (const float *)part, nb, cols, db);
    return hipGetLastError();
}

}  // namespace quan
