// Mixed-radix C-point FFT for channel counts that are not powers of two
// (C = 2^a 3^b 5^c 7^d): the DFT of Sec. 2, Eq. (2), unnormalised, natural
// bin order; the inverse (exp(+...)) as conjugate in, conjugate out.
//
// Stockham autosort, one pass per radix of the schedule. A pass of radix R
// and stride L (the product of the earlier radices) lets butterfly j
// (0 <= j < C/R) read elements j + i*C/R, multiply element i by W_{RL}^{ik}
// (k = j mod L), run an R-point DFT and write element i to
// (j - k) R + k + i L. The first pass reads the row from HBM and the last
// writes it there, both coalesced; in between the row lives in one padded LDS
// buffer: a lane holds the inputs of all its butterflies before any lane
// writes. Twiddles come from a table per pass
// laid out [i][k], so that neighbouring lanes read neighbouring entries.
//
// Radices up to 16, composites of coprime factors (6, 10, 12, 14, 15) by the
// prime-factor map, so without inner twiddles: 3072 channels take three
// passes (16, 16, 12), 1344 three (14, 12, 8), 6144 four (12, 8, 8, 8). With
// the factors 16, 8, 4, 2, 7, 5, 3 one by one (3072: 16, 16, 4, 3), two LDS
// buffers per row, unpadded, and a division by L in the lane, the transforms
// of 2^27 samples took 686 us at 3072 channels (now 432, 5.0 TB/s), 952 at
// 6144 (478) and 608 at 1536 (433). Bound: HBM and, above 4096 channels, the
// barriers of a fourth pass.
//
// A group of G lanes owns one row: as many as the pass with the most
// butterflies per gf_butterflies(R) asks for, rounded to a power of two up to
// a wave (several rows per block of 256 lanes), to whole waves above (one row
// per block).
//
// Stores and lines. A group that writes less than a 128-byte line at a time
// stores through L2, which gathers the lines: groups of fewer than 16 lanes
// (96 channels, 2^20 spectra: non-temporal 935 us, plain 389; from 16 lanes on
// non-temporal is the faster, 240 channels 286 to 303). So does a group of 16
// whose rows start off the 64-byte sectors and whose last pass gives a lane
// several butterflies: the pieces of a line are then written a butterfly
// apart. T = 1, 2^26 samples, FIR and transform, with a wave per row and one
// radix per factor, with non-temporal stores, and now: 175 channels 616, 806,
// 547 us; 147 660, 779, 561; 125 698, 780, 548; 162 610, 665, 502. (200
// channels, on the sectors, 520, 424 and 448 with plain stores; 168, one
// butterfly a lane, 548, 432 and 463.)
// Rows off the lines gain from one sweep per pass too: groups of 32 take a
// wave where every pass then has work for most lanes (343 channels 498, 582,
// 504; 294 544, 526, 490; 250, whose first pass would use 25 lanes, 529, 506,
// 528 with a wave).
#include <algorithm>

#include "fft_device.h"
#include "launch.h"

namespace pfb {

// Butterflies of radix R per lane, at most: one from radix 9 up (two of 15
// with their twiddles would take all registers of two waves per SIMD), up to
// 16 elements below.
constexpr int gf_butterflies(int R) { return R > 8 ? 1 : 16 / R; }

// cos(2 pi m / R) and sin(2 pi m / R) for the odd radices.
template <int R> struct OddTw;
template <> struct OddTw<3> {
    static constexpr float c[3] = {1.0f, -0.5f, -0.5f};
    static constexpr float s[3] = {0.0f, 0.86602540378443865f, -0.86602540378443865f};
};
template <> struct OddTw<5> {
    static constexpr float c[5] = {1.0f, 0.30901699437494742f, -0.80901699437494742f, -0.80901699437494742f,
                                   0.30901699437494742f};
    static constexpr float s[5] = {0.0f, 0.95105651629515357f, 0.58778525229247314f, -0.58778525229247314f,
                                   -0.95105651629515357f};
};
template <> struct OddTw<7> {
    static constexpr float c[7] = {1.0f, 0.62348980185873353f, -0.22252093395631440f, -0.90096886790241913f,
                                   -0.90096886790241913f, -0.22252093395631440f, 0.62348980185873353f};
    static constexpr float s[7] = {0.0f, 0.78183148246802981f, 0.97492791218182361f, 0.43388373911755812f,
                                   -0.43388373911755812f, -0.97492791218182361f, -0.78183148246802981f};
};

// R-point DFT (R odd) in place, exp(-2 pi i nk / R), by symmetric pairs:
// with a_n = v_n + v_{R-n}, b_n = v_n - v_{R-n} (n = 1..(R-1)/2),
//   P_k = v_0 + sum_n cos(2 pi nk/R) a_n,  Q_k = sum_n sin(2 pi nk/R) b_n,
//   X_k = P_k - i Q_k,  X_{R-k} = P_k + i Q_k.
template <int R> __device__ __forceinline__ void dft_odd(float2 *v)
{
    constexpr int H = (R - 1) / 2;
    float2 a[H + 1], b[H + 1];
    float2 x0 = v[0];
    sfor<H>([&](auto nc) PFB_INLINE {
        constexpr int n = decltype(nc)::value + 1;
        a[n] = cadd(v[n], v[R - n]);
        b[n] = csub(v[n], v[R - n]);
    });
    float2 s0 = x0;
    sfor<H>([&](auto nc) PFB_INLINE { s0 = cadd(s0, a[decltype(nc)::value + 1]); });
    float2 out[R];
    out[0] = s0;
    sfor<H>([&](auto kc) PFB_INLINE {
        constexpr int k = decltype(kc)::value + 1;
        float px = x0.x, py = x0.y, qx = 0.0f, qy = 0.0f;
        sfor<H>([&](auto nc) PFB_INLINE {
            constexpr int n = decltype(nc)::value + 1;
            constexpr float c = OddTw<R>::c[(n * k) % R];
            constexpr float s = OddTw<R>::s[(n * k) % R];
            px = __builtin_fmaf(c, a[n].x, px);
            py = __builtin_fmaf(c, a[n].y, py);
            qx = __builtin_fmaf(s, b[n].x, qx);
            qy = __builtin_fmaf(s, b[n].y, qy);
        });
        out[k] = make_float2(px + qy, py - qx);     // P - iQ
        out[R - k] = make_float2(px - qy, py + qx); // P + iQ
    });
    sfor<R>([&](auto i) PFB_INLINE { v[i] = out[i]; });
}

template <int R> __device__ __forceinline__ void dft_any(float2 *v);

constexpr int inverse_mod(int a, int n)
{
    for (int x = 1; x < n; ++x)
        if (a * x % n == 1)
            return x;
    return 0;
}

// N1 * N2 points, N1 and N2 coprime: with n = N2 n1 + N1 n2 and
// k = N2 (N2^-1 mod N1) k1 + N1 (N1^-1 mod N2) k2 (all mod N1 N2),
// W_N^{nk} = W_N1^{n1 k1} W_N2^{n2 k2}.
template <int N1, int N2> __device__ __forceinline__ void dft_pfa(float2 *v)
{
    constexpr int N = N1 * N2, E1 = N2 * inverse_mod(N2 % N1, N1), E2 = N1 * inverse_mod(N1 % N2, N2);
    float2 a[N2][N1];
    sfor<N2>([&](auto n2) PFB_INLINE {
        sfor<N1>([&](auto n1) PFB_INLINE {
            a[n2][n1] = v[(N2 * decltype(n1)::value + N1 * decltype(n2)::value) % N];
        });
        dft_any<N1>(a[n2]);
    });
    sfor<N1>([&](auto k1) PFB_INLINE {
        float2 b[N2];
        sfor<N2>([&](auto n2) PFB_INLINE { b[n2] = a[n2][k1]; });
        dft_any<N2>(b);
        sfor<N2>([&](auto k2) PFB_INLINE {
            v[(E1 * decltype(k1)::value + E2 * decltype(k2)::value) % N] = b[k2];
        });
    });
}

template <int R> __device__ __forceinline__ void dft_any(float2 *v)
{
    if constexpr (R == 3 || R == 5 || R == 7)
        dft_odd<R>(v);
    else if constexpr (R == 6)
        dft_pfa<2, 3>(v);
    else if constexpr (R == 10)
        dft_pfa<2, 5>(v);
    else if constexpr (R == 12)
        dft_pfa<4, 3>(v);
    else if constexpr (R == 14)
        dft_pfa<2, 7>(v);
    else if constexpr (R == 15)
        dft_pfa<3, 5>(v);
    else
        Dft<R>::run(v);
}

// Place of element idx in the row's LDS buffer.
__device__ __forceinline__ int gf_pad(int idx) { return idx + (idx >> 4); }

// Element idx of a row at a (wave-uniform) base: a 32-bit offset per lane.
template <class T> __device__ __forceinline__ T &gf_at(T *base, uint32_t idx)
{
    return *(T *)((__attribute__((address_space(1))) char *)(uintptr_t)base + idx * 8u);
}

// One pass of radix R over the row; MULTI: the group spans several waves.
template <int R, bool FIRST, bool LAST, bool INV, bool MULTI>
__device__ __forceinline__ void gf_pass(const GfftPass ps, int C, int G, bool nt, int lane, const float2 *in,
                                        float2 *out, float2 *row, const float2 *tw)
{
    constexpr int NB = gf_butterflies(R); // C/R <= NB * G
    const int CR = C / R, L = ps.stride;
    float2 v[NB][R];
    int o[NB];
    sfor<NB>([&](auto q) PFB_INLINE {
        const int j = lane + G * decltype(q)::value;
        if (j < CR) {
            if constexpr (FIRST) {
                o[q] = j * R;
                sfor<R>([&](auto i) PFB_INLINE {
                    const float2 z = gf_at(in, (uint32_t)(j + decltype(i)::value * CR));
                    v[q][i] = INV ? conj2(z) : z;
                });
            } else {
                const int k = j - (int)__umulhi((uint32_t)j, ps.magic) * L;
                o[q] = (j - k) * R + k;
                float2 w[R];
                sfor<R - 1>([&](auto i) PFB_INLINE { w[i + 1] = gf_at(tw, (uint32_t)(ps.tw + k + (decltype(i)::value + 1) * L)); });
                sfor<R>([&](auto i) PFB_INLINE { v[q][i] = row[gf_pad(j + decltype(i)::value * CR)]; });
                sfor<R - 1>([&](auto i) PFB_INLINE { v[q][i + 1] = cmul(v[q][i + 1], w[i + 1]); });
            }
            dft_any<R>(v[q]);
            if constexpr (LAST) // (j - k) R + k is j: L R = C
                sfor<R>([&](auto i) PFB_INLINE {
                    float2 *d = &gf_at(out, (uint32_t)(j + decltype(i)::value * CR));
                    const float2 z = INV ? conj2(v[q][i]) : v[q][i];
                    if (MULTI || nt)
                        store_nt(d, z);
                    else // less than a line at a time
                        *d = z;
                });
        }
        // one butterfly's addresses and twiddles at a time in registers
        __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (!LAST) {
        if constexpr (!FIRST)
            group_sync<MULTI ? 128 : 64>(); // every lane has read before any lane writes
        sfor<NB>([&](auto q) PFB_INLINE {
            if (lane + G * decltype(q)::value < CR)
                sfor<R>([&](auto i) PFB_INLINE { row[gf_pad(o[q] + decltype(i)::value * L)] = v[q][i]; });
        });
        group_sync<MULTI ? 128 : 64>();
    }
}

template <bool FIRST, bool LAST, bool INV, bool MULTI>
__device__ __forceinline__ void gf_pass_any(const GfftPass ps, int C, int G, bool nt, int lane, const float2 *in,
                                            float2 *out, float2 *row, const float2 *tw)
{
#define PFB_GF(R)                                                                                            \
    case R: gf_pass<R, FIRST, LAST, INV, MULTI>(ps, C, G, nt, lane, in, out, row, tw); break;
    switch (ps.radix) {
        PFB_GF(16)
        PFB_GF(15)
        PFB_GF(14)
        PFB_GF(12)
        PFB_GF(10)
        PFB_GF(8)
        PFB_GF(7)
        PFB_GF(6)
        PFB_GF(5)
        PFB_GF(4)
        PFB_GF(3)
    default:
        gf_pass<2, FIRST, LAST, INV, MULTI>(ps, C, G, nt, lane, in, out, row, tw);
    }
#undef PFB_GF
}

// MAXT: threads per block at most (256: groups within a wave).
template <bool INV, int MAXT>
__global__ __launch_bounds__(MAXT) void gfft_kernel(FftArgs a, GfftSched s)
{
    constexpr bool MULTI = MAXT > 256;
    extern __shared__ float2 gf_lds[];
    const int C = s.C, G = s.group;
    const int grp = MULTI ? 0 : (int)threadIdx.x / G;
    const int lane = MULTI ? (int)threadIdx.x : (int)threadIdx.x % G;
    const int64_t r0 = (int64_t)blockIdx.x * s.rows_per_block + grp;
    // MULTI: one row per block, so the exit is block-uniform; otherwise a
    // group past the last row may leave, there is no block barrier
    if (r0 >= a.nrows)
        return;
    const int64_t g = r0 / a.rows_per_group, r = r0 % a.rows_per_group;
    const float2 *in = a.in + g * a.in_gstride + r * C;
    float2 *out = a.out + g * a.out_gstride + r * C;
    float2 *row = gf_lds + grp * (C + C / 16 + 1);
    gf_pass_any<true, false, INV, MULTI>(s.pass[0], C, G, s.nt, lane, in, out, row, a.tw);
    for (int p = 1; p + 1 < s.npass; ++p) {
        // opaque: every radix's addresses would be hoisted out of the loop
        int ln = lane;
        asm volatile("" : "+v"(ln));
        gf_pass_any<false, false, INV, MULTI>(s.pass[p], C, G, s.nt, ln, in, out, row, a.tw);
    }
    gf_pass_any<false, true, INV, MULTI>(s.pass[s.npass - 1], C, G, s.nt, lane, in, out, row, a.tw);
}

// The fewest radices whose product is `rem`, none above `most`; of those the
// smallest sum (the flattest schedule). Returns the count, or 0.
static int gfft_factor(int rem, int most, int depth, int *best, int *best_sum, int sum, int *cur, int n, int found)
{
    if (rem == 1) {
        if (found == 0 || n < found || (n == found && sum < *best_sum)) {
            std::copy(cur, cur + n, best);
            *best_sum = sum;
            return n;
        }
        return found;
    }
    if (n == depth || (found && n + 1 > found))
        return found;
    for (int r : {16, 15, 14, 12, 10, 8, 7, 6, 5, 4, 3, 2})
        if (r <= most && rem % r == 0) {
            cur[n] = r;
            found = gfft_factor(rem / r, r, depth, best, best_sum, sum + r, cur, n + 1, found);
        }
    return found;
}

// Radix schedule of a 7-smooth C (false if C has another prime factor).
bool gfft_schedule(int C, GfftSched *s)
{
    if (C < 17 || C > 8192)
        return false; // the kernel's first and last passes are distinct
    int radix[GF_MAX_PASS], cur[GF_MAX_PASS], sum = 0;
    const int np = gfft_factor(C, 16, GF_MAX_PASS, radix, &sum, 0, cur, 0, 0);
    if (np < 2)
        return false;
    GfftSched t{};
    t.C = C;
    t.npass = np;
    int L = 1;
    for (int p = 0; p < np; ++p) {
        GfftPass &q = t.pass[p];
        q.radix = radix[p];
        q.stride = L;
        q.magic = (uint32_t)((((uint64_t)1 << 32) + (uint64_t)L - 1) / (uint64_t)L); // 0 for L = 1, unused
        q.tw = t.tw_entries;
        if (p > 0)
            t.tw_entries += radix[p] * L;
        L *= radix[p];
    }
    int lanes = 1;
    for (int p = 0; p < np; ++p) {
        const int per = radix[p] * gf_butterflies(radix[p]);
        lanes = std::max(lanes, (C + per - 1) / per);
    }
    const int first = C / radix[0], last = C / radix[np - 1]; // butterflies of the largest and the smallest radix
    if (C % 16 != 0 && lanes > 16 && lanes <= 32 && first <= 64 && first >= (C % 8 != 0 ? 35 : 48))
        lanes = 64;
    if (lanes <= 64) {
        t.group = 1;
        while (t.group < lanes)
            t.group *= 2;
        t.rows_per_block = 256 / t.group;
    } else {
        t.group = (lanes + 63) / 64 * 64;
        t.rows_per_block = 1;
    }
    t.nt = t.group > 16 || (t.group == 16 && (C % 8 == 0 || last <= 16));
    *s = t;
    return true;
}

hipError_t launch_gfft(const FftArgs &a, const GfftSched &s, bool inv, hipStream_t st)
{
    const int64_t blocks = (a.nrows + s.rows_per_block - 1) / s.rows_per_block;
    if (blocks <= 0)
        return hipSuccess;
    const size_t lds = (size_t)s.rows_per_block * (s.C + s.C / 16 + 1) * sizeof(float2);
    const dim3 grid((unsigned)blocks), block((unsigned)(s.group * s.rows_per_block));
    auto k = s.group <= 64   ? (inv ? gfft_kernel<true, 256> : gfft_kernel<false, 256>)
             : s.group <= 512 ? (inv ? gfft_kernel<true, 512> : gfft_kernel<false, 512>)
                              : (inv ? gfft_kernel<true, 1024> : gfft_kernel<false, 1024>);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k, grid, block, lds, st, a, s);
    return hipGetLastError();
}

} // namespace pfb
