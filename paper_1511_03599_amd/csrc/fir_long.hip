// Polyphase FIR for tap counts beyond the register window (T > 64), and for
// 33 to 64 taps where it is the faster one (fir_segments_pay in api.hip): the
// FIR of Algorithm 1, y[s][c] = sum_{t<T} h[t][c] x[s+t][c].
//
// One wave owns 64 adjacent channels (one per lane) of a tile of N = 16
// filtered spectra and keeps the tile's N complex sums in registers. It walks
// the taps in segments of N, down the tile once per segment. The register
// window of N raw rows slides on from one segment to the next: the N - 1 rows
// that a segment starts with are those that the one before ended on, so a
// tile reads each of its N + T - 1 raw rows once. Each sum takes its taps in
// ascending order from one accumulator, so the result is the sequential sum a
// single window of T taps would give. Zero taps fill the segments, a.shift of
// them in front, the others behind: for finite samples they add exact zeros,
// an infinity or NaN under one of them makes the sum NaN. Rows are shared by
// T / N tiles; the caches serve the re-reads.
//
// Rows, taps and stores go through bounded views of one row's 64 channels,
// empty outside the stream, the filter or the tile: every load is
// unconditional, so a wait covers no more than the row that enters the
// window. The next segment's taps are loaded while this one runs.
//
// Bound: VALU, 2T FMAs per sample: 65-85% of it at 2.3 GHz in large calls; the
// rest is moves, conversions and the waits that three waves per SIMD leave. With
// segments and tiles of 32, whose window was loaded again for every segment
// and whose registers allowed two waves (one for float16): 1024 channels,
// 65536 spectra, 128 taps complex64 706 -> 711 us (the chip's power limit),
// int8 605 -> 537, 192 taps complex64 976 -> 909; 4096 channels, 104 taps,
// 8354 spectra float16 464 -> 272; 256 channels, 100 taps, 3000 spectra
// complex64 46 -> 17. The sliding window with N = 32 does not fit the
// registers of two waves (788 us for the first of these).
#include "device_common.h"
#include "launch.h"

namespace pfb {

constexpr unsigned FIR_LONG_GRID = 1 << 20; // workgroups along x (a dimension holds under 2^32 threads)

// LEAD: a.shift zero taps come first (the counters that keep them and the rows
// before the stream out cost long filters 5 to 10%).
template <int DT, bool LEAD> __global__ __launch_bounds__(256, 3) void fir_long_kernel(FirArgs a)
{
    constexpr int N = FIR_LONG_ROWS;
    constexpr int D = 4; // rows in flight ahead of the window
    constexpr int SB = SampleBytes<DT>::value;
    static_assert(N % D == 0, "the ring repeats with the segments");
    // scalar task index: tile, row and address bases stay in scalar registers
    const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t gw = block * (blockDim.x >> 6) + wave_id_uniform();
    const int64_t total = (int64_t)a.B * a.n_tiles * a.n_cchunks;
    if (gw >= total)
        return;
    const int cch = (int)(gw % a.n_cchunks);
    const int64_t rest = gw / a.n_cchunks;
    const int tile = (int)(rest % a.n_tiles);
    const int b = (int)(rest / a.n_tiles);
    const int lane = lane_id();
    const int cw = a.C - cch * 64 < 64 ? a.C - cch * 64 : 64; // channels of this wave
    const int64_t s_begin = a.out_first + (int64_t)tile * N;
    const int64_t left_out = a.out_first + a.out_count - s_begin;
    const int nout = (int)(left_out < N ? left_out : N);

    // the next raw row and tap row to load, and how many there are; `lead`
    // of the rows lie before the stream
    const int shift = LEAD ? a.shift : 0;
    const int64_t row_bytes = (int64_t)a.C * SB, tap_bytes = (int64_t)a.C * 4;
    const char *xp = reinterpret_cast<const char *>(a.x) +
                     ((int64_t)b * a.in_bstride + (s_begin - shift) * a.C + (int64_t)cch * 64) * SB;
    const char *hp_next = reinterpret_cast<const char *>(a.h) + (int64_t)cch * 64 * 4 - shift * tap_bytes;
    const int64_t left_in = a.in_rows - s_begin + shift;
    int rows_left = (int)(left_in < 0x40000000 ? left_in : 0x40000000);
    int lead = s_begin < shift ? shift - (int)s_begin : 0, taps_left = a.T + shift;
    auto ld = [&](Packed<DT, 1> &o) PFB_INLINE {
        buf_load_packed<DT, 1>(buf_view(xp, (!LEAD || lead <= 0) && rows_left > 0 ? cw * SB : 0), lane * SB, o);
        xp += row_bytes;
        --rows_left;
        --lead;
    };
    auto ld_tap = [&](float &o) PFB_INLINE {
        Packed<DT_CI16, 1> t; // 4 bytes
        buf_load_packed<DT_CI16, 1>(buf_view(hp_next, taps_left > 0 && (!LEAD || taps_left <= a.T) ? cw * 4 : 0), lane * 4, t);
        o = __uint_as_float(t.w[0]);
        hp_next += tap_bytes;
        --taps_left;
    };

    float2 acc[N];
    sfor<N>([&](auto o) PFB_INLINE { acc[o] = make_float2(0.0f, 0.0f); });
    float hp[N], hn[N];
    float2 w[N][1];
    Packed<DT, 1> pf[D];
    sfor<N>([&](auto j) PFB_INLINE { ld_tap(hp[j]); });
    {
        Packed<DT, 1> first[N - 1];
        sfor<N - 1>([&](auto j) PFB_INLINE { ld(first[j]); });
        sfor<D>([&](auto k) PFB_INLINE { ld(pf[k]); });
        sfor<N - 1>([&](auto j) PFB_INLINE { unpack<DT, 1>(first[j], w[j]); });
    }
#pragma unroll 1
    for (int g = (a.T + shift + N - 1) / N; g > 0; --g) {
        // sum o reads window rows o + j, j < N, of which row o + N - 1 is new
        sfor<N>([&](auto oc) PFB_INLINE {
            constexpr int o = decltype(oc)::value;
            unpack<DT, 1>(pf[o % D], w[(o + N - 1) % N]);
            ld(pf[o % D]);
            if constexpr (2 * o < N) {
                ld_tap(hn[2 * o]);
                ld_tap(hn[2 * o + 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
            float ar = acc[o].x, ai = acc[o].y;
            sfor<N>([&](auto jc) PFB_INLINE {
                constexpr int j = decltype(jc)::value;
                ar = __builtin_fmaf(hp[j], w[(o + j) % N][0].x, ar);
                ai = __builtin_fmaf(hp[j], w[(o + j) % N][0].y, ai);
            });
            acc[o] = make_float2(ar, ai);
        });
        sfor<N>([&](auto j) PFB_INLINE { hp[j] = hn[j]; });
    }
    float2 *yp = a.y + (int64_t)b * a.y_bstride + (s_begin - a.out_first) * a.C + (int64_t)cch * 64;
    sfor<N>([&](auto oc) PFB_INLINE {
        constexpr int o = decltype(oc)::value;
        const float2 v[1] = {acc[o]};
        buf_store_c64_nt<1>(buf_view(yp, o < nout ? cw * 8 : 0), lane * 8, v);
        yp += a.C;
    });
}

template <bool LEAD> static hipError_t launch_fir_long_lead(const FirArgs &a, int dtype, hipStream_t st)
{
    const int64_t waves = (int64_t)a.B * a.n_tiles * a.n_cchunks;
    const int64_t blocks = (waves + 3) / 4;
    if (blocks <= 0)
        return hipSuccess;
    const unsigned gx = (unsigned)(blocks < FIR_LONG_GRID ? blocks : FIR_LONG_GRID);
    const dim3 grid(gx, (unsigned)((blocks + gx - 1) / gx)), block(256);
    switch (dtype) {
    case DT_C64: hipLaunchKernelGGL((fir_long_kernel<DT_C64, LEAD>), grid, block, 0, st, a); break;
    case DT_CI16: hipLaunchKernelGGL((fir_long_kernel<DT_CI16, LEAD>), grid, block, 0, st, a); break;
    case DT_CI8: hipLaunchKernelGGL((fir_long_kernel<DT_CI8, LEAD>), grid, block, 0, st, a); break;
    case DT_CF16: hipLaunchKernelGGL((fir_long_kernel<DT_CF16, LEAD>), grid, block, 0, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fir_long(FirArgs a, int dtype, hipStream_t st)
{
    a.SB = FIR_LONG_ROWS;
    a.n_tiles = (int)((a.out_count + FIR_LONG_ROWS - 1) / FIR_LONG_ROWS);
    a.n_cchunks = (int)(((int64_t)a.C + 63) / 64);
    return a.shift > 0 ? launch_fir_long_lead<true>(a, dtype, st) : launch_fir_long_lead<false>(a, dtype, st);
}

} // namespace pfb
