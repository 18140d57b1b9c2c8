// FIR + FFT in one launch for the shapes whose register window does not fit
// one workgroup (fused_launch.h covers C in {256, 512, 1024} at T <= 16), and
// for the polarisation-interleaved sub-bands. Instantiated per input type and
// group of sizes in separate translation units (block_<type>_<group>.hip).
//
// A persistent workgroup of 512 threads takes blocks of filtered spectra.
// The LDS holds the filtered values of R of them (R * C = 16384 samples);
// a block is H * R spectra, H = 2 from C = 1024. Per block:
//   1. FIR: a thread owns V adjacent columns of RT2 = H * RT rows and walks
//      the RT2 + TP - 1 raw rows they need, one sum per row and column in
//      registers. Every raw sample is loaded and converted once per thread
//      that needs it and the taps are read again for every block, where the
//      register window reads both once: L2 serves the difference, because
//      the blocks that share raw rows run at the same time on one XCD and
//      the taps are the same for all. The first R rows go to the LDS, the
//      other half waits in registers (32 sums per thread): with H = 2 a raw
//      row is read (2R + TP - 1) / 2R times instead of (R + TP - 1) / R, and
//      the taps half as often.
//   2. FFT of the R rows in the LDS, the last pass writing the spectra to
//      HBM; then the waiting half takes its place.
// The filtered spectra never reach HBM: 16 bytes per complex64 sample
// instead of 32 for a FIR launch and an FFT launch.
//
// The raw rows form one sequence over all passes and blocks of a workgroup,
// and a ring of D rows per thread is in flight ahead of the sums, across the
// transforms too. Every load goes through a bounded view, which returns
// zeros outside the stream, so no load sits under a branch.
//
// Bound: one workgroup per CU (LDS), two waves per SIMD, so FIR and FFT
// phases of a CU do not overlap; at 4096 channels, 16 taps and int8 input the
// VALU issues 64% of the time (86 operations per sample). Measured against
// FIR + FFT launches (2^27 samples, 16 taps): 4096 channels int8 0.66 -> 0.39
// ms, complex64 0.78 -> 0.52; 2048 channels complex64 0.79 -> 0.50; 1024
// channels, 32 taps, 2^26 samples 0.40 -> 0.27; 8 sub-bands of 4096 channels,
// int8, 2^27 samples 0.92 -> 0.42. With H = 1: 0.49, 0.65, 0.53, 0.29, 0.60.
// Two workgroups of half the rows and threads per CU, which would overlap
// their phases, read more through L2 and were slower (4096 channels int8
// 0.48, complex64 0.68 with H = 2). Blocks dealt to the XCDs one by one
// instead of in runs: 2048 channels complex64 0.78 against 0.52 (H = 1).
//
// Registers: 256, the most that two waves per SIMD leave. The 16-tap windows
// of four columns spill beyond them: int16 13, 13 and 15 and float16 15, 9
// and 13 registers at 2048, 4096 and 8192 channels, int8 7 at 8192 (32 to 64
// bytes of scratch a lane); no other instance does.
//
// Sums take their taps in ascending order from one accumulator, with the taps
// zero-padded at the front to TP, and the transform's radices, twiddles and
// order of operations are the split path's: both give the same bits (at 33 to
// 64 taps for finite samples: the split path's long-tap FIR pads less).
#pragma once

#include "fft_device.h"
#include "launch.h"

namespace pfb {

constexpr int block_ring(int lp, int most)
{
    for (int d = most; d > 1; --d)
        if (d < lp && lp % d == 0)
            return d;
    return 1;
}

// Transforms that span several waves (C >= 2048: passes of radix R, R and Q).
// Element c of a row sits in sub-row c mod Q at place c / Q. Butterfly j of
// the first pass feeds only second-pass butterflies whose inputs all come
// from butterflies of the same j mod Q, so the first two passes are Q
// independent R*R-point transforms of R lanes each, inside a wave and
// without a barrier; the last pass combines place j of all sub-rows. The
// spacing of the sub-rows spreads adjacent columns over the LDS banks.
// (With the split path's form, a barrier around every pass, the transforms
// of a block took 334 us per 2^27 samples at 4096 channels; now 226.)
template <int LOG2C> struct BigFft {
    static constexpr int R = fft_elems_per_lane(LOG2C);
    static constexpr int RR = R * R;
    static constexpr int Q = (1 << LOG2C) / RR;
    static constexpr int SUB = RR + RR / 16 + (Q == 4 ? 4 : 2);
    static constexpr int ROW = Q * SUB;
    static_assert(Q == 4 || Q == 8, "radices R, R, Q");
};

constexpr int BLOCK_NT = 512;          // threads per workgroup
constexpr int BLOCK_SAMPLES = 16384;   // filtered samples in the LDS

// POL: the columns of a row are the channels of one sub-band with two
// interleaved polarisations; a block then holds both polarisations.
template <int DT, int TP, int LOG2C, bool POL> struct BlockShape {
    static constexpr int C = 1 << LOG2C;
    static constexpr int NT = BLOCK_NT;
    static constexpr int H = LOG2C >= 10 ? 2 : 1;
    static constexpr int TROWS = BLOCK_SAMPLES / C;       // transforms in the LDS
    static constexpr int R = POL ? TROWS / 2 : TROWS;     // filtered spectra in the LDS
    // columns per thread: 16-byte complex64 loads and 8-byte ones of the
    // smaller types (4096 channels, int8: four columns 0.46 ms, two 0.50, at
    // H = 1); one where the taps of two would not fit
    static constexpr int V = POL ? 2 : TP > 16 ? 1 : LOG2C >= 11 && DT != DT_C64 ? 4 : 2;
    static constexpr int HV = POL ? 1 : V;                // channels per thread (taps)
    static constexpr int RT = R < 16 ? R : 16;            // LDS rows per thread
    static constexpr int RT2 = H * RT;                    // sums per thread and column
    static constexpr int R2 = H * R;                      // filtered spectra per block
    static constexpr int COLG = POL ? C : C / V;          // column groups per row
    static constexpr int PASSES = COLG * (R / RT) / NT;
    static constexpr int L = RT2 + TP - 1;                // raw rows per thread and pass
    static constexpr int LP = RT2 + TP;                   // ring steps per pass
    static constexpr int D = block_ring(LP, H == 1 || POL ? 12 : 8);
    static constexpr int G = FftLanes<LOG2C>::G;
    static constexpr int NG = NT / G;                     // transforms at once
    static constexpr int ROUNDS = TROWS / NG;
    static constexpr bool BIG = LOG2C >= 11;
    using S = FftShape<LOG2C, G>;
    using BF = BigFft<BIG ? LOG2C : 11>;
    static constexpr int ROW = BIG ? BF::ROW : S::PADDED; // LDS float2 per transform
    static constexpr int TWN = BIG ? BF::RR : fft_tw_entries<LOG2C>();
    static_assert(R >= 1 && PASSES >= 1 && PASSES * NT == COLG * (R / RT), "FIR shape");
    static_assert(H == 1 || R == RT, "the waiting rows are the thread's own");
    static_assert(BIG || (NG >= 1 && ROUNDS * NG == TROWS), "transform rounds");

    // place of column c in its LDS row
    static __device__ __forceinline__ int at(int c)
    {
        if constexpr (BIG)
            return (c % BF::Q) * BF::SUB + S::pad(c / BF::Q);
        else
            return S::pad(c);
    }
};

// Transforms of the first `nout` spectra in the LDS, into spectra s0, s0 + 1,
// ... of stream or sub-band `unit`. tws: the LDS twiddles (big transforms:
// those of the second pass); tw2: the thread's last-pass twiddles.
template <class K, int JPT, bool POL, int LOG2C>
__device__ __forceinline__ void block_transform(const BlockArgs &a, float2 *lds, const float2 *tws,
                                                const float2 (&tw2)[JPT][K::BF::Q - 1], int64_t unit, int64_t s0,
                                                int nout)
{
    constexpr int C = K::C, NT = K::NT;
    using S = typename K::S;
    using BF = typename K::BF;
    const int t = (int)threadIdx.x;
    // the view of the rows' spectra, and bytes between them; spectra from
    // `nout` on lie outside it, so every store is issued unconditionally and
    // the next block's first rows are waited for without waiting for the
    // stores issued after them
    const int ystep = (int)(POL ? a.nsub * (2 * C) : (int64_t)C) * 8;
    const BufView vy = buf_view(POL ? a.Y + (s0 * a.nsub + unit) * (2 * C) : a.Y + (unit * a.S + s0) * C,
                                (int64_t)(nout - 1) * ystep + (POL ? 2 * C : C) * 8);
    if constexpr (K::BIG) {
        constexpr int R = BF::R, RR = BF::RR, Q = BF::Q, RSTEP = R + R / 16;
        constexpr int SUBS = K::TROWS * Q, AT = NT / R;
        static_assert(SUBS % AT == 0 && 64 % R == 0, "sub-row rounds");
#pragma unroll 1
        for (int base = 0; base < SUBS; base += AT) {
            const int sb = base + t / R;
            int l = t % R;
            asm volatile("" : "+v"(l)); // addresses formed here, not hoisted
            float2 *row = lds + (sb / Q) * K::ROW + (sb % Q) * BF::SUB;
            const int pl = S::pad(l);
            float2 v[R];
            sfor<R>([&](auto i) PFB_INLINE { v[i] = row[pl + decltype(i)::value * RSTEP]; });
            Dft<R>::run(v);
            float2 *w = row + l * RSTEP;
            sfor<R>([&](auto i) PFB_INLINE { w[decltype(i)::value + decltype(i)::value / 16] = v[i]; });
            group_sync<64>();
            sfor<R>([&](auto i) PFB_INLINE { v[i] = row[pl + decltype(i)::value * RSTEP]; });
            sfor<R - 1>([&](auto ic) PFB_INLINE {
                constexpr int i = decltype(ic)::value + 1;
                v[i] = cmul(v[i], tws[i * R + l]);
            });
            Dft<R>::run(v);
            sfor<R>([&](auto i) PFB_INLINE { row[pl + decltype(i)::value * RSTEP] = v[i]; });
        }
        lds_barrier();
        // last pass: a thread takes place j of every JG-th row (or pair of
        // polarisations), so its twiddles stay in registers for all blocks
        constexpr int JG = NT > RR ? NT / RR : 1;
        constexpr int PR = POL ? 2 : 1;
        static_assert(K::TROWS % (JG * PR) == 0, "rows per thread group");
        sfor<JPT>([&](auto jc) PFB_INLINE {
            int j = t % RR + decltype(jc)::value * NT;
            asm volatile("" : "+v"(j));
            const int pj = S::pad(j);
            sfor<K::TROWS / JG / PR>([&](auto rc) PFB_INLINE {
                const int rp = decltype(rc)::value * JG + t / RR % JG;
                float2 v[PR][Q];
                sfor<PR>([&](auto pc) PFB_INLINE {
                    const float2 *row = lds + (rp * PR + decltype(pc)::value) * K::ROW + pj;
                    sfor<Q>([&](auto i) PFB_INLINE { v[pc][i] = row[decltype(i)::value * BF::SUB]; });
                    sfor<Q - 1>([&](auto i) PFB_INLINE { v[pc][i + 1] = cmul(v[pc][i + 1], tw2[jc][i]); });
                    Dft<Q>::run(v[pc]);
                });
                const int o = rp * ystep + j * (PR * 8);
                sfor<Q>([&](auto i) PFB_INLINE {
                    float2 z[PR];
                    sfor<PR>([&](auto pc) PFB_INLINE { z[pc] = v[pc][i]; });
                    buf_store_c64_nt<PR>(vy, o + decltype(i)::value * PR * RR * 8, z);
                });
            });
        });
    } else {
        constexpr int G = K::G;
        const int gid = t / G;
#pragma unroll 1
        for (int round = 0; round < K::ROUNDS; ++round) {
            const int tr = round * K::NG + gid;
            float2 *row = lds + tr * K::ROW;
            const int sr = POL ? tr / 2 : tr;
            const int o = sr * ystep + (POL ? tr % 2 * 8 : 0);
            int ln = t % G;
            asm volatile("" : "+v"(ln));
            float2 v[S::E];
            if constexpr (LOG2C >= 7)
                fft_gather_first_lds<LOG2C, G>(ln, row, v);
            else
                fft_gather_first<LOG2C, G>(ln, [&](int idx) { return row[S::pad(idx)]; }, v);
            fft_passes<LOG2C, G, false, true, true>(ln, row, tws, v, [&](int idx, float2 z) {
                const float2 z1[1] = {z};
                if constexpr (G >= 16 && !POL) {
                    buf_store_c64_nt<1>(vy, o + idx * 8, z1);
                } else { // less than a line at a time: L2 gathers it
                    const v2u_t w = {__float_as_uint(z.x), __float_as_uint(z.y)};
                    __builtin_amdgcn_raw_buffer_store_b64(w, vy.r, o + idx * (POL ? 16 : 8), 0, 0);
                }
            });
        }
    }
}

template <int DT, int TP, int LOG2C, bool POL>
__global__ __launch_bounds__(BLOCK_NT) void block_kernel(BlockArgs a)
{
    using K = BlockShape<DT, TP, LOG2C, POL>;
    using BF = typename K::BF;
    constexpr int C = K::C, NT = K::NT, H = K::H, R = K::R, R2 = K::R2, RT = K::RT, RT2 = K::RT2;
    constexpr int V = K::V, HV = K::HV, L = K::L, LP = K::LP, D = K::D;
    constexpr int SB = SampleBytes<DT>::value;
    __shared__ __attribute__((aligned(16))) float2 lds[K::TROWS * K::ROW];
    __shared__ float2 tws[K::TWN];

    // this workgroup's blocks q, q + grid, ...: runs of consecutive blocks
    // per XCD (workgroup ids go round the eight XCDs)
    const int64_t total = a.n_blocks * a.units;
    const int grid = (int)gridDim.x;
    int64_t q = grid % 8 == 0 ? ((int)blockIdx.x % 8) * (grid / 8) + (int)blockIdx.x / 8 : (int)blockIdx.x;
    if (q >= total)
        return;

    const int t = (int)threadIdx.x;
    const int off = TP - a.T;
    const int64_t in_rows = a.S + a.T - 1;
    const int rb = (int)((POL ? (int64_t)2 * C * a.nsub : C) * SB); // bytes of a raw row
    constexpr int SEG = (POL ? 2 : 1) * C * SB;                      // bytes of it that a block reads
    const BufView vh = buf_view(a.h, (int64_t)a.T * C * 4);

    // twiddles; the LDS ones are read after the first barrier
    constexpr int JPT = BF::RR > NT ? BF::RR / NT : 1;
    float2 tw2[JPT][BF::Q - 1];
    if constexpr (K::BIG) {
        for (int e = t; e < BF::RR; e += NT)
            tws[(e % BF::R) * BF::R + e / BF::R] = a.tw[e];
        sfor<JPT>([&](auto jc) PFB_INLINE {
            const float2 *w = a.tw + BF::RR + (t % BF::RR + decltype(jc)::value * NT) * BF::Q + 1;
            sfor<BF::Q - 1>([&](auto i) PFB_INLINE { tw2[jc][i] = w[decltype(i)::value]; });
        });
    } else {
        stage_twiddles_lds<LOG2C>(tws, a.tw, t, NT);
    }

    // block q -> stream (or sub-band) and first spectrum
    struct Blk {
        int64_t unit, s0;
    };
    auto blk_of = [&](int64_t i) PFB_INLINE -> Blk { return {i / a.n_blocks, (i % a.n_blocks) * R2}; };
    // the view of a block's raw rows s0 - off, ... that lie in the stream,
    // and the offset of row s0 - off in it (negative before the stream)
    auto view_of = [&](const Blk &k, int &first) PFB_INLINE -> BufView {
        const int64_t r0 = k.s0 - off, rv = r0 < 0 ? 0 : r0;
        const int64_t nr = in_rows - rv < R2 + TP ? in_rows - rv : R2 + TP;
        first = (int)(r0 - rv) * rb;
        return buf_view(reinterpret_cast<const char *>(a.x) + rv * rb + k.unit * (POL ? SEG : in_rows * rb),
                        (nr - 1) * rb + SEG);
    };
    // a thread's column group and first LDS row in pass p, formed where they
    // are used (opaque thread index: hoisted, the unrolled passes' addresses
    // exhaust the registers)
    auto task_of = [&](int p) PFB_INLINE {
        int x = t;
        asm volatile("" : "+v"(x));
        return p * NT + x;
    };
    auto colg_of = [&](int p) PFB_INLINE { return task_of(p) % K::COLG; };
    auto row0_of = [&](int p) PFB_INLINE { return task_of(p) / K::COLG * RT; };
    auto voff_of = [&](int p, int first) PFB_INLINE { return first + row0_of(p) * rb + colg_of(p) * (V * SB); };
    auto hoff_of = [&](int p) PFB_INLINE { return colg_of(p) * (HV * 4); };
    // tap j of the padded filter (zero below `off`: outside the view)
    float hp[TP][HV];
    auto load_tap = [&](auto jc, int hoff) PFB_INLINE {
        constexpr int j = decltype(jc)::value;
        Packed<DT_CI16, HV> w; // 4 bytes each
        buf_load_packed<DT_CI16, HV>(vh, hoff + (j - off) * (C * 4), w);
        sfor<HV>([&](auto k) PFB_INLINE { hp[j][k] = __uint_as_float(w.w[k]); });
    };
    // column k of LDS spectrum row r
    auto put = [&](int r, int cg, auto kc, float2 v) PFB_INLINE {
        constexpr int k = decltype(kc)::value;
        if constexpr (POL)
            lds[(r * 2 + k) * K::ROW + K::at(cg)] = v;
        else
            lds[r * K::ROW + K::at(cg * V + k)] = v;
    };

    Packed<DT, V> pf[D]; // the ring: raw rows in flight, still packed
    Blk cur = blk_of(q);
    int first;
    BufView vx = view_of(cur, first);
    int voff = voff_of(0, first);
    sfor<TP>([&](auto j) PFB_INLINE { load_tap(j, hoff_of(0)); });
    static_assert(D <= L, "ring depth");
    // issued in the order of their use: a wait inside the loop counts from
    // the order of the loads on every path to it
    __builtin_amdgcn_sched_barrier(0);
    sfor<D>([&](auto i) PFB_INLINE {
        buf_load_packed<DT, V>(vx, voff + decltype(i)::value * rb, pf[i]);
        __builtin_amdgcn_sched_barrier(0);
    });

    for (;;) {
        const int64_t qn = q + grid;
        const bool more = qn < total;
        const Blk nxt = blk_of(more ? qn : q); // the last block prefetches its own rows again, unused
        int nfirst;
        const BufView vn = view_of(nxt, nfirst);
        float2 hold[H > 1 ? K::PASSES : 1][RT][V];
        auto fir_pass = [&](auto pc) PFB_INLINE {
            const int p = (int)pc;
            const bool lastp = p + 1 == K::PASSES;
            const BufView vnext = lastp ? vn : vx;
            const int pn = lastp ? 0 : p + 1;
            const int voffn = voff_of(pn, lastp ? nfirst : first);
            const int hoffn = hoff_of(pn);
            float2 acc[RT2][V];
            sfor<RT2>([&](auto r) PFB_INLINE {
                sfor<V>([&](auto k) PFB_INLINE { acc[r][k] = make_float2(0.0f, 0.0f); });
            });
            // step i: raw row i enters the sums of rows i - TP + 1 .. i, and
            // row i + D is requested into its slot (step LP - 1 has no row:
            // it keeps the slots of all passes alike)
            sfor<LP>([&](auto ic) PFB_INLINE {
                constexpr int i = decltype(ic)::value;
                float2 xv[V];
                // loads stay in the order they are waited for, and in step
                // with the sums (free to move, they gathered at the end of
                // a pass: 1024 channels, 32 taps 0.281 -> 0.266 ms, 8
                // sub-bands 0.438 -> 0.417)
                if constexpr (i % 2 == 0)
                    __builtin_amdgcn_sched_barrier(0);
                if constexpr (i < L)
                    unpack<DT, V>(pf[i % D], xv);
                if constexpr (i + D < L)
                    buf_load_packed<DT, V>(vx, voff + (i + D) * rb, pf[i % D]);
                else if constexpr (i + D >= LP)
                    buf_load_packed<DT, V>(vnext, voffn + (i + D - LP) * rb, pf[i % D]);
                if constexpr (i < L) {
                    sfor<RT2>([&](auto rc) PFB_INLINE {
                        constexpr int r = decltype(rc)::value, j = i - r;
                        if constexpr (j >= 0 && j < TP) {
                            sfor<V>([&](auto kc) PFB_INLINE {
                                constexpr int k = decltype(kc)::value;
                                const float h = hp[j][HV == 1 ? 0 : k];
                                acc[r][k].x = __builtin_fmaf(h, xv[k].x, acc[r][k].x);
                                acc[r][k].y = __builtin_fmaf(h, xv[k].y, acc[r][k].y);
                            });
                        }
                    });
                    // a tap's last row makes room for the next pass's tap
                    if constexpr (K::PASSES > 1 && i >= RT2 - 1)
                        load_tap(std::integral_constant<int, i - (RT2 - 1)>{}, hoffn);
                }
            });
            const int cg = colg_of(p), row0 = row0_of(p);
            sfor<RT>([&](auto r) PFB_INLINE {
                sfor<V>([&](auto k) PFB_INLINE {
                    put(row0 + decltype(r)::value, cg, k, acc[r][k]);
                    if constexpr (H > 1)
                        hold[decltype(pc)::value][r][k] = acc[RT + decltype(r)::value][k];
                });
            });
            vx = vnext;
            voff = voffn;
        };
        if constexpr (H > 1) {
            sfor<K::PASSES>([&](auto pc) PFB_INLINE { fir_pass(pc); });
        } else {
#pragma unroll 1
            for (int p = 0; p < K::PASSES; ++p)
                fir_pass(p);
        }
        const int nrows = (int)(a.S - cur.s0 < R2 ? a.S - cur.s0 : R2);
        // left at the end of an iteration only: every path to the next block
        // then issues stores after that block's prefetched rows
#pragma unroll 1
        for (int half = 0;;) {
            if constexpr (H > 1) {
                if (half == 1) {
                    lds_barrier(); // the first half's transforms are done
                    sfor<K::PASSES>([&](auto pc) PFB_INLINE {
                        const int cg = colg_of(decltype(pc)::value);
                        sfor<RT>([&](auto r) PFB_INLINE {
                            sfor<V>([&](auto k) PFB_INLINE { put(decltype(r)::value, cg, k, hold[pc][r][k]); });
                        });
                    });
                }
            }
            lds_barrier();
            const int left = nrows - half * R;
            block_transform<K, JPT, POL, LOG2C>(a, lds, tws, tw2, cur.unit, cur.s0 + half * R, left < R ? left : R);
            if (++half == H || half * R >= nrows)
                break;
        }
        lds_barrier(); // the LDS rows are free for the next block
        if (!more)
            break;
        q = qn;
        cur = nxt;
        first = nfirst;
    }
}

template <int DT, int TP, int LOG2C, bool POL> hipError_t launch_block_t(BlockArgs a, hipStream_t st)
{
    using K = BlockShape<DT, TP, LOG2C, POL>;
    a.n_blocks = (a.S + K::R2 - 1) / K::R2;
    const int64_t total = a.n_blocks * a.units;
    if (total <= 0)
        return hipSuccess;
    // One workgroup per CU, and a multiple of the eight XCDs where the CUs allow
    // it, the last of them with no block: runs of neighbouring blocks on one
    // XCD for every count (8192 channels, 16 taps, complex64: 165 blocks dealt
    // one by one 45.8 us, in runs 37.6).
    const int64_t cus = a.num_cus > 0 ? a.num_cus : 256;
    int64_t grid = total < cus ? total : cus;
    if ((grid + 7) / 8 * 8 <= cus)
        grid = (grid + 7) / 8 * 8;
    hipLaunchKernelGGL((block_kernel<DT, TP, LOG2C, POL>), dim3((unsigned)grid), dim3(BLOCK_NT), 0, st, a);
    return hipGetLastError();
}

// Windows from TP0 to TP1 taps.
template <int DT, int LOG2C, bool POL, int TP0, int TP1>
hipError_t launch_block_c(const BlockArgs &a, int tp, hipStream_t st)
{
    if (tp == TP0)
        return launch_block_t<DT, TP0, LOG2C, POL>(a, st);
    if constexpr (TP0 < TP1)
        return launch_block_c<DT, LOG2C, POL, 2 * TP0, TP1>(a, tp, st);
    else
        return hipErrorInvalidValue;
}

// The sizes of one translation unit each (block_supported in block.hip).
template <int DT> hipError_t launch_block_small(const BlockArgs &a, int tp, int log2c, hipStream_t st)
{
    switch (log2c) {
    case 5: return launch_block_c<DT, 5, false, 4, 64>(a, tp, st);
    case 6: return launch_block_c<DT, 6, false, 4, 64>(a, tp, st);
    case 7: return launch_block_c<DT, 7, false, 4, 64>(a, tp, st);
    case 8: return launch_block_c<DT, 8, false, 32, 64>(a, tp, st);
    case 9: return launch_block_c<DT, 9, false, 32, 64>(a, tp, st);
    case 10: return launch_block_c<DT, 10, false, 32, 64>(a, tp, st);
    default: return hipErrorInvalidValue;
    }
}
template <int DT> hipError_t launch_block_large(const BlockArgs &a, int tp, int log2c, hipStream_t st)
{
    switch (log2c) {
    case 11: return launch_block_c<DT, 11, false, 4, 32>(a, tp, st);
    case 12: return launch_block_c<DT, 12, false, 4, 32>(a, tp, st);
    case 13: return launch_block_c<DT, 13, false, 4, 16>(a, tp, st);
    default: return hipErrorInvalidValue;
    }
}
template <int DT> hipError_t launch_block_pol(const BlockArgs &a, int tp, int log2c, hipStream_t st)
{
    switch (log2c) {
    case 9: return launch_block_c<DT, 9, true, 4, 32>(a, tp, st);
    case 10: return launch_block_c<DT, 10, true, 4, 32>(a, tp, st);
    case 11: return launch_block_c<DT, 11, true, 4, 32>(a, tp, st);
    case 12: return launch_block_c<DT, 12, true, 4, 32>(a, tp, st);
    default: return hipErrorInvalidValue;
    }
}

} // namespace pfb
