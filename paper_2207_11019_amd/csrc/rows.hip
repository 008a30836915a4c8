// Contractions by filter rows in pieces of a few channels: forward and data gradient of bf16 filters three or five taps wide (stride 1, the
// output as wide as the input), two- and three-dimensional, whose channels are no whole K tiles of 64.
//
//   C[M][N] = A[M][K] * B[N][K]^T,  K over (filter row, piece of channels, tap of the row, channel); operands as in igemm.hip
//
// What bounds such layers is the path from the L2 through the LDS to the matrix cores, not the products.  In chunks across taps
// (igemm_kernel, KT_CHUNKS) a tile's pixels are loaded anew for each tap, every lane looking its chunk's tap up.  Here a
// stage of LDS holds the pixels that a filter row of the tile meets, once, and the taps of weights of that row, P chunks of 16 bytes (8 channels)
// each, P = 4 or 6: which tap that is is wave-uniform, a tap is another row of LDS to read from (a row of zeros where it lies beside the image).
// Two stages, one workgroup barrier each.  A stage of 256x64 tiles is 29 KB for 96 values of K where 64 of them took 40.
//
// Measured (us, chunks across taps / here): 64 x 32^2 x 32 channels 7.6 / 5.0 (159 -> 243 TFLOP/s), 128 x 28^2 x 160 83 / 54
// (557 -> 856 TFLOP/s); per step: volumetric 1585 / 1509, ResNet of width 32 on 40x40 1184 / 1105.
//
// LDS rows are 16 P bytes.  Sixteen lanes read one chunk of 16 consecutive rows at a time, 256 bytes: the chunks of a row change places
// by the row (swz) so that they fall on distinct banks.
#include "contraction.h"
#include "lds_dma.h"
#include <type_traits>

namespace lpm {

template <int P>
__device__ __forceinline__ int swz(int r) { return P == 4 ? (r >> 2) & 3 : (r >> 3) & 1; }

// LDS of a stage in units of 1 KB, what a wavefront loads at a time: the pixels of the tile's rows and of those before and behind them,
// and a row of zeros; the weights
constexpr int rows_a_units(int taps, int P, int BM) { return ((BM + taps) * P + 63) / 64; }
constexpr int rows_stage(int taps, int P, int BM, int BN) { return (rows_a_units(taps, P, BM) + taps * BN * P / 64) * 1024; }

template <int TAPS, int P, int BM, int BN, int WGM, int WGN, int LA, int MODE>
__global__ void __launch_bounds__(WGM * WGN * 64, 2) rows_kernel(const IgemmArgs p) {
    constexpr int NW = WGM * WGN, WTM = BM / WGM, WTN = BN / WGN, MI = WTM / 32, NI = WTN / 32, ROWB = P * 16;
    constexpr int UA = rows_a_units(TAPS, P, BM), U = UA + TAPS * BN * P / 64, STAGE = U * 1024, NL = (U + NW - 1) / NW;      // units, loads of a wavefront
    constexpr int KS = TAPS * P / 2, SETS = KS > 9 ? 5 : KS, SIDE = TAPS / 2;      // steps of 16 values of K, sets of their operands
    static_assert(TAPS * BN * P % 64 == 0 && LA < SETS && KS % SETS == 0, "layout");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int nt = (p.N + BN - 1) / BN, tm = div_by(tile, p.dNt), n0 = (tile - tm * nt) * BN, m0 = tm * BM, rows = p.M;

    const int Cc = p.Ci / 8, G = (Cc + P - 1) / P, nk = p.Kd * p.Kh * G;       // chunks and pieces of a tap's channels, stages
    const bool ragged = G * P != Cc;
    const unsigned tapC = (unsigned)p.Ci * 2u;
    constexpr int SG = MODE == MODE_FWD ? 1 : -1;                               // the pixels move with the filter or against it
    const unsigned aH = (unsigned)SG * tapC * (unsigned)p.Wi, aD = aH * (unsigned)p.Hi;
    // (the buffer begins early by what the first filter row of the first pixel lies before it, so that no offset is negative)
    const unsigned span = (unsigned)((p.Kd - 1) * p.Hi + p.Kh - 1) * (unsigned)p.Wi * tapC;
    const unsigned bias = MODE == MODE_FWD ? (unsigned)(p.pad_d * p.Hi + p.pad) * (unsigned)p.Wi * tapC : span;
    u32x4_ rsA = buffer_words((const unsigned char*)p.A - bias, p.a_bytes + bias), rsB = buffer_words(p.B, p.b_bytes);

    // ---- loader state.  Unit u of a stage is chunks 64 u .. 64 u + 63 of its rows.  msk: bit 0: the chunk exists in the last piece of a
    // tap's channels; 12..23, 24..31: the filter rows and slices that meet the pixel inside the image
    unsigned off[NL], msk[NL], cur[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int u = i * NW + wave;
        if (i * NW + NW <= UA || (i * NW < UA && u < UA)) {
            const int idx = u * 64 + lane, r = idx / P, c = (idx - r * P) ^ swz<P>(r), row = m0 - SIDE + r;
            const bool ok = (row >= 0) & (row < rows) & (r < BM + 2 * SIDE);
            const int rr = ok ? row : 0, t = div_by(rr, p.dWr), wq = rr - t * p.Wr;
            int n = div_by(t, p.dHr), d0 = 0;
            const int hq = t - n * p.Hr, h0 = MODE == MODE_FWD ? hq - p.pad : hq + p.pad;
            unsigned m = (MODE == MODE_FWD ? tap_bits(max(0, -h0), min(p.Kh, p.Hi - h0)) : tap_bits(max(0, h0 - p.Hi + 1), min(p.Kh, h0 + 1))) << 12;
            if (p.Kd > 1 || p.Dr > 1 || p.Di > 1) {
                const int ns = div_by(n, p.dDr), dq = n - ns * p.Dr;
                n = ns;
                d0 = MODE == MODE_FWD ? dq - p.pad_d : dq + p.pad_d;
                m |= (MODE == MODE_FWD ? tap_bits(max(0, -d0), min(p.Kd, p.Di - d0)) : tap_bits(max(0, d0 - p.Di + 1), min(p.Kd, d0 + 1))) << 24;
            } else m |= 1u << 24;
            msk[i] = ok ? m | (unsigned)(c < Cc - (G - 1) * P) : 0u;
            off[i] = (unsigned)(((n * p.Di + d0) * p.Hi + h0) * p.Wi + wq) * tapC + (MODE == MODE_FWD ? bias : 0u) + (unsigned)c * 16u;
        } else {
            const int idx = (u - UA) * 64 + lane, r = idx / P, c = (idx - r * P) ^ swz<P>(r), s = r / BN, n = r - s * BN;
            msk[i] = 0xfffff000u | (unsigned)(c < Cc - (G - 1) * P);
            off[i] = (unsigned)(n0 + n) * p.b_pitch + (unsigned)s * tapC + (unsigned)c * 16u;       // (rows past N lie past the buffer's end)
        }
    }
    // the stage to be loaded next: filter row and slice, pieces left of it, rows left, wave-uniform offsets
    int kh = 0, g_left = G, row_left = p.Kd * p.Kh;
    unsigned la = MODE == MODE_FWD ? 0u : span, lb = 0, on = ROWB;
    const unsigned last = ragged ? 1u : 0u;
    unsigned bit = (1u << 24) | (1u << 12) | (G == 1 ? last : 0u);
    auto aim = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NL; ++i) cur[i] = (msk[i] & bit) == bit ? off[i] : OOB;
    };
    aim();
    // (past the last stage the buffers count as empty)
    auto next_stage = [&]() __attribute__((always_inline)) {
        if (--g_left > 0) {
            la += on; lb += on;
            if (g_left == 1 && ragged) { bit |= 1u; aim(); }
            return;
        }
        if (--row_left <= 0) {
            rsA.z = 0; rsB.z = 0; la = 0; lb = 0; on = 0;
            g_left = row_left = 0x7fffffff;
            bit = 0x80000000u;
            return;
        }
        const unsigned back = (unsigned)(G - 1) * ROWB;
        lb += (unsigned)TAPS * tapC - back;
        la += aH - back;
        bit &= ~1u;
        if (++kh < p.Kh) bit = ((bit & 0xfff000u) << 1) | (bit & 0xff000000u);
        else { kh = 0; la += aD - aH * (unsigned)p.Kh; bit = ((bit & 0xff000000u) << 1) | 0x1000u; }
        if (G == 1) bit |= last;
        g_left = G;
        aim();
    };
    const bool more = wave < U % NW;                       // this wavefront has NL loads a stage, not one less
    auto issue = [&](int st, int part) __attribute__((always_inline)) {
        unsigned char* sp = lds + st * STAGE + wave * 1024;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            if (i * KS / NL != part) continue;
            const bool a = i * NW + NW <= UA || (i * NW < UA && i * NW + wave < UA);
            u32x4_ rs = rsB;
            if (i * NW + NW <= UA) rs = rsA;
            else if (i * NW < UA) {            // (a step that both tensors share, each wavefront one of them)
#pragma unroll
                for (int k = 0; k < 4; ++k) rs[k] = (unsigned)__builtin_amdgcn_readfirstlane((int)(a ? rsA[k] : rsB[k]));
            }
            if ((i + 1) * NW <= U || more) load_to_lds16s(rs, sp + i * NW * 1024, cur[i], a ? la : lb);
        }
        if (part == KS - 1) next_stage();
    };

    // (the first stage is on its way before anything else is worked out)
#pragma unroll
    for (int q = 0; q < KS; ++q) issue(0, q);
    __builtin_amdgcn_sched_barrier(0);

    f32x16 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;

    // operand addresses in a stage: row lane % 32 of the wavefront's part, chunk 2j + lane / 32 of a tap's piece
    const int wm = wave / WGN, wn = wave - wm * WGN, rl = lane & 31, kq = lane >> 5;
    auto piece = [](unsigned o, int j) __attribute__((always_inline)) { return P == 6 ? o + (unsigned)j * 32u : o ^ ((unsigned)j << 5); };
    unsigned oA[TAPS][MI], oB[P / 2];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
        const int at = wm * WTM + mi * 32 + rl, row = m0 + at, w = row - div_by(row, p.dWr) * p.Wr;
#pragma unroll
        for (int s = 0; s < TAPS; ++s) {
            const bool out = s != SIDE && (unsigned)(w + s - SIDE) >= (unsigned)p.Wr;
            const int r = out ? BM + 2 * SIDE : at + s;
            oA[MODE == MODE_FWD ? s : TAPS - 1 - s][mi] = (unsigned)(r * ROWB + ((kq ^ swz<P>(r)) << 4));
        }
    }
#pragma unroll
    for (int j = 0; j < P / 2; ++j) oB[j] = piece((unsigned)(UA * 1024 + (wn * WTN + rl) * ROWB + ((kq ^ swz<P>(rl)) << 4)), j);

    struct Frag { uint4 a[MI], b[NI]; };
    Frag f[SETS];
    auto read = [&](int st, int ks) __attribute__((always_inline)) {
        const int s = ks / (P / 2), j = ks - s * (P / 2);
        const unsigned char* sp = lds + st * STAGE;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) f[ks % SETS].a[mi] = *reinterpret_cast<const uint4*>(sp + piece(oA[s][mi], j));
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) f[ks % SETS].b[ni] = *reinterpret_cast<const uint4*>(sp + oB[j] + (s * BN + ni * 32) * ROWB);
    };
    auto multiply = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f[ks % SETS].b[ni]), __builtin_bit_cast(bf16x8, f[ks % SETS].a[mi]), acc[mi][ni], 0, 0, 0);
    };
    // The next stage has landed, and the last operands of the present one have arrived: what is loaded behind the barrier goes where it lies.
    auto meet = [&]() __attribute__((always_inline)) {
        LPM_WAIT_VM(0);
        __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    constexpr int EN = NI <= 2 ? NI : 1;           // (the epilogue takes one or two columns of 32 channels at a time)
    typedef Epilogue<bf16_t, MI, EN, MODE> Ep;
    Ep ep;
    const int er0 = m0 + wm * WTM, ec0 = n0 + wn * WTN;
    constexpr bool early = Ep::R <= 2 && EN == NI;             // (the epilogue's operands arrive under the main loop where the registers allow)
    if (early) ep.load(p, er0, ec0, rows, lane, 0, 0, 0, 0, 0, 0);
    meet();
#pragma unroll
    for (int q = 0; q < LA; ++q) {
        issue(1, q);
        read(0, q);
    }
    // A stage's products, the operands read LA steps ahead, and from the meeting on the loads of the stage after the next, over KS steps.
    int it = 0;
    auto step = [&](auto index) __attribute__((always_inline)) {        // false: that was the last stage
        constexpr int u = decltype(index)::value;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (s == KS - LA) meet();
            if (s < KS - LA) read(u, s + LA);
            else read(1 - u, s + LA - KS);
            __builtin_amdgcn_sched_barrier(0);
            multiply(s);
            if (s < KS - LA) issue(1 - u, s + LA);
            else issue(u, s + LA - KS);
            __builtin_amdgcn_sched_barrier(0);
        }
        return ++it < nk;
    };
    while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {}
    LPM_WAIT_VM(0);
    __syncthreads();                            // the stages are dead: the epilogue takes them

    float* area = reinterpret_cast<float*>(lds) + wave * MI * Ep::PIECE;
#pragma unroll
    for (int n = 0; n < NI; n += EN) {
        const int col = ec0 + n * 32;
        if (!early) ep.load(p, er0, col, rows, lane, 0, 0, 0, 0, 0, 0);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < EN; ++ni)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4*>(area + mi * Ep::PIECE + rl * Ep::PITCH + ni * 32 + q * 8 + kq * 4) =
                        make_float4(acc[mi][n + ni][4 * q], acc[mi][n + ni][4 * q + 1], acc[mi][n + ni][4 * q + 2], acc[mi][n + ni][4 * q + 3]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        ep.store(p, area, er0, col, rows, lane, 0, 0, 0, 0, 0, 0);
        if constexpr (MODE == MODE_FWD) if (p.fwd_pool && p.Wr == 32) {
            __syncthreads();
            if constexpr (MI == 1) {
                if (!(wm & 1)) ep.pool32(p, area, area + WGN * Ep::PIECE, er0, col, rows, lane);
            } else {
#pragma unroll
                for (int mi = 0; mi < MI; mi += 2) ep.pool32(p, area + mi * Ep::PIECE, area + (mi + 1) * Ep::PIECE, er0 + mi * 32, col, rows, lane);
            }
            if (EN < NI) __syncthreads();          // (another wavefront's area was read)
        }
    }
}

template <int TAPS, int P, int BM, int BN, int WGM, int WGN, int LA, int MODE>
static hipError_t go(const IgemmArgs& a, hipStream_t st) {
    constexpr int stages = 2 * rows_stage(TAPS, P, BM, BN), cols = BN / WGN, epilogue = BM * WGN * ((cols <= 64 ? cols : 32) + 4) * 4, bytes = stages > epilogue ? stages : epilogue;
    static_assert(bytes <= 160 * 1024, "LDS of a CU");
    static DeviceSet done;
    const hipError_t attr = allow_lds(rows_kernel<TAPS, P, BM, BN, WGM, WGN, LA, MODE>, bytes, done);
    if (attr != hipSuccess) return attr;
    IgemmArgs b = a;
    const int nt = (a.N + BN - 1) / BN;
    b.dNt = fast_div(nt);
    launch_last(rows_kernel<TAPS, P, BM, BN, WGM, WGN, LA, MODE>, dim3((unsigned)((a.M + BM - 1) / BM * nt)), dim3(WGM * WGN * 64), bytes, st, b);
    return hipGetLastError();
}

// ---- which calls come here, and on which tiles
static int64_t tiles(const IgemmArgs& a, int bm, int bn) { return ((int64_t)a.M + bm - 1) / bm * ((a.N + bn - 1) / bn); }
static int padded(int n, int unit) { return (n + unit - 1) / unit * unit; }

// Chunks of a piece: 32 channels, or 48 where that leaves fewer of the last piece empty -- as many where both do, and 32-channel pieces would
// not be whole (80 channels, 16 x 32^2: 7.5 / 6.7 us; 96, 13 x 24^2: 5.5 / 5.6).
static int chunks_of(int ci) {
    const int p4 = padded(ci, 32), p6 = padded(ci, 48);
    return p6 < p4 || (p6 == p4 && ci % 32) ? 6 : 4;
}

// 128x96 tiles: where they pad fewer channels
static bool by96(const IgemmArgs& a) { return a.N > 64 && padded(a.N, 96) < padded(a.N, 64) && tiles(a, 128, 96) >= 300; }

// keep_order: the sums are to be those of chunks across taps -- a tap's channels in one piece, in whole steps of 16
bool rows_take(const IgemmArgs& a, bool keep_order) {
    if ((a.Kw != 3 && a.Kw != 5) || a.stride != 1 || a.pad != a.Kw / 2 || a.Ci % 8 || a.Ci < 16) return false;
    // Whole K tiles are better where they are (16 x 14^2 x 256 8.5 / 9.2 us) but for outputs that fill half a tile (24 x 112^2, 64 -> 8 33.3 / 18.6).
    if (a.Ci % 64 == 0 && (keep_order || a.N > 32)) return false;
    // A block walks its reduction alone.  With less than a tile for each CU that takes as long or longer than on 64x64 tiles in chunks from some 80 taps of
    // a piece on: alone, us, there / here: 24 x 6^2, 280 -> 720 channels (18 stages of three) 11.7 / 9.6, 3 x 38^2, 224 -> 208 (21) 12.0 / 8.9, 22 x 7^2, 360 -> 520
    // (24) 13.8 / 11.4, 4 x 16^2, 360 -> 608 15.4 / 15.2; 5 x 15^2, 456 -> 528 (30) 20.0 / 18.4, 23 x 8^2, 400 -> 536 (39) 15.7 / 20.5, 5 x 18^2, 480 -> 544 (45) 17.9 / 23.6;
    // 5x5 filters 4 x 28^2, 136 -> 264 (15 of five) 15.2 / 11.5, 24 x 7^2, 120 -> 760 (20) 15.0 / 15.7.  More tiles: 64 x 7^2 x 480, 375 of them, 25.2 / 23.2.
    // A third of the pieces empty (72 channels) is more than is gained (32 x 28^2: 9.2 / 9.6, 5x5 14.9 / 16.8) but for few channels (24: 5.7 / 4.1).
    const int P = chunks_of(a.Ci);
    if (keep_order && (a.Ci % 16 || a.Ci > P * 8)) return false;
    const int pieces = (a.Ci / 8 + P - 1) / P;
    if (a.Ci > 48 && 4 * 8 * P * pieces > 5 * a.Ci) return false;
    const int taps = a.Kd * a.Kh * a.Kw;
    // Of 16 channels half a piece is empty.  Where the outputs fill no more than half a tile of 64 the products there are half padding, too (256x32, volumes
    // 16 -> 16 to 32 channels, from 512 tiles of 128x32 on: 1874 / 1038 for 40 sizes together; with fewer than 128, 60 sizes, 315 / 356).  Where they fill it:
    // 3x3 up to 1.2 times faster, up to 1.2 times slower from 384 tiles of 128x128 on (49152 rows, 16 -> 480: 22.9 / 27.5); 5x5 with more than 64
    // outputs 552 / 552 (39 sizes); volumes 1.1 times slower (4 x 2 x 101 x 104, 16 -> 224: 32.1 / 41.1).
    const bool fill = a.N % 128 == 0 || a.N % 128 > 64, large = fill && tiles(a, 128, 128) >= 384;
    if (2 * a.Ci <= 8 * P) {
        if (a.N <= 32 ? taps > 25 && tiles(a, 128, 32) < 128 : taps > 9 ? taps > 25 || a.N > 64 : large) return false;
    }
    // Pieces of 48 go on 128x32 tiles or 128x96.  Against two blocks of 128x128 or one of 256x128 to a CU the former read their pixels too often: 55 sizes
    // 2113 / 2320 (38 x 37^2, 360 -> 208 98 / 123, 6 x 42^2, 432 -> 384 43 / 54).  Nor against a round of CUs that 128x128 tiles fill to four fifths, but for
    // up to 96 outputs (48 channels 3x3, tiles of 128x128: 176 9.5 / 7.5, 219 8.4 / 9.4, 252 9.1 / 10.0, 259 13.8 / 10.5; 80 outputs, 192 8.1 / 7.2; 5x5, 72, 254 12.9 / 11.7).
    const int64_t t128 = tiles(a, 128, 128);
    if (P == 6 && (large || (fill && a.N > 96 && t128 >= 205 && t128 <= 256)) && !by96(a)) return false;
    return tiles(a, 128, 32) >= 256 || taps * pieces <= 80;
}

template <int TAPS, int MODE>
static hipError_t go_mode(const IgemmArgs& a, hipStream_t st) {
    // Alone, us, chunks across taps / here.  128x32 tiles of four wavefronts down the rows, two stages (30 KB): three and more blocks share a CU.
    // 64 x 32^2 x 32 channels 7.6 / 5.0, 24 x 27^2 x 96 -> 160 13.7 / 10.0 (data gradient 15.0 / 9.8), 8 x 28^2 x 160 9.5 / 7.2.
    // 256x32 where there are enough of them (from 800 of 128x32 on; 128x32 / 256x32: 980: 18.5 / 16.1, 1176: 16.3 / 14.6, 686: 18.2 / 17.1, 685:
    // 10.0 / 10.2, 343: 11.2 / 11.8).  256x64 of eight wavefronts where one round of CUs takes them all and is more than half full (207 of them:
    // 10.0 / 9.2, 196: 17.1 / 15.2, 144: 19.3 / 16.1, 138: 9.7 / 11.4, 98: 8.3 / 9.9), of four, 64x64 each, over several rounds (392: 26.7 / 21.6,
    // 980: 56.3 / 47.9, 343: 49.5 / 46.0, 294: 16.1 / 19.5).  128x96 where that pads fewer channels (450: 15.2 / 13.6, 392: 14.6 / 12.8, 137: 9.7 / 11.1).
    // 5x5 filters on the same lines: 24 x 27^2 x 96 -> 160 27.6 / 18.5 (33.4 / 21.7), 4 x 30^2 x 360 -> 480 57.7 / 45.7, 8 x 56^2 x 24 -> 48 7.4 / 6.3 (9.6 / 5.6).
    const bool wide = by96(a);
    if (chunks_of(a.Ci) == 6) {
        if (wide) return go<TAPS, 6, 128, 96, 4, 1, 4, MODE>(a, st);
        return go<TAPS, 6, 128, 32, 4, 1, 4, MODE>(a, st);
    }
    if (wide) return go<TAPS, 4, 128, 96, 4, 1, 3, MODE>(a, st);
    const int64_t t64 = tiles(a, 256, 64);
    if (a.N > 32 && t64 >= 340) return go<TAPS, 4, 256, 64, 4, 1, 3, MODE>(a, st);
    if (a.N > 32 && t64 >= 140 && t64 <= 256) return go<TAPS, 4, 256, 64, 4, 2, 3, MODE>(a, st);
    if (tiles(a, 128, 32) >= 800) return go<TAPS, 4, 256, 32, 4, 1, 3, MODE>(a, st);
    return go<TAPS, 4, 128, 32, 4, 1, 3, MODE>(a, st);
}

hipError_t launch_rows(int mode, const IgemmArgs& a, hipStream_t st) {
    if (a.Kw == 5) return mode == MODE_FWD ? go_mode<5, MODE_FWD>(a, st) : mode == MODE_DGRAD ? go_mode<5, MODE_DGRAD>(a, st) : go_mode<5, MODE_UNPOOL>(a, st);
    return mode == MODE_FWD ? go_mode<3, MODE_FWD>(a, st) : mode == MODE_DGRAD ? go_mode<3, MODE_DGRAD>(a, st) : go_mode<3, MODE_UNPOOL>(a, st);
}

}  // namespace lpm
