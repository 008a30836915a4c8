// Weight gradient (eq. 8) on the matrix cores, bfloat16 and float layers, two- and three-dimensional, fp32 accumulation.
//
//   dW[co][tap][ci] = sum over output pixels q of dz[q][co] * x[pixel(q, tap)][ci]
//
// The reduction index is the output pixel, and both operands are stored with the pixel outermost (dz [m][Do][Ho][Wo][Cout],
// x [m][D][H][W][Cin]).  A K tile is a run of pixels: its rows -- 32, 64 or 128 channels each -- are copied as they lie in memory,
// straight from global memory to LDS, through a ring of NST stages with one workgroup barrier per tile; rows outside the image
// or the channel range load zeros through the buffer bounds check.
//   bf16   The matrix operands are fetched with the LDS transpose read of gfx950 (16-bit elements, 64 bits per lane): in every
//          group of 16 lanes, lane i supplies the address of 4 consecutive elements of a row and receives element (i % 4) of the
//          rows supplied by lanes 4j + i/4, j = 0..3 -- a column of 4 rows.
//   float  v_mfma_f32_32x32x2_f32 takes one value per lane, channel lane % 32 of pixel lane / 32: a plain 4-byte LDS read.
// Blocks own BM output x BN input channels and one filter tap, or the three taps of a row of a 3x3 stride-1 filter:
//   LIN    1x1 filter, stride 1: a K tile is 64 (float: 32) consecutive pixels of both tensors.
//   PIX    one tap of any other filter: consecutive output pixels, each with its input pixel.
//   ROW3   a filter row: a K tile is eight segments of 8 pixels of an output row; the ten input pixels a segment meets are
//          loaded once, fetched once and shifted by one and two pixels with v_alignbit, so the LDS transpose reads serve three
//          times the products.
//          Layers of up to 32 x 32 channels (ROW3_32): tiles of that size and K tiles of 128 pixels, one wavefront for 16 of them each.  On
//          64 x 64 tiles three wavefronts of four multiplied zeros (per step, us: volumetric 1497 -> 1395, ResNet of width 32 on 40x40
//          1105 -> 1069; dW off from 64 bits by 3.7 to 4.5e-8 of its norm, 4.3 to 6.4e-8 on 64 x 64 tiles).
// Where PIX and ROW3 find a pixel or segment -- byte offsets and which of its pixels exist -- is worked out by one thread each,
// some hundred at a time, and kept in LDS: the loader's address arithmetic, a dozen instructions per load when every lane
// followed its own pixel from tile to tile, had taken more issue slots than the matrix instructions.
// Eight wavefronts: two groups of four (ROW3_32: eight of one) share the block's tile of dW, each with its part of every K tile, and add their sums through
// LDS at the end (one group per SIMD left the latencies of LDS and barrier uncovered: a launch is about one block per CU).
// The pixel range may be split over blocks; the partial results are summed by wgrad_reduce_batch in a fixed order.
// Measured alone with its reduction (us; four wavefronts, addresses followed lane by lane -> this): 3x3 256 -> 256 channels, 128
// images of 14x14 65.7 -> 47.5, 16 images 21.4 -> 18.7; 4 x 224^2 64 -> 64 34.7 -> 26.7; 1x1 1024 -> 256, 128 x 14^2 39.8 -> 28.7, now 24.7.
// Three stages for the 64-channel tiles: with four (or records for a longer run of pixels) the launch is faster alone, but
// the other streams' blocks no longer fit the CU beside it (R50 conv4_x at 64: 1.85 -> 1.89 ms per step).  Four for the
// 128-channel tiles and for filter rows over 64 K tiles and more, where the loads in flight count for more.
#include "lpm_internal.h"
#include "elem.h"
#include "lds_dma.h"
#include <algorithm>
#include <cmath>

namespace lpm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef short short4_ __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_ __attribute__((ext_vector_type(2)));

constexpr unsigned WG_OOB = 0xffffffffu;

struct WgArgs {
    const void* X;
    const void* DZ;
    float* out;            // dW, or the partials base when splits > 1
    float* db;             // bias gradient (sum of dz over the pixels), or NULL
    const float* rscale;   // the layer's per-channel scale, or NULL: row co of dW is multiplied by it (dz is the gradient before the scale)
    size_t part_stride;    // floats between the partials of consecutive splits (>= Cout*K + Cout)
    unsigned dz_bytes, x_bytes;
    int Cout, Cin, Kh, Kw, Kd, H, W, D, Ho, Wo, Do, stride, pad, pad_d;
    FastDiv dTW, dHo, dDo;
    int TW;                // units per output row: Wo pixels or ceil(Wo / 8) segments (ROW3)
    int units;             // m * Do * Ho * TW
    int kt_total, kt_per_split, splits;
    int accumulate;
    int co_tiles, ci_tiles, tap_groups, g2, kind;
    FastDiv dCi, dGroups, dG2, dKw, dAll;      // tiles along Cin, tap groups, those of a filter slice, taps of a filter row, tiles of dW
};

// four rows of the column a lane ends up with (see above)
__device__ __forceinline__ u32x2_ tr4(const unsigned char* p) {
    return __builtin_bit_cast(u32x2_, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_*)(p)));
}

enum { LIN = 0, PIX = 1, ROW3 = 3, ROW3_32 = 4 /* of 32 x 32 channels */ };

// pixels of a K tile
constexpr int wg_pixels(int es, int bm) { return es == 4 ? 32 : bm == 32 ? 128 : 64; }

// Where 16-byte chunk c of row r of an operand lies in an LDS row of P bytes, and which chunk lies at position c (its own inverse).
// 16 lanes of a transpose read take 32 bytes each of four consecutive rows: of 256-byte rows (128 channels) all four share their
// banks, so the rows' 64-byte quarters change places by the row (1x1 1024 -> 256 channels, 128 x 14^2, alone 28.3 -> 24.7 us; per step, R50
// conv4_x at 16 / 128 samples 1655 -> 1621, 6596 -> 6390).  Rows of 128 bytes take as long either way, and so do float's.
template <int ES, int P>
__device__ __forceinline__ int place(int c, int r) { return ES == 2 && P == 256 ? c ^ ((r & 3) << 2) : c; }

// One block: tile `tile` of dW (all of them, tap groups included) over pixel range `split`.
template <typename E, int BM, int BN, int KIND, int NST>
__device__ __forceinline__ void wgrad_tile(const WgArgs p, int tile, const int split) {
    constexpr int TAPS = KIND == ROW3 ? 3 : 1, WGM = BM == 32 ? 1 : 2, WGN = BN == 32 ? 1 : 2, WPG = WGM * WGN, GROUPS = 8 / WPG;
    constexpr int ES = sizeof(E), T = 512, KT = wg_pixels(ES, BM);
    constexpr int WTM = BM / WGM, WTN = BN / WGN, MI = WTM / 32, NI = WTN / 32;
    constexpr int HX = 10;                                                    // input pixels of a segment
    constexpr int PA = BM * ES, PB = BN * ES;                                 // bytes of an LDS row
    constexpr int A_BYTES = KT * PA;
    constexpr int B_ROWS = KIND == ROW3 ? KT / 8 * HX : KT;
    constexpr int A_LD = A_BYTES / (T * 16), B_LD = (B_ROWS * PB + T * 16 - 1) / (T * 16), LPT = A_LD + B_LD;
    constexpr int STAGE = A_BYTES + B_ROWS * PB;                              // (loads past the last row go to a dump of 1 KB)
    constexpr int KU = KIND == ROW3 ? KT / 8 : KT;                                 // units per K tile
    constexpr int CT = ES == 2 && KIND != ROW3 ? 8 : 16, CU = CT * KU;         // K tiles and units of a chunk of unit records
    constexpr int KSW = KT * ES / 32 / GROUPS;                                // K steps of a tile per wavefront
    static_assert(KIND != ROW3 || ES == 2, "filter rows: bf16");
    static_assert(A_LD * T * 16 == A_BYTES && CT % 2 == 0 && CT >= 8 && NST <= 4 && CU <= T && (B_ROWS * PB) % 1024 == 0, "layout");
    constexpr int DUMP = KIND == ROW3 ? 1024 : 0;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];      // NST stages, the dump, two chunks of records
    unsigned* rec1 = reinterpret_cast<unsigned*>(lds + NST * STAGE);          // PIX: offset of the input pixel, or none
    uint4* rec3 = reinterpret_cast<uint4*>(lds + NST * STAGE + DUMP);                // ROW3: dz offset, its pixels; x offset, mask of its pixels
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int tq = div_by(tile, p.dCi), ci_t = tile - tq * p.ci_tiles, co_t = div_by(tq, p.dGroups), grp = tq - co_t * p.tap_groups;
    const int co0 = co_t * BM, ci0 = ci_t * BN;
    const int kd = div_by(grp, p.dG2), grp2 = grp - kd * p.g2;      // filter slice, tap group inside it
    const int kh = TAPS == 3 ? grp2 : div_by(grp2, p.dKw), kw = TAPS == 3 ? 0 : grp2 - kh * p.Kw;
    const int kt0 = split * p.kt_per_split, nk = min(p.kt_total, kt0 + p.kt_per_split) - kt0;

    u32x4_ rsD = buffer_words(p.DZ, p.dz_bytes), rsX = buffer_words(p.X, p.x_bytes);

    // ---- unit records of chunk c, one per thread
    const unsigned cA = (unsigned)(p.Cout * ES), cB = (unsigned)(p.Cin * ES);
    auto fill = [&](int c) __attribute__((always_inline)) {
        if (KIND == LIN || tid >= CU) return;
        const int u = (kt0 + c * CT) * KU + tid, end = min(p.units, (kt0 + nk) * KU);
        const bool in = u < end;
        const int uu = in ? u : 0, q = div_by(uu, p.dTW), w = uu - q * p.TW, n = div_by(q, p.dHo), h = q - n * p.Ho;
        int img = n;
        bool ok = in;
        if (p.D > 1 || p.Do > 1 || p.Kd > 1) {           // n counts (sample, output slice) pairs
            const int ns = div_by(n, p.dDo), d = (n - ns * p.Do) * p.stride + kd - p.pad_d;
            ok = ok & ((unsigned)d < (unsigned)p.D);
            img = ns * p.D + d;
        }
        const int y = h * p.stride + kh - p.pad;
        ok = ok & ((unsigned)y < (unsigned)p.H);
        if (KIND == ROW3) {
            const int x0 = w * 8 - p.pad, lo = max(0, -x0), hi = min(HX, p.W - x0);
            rec3[(c & 1) * CU + tid] = make_uint4((unsigned)((n * p.Ho + h) * p.Wo + w * 8) * cA, in ? (unsigned)min(8, p.Wo - w * 8) : 0u,
                                                 (unsigned)((img * p.H + y) * p.W + x0) * cB, ok && hi > lo ? (1u << hi) - (1u << lo) : 0u);
        } else {
            const int x = w * p.stride + kw - p.pad;
            rec1[(c & 1) * CU + tid] = ok && (unsigned)x < (unsigned)p.W ? (unsigned)((img * p.H + y) * p.W + x) * cB : WG_OOB;
        }
    };
    // ---- loader state: the lane's row and channel in a K tile
    unsigned a_off[A_LD], b_off[B_LD];
    int a_px[A_LD], b_u[B_LD], b_in[B_LD];
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
        const int idx = i * T + tid, r = idx / (PA / 16), ch = co0 + place<ES, PA>(idx - r * (PA / 16), r) * (16 / ES);
        a_px[i] = ch < p.Cout ? r & 7 : 8;                        // ROW3: pixel of the segment (8: none)
        a_off[i] = KIND == ROW3 ? (unsigned)((r & 7) * p.Cout + ch) * ES : ch < p.Cout ? (unsigned)(r * p.Cout + ch) * ES : WG_OOB;
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        const int idx = i * T + tid, r = idx / (PB / 16), ch = ci0 + place<ES, PB>(idx - r * (PB / 16), r) * (16 / ES);
        const bool ok = r < B_ROWS && ch < p.Cin;
        b_u[i] = KIND == ROW3 ? min(r / HX, KU - 1) : r;
        b_in[i] = KIND == ROW3 ? (ok ? r - r / HX * HX : 31) : 0;                     // (bit 31 of a mask is never set)
        b_off[i] = KIND == ROW3 ? (unsigned)(b_in[i] * p.Cin + ch) * ES : KIND == LIN ? (ok ? (unsigned)(r * p.Cin + ch) * ES : WG_OOB)
                                                                                      : (ok ? (unsigned)ch * ES : WG_OOB);
    }
    // the records of the K tile to be loaded next, and its wave-uniform offsets (LIN; dz of PIX)
    int tl = 0;
    uint2 ra[KIND == ROW3 ? A_LD : 1], rb[KIND == ROW3 ? B_LD : 1];
    unsigned rp_[KIND == PIX ? B_LD : 1];
    unsigned sA = (unsigned)kt0 * (unsigned)KT * cA, sB = (unsigned)kt0 * (unsigned)KT * cB;
    auto look_up = [&]() __attribute__((always_inline)) {
        const int u0 = (tl * KU) & (2 * CU - 1);
        if constexpr (KIND == ROW3) {
#pragma unroll
            for (int i = 0; i < A_LD; ++i) ra[i] = *reinterpret_cast<const uint2*>(&rec3[u0 + ((i * T + tid) / (PA / 16) >> 3)]);
#pragma unroll
            for (int i = 0; i < B_LD; ++i) rb[i] = *(reinterpret_cast<const uint2*>(&rec3[u0 + b_u[i]]) + 1);
        } else if constexpr (KIND == PIX) {
#pragma unroll
            for (int i = 0; i < B_LD; ++i) rp_[i] = rec1[u0 + b_u[i]];
        }
    };
    // The loads of a tile come in four parts, put behind matrix instructions by the loop below.  Past the last tile nothing is
    // in range: zeros arrive, and the number of loads in flight stays what the waits assume.
    bool live = false;
    auto issue = [&](int st, int part) __attribute__((always_inline)) {
        unsigned char* sp = lds + st * STAGE + wave * 1024;
        if (part == 0 && KIND != ROW3) {
            live = tl < nk;
            rsD.z = live ? p.dz_bytes : 0u;
            if (KIND == LIN) rsX.z = live ? p.x_bytes : 0u;
        }
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            if (i * 4 / LPT != part) continue;
            if constexpr (KIND == ROW3) load_to_lds16(rsD, sp + i * T * 16, a_px[i] < (int)ra[i].y ? a_off[i] + ra[i].x : WG_OOB);
            else load_to_lds16s(rsD, sp + i * T * 16, a_off[i], live ? sA : 0u);
        }
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            if ((i + A_LD) * 4 / LPT != part) continue;
            unsigned char* d = sp + A_BYTES + i * T * 16;
            if (KIND == ROW3 && (i * T + wave * 64) * 16 >= B_ROWS * PB) d = lds + NST * STAGE;
            if constexpr (KIND == ROW3) load_to_lds16(rsX, d, (rb[i].y >> b_in[i]) & 1u ? b_off[i] + rb[i].x : WG_OOB);
            else if constexpr (KIND == PIX) load_to_lds16(rsX, d, ((rp_[i] != WG_OOB) & (b_off[i] != WG_OOB)) ? b_off[i] + rp_[i] : WG_OOB);
            else load_to_lds16s(rsX, d, b_off[i], live ? sB : 0u);
        }
        if (part == 3) {
            ++tl;
            sA += (unsigned)KT * cA;
            if (KIND == LIN) sB += (unsigned)KT * cB;
            look_up();
        }
    };

    f32x16 acc[TAPS][MI][NI];
#pragma unroll
    for (int t = 0; t < TAPS; ++t)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[t][mi][ni][i] = 0.f;
    // the blocks of tap group 0 / Cin tile 0 also sum dz over the pixels (the bias gradient): the wavefronts of the first column
    // add up the operands they hold anyway, a channel per lane
    const int wk = wave / WPG, wm = (wave - wk * WPG) / WGN, wn = wave % WGN;
    const bool do_bias = p.db != nullptr && grp == 0 && ci_t == 0 && wn == 0;
    float bsum[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) bsum[mi] = 0.f;

    // operand addresses.  bf16: reduction rows (lane / 32) * 8 + (lane % 16) / 4 (+ 4 for the second read), columns
    // (lane / 16 % 2) * 16 + (lane % 4) * 4 .. + 3 of 32 -- each lane ends up with column lane % 32.  float: row lane / 32.
    const int tr_row = (lane & 15) >> 2, tr_col = (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
    const int rl = lane & 31, kq = lane >> 5;
    // (K steps and a step's further reads lie multiples of four rows apart: the lane's first row is enough for place().)
    unsigned fa[MI], fb[NI];
    const int ra0 = ES == 2 ? kq * 8 + tr_row : kq, rb0 = ES == 2 ? kq * (KIND == ROW3 ? HX : 8) + tr_row : kq;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
        fa[mi] = (unsigned)(ra0 * PA + place<ES, PA>(wm * WTM / (16 / ES) + mi * (32 * ES / 16), ra0) * 16 + (ES == 2 ? tr_col : rl * 4));
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
        fb[ni] = (unsigned)(A_BYTES + rb0 * PB + place<ES, PB>(wn * WTN / (16 / ES) + ni * (32 * ES / 16), rb0) * 16 + (ES == 2 ? tr_col : rl * 4));

    // two operand sets: the next K tile is read from LDS while the matrix cores work on the present one
    struct Frag { unsigned a[KSW][MI][4], b[KSW][NI][TAPS == 3 ? 6 : 4]; };
    const int kw0 = wk * KSW;                // the wavefront's first K step
    auto read = [&](Frag& f, int st, int ks) __attribute__((always_inline)) {
        const unsigned char* sp = lds + st * STAGE;
        const int ka = kw0 + ks;
        if constexpr (ES == 2) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const unsigned char* q = sp + fa[mi] + ka * 16 * PA;
                const u32x2_ v0 = tr4(q), v1 = tr4(q + 4 * PA);
                f.a[ks][mi][0] = v0.x; f.a[ks][mi][1] = v0.y; f.a[ks][mi][2] = v1.x; f.a[ks][mi][3] = v1.y;
            }
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const unsigned char* q = sp + fb[ni] + ka * (TAPS == 3 ? 2 * HX : 16) * PB;
                const u32x2_ v0 = tr4(q), v1 = tr4(q + 4 * PB);
                f.b[ks][ni][0] = v0.x; f.b[ks][ni][1] = v0.y; f.b[ks][ni][2] = v1.x; f.b[ks][ni][3] = v1.y;
                if constexpr (TAPS == 3) {
                    const u32x2_ v2 = tr4(q + 8 * PB);
                    f.b[ks][ni][4] = v2.x; f.b[ks][ni][5] = v2.y;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) f.a[ks][mi][j] = *reinterpret_cast<const unsigned*>(sp + fa[mi] + (ka * 8 + j * 2) * PA);
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) f.b[ks][ni][j] = *reinterpret_cast<const unsigned*>(sp + fb[ni] + (ka * 8 + j * 2) * PB);
            }
        }
    };
    auto frag8 = [](unsigned x, unsigned y, unsigned z, unsigned w) __attribute__((always_inline)) { return __builtin_bit_cast(bf16x8, make_uint4(x, y, z, w)); };
    auto multiply = [&](const Frag& f, int ks) __attribute__((always_inline)) {
        if constexpr (ES == 2) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const unsigned (&b)[TAPS == 3 ? 6 : 4] = f.b[ks][ni];
                bf16x8 bt[TAPS];
                bt[0] = frag8(b[0], b[1], b[2], b[3]);
                if constexpr (TAPS == 3) {           // pixels x .. x+7, x+1 .. x+8, x+2 .. x+9 of the segment's input row, two per word
                    bt[1] = frag8(__builtin_amdgcn_alignbit(b[1], b[0], 16), __builtin_amdgcn_alignbit(b[2], b[1], 16),
                                  __builtin_amdgcn_alignbit(b[3], b[2], 16), __builtin_amdgcn_alignbit(b[4], b[3], 16));
                    bt[2] = frag8(b[1], b[2], b[3], b[4]);
                    // (the fetch's unused half stays allocated until here: reusing its register would wait for the fetch)
                    asm volatile("" : : "v"(b[5]));
                }
#pragma unroll
                for (int t = 0; t < TAPS; ++t)
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi)
                        acc[t][mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag8(f.a[ks][mi][0], f.a[ks][mi][1], f.a[ks][mi][2], f.a[ks][mi][3]), bt[t], acc[t][mi][ni], 0, 0, 0);
            }
            if (do_bias) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        bsum[mi] += __uint_as_float(f.a[ks][mi][k] << 16) + __uint_as_float(f.a[ks][mi][k] & 0xffff0000u);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
                        acc[0][mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(f.a[ks][mi][j]), __uint_as_float(f.b[ks][ni][j]), acc[0][mi][ni], 0, 0, 0);
                if (do_bias) {
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) bsum[mi] += __uint_as_float(f.a[ks][mi][j]);
                }
            }
        }
    };
    // a tile has landed once only the loads of the NST - 2 tiles behind it are outstanding; every wavefront's earlier operand
    // reads are complete then, too, so the stage they came from may be loaded again after the barrier
    auto meet = [&]() __attribute__((always_inline)) {
        LPM_WAIT_VM(LPT * (NST - 2));
        __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    if (nk > 0) {
        fill(0);
        if (KIND != LIN) __syncthreads();
        look_up();
#pragma unroll
        for (int i = 0; i < NST - 1; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) issue(i, q);
        Frag f0, f1;
        meet();
#pragma unroll
        for (int q = 0; q < 4; ++q) issue(NST - 1, q);
#pragma unroll
        for (int ks = 0; ks < KSW; ++ks) read(f0, 0, ks);
        int st = 0;
        auto half = [&](const Frag& cur, Frag& nxt) __attribute__((always_inline)) {
            const int st1 = st == NST - 1 ? 0 : st + 1;
            meet();
            read(nxt, st1, 0);
#pragma unroll
            for (int ks = 0; ks < KSW; ++ks) {
                __builtin_amdgcn_sched_barrier(0);
                if (ks + 1 < KSW) read(nxt, st1, ks + 1);
                multiply(cur, ks);
#pragma unroll
                for (int q = ks * 4 / KSW; q < (ks + 1) * 4 / KSW; ++q) issue(st, q);
            }
            __builtin_amdgcn_sched_barrier(0);
            st = st1;
        };
        // A chunk's records are written while the chunk before is worked on: the one before that, in the same place, has been
        // loaded (loads run NST - 1 tiles ahead), and at least CT - NST barriers pass until the first is read.
        for (int c = 0, it = 0; it < nk; ++c) {
            fill(c + 1);
            const int e = KIND == LIN ? nk : min(nk, it + CT);
            for (; it < e; it += 2) {            // (an odd count ends with a tile of zeros)
                half(f0, f1);
                half(f1, f0);
            }
        }
        LPM_WAIT_VM(0);
    }

    // the second half of the groups hands its sums to the first, until one is left
    __syncthreads();
#pragma unroll
    for (int g = GROUPS / 2; g > 0; g >>= 1) {
        const int slot = wk >= g ? wave - g * WPG : wave;
        float4* ex = reinterpret_cast<float4*>(lds) + slot * (TAPS * MI * NI * 4 * 64) + lane;
        float* exb = reinterpret_cast<float*>(lds + 4 * TAPS * MI * NI * 4096) + slot * (MI * 64) + lane;
        static_assert(4 * TAPS * MI * NI * 4096 + 4 * MI * 256 <= NST * STAGE, "the sums fit the dead stages");
        if (wk >= g && wk < 2 * g) {
#pragma unroll
            for (int t = 0; t < TAPS; ++t)
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            ex[(((t * MI + mi) * NI + ni) * 4 + q) * 64] = make_float4(acc[t][mi][ni][4 * q], acc[t][mi][ni][4 * q + 1], acc[t][mi][ni][4 * q + 2], acc[t][mi][ni][4 * q + 3]);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) exb[mi * 64] = bsum[mi];
        }
        __syncthreads();
        if (wk >= g) {
            if (g == 1) return;
        } else {
#pragma unroll
            for (int t = 0; t < TAPS; ++t)
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float4 v = ex[(((t * MI + mi) * NI + ni) * 4 + q) * 64];
                            acc[t][mi][ni][4 * q] += v.x; acc[t][mi][ni][4 * q + 1] += v.y; acc[t][mi][ni][4 * q + 2] += v.z; acc[t][mi][ni][4 * q + 3] += v.w;
                        }
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) bsum[mi] += exb[mi * 64];
        }
        if (g > 1) __syncthreads();
    }

    // accumulator element i of a lane: row (i / 4) * 8 + (lane / 32) * 4 + i % 4, column lane % 32
    const int KhKw = p.Kd * p.Kh * p.Kw;             // all taps of the filter
    const size_t total = (size_t)p.Cout * KhKw * p.Cin;
    const bool whole = p.splits == 1;
    float* out = p.out + (whole ? 0 : (size_t)split * p.part_stride);
    const int rq = kq * 4;
    if (do_bias) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const float v = bsum[mi] + __shfl_xor(bsum[mi], 32);           // the two halves of the pixels
            const int co = co0 + wm * WTM + mi * 32 + rl;
            if (kq || co >= p.Cout) continue;
            if (!whole) out[total + co] = v;
            else p.db[co] = p.accumulate ? p.db[co] + v : v;
        }
    }
    // Stores through a buffer resource: rows past the last output channel lie past the buffer's end.  (The row is part of the
    // lane's offset: as a wave-uniform offset beside it, 27 rows exceed the buffer of a layer with fewer output channels, and the
    // bounds check would have to survive a negative length.)
    const unsigned pitch = (unsigned)(KhKw * p.Cin) * 4u;
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(out, 0, (unsigned)p.Cout * pitch, 0x00020000);
#pragma unroll
    for (int t = 0; t < TAPS; ++t) {
        const int tap = (kd * p.Kh + kh) * p.Kw + (TAPS == 3 ? t : kw);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const int ci = ci0 + wn * WTN + ni * 32 + rl, cb = co0 + wm * WTM + mi * 32 + rq;
                if (ci >= p.Cin) continue;
                const unsigned vo = (unsigned)cb * pitch + (unsigned)(tap * p.Cin + ci) * 4u;
                f32x16 v = acc[t][mi][ni];
                if (whole && p.rscale) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] *= p.rscale[min(cb + (i >> 2) * 8 + (i & 3), p.Cout - 1)];
                }
                if (whole && p.accumulate) {         // all the loads before the first use
                    float old[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        old[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ro, vo + (unsigned)((i >> 2) * 8 + (i & 3)) * pitch, 0, 0));
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] += old[i];
                }
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[i]), ro, vo + (unsigned)((i >> 2) * 8 + (i & 3)) * pitch, 0, 0);
            }
    }
}

// --------------------------------------------------------------------------------------------------
// The weight gradients of several layers in one launch: the blocks of all of them fill the card together, so a layer need not be
// cut into as many pixel ranges as would do that alone (partial sums written, and read by the reduction), tiles of dW may be
// larger, and the host enqueues one kernel behind one event where it had one of each per layer -- a wait for an event of
// another stream is 10 us of host time.  Per step with a launch per layer / with groups, in us: ResNet-18/CIFAR 3259 / 2873, its
// width-48 form 2693 / 2445, R50 conv4_x at 64 1711 / 1660, volumetric 1738 / 1690, VGG-16/CIFAR 1869 / 1857,
// VGG-16/224 6706 / 6666.
// Registers: at most 128 for the 64-channel tiles, so that two wavefronts of a block, a contraction's and another stream's
// fit a SIMD's 512 (131 instead of 119 cost ResNet-18/CIFAR 2.5 %); the arguments come by value, by reference they cost those twelve.
struct WgGroup {
    int count;
    int first[LPM_WGRAD_GROUP];              // first block of every layer, INT_MAX past the last
    WgArgs d[LPM_WGRAD_GROUP];
};

// Tiles of 64 x 64 channels, by filter rows also of 32 x 32; BIG: 128 x 128 (see plan_group).
template <typename E, bool BIG>
__global__ void __launch_bounds__(512, BIG ? 3 : 4) wgrad_many(const WgGroup a) {
    const int v = xcd_remap((int)blockIdx.x, (int)gridDim.x);      // (as below)
    int k = 0;
#pragma unroll
    for (int j = 1; j < LPM_WGRAD_GROUP; ++j) k += v >= a.first[j];      // (a sum, not a search: no load waits for the one before)
    const WgArgs& p = a.d[k];
    const int local = v - a.first[k], n = p.co_tiles * p.ci_tiles * p.tap_groups, split = div_by(local, p.dAll), tile = local - split * n;
    constexpr int B = BIG ? 128 : 64, NST = BIG ? 4 : 3;
    if (p.kind == LIN) wgrad_tile<E, B, B, LIN, NST>(p, tile, split);
    else if (p.kind == PIX) wgrad_tile<E, B, B, PIX, NST>(p, tile, split);
    else if constexpr (sizeof(E) == 2 && !BIG) {
        if (p.kind == ROW3_32) wgrad_tile<E, 32, 32, ROW3, NST>(p, tile, split);
        else wgrad_tile<E, 64, 64, ROW3, NST>(p, tile, split);
    }
}
template <typename E, int BM, int BN, int KIND, int NST>
__global__ void __launch_bounds__(512, BM <= 64 ? 4 : 3) wgrad_mm(WgArgs p) {
    // all blocks of one pixel range go to one XCD (they read the same dz and x rows)
    const int v = xcd_remap((int)(blockIdx.z * gridDim.x + blockIdx.x), (int)(gridDim.x * gridDim.z)), split = v / (int)gridDim.x;
    wgrad_tile<E, BM, BN, KIND, NST>(p, v - split * (int)gridDim.x, split);
}
constexpr int wg_lds(int es, int bm, int bn, int kind, int nst) {
    const int kt = wg_pixels(es, bm);
    return nst * (kt * bm * es + (kind == ROW3 ? kt / 8 * 10 : kt) * bn * es) + (kind == LIN ? 0 : kind == ROW3 ? 1024 + kt * 4 * 16 : 1024 * 4);
}

struct WgPlan { int kind, big, groups, co_tiles, ci_tiles, TW, kt_total, kt_per, splits; };

static WgPlan plan_tiles(int dtype, const ConvGeom& g) {
    WgPlan pl{};
    const int tx = (g.Wo + 7) / 8;
    // a filter row per block where the row segments are mostly real pixels
    const bool row3 = dtype == LPM_BF16 && g.Kh == 3 && g.Kw == 3 && g.stride == 1 && g.Wo * 10 >= tx * 8 * 8;
    // 32 x 32 channels: the wavefronts that the rest of a 64 x 64 tile would idle take pixels instead, eight groups of them
    const bool half = row3 && g.Cout <= 32 && g.Cin <= 32;
    pl.kind = half ? ROW3_32 : row3 ? ROW3 : g.taps() == 1 && g.stride == 1 && g.pad == 0 && g.pad_d == 0 ? LIN : PIX;
    pl.groups = g.taps() / (row3 ? 3 : 1);
    pl.TW = row3 ? tx : g.Wo;
    const int64_t units = (int64_t)g.m * g.Do * g.Ho * pl.TW, ku = half ? 16 : row3 ? 8 : dtype == LPM_BF16 ? 64 : 32;
    pl.kt_total = (int)((units + ku - 1) / ku);
    pl.co_tiles = (g.Cout + 63) / 64;
    pl.ci_tiles = (g.Cin + 63) / 64;
    return pl;
}
static WgPlan big_tiles(const ConvGeom& g, WgPlan pl) {
    pl.big = 1;
    pl.co_tiles = (g.Cout + 127) / 128;
    pl.ci_tiles = (g.Cin + 127) / 128;
    return pl;
}
static int64_t wg_tiles(const WgPlan& pl) { return (int64_t)pl.co_tiles * pl.ci_tiles * pl.groups; }
static void set_splits(WgPlan& pl, int64_t sp) {
    pl.kt_per = (int)((pl.kt_total + sp - 1) / sp);
    pl.splits = (pl.kt_total + pl.kt_per - 1) / pl.kt_per;
}
// at least eight K tiles per block, four where that leaves fewer than eight ranges: every range costs a pass over dW
static int64_t most_splits(const ConvGeom& g, const WgPlan& pl) {
    const int64_t out_bytes = ((int64_t)g.Cout * g.K() + g.Cout) * 4;
    return std::min<int64_t>(std::max(std::max(1, pl.kt_total / 8), std::min(8, pl.kt_total / 4)), std::max<int64_t>(1, (64ll << 20) / out_bytes));
}

// One layer's launch.  A block per CU when it has the card to itself.  Beside the forward and data-phase kernels the CUs it leaves
// are not idle, and every block writes partial sums that the reduction reads: 192 blocks, 128 of the four times larger tiles.
// Per step with 256 / 192 / 128 for both, in us: ResNet-18/CIFAR 3440 / 3360 / 3304, VGG-16/224 6850 / 6805 / 6918, volumetric
// 1758 / 1764 / 1798; 128-channel tiles alone at 128: R50 conv4_x at 512 7240 -> 7066.
static WgPlan plan_wgrad(int dtype, const ConvGeom& g, bool shared) {
    WgPlan pl = plan_tiles(dtype, g);
    if (dtype == LPM_BF16 && pl.kind < ROW3 && g.Cout >= 128 && g.Cin >= 128 && wg_tiles(big_tiles(g, pl)) * std::max(1, pl.kt_total / 16) >= 192) pl = big_tiles(g, pl);
    const int64_t base = wg_tiles(pl), want = shared ? (pl.big ? 128 : 192) : 256;
    int64_t sp = std::max<int64_t>(1, want / base);
    if (base * sp < want * 3 / 4) sp = std::max<int64_t>(sp, want * 7 / 4 / base);
    set_splits(pl, std::min(sp, most_splits(g, pl)));
    return pl;
}
// pixel ranges that the scratch of a layer holds partial sums of
static int room_for(int dtype, const ConvGeom& g) { return std::max(plan_wgrad(dtype, g, false).splits, plan_wgrad(dtype, g, true).splits); }

// Several layers' launch: cut so that some 192 blocks have the same share of the K tiles, a K tile of a filter row counting twice
// (128 / 256: within 1 %, either way).  Large tiles, in a launch of their own, where the layers that can have them make 192 blocks
// of 16 K tiles, and then 64 blocks: few and long, they leave CUs to the other streams (R50 conv4_x at 64, per step: small tiles 1715 us,
// large ones on 128 / 96 / 64 blocks 1703 / 1690 / 1655; filter rows of 128 x 64 channels as well 1670, but 1 % more on VGG-16/224).
// Fewer ranges are longer fp32 sums.  Against 64 bits a 1x1 layer's dW is off by 1.3e-7 of its 2-norm in four ranges of 49 K tiles and by 2.3e-7
// in one (16 x 14^2 pixels), by 1.6e-7 and 2.9e-7 in one of 74, the most seen; the lone launch at 48 x 14^2 by 2.3e-7.  With the lone launches' ranges R50
// conv4_x takes 1 to 7 % more per step at 12 to 64 samples, ResNet-18/CIFAR 5 to 8, VGG-16/224 2 to 4, float ResNet-18 1 to 3.
static void plan_group(int dtype, const WgradTask* t, int n, WgPlan* pl) {
    auto cost = [](const WgPlan& p) { return (p.kind == ROW3 || p.big ? 2. : 1.) * p.kt_total; };
    auto large = [&](int i) { return dtype == LPM_BF16 && pl[i].kind < ROW3 && t[i].g.Cout >= 128 && t[i].g.Cin >= 128; };
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        pl[i] = plan_tiles(dtype, t[i].g);
        if (large(i)) blocks += wg_tiles(big_tiles(t[i].g, pl[i])) * std::max(1, pl[i].kt_total / 16);
    }
    double work[2] = {0, 0};
    for (int i = 0; i < n; ++i) {
        if (blocks >= 192 && large(i)) pl[i] = big_tiles(t[i].g, pl[i]);
        work[pl[i].big] += cost(pl[i]) * wg_tiles(pl[i]);
    }
    for (int i = 0; i < n; ++i) {
        const int64_t sp = (int64_t)std::ceil(cost(pl[i]) * (pl[i].big ? 64 : 192) / work[pl[i].big] - .05);
        set_splits(pl[i], std::max<int64_t>(1, std::min<int64_t>({sp, most_splits(t[i].g, pl[i]), room_for(dtype, t[i].g)})));
    }
}

// channel counts in whole 16-byte chunks, 32-bit byte offsets (with the rows a last K tile reaches past the end)
bool wgrad_mm_ok(int dtype, const ConvGeom& g) {
    const int es = dtype == LPM_BF16 ? 2 : 4;
    const int64_t lim = ((int64_t)1 << 32) - 1, slack = 4 * 64 + (int64_t)g.Ho * g.Wo, slack_in = (int64_t)2 * g.D * g.H * g.W + 4 * 64;
    return (g.Cin * es) % 16 == 0 && (g.Cout * es) % 16 == 0 && (g.rows_out() + slack) * g.Cout * es < lim &&
           (g.rows_in() + slack_in) * g.Cin * es < lim && (int64_t)(g.Cout + 128) * g.K() < ((int64_t)1 << 30);
}

static size_t wg_stride(const ConvGeom& g) { return ((size_t)g.Cout * g.K() + g.Cout + 3) & ~(size_t)3; }      // (16-byte loads in the reduction)
size_t wgrad_mm_ws_bytes(int dtype, const ConvGeom& g) {
    const int splits = room_for(dtype, g);
    return splits > 1 ? (size_t)splits * wg_stride(g) * sizeof(float) : 0;
}

static WgArgs wg_args(int dtype, const WgradTask& t, const WgPlan& pl) {
    const ConvGeom& g = t.g;
    const int es = dtype == LPM_BF16 ? 2 : 4;
    WgArgs a{};
    a.X = t.x; a.DZ = t.dz;
    a.out = pl.splits > 1 ? (float*)t.ws : t.dw;
    a.db = t.db; a.rscale = t.rscale;
    a.part_stride = wg_stride(g);
    a.dz_bytes = (unsigned)(g.rows_out() * g.Cout * es); a.x_bytes = (unsigned)(g.rows_in() * g.Cin * es);
    a.Cout = g.Cout; a.Cin = g.Cin; a.Kh = g.Kh; a.Kw = g.Kw; a.Kd = g.Kd;
    a.H = g.H; a.W = g.W; a.D = g.D; a.Ho = g.Ho; a.Wo = g.Wo; a.Do = g.Do;
    a.stride = g.stride; a.pad = g.pad; a.pad_d = g.pad_d;
    a.TW = pl.TW;
    a.dTW = fast_div(pl.TW); a.dHo = fast_div(g.Ho); a.dDo = fast_div(g.Do);
    a.units = (int)((int64_t)g.m * g.Do * g.Ho * pl.TW);
    a.kt_total = pl.kt_total; a.kt_per_split = pl.kt_per; a.splits = pl.splits;
    a.accumulate = t.accumulate;
    a.co_tiles = pl.co_tiles; a.ci_tiles = pl.ci_tiles; a.tap_groups = pl.groups; a.kind = pl.kind;
    a.g2 = pl.groups / a.Kd;
    a.dCi = fast_div(pl.ci_tiles); a.dGroups = fast_div(pl.groups); a.dG2 = fast_div(a.g2); a.dKw = fast_div(g.Kw);
    a.dAll = fast_div((int)wg_tiles(pl));
    return a;
}

template <typename E, int BM, int BN, int KIND, int NST>
static hipError_t go(const WgArgs& a, const WgPlan& pl, hipStream_t st) {
    constexpr int bytes = wg_lds(sizeof(E), BM, BN, KIND, NST);
    static DeviceSet done;
    const hipError_t attr = allow_lds(wgrad_mm<E, BM, BN, KIND, NST>, bytes, done);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((wgrad_mm<E, BM, BN, KIND, NST>), dim3((unsigned)wg_tiles(pl), 1, pl.splits), dim3(512), bytes, st, a);
    return hipGetLastError();
}
static hipError_t run_one(int dtype, const WgradTask& t, const WgPlan& pl, hipStream_t st) {
    const WgArgs a = wg_args(dtype, t, pl);
    if (dtype == LPM_F32) return pl.kind == LIN ? go<float, 64, 64, LIN, 3>(a, pl, st) : go<float, 64, 64, PIX, 3>(a, pl, st);
    if (pl.kind == ROW3_32) return go<bf16_t, 32, 32, ROW3, 3>(a, pl, st);
    if (pl.kind == ROW3) return pl.kt_per >= 64 ? go<bf16_t, 64, 64, ROW3, 4>(a, pl, st) : go<bf16_t, 64, 64, ROW3, 3>(a, pl, st);
    if (pl.big) return pl.kind == LIN ? go<bf16_t, 128, 128, LIN, 4>(a, pl, st) : go<bf16_t, 128, 128, PIX, 4>(a, pl, st);
    return pl.kind == LIN ? go<bf16_t, 64, 64, LIN, 3>(a, pl, st) : go<bf16_t, 64, 64, PIX, 3>(a, pl, st);
}
template <typename E, bool BIG>
static hipError_t go_many(const WgradTask* t, const WgPlan* pl, int n, hipStream_t st) {
    constexpr int B = BIG ? 128 : 64, NST = BIG ? 4 : 3, ES = sizeof(E);
    constexpr int kinds[5] = {wg_lds(ES, B, B, LIN, NST), wg_lds(ES, B, B, PIX, NST), 0, ES == 2 && !BIG ? wg_lds(ES, 64, 64, ROW3, NST) : 0, ES == 2 && !BIG ? wg_lds(ES, 32, 32, ROW3, NST) : 0};
    WgGroup a{};
    int blocks = 0, bytes = 0;
    for (int i = 0; i < n; ++i) {
        if ((bool)pl[i].big != BIG) continue;
        a.first[a.count] = blocks;
        a.d[a.count++] = wg_args(ES == 2 ? LPM_BF16 : LPM_F32, t[i], pl[i]);
        blocks += (int)(wg_tiles(pl[i]) * pl[i].splits);
        bytes = std::max(bytes, kinds[pl[i].kind]);
    }
    if (!a.count) return hipSuccess;
    for (int i = a.count; i < LPM_WGRAD_GROUP; ++i) a.first[i] = 0x7fffffff;
    static DeviceSet done;
    const hipError_t attr = allow_lds(wgrad_many<E, BIG>, std::max({kinds[LIN], kinds[PIX], kinds[ROW3], kinds[ROW3_32]}), done);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((wgrad_many<E, BIG>), dim3((unsigned)blocks), dim3(512), bytes, st, a);
    return hipGetLastError();
}
static ReduceDesc reduction(const WgradTask& t, const WgPlan& pl) {
    const ConvGeom& g = t.g;
    if (pl.splits == 1) return ReduceDesc{};
    return ReduceDesc{(const float*)t.ws, wg_stride(g), pl.splits, t.dw, (int64_t)g.Cout * g.K(), t.db, t.db ? g.Cout : 0, t.rscale, g.K(), t.accumulate};
}

hipError_t wgrad_mm_launch(int dtype, const WgradTask& t, hipStream_t st) {
    const WgPlan pl = plan_wgrad(dtype, t.g, false);
    const hipError_t e = run_one(dtype, t, pl, st);
    const ReduceDesc d = reduction(t, pl);
    if (e != hipSuccess || d.splits == 0) return e;
    return launch_reduce_batch(&d, 1, st);      // (the kernel that also reduces the layers of a group: the same order)
}
hipError_t wgrad_mm_group(int dtype, const WgradTask* t, int n, hipStream_t st, ReduceDesc* red) {
    if (n > LPM_WGRAD_GROUP) return hipErrorInvalidValue;
    WgPlan pl[LPM_WGRAD_GROUP];
    hipError_t e;
    if (n == 1) {
        pl[0] = plan_wgrad(dtype, t[0].g, true);
        e = run_one(dtype, t[0], pl[0], st);
    } else {
        plan_group(dtype, t, n, pl);
        e = dtype == LPM_F32 ? go_many<float, false>(t, pl, n, st) : go_many<bf16_t, false>(t, pl, n, st);
        if (e == hipSuccess && dtype == LPM_BF16) e = go_many<bf16_t, true>(t, pl, n, st);
    }
    for (int i = 0; i < n; ++i) red[i] = reduction(t[i], pl[i]);
    return e;
}

}  // namespace lpm
