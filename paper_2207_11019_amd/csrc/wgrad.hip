// Weight gradient (eq. 8) on the matrix cores, bfloat16 and float layers, two- and three-dimensional, fp32 accumulation.
//
//   dW[co][tap][ci] = sum over output pixels q of dz[q][co] * x[pixel(q, tap)][ci]
//
// The reduction index is the output pixel, and both operands are stored with the pixel outermost (dz [m][Do][Ho][Wo][Cout],
// x [m][D][H][W][Cin]).  A K tile is a run of pixels: its rows -- 64 or 128 channels each -- are copied as they lie in memory,
// straight from global memory to LDS, through a ring of NST stages with one workgroup barrier per tile; rows outside the image
// or the channel range load zeros through the buffer bounds check.
//   bf16   The matrix operands are fetched with the LDS transpose read of gfx950 (16-bit elements, 64 bits per lane): in every
//          group of 16 lanes, lane i supplies the address of 4 consecutive elements of a row and receives element (i % 4) of the
//          rows supplied by lanes 4j + i/4, j = 0..3 -- a column of 4 rows.
//   float  v_mfma_f32_32x32x2_f32 takes one value per lane, channel lane % 32 of pixel lane / 32: a plain 4-byte LDS read.
// Blocks own BM output x BN input channels and one filter tap (TAPS = 1: K tiles of 64 -- float: 32 -- consecutive output pixels),
// or the three taps of a row of a 3x3 stride-1 filter (TAPS = 3: K tiles of eight segments of 8 pixels of an output row; the ten
// input pixels a segment meets are loaded once, fetched once and shifted by one and two pixels with v_alignbit, so the LDS
// transpose reads, which bound the single-tap form at 64x64 channels, serve three times the products).
// The pixel range may be split over blocks; the partial results are summed by wgrad_reduce_batch in a fixed order.
#include "lpm_internal.h"
#include "elem.h"
#include "lds_dma.h"
#include <algorithm>

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
    FastDiv dTW, dHo;
    int TW;                // units per output row: Wo pixels (TAPS = 1) or ceil(Wo / 8) segments (TAPS = 3)
    int kt_total, kt_per_split, splits;
    int accumulate;
    int co_tiles, ci_tiles, tap_groups;
};

// four rows of the column a lane ends up with (see above)
__device__ __forceinline__ u32x2_ tr4(const unsigned char* p) {
    return __builtin_bit_cast(u32x2_, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_*)(p)));
}

template <typename E, int BM, int BN, int WGM, int WGN, int TAPS, int NST, int OCC>
__global__ void __launch_bounds__(WGM * WGN * 64, OCC) wgrad_mm(WgArgs p) {
    constexpr int ES = sizeof(E), T = WGM * WGN * 64, KT = ES == 2 ? 64 : 32;
    constexpr int WTM = BM / WGM, WTN = BN / WGN, MI = WTM / 32, NI = WTN / 32;
    constexpr int HX = 10;                                                    // input pixels of a segment
    constexpr int PA = BM * ES, PB = BN * ES;                                 // bytes of an LDS row
    constexpr int CA = PA / 16, CB = PB / 16;                                 // chunks of a row
    constexpr int A_BYTES = KT * PA;
    constexpr int B_ROWS = TAPS == 3 ? 8 * HX : KT;
    constexpr int A_LD = A_BYTES / (T * 16), B_LD = (B_ROWS * PB + T * 16 - 1) / (T * 16), LPT = A_LD + B_LD;
    constexpr int STAGE = A_BYTES + B_LD * T * 16;
    constexpr int KU = TAPS == 3 ? 8 : KT;                                    // units per K tile
    static_assert(TAPS == 1 || ES == 2, "filter rows: bf16");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];      // NST stages
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // all blocks of one pixel range go to one XCD (they read the same dz and x rows)
    const int v_id = xcd_remap((int)(blockIdx.z * gridDim.x + blockIdx.x), (int)(gridDim.x * gridDim.z));
    const int split = v_id / (int)gridDim.x;
    int tile = v_id - split * (int)gridDim.x;
    const int ci_t = tile % p.ci_tiles; tile /= p.ci_tiles;
    const int grp = tile % p.tap_groups;
    const int co_t = tile / p.tap_groups;
    const int co0 = co_t * BM, ci0 = ci_t * BN;
    const int g2d = p.tap_groups / p.Kd, kd = grp / g2d, grp2 = grp - kd * g2d;      // filter slice, tap group inside it
    const int kh = TAPS == 3 ? grp2 : grp2 / p.Kw, kw = TAPS == 3 ? 0 : grp2 % p.Kw;
    const int kt0 = split * p.kt_per_split, nk = min(p.kt_total, kt0 + p.kt_per_split) - kt0;

    u32x4_ rsD = buffer_words(p.DZ, p.dz_bytes), rsX = buffer_words(p.X, p.x_bytes);

    // ---- loader state.  The K tile's addresses move by constants from tile to tile, with a correction where a unit passes the
    // end of an output row or image: no multiplication per load.
    const int step_q = div_by(KU, p.dTW), step_w = KU - step_q * p.TW, step_n = div_by(step_q, p.dHo), step_h = step_q - step_n * p.Ho;
    auto locate = [&](int u, int& w, int& h, int& n) __attribute__((always_inline)) {
        const int q = div_by(u, p.dTW);
        w = u - q * p.TW; n = div_by(q, p.dHo); h = q - n * p.Ho;
    };
    const int UW = TAPS == 3 ? 8 : 1;                 // output pixels of a unit
    // dz, TAPS = 1: rows are consecutive in memory; a row past the last pixel lies past the buffer's end.
    // TAPS = 3: load i of a wavefront is segment i * T/64 + wave of the tile, pixel lane / 8
    unsigned a_off[A_LD], a_s[TAPS == 3 ? A_LD : 1];
    int aw[TAPS == 3 ? A_LD : 1], ah[TAPS == 3 ? A_LD : 1];
    const unsigned cA = (unsigned)(p.Cout * ES);
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
        const int idx = i * T + tid, r = idx / CA, c = idx - r * CA, ch = co0 + c * (16 / ES);
        if (TAPS == 3) {
            int an;
            locate(kt0 * KU + i * (T / 64) + wave, aw[i], ah[i], an);
            a_s[i] = (unsigned)((an * p.Ho + ah[i]) * p.Wo + aw[i] * 8) * cA;
            a_off[i] = ch < p.Cout ? (unsigned)((r & 7) * p.Cout + ch) * ES : WG_OOB;
        } else {
            a_off[i] = ch < p.Cout ? (unsigned)(r * p.Cout + ch) * ES : WG_OOB;
        }
    }
    if (TAPS == 1) a_s[0] = (unsigned)kt0 * (unsigned)KT * cA;
    const unsigned dA = (unsigned)((step_n * p.Ho + step_h) * p.Wo + step_w * 8) * cA, dAw = (unsigned)(p.Wo - p.TW * 8) * cA;
    // x: a row per pixel.  bx, by: input coordinates under the block's tap; thr: bx of the first unit past the output row
    unsigned b_off[B_LD];
    int bx[B_LD], by[B_LD], bn[B_LD], thr[TAPS == 3 ? B_LD : 1];
    const unsigned cB = (unsigned)(p.Cin * ES);
    const bool vol = p.D > 1 || p.Do > 1;
    const int sx = UW * p.stride, ylim = p.Ho * p.stride + kh - p.pad;
    if (TAPS == 1) thr[0] = p.TW * sx + kw - p.pad;
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        const int idx = i * T + tid, r = idx / CB, c = idx - r * CB, ch = ci0 + c * (16 / ES);
        const int seg = TAPS == 3 ? r / HX : r, in = TAPS == 3 ? r - seg * HX - p.pad : kw - p.pad;
        const bool ok = r < B_ROWS && ch < p.Cin;
        int w, h, n;
        locate(kt0 * KU + (r < B_ROWS ? seg : 0), w, h, n);
        bx[i] = ok ? w * sx + in : -(1 << 30);       // (a chunk that loads nothing stays left of every image)
        if (TAPS == 3) thr[i] = p.TW * sx + in;
        by[i] = h * p.stride + kh - p.pad;
        bn[i] = n;
        // volumes: the image (slice) is found anew for every tile, the offset is the one inside it
        b_off[i] = (unsigned)(((vol ? 0 : n) * p.H + by[i]) * p.W + w * sx + in) * cB + (unsigned)ch * ES;
    }
    const unsigned dB = (unsigned)(((vol ? 0 : step_n) * p.H + step_h * p.stride) * p.W + step_w * sx) * cB;
    const unsigned dBw = (unsigned)(p.stride * p.W - p.TW * sx) * cB;                                    // unit wraps to the next output row
    const unsigned dBh = (unsigned)((vol ? 0 : p.H) - p.Ho * p.stride) * (unsigned)p.W * cB;             // row wraps to the next image
    // The loads of a tile come in four parts, each behind a few matrix instructions of the loop below.  Past the last tile the
    // buffers count as empty: zeros arrive, and the number of loads in flight stays what the waits assume.
    int left = nk;
    bool live = false;
    auto issue = [&](int st, int part) __attribute__((always_inline)) {
        unsigned char* sp = lds + st * STAGE + wave * 1024;
        if (part == 0) {
            live = left > 0;
            --left;
            rsD.z = live ? p.dz_bytes : 0u;
            rsX.z = live ? p.x_bytes : 0u;
        }
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            if (i * 4 / LPT != part) continue;
            if (TAPS == 3) {
                load_to_lds16s(rsD, sp + i * T * 16, (lane >> 3) < p.Wo - aw[i] * 8 ? a_off[i] : WG_OOB, live ? a_s[i] : 0u);
                aw[i] += step_w; ah[i] += step_h; a_s[i] += dA;
                if (aw[i] >= p.TW) { aw[i] -= p.TW; ++ah[i]; a_s[i] += dAw; }
                if (ah[i] >= p.Ho) ah[i] -= p.Ho;
            } else load_to_lds16s(rsD, sp + i * T * 16, a_off[i], live ? a_s[0] : 0u);
        }
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            if ((i + A_LD) * 4 / LPT != part) continue;
            bool ok = ((unsigned)by[i] < (unsigned)p.H) & ((unsigned)bx[i] < (unsigned)p.W);
            unsigned off = b_off[i];
            if (vol) {                               // bn counts (sample, output slice) pairs
                const int ns = bn[i] / p.Do, d = (bn[i] - ns * p.Do) * p.stride + kd - p.pad_d;
                ok = ok & ((unsigned)d < (unsigned)p.D);
                off += (unsigned)((ns * p.D + d) * p.H * p.W) * cB;
            }
            load_to_lds16(rsX, sp + A_BYTES + i * T * 16, ok ? off : WG_OOB);      // (images past the last lie past the buffer's end)
            bx[i] += step_w * sx; by[i] += step_h * p.stride; b_off[i] += dB;
            if (vol) bn[i] += step_n;
            const bool ww = bx[i] >= thr[TAPS == 3 ? i : 0];
            bx[i] -= ww ? p.TW * sx : 0; by[i] += ww ? p.stride : 0; b_off[i] += ww ? dBw : 0u;
            const bool hw = by[i] >= ylim;
            by[i] -= hw ? p.Ho * p.stride : 0; b_off[i] += hw ? dBh : 0u;
            if (vol) bn[i] += hw ? 1 : 0;
        }
        if (TAPS == 1 && part == 3) a_s[0] += (unsigned)KT * cA;
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
    const int wm = wave / WGN, wn = wave - wm * WGN;
    const bool do_bias = p.db != nullptr && grp == 0 && ci_t == 0 && wn == 0;
    float bsum[MI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) bsum[mi] = 0.f;

    // operand addresses.  bf16: reduction rows (lane / 32) * 8 + (lane % 16) / 4 (+ 4 for the second read), columns
    // (lane / 16 % 2) * 16 + (lane % 4) * 4 .. + 3 of 32 -- each lane ends up with column lane % 32.  float: row lane / 32.
    const int tr_row = (lane & 15) >> 2, tr_col = (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
    const int rl = lane & 31, kq = lane >> 5;
    const unsigned fa = ES == 2 ? (unsigned)((kq * 8 + tr_row) * PA + wm * WTM * 2 + tr_col) : (unsigned)(kq * PA + (wm * WTM + rl) * 4);
    const unsigned fb = A_BYTES + (ES == 2 ? (unsigned)((kq * (TAPS == 3 ? HX : 8) + tr_row) * PB + wn * WTN * 2 + tr_col)
                                           : (unsigned)(kq * PB + (wn * WTN + rl) * 4));

    // two operand sets: the next K tile is read from LDS while the matrix cores work on the present one
    struct Frag { unsigned a[4][MI][4], b[4][NI][TAPS == 3 ? 6 : 4]; };
    auto read = [&](Frag& f, int st, int ks) __attribute__((always_inline)) {
        const unsigned char* sp = lds + st * STAGE;
        if constexpr (ES == 2) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const unsigned char* q = sp + fa + ks * 16 * PA + mi * 64;
                const u32x2_ v0 = tr4(q), v1 = tr4(q + 4 * PA);
                f.a[ks][mi][0] = v0.x; f.a[ks][mi][1] = v0.y; f.a[ks][mi][2] = v1.x; f.a[ks][mi][3] = v1.y;
            }
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const unsigned char* q = sp + fb + ks * (TAPS == 3 ? 2 * HX : 16) * PB + ni * 64;
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
                for (int mi = 0; mi < MI; ++mi) f.a[ks][mi][j] = *reinterpret_cast<const unsigned*>(sp + fa + (ks * 8 + j * 2) * PA + mi * 128);
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) f.b[ks][ni][j] = *reinterpret_cast<const unsigned*>(sp + fb + (ks * 8 + j * 2) * PB + ni * 128);
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
#pragma unroll
        for (int i = 0; i < NST - 1; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) issue(i, q);
        Frag f0, f1;
        meet();
#pragma unroll
        for (int q = 0; q < 4; ++q) issue(NST - 1, q);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) read(f0, 0, ks);
        int st = 0;
        auto half = [&](const Frag& cur, Frag& nxt) __attribute__((always_inline)) {
            const int st1 = st == NST - 1 ? 0 : st + 1;
            meet();
            read(nxt, st1, 0);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                __builtin_amdgcn_sched_barrier(0);
                if (ks < 3) read(nxt, st1, ks + 1);
                multiply(cur, ks);
                issue(st, ks);
            }
            __builtin_amdgcn_sched_barrier(0);
            st = st1;
        };
        for (int it = 0; it < nk; it += 2) {     // (an odd count ends with a tile of zeros)
            half(f0, f1);
            half(f1, f0);
        }
        LPM_WAIT_VM(0);
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
    // stores through a buffer resource: the lane's offset is fixed, an element adds a wave-uniform row offset, and rows past the
    // last output channel lie past the buffer's end
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
                const unsigned vo = ci < p.Cin ? (unsigned)cb * pitch + (unsigned)(tap * p.Cin + ci) * 4u : WG_OOB;
                f32x16 v = acc[t][mi][ni];
                if (whole && p.rscale) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] *= p.rscale[min(cb + (i >> 2) * 8 + (i & 3), p.Cout - 1)];
                }
                if (whole && p.accumulate) {         // all the loads before the first use
                    float old[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        old[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ro, vo, (unsigned)((i >> 2) * 8 + (i & 3)) * pitch, 0));
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] += old[i];
                }
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[i]), ro, vo, (unsigned)((i >> 2) * 8 + (i & 3)) * pitch, 0);
            }
    }
}

// --------------------------------------------------------------------------------------------------
struct WgPlan { int taps, big, groups, co_tiles, ci_tiles, TW, kt_total, kt_per, splits; };

static WgPlan plan_wgrad(int dtype, const ConvGeom& g) {
    WgPlan pl{};
    const int tx = (g.Wo + 7) / 8;
    // a filter row per block where the row segments are mostly real pixels
    const bool row3 = dtype == LPM_BF16 && g.Kh == 3 && g.Kw == 3 && g.stride == 1 && g.Wo * 10 >= tx * 8 * 8;
    pl.taps = row3 ? 3 : 1;
    pl.groups = g.taps() / pl.taps;
    pl.TW = row3 ? tx : g.Wo;
    const int64_t units = (int64_t)g.m * g.Do * g.Ho * pl.TW, ku = row3 ? 8 : dtype == LPM_BF16 ? 64 : 32;
    pl.kt_total = (int)((units + ku - 1) / ku);
    pl.big = dtype == LPM_BF16 && !row3 && g.Cout >= 128 && g.Cin >= 128 &&
             (int64_t)((g.Cout + 127) / 128) * ((g.Cin + 127) / 128) * pl.groups * std::max(1, pl.kt_total / 16) >= 192;
    const int t = pl.big ? 128 : 64;
    pl.co_tiles = (g.Cout + t - 1) / t;
    pl.ci_tiles = (g.Cin + t - 1) / t;
    const int64_t base = (int64_t)pl.co_tiles * pl.ci_tiles * pl.groups;
    const int64_t out_bytes = ((int64_t)g.Cout * g.K() + g.Cout) * 4;
    int64_t sp = std::max<int64_t>(1, 256 / base);
    if (base * sp < 192) sp = std::max<int64_t>(sp, 448 / base);
    // at least eight K tiles per block, four where that leaves fewer than eight ranges: every range costs a pass over dW
    sp = std::min<int64_t>(sp, std::max(std::max(1, pl.kt_total / 8), std::min(8, pl.kt_total / 4)));
    sp = std::min<int64_t>(sp, std::max<int64_t>(1, (64ll << 20) / out_bytes));
    pl.kt_per = (int)((pl.kt_total + sp - 1) / sp);
    pl.splits = (pl.kt_total + pl.kt_per - 1) / pl.kt_per;
    return pl;
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
    const WgPlan pl = plan_wgrad(dtype, g);
    return pl.splits > 1 ? (size_t)pl.splits * wg_stride(g) * sizeof(float) : 0;
}

template <typename E, int BM, int BN, int WGM, int WGN, int TAPS, int NST, int OCC>
static hipError_t go(const WgArgs& a, const WgPlan& pl, hipStream_t st) {
    constexpr int ES = sizeof(E), T = WGM * WGN * 64, KT = ES == 2 ? 64 : 32, rows = TAPS == 3 ? 80 : KT;
    constexpr int stage = KT * BM * ES + (rows * BN * ES + T * 16 - 1) / (T * 16) * (T * 16), bytes = NST * stage;
    static const hipError_t attr = hipFuncSetAttribute((const void*)wgrad_mm<E, BM, BN, WGM, WGN, TAPS, NST, OCC>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((wgrad_mm<E, BM, BN, WGM, WGN, TAPS, NST, OCC>), dim3((unsigned)(pl.co_tiles * pl.ci_tiles * pl.groups), 1, pl.splits),
                       dim3(T), bytes, st, a);
    return hipGetLastError();
}

hipError_t wgrad_mm_launch(int dtype, const ConvGeom& g, const void* x, const void* dz, float* dw, float* dbias, const float* rscale,
                           int accumulate, void* ws, hipStream_t st, ReduceDesc* deferred) {
    const int es = dtype == LPM_BF16 ? 2 : 4;
    const WgPlan pl = plan_wgrad(dtype, g);
    WgArgs a{};
    a.X = x; a.DZ = dz;
    a.out = pl.splits > 1 ? (float*)ws : dw;
    a.db = dbias; a.rscale = rscale;
    a.part_stride = wg_stride(g);
    a.dz_bytes = (unsigned)(g.rows_out() * g.Cout * es); a.x_bytes = (unsigned)(g.rows_in() * g.Cin * es);
    a.Cout = g.Cout; a.Cin = g.Cin; a.Kh = g.Kh; a.Kw = g.Kw; a.Kd = g.Kd;
    a.H = g.H; a.W = g.W; a.D = g.D; a.Ho = g.Ho; a.Wo = g.Wo; a.Do = g.Do;
    a.stride = g.stride; a.pad = g.pad; a.pad_d = g.pad_d;
    a.TW = pl.TW;
    a.dTW = fast_div(pl.TW); a.dHo = fast_div(g.Ho);
    a.kt_total = pl.kt_total; a.kt_per_split = pl.kt_per; a.splits = pl.splits;
    a.accumulate = accumulate;
    a.co_tiles = pl.co_tiles; a.ci_tiles = pl.ci_tiles; a.tap_groups = pl.groups;
    hipError_t e;
    if (dtype == LPM_F32) e = go<float, 64, 64, 2, 2, 1, 3, 2>(a, pl, st);
    else if (pl.taps == 3) e = go<bf16_t, 64, 64, 2, 2, 3, 3, 2>(a, pl, st);
    else if (pl.big) e = go<bf16_t, 128, 128, 2, 2, 1, 2, 2>(a, pl, st);
    else e = go<bf16_t, 64, 64, 2, 2, 1, 3, 2>(a, pl, st);
    if (e != hipSuccess || pl.splits == 1) return e;
    const int64_t n = (int64_t)g.Cout * g.K();
    const int nb = dbias ? g.Cout : 0;
    // one reduction kernel whether it runs now or batched with the stage's other layers: the same summation order
    const ReduceDesc d{(const float*)ws, a.part_stride, pl.splits, dw, n, dbias, nb, rscale, g.K(), accumulate};
    if (deferred) { *deferred = d; return hipSuccess; }
    return launch_reduce_batch(&d, 1, st);
}

}  // namespace lpm
