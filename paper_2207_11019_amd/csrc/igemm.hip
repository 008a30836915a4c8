// Implicit-GEMM contractions for gfx950 on the matrix cores: convolution forward (eq. 1) and data gradient (eq. 9) of
// bfloat16 and float layers, two- and three-dimensional, fp32 accumulation.
//
//   C[M][N] = A[M][K] * B[N][K]^T
//   forward  rows = output pixels, A gathered from x  [m][D][H][W][Cin],    B = w  [Cout][taps][Cin]
//   dgrad    rows = input pixels,  A gathered from dz [m][Do][Ho][Wo][Cout], B = wt [Cin][taps][Cout] (bf16), or, for float
//            layers, which keep no transposed copy, w [Cout][taps][Cin] read with its reduction index outermost
//   K runs over (filter tap, channel).  A strided data gradient goes by residue class (d, h, w modulo the stride) of the
//   input pixel: a class meets the taps of matching parity only, and its rows are written back to their pixels.
//
// Structure.  A K tile is 128 bytes of K (64 bf16 or 32 float values) of BM rows of A and BN rows of B, copied straight from
// global memory to LDS (buffer_load ... lds: no registers, no LDS stores), through a ring of NST stages with one workgroup
// barrier per tile.  LDS rows are 128 bytes without padding; chunk c (16 bytes) of row r lies at position c ^ (r / 2 % 8), so the
// operand reads of a wavefront (one chunk of 32 consecutive rows per half) fall on distinct banks: two rows span the 64 of them,
// and rows of one parity share theirs (with c ^ (r % 8) half of them idled: 0.94 M conflict cycles in a launch of 3x3 256 -> 256
// at 16 x 14^2, 0.01 M so, tap by tap; by filter rows, below, it has 0.26 M, of the lanes that read the row of zeros; 128x128 tiles, 128 x 14^2 x 256
// channels 3x3: 36.3 -> 34.6 us).  Out-of-range chunks -- padding taps, ragged
// rows -- load zeros through the buffer bounds check.  Whether a row meets a tap is one bit test against a mask made once per row.
// A channel count that is a multiple of 128 bytes lets a whole K tile lie in one tap (UNI): the tap is wave-uniform.
// Otherwise every lane follows its own chunk's tap through a table in LDS, so any multiple of 16 bytes of channels works.
// bf16 filters three taps wide, stride 1, in whole K tiles a tap (KT_ROW): the three taps of a filter row meet the same pixels but for one
// at either end, so the tile's pixels are loaded once for all three, into a ring of their own, and a tap is another row of LDS to read
// from: a third fewer bytes from L2 per product on 64x64 tiles, two fifths on 128x64.  Where a tap lies beside the image the reader
// takes a row of zeros.  Alone, us: 4 x 224^2 64 -> 64 33.1 -> 28.5, 16 x 32^2 x 64 5.4 -> 5.1; the others keep their time alone and
// leave the L2 to the streams beside them.
//
// What is neither goes by filter rows in pieces of 32 or 48 channels where it can (rows.hip; in_pieces below).
//
// The matrix instructions are v_mfma_f32_32x32x16_bf16 (a lane supplies 8 consecutive K values of row lane % 32) and
// v_mfma_f32_32x32x2_f32 (one value; four instructions share a 16-byte chunk, the K order inside a chunk being the same
// permutation for both operands).  The weights are the instruction's first operand: accumulator element i of a lane is output
// channel (i/4)*8 + (lane/32)*4 + i%4 of pixel lane % 32, four consecutive channels at a time.
#include "contraction.h"
#include "lds_dma.h"
#include <algorithm>
#include <cstring>
#include <utility>

namespace lpm {

// Chunks per lane whose epilogue operands are held across the main loop.  Two: the 64x64 tile (124 registers, 140 of a data
// gradient).  With the wider tiles too they gained alone, but fewer of the other streams' wavefronts fitted beside
// them: VGG-16/224 7.05 -> 7.18 ms per step.
constexpr int EARLY_ROWS = 2;

// partial tiles pass between blocks on different XCDs: stores go through to memory, loads do not hit a stale line
constexpr int AUX_AGENT = 16;

// layout of B: [N][K] rows; K outermost; K outermost and scaled
enum { BT_NONE = 0, BT_PLAIN = 1, BT_SCALED = 2 };

// f(0), f(1), ... until one of them is false
template <typename F, int... I>
__device__ __forceinline__ bool round_of(F& f, std::integer_sequence<int, I...>) { return (f(std::integral_constant<int, I>{}) && ...); }

// What a K tile is: chunks that follow their taps lane by lane; 64 (float: 32) channels of one tap; the same, the taps of a filter row
// one after the other
enum { KT_CHUNKS = 0, KT_TAP = 1, KT_ROW = 2 };

// KT_ROW: filter rows that are read or being loaded at a time, while tile t + 1 is read and tile t + nst (and a part of the row behind
// it) is loaded, whatever t
constexpr int row_stages(int nst) { return (nst + 3) / 3 + 1; }

// Block bx of the gx tiles' blocks, part bz of a split reduction.
template <typename E, int BM, int BN, int WGM, int WGN, int KG, int NST, int MODE, int KIND, int BT>
__device__ __forceinline__ void igemm_block(const IgemmArgs& p, const int bx, const int gx, const int bz) {
    constexpr int ES = sizeof(E), T = WGM * WGN * KG * 64, RS = T / 8;        // rows a load step covers
    constexpr int WTM = BM / WGM, WTN = BN / WGN, MI = WTM / 32, NI = WTN / 32;
    constexpr int KSW = 4 / KG;              // KG groups of wavefronts share the K steps of every tile; the first one ends up with the sums
    constexpr bool UNI = KIND != KT_CHUNKS, ROW = KIND == KT_ROW;
    // ROW: the pixels that a filter row of the tile meets, each of them once: one more at either end, whole pieces of eight
    constexpr int A_ROWS = ROW ? BM + 8 : BM, A_N = (A_ROWS + RS - 1) / RS;            // A_N load steps,
    constexpr int A_LD = ROW ? (A_N + 2) / 3 : A_N, B_LD = BN / RS, LPT = A_LD + B_LD;  // a third of them with every K tile
    constexpr int A_BYTES = A_ROWS * 128, NSTA = ROW ? row_stages(NST) : NST;
    constexpr int STAGE = ROW ? BN * 128 : A_BYTES + BN * 128, B_AT = ROW ? NSTA * A_BYTES : A_BYTES;      // ROW: a ring for A and one for B
    constexpr int STAGES = ROW ? B_AT + NST * STAGE + 1024 : NST * STAGE;                                   // ... and 1 KB for load steps past A's end
    static_assert(!BT || ES == 4, "float data gradient only");
    static_assert(!ROW || (ES == 2 && MODE != MODE_DGRAD_S), "filter rows: bf16, stride 1");
    // BT: B is read with its reduction index outermost; BT_SCALED: and multiplied by kscale, kept in LDS, on its way to the
    // matrix cores (the dz of a float layer with a scale is stored without it; 16 multiplications per 16 products)
    constexpr bool KS = BT == BT_SCALED;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];      // NST stages [+ tap table] [+ kscale]
    int4* tab = reinterpret_cast<int4*>(lds + STAGES);
    float* ksc = reinterpret_cast<float*>(lds + STAGES + (UNI ? 0 : MAX_TAB * 16));

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (strided: the residue classes differ in work, so their tiles stay in launch order, which deals them to the XCDs in turn)
    const int tile = MODE == MODE_DGRAD_S ? bx : xcd_remap(bx, gx);
    const int nt = (p.N + BN - 1) / BN, tm = div_by(tile, p.dNt), n0 = (tile - tm * nt) * BN;
    int m0 = tm * BM;
    int kt0 = bz * p.kt_per_split, kt1 = min(p.kt_total, kt0 + p.kt_per_split);
    int nkd = p.Kd, nkh = p.Kh, nkw = p.Kw, kd0 = 0, kh0 = 0, kw0 = 0, kstep = 1;      // taps visited: first and count per axis
    int ph = 0, pw = 0, pd = 0, Hc = p.Hr, Wc = p.Wr, Dc = p.Dr, rows = p.M;           // residue class of the rows and its extent
    int oh = p.pad, ow = p.pad, od = p.pad_d;
    const int Cc = p.Ci * ES / 16;                                                      // chunks per tap
    if (MODE == MODE_DGRAD_S) {
        // (divisions by the stride and by a class's extents are multiplications, the class's number a sum: an instruction sequence each, with
        // its own wait for its arguments, they had taken 1.5 us before the first load)
        const int s_ = p.stride;
        int c = 0;
#pragma unroll
        for (int k = 1; k < 16; ++k) c += tm >= p.cls_tile0[k];      // (past the last class they hold the number of tiles)
        const int pq = div_by(c, p.dS);
        pw = c - pq * s_;
        pd = div_by(pq, p.dS);
        ph = pq - pd * s_;
        Hc = div_by(p.Hr - ph + s_ - 1, p.dS); Wc = div_by(p.Wr - pw + s_ - 1, p.dS);
        Dc = p.Dr > 1 ? div_by(p.Dr - pd + s_ - 1, p.dS) : 1;
        rows = p.images * Dc * Hc * Wc;
        m0 = (tm - p.cls_tile0[c]) * BM;
        kstep = s_;
        // output pixel = class coordinate + (ph + pad - kh) / stride, an exact quotient that falls by one per visited tap
        oh = div_by(ph + p.pad, p.dS); ow = div_by(pw + p.pad, p.dS); od = div_by(pd + p.pad_d, p.dS);
        kh0 = ph + p.pad - oh * s_; kw0 = pw + p.pad - ow * s_;
        kd0 = pd + p.pad_d - od * s_;
        nkh = kh0 < p.Kh ? div_by(p.Kh - kh0 + s_ - 1, p.dS) : 0;
        nkw = kw0 < p.Kw ? div_by(p.Kw - kw0 + s_ - 1, p.dS) : 0;
        nkd = kd0 < p.Kd ? div_by(p.Kd - kd0 + s_ - 1, p.dS) : 0;
        kt0 = 0;
        kt1 = (nkd * nkh * nkw * Cc + 7) / 8;
        if (p.splits > 1) {
            const int per = (kt1 + p.splits - 1) / p.splits;
            kt0 = bz * per;
            kt1 = min(kt1, kt0 + per);
        }
    }
    const int ntap = nkd * nkh * nkw, nk = max(0, kt1 - kt0);
    const unsigned tapC = (unsigned)p.Ci * ES;                       // bytes of one tap's channels
    // byte steps of one visited tap along w, h, d: A moves with the filter (forward) or against it (data gradient)
    constexpr int SG = MODE == MODE_FWD ? 1 : -1;
    const unsigned aW = (unsigned)SG * tapC, aH = aW * (unsigned)p.Wi, aD = aH * (unsigned)p.Hi;
    // (BT: B's rows are the gathered channels, a tap is a column offset)
    const unsigned bTap = BT ? (unsigned)p.N * ES : tapC;
    const unsigned bW = bTap * kstep, bH = bW * (unsigned)p.Kw, bD = bH * (unsigned)p.Kh;
    const unsigned b0 = bTap * (unsigned)((kd0 * p.Kh + kh0) * p.Kw + kw0);

    // A's buffer starts `bias` bytes early, so that the offset of a row's tap (0,0) -- outside the image where there is
    // padding -- and the tap's own are both non-negative: lane offset + wave-uniform offset.  (Chunks whose tap misses the
    // image never use them.)
    // (ROW: a row's offset is that of the middle tap)
    const unsigned span = (unsigned)((((nkd - 1) * p.Hi + (nkh - 1)) * p.Wi + (ROW ? 0 : nkw - 1))) * tapC;      // from the first tap to the last
    const unsigned bias = MODE == MODE_FWD ? (unsigned)((od * p.Hi + oh) * p.Wi + (ROW ? 0 : ow)) * tapC : (ntap ? span : 0u);
    const unsigned aoff0 = MODE == MODE_FWD ? 0u : (ntap ? span : 0u);           // wave-uniform offset of the first tap
    u32x4_ rsA = buffer_words((const unsigned char*)p.A - bias, p.a_bytes + bias), rsB = buffer_words(p.B, p.b_bytes);

    if (!UNI) {
        for (int t = tid; t < ntap; t += T) {
            const int td = t / (nkh * nkw), r = t - td * (nkh * nkw), th = r / nkw, tw = r - th * nkw;
            tab[t] = make_int4((int)(aoff0 + td * aD + th * aH + tw * aW), (int)(b0 + td * bD + th * bH + tw * bW),
                               p.free_taps ? 1 : (int)((1u << (24 + td)) | (1u << (12 + th)) | (1u << tw)), 0);
        }
    }
    if (KS) {
        for (int c = tid; c < p.Ci; c += T) ksc[c] = p.kscale[c];      // (the first K tile's barrier makes it visible)
    }
    // ---- loader state.  Lane l of a load fills chunk position l % 8 of row r = 8 * wave + l / 8 (a load step is a multiple of 16
    // rows): it fetches chunk (l % 8) ^ (r / 2 % 8)
    const int lrow = lane >> 3, kcol = (lane & 7) ^ ((wave & 1) * 4 + (lrow >> 1));
    unsigned a_base[A_N], a_msk[A_N], b_off[B_LD];
    FastDiv dWc{}, dHc{}, dDc{};
    if (MODE == MODE_DGRAD_S) {
        dWc = p.dWc[Wc - div_by(p.Wr, p.dS)];
        dHc = p.dHc[Hc - div_by(p.Hr, p.dS)];
        if (p.Dr > 1) dDc = p.dDc[Dc - div_by(p.Dr, p.dS)];
    }
#pragma unroll
    for (int i = 0; i < A_N; ++i) {
        const int pos = i * RS + wave * 8 + lrow, row = ROW ? m0 - 1 + pos : m0 + pos;
        const bool ok = ROW ? (row >= 0) & (row < rows) & (pos < BM + 2) : row < rows;
        const int rr = ok ? row : 0;
        int wq, hq, n, dq = 0;
        if (MODE == MODE_DGRAD_S) {
            const int t = div_by(rr, dWc);
            wq = rr - t * Wc;
            n = div_by(t, dHc);
            hq = t - n * Hc;
            if (p.Dr > 1) { const int ns = div_by(n, dDc); dq = n - ns * Dc; n = ns; }
        } else {
            const int t = div_by(rr, p.dWr);
            wq = rr - t * p.Wr;
            n = div_by(t, p.dHr);
            hq = t - n * p.Hr;
            if (p.Dr > 1) { const int ns = div_by(n, p.dDr); dq = n - ns * p.Dr; n = ns; }
        }
        const bool fwd = MODE == MODE_FWD;
        const int h0 = fwd ? hq * p.stride - oh : hq + oh, w0 = ROW ? wq : fwd ? wq * p.stride - ow : wq + ow;
        int d0 = 0;
        unsigned m = 0xffffffffu;
        if (!p.free_taps) {
            m = fwd ? (tap_bits(max(0, -h0), min(nkh, p.Hi - h0)) << 12) | tap_bits(max(0, -w0), min(nkw, p.Wi - w0))
                    : (tap_bits(max(0, h0 - p.Hi + 1), min(nkh, h0 + 1)) << 12) | tap_bits(max(0, w0 - p.Wi + 1), min(nkw, w0 + 1));
            if (ROW) m = (m & 0xfff000u) | 1u;             // (along the image row the reader masks)
            m |= 1u << 24;
        }
        if (p.Kd > 1 || p.Dr > 1 || p.Di > 1) {
            d0 = fwd ? dq * p.stride - od : dq + od;
            if (!p.free_taps) m = (m & 0xffffffu) | ((fwd ? tap_bits(max(0, -d0), min(nkd, p.Di - d0)) : tap_bits(max(0, d0 - p.Di + 1), min(nkd, d0 + 1))) << 24);
        }
        a_msk[i] = ok ? m : 0u;
        a_base[i] = (unsigned)(((n * p.Di + d0) * p.Hi + h0) * p.Wi + w0) * tapC + (MODE == MODE_FWD ? bias : 0u) + (UNI ? (unsigned)kcol * 16u : 0u);
    }
    // BT: chunk (lane) of the K tile [32 reduction rows][BN channels]
    int bt_k[BT ? B_LD : 1], bt_t[BT ? B_LD : 1];          // channel and (non-UNI) tap of the reduction row
    const int kt_ch = 128 / ES;
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        if (BT) {
            const int idx = i * T + tid, kr = idx / (BN / 4), cc = idx - kr * (BN / 4);
            b_off[i] = n0 + cc * 4 < p.N ? (unsigned)(n0 + cc * 4) * ES + (UNI ? (unsigned)kr * p.b_pitch : 0u) : OOB;
            const int k = kt0 * kt_ch + kr;
            bt_t[i] = k / p.Ci; bt_k[i] = k - bt_t[i] * p.Ci;
        } else {
            b_off[i] = (unsigned)(n0 + i * RS + wave * 8 + lrow) * p.b_pitch + (UNI ? (unsigned)kcol * 16u : 0u);       // (rows past N lie past the buffer's end)
        }
    }
    // cursor of the next K tile: UNI: tap (wave-uniform) and how many K tiles follow in it; else the lane's chunk and its tap
    int c_td = 0, c_th = 0, c_tw = 0;
    // ROW: all three in filter rows for K tiles, the same for taps; B counts for itself, A's loads run ahead
    int per = nk, run = nk;                  // K tiles of a tap, K tiles until the tap changes or the reduction ends
    unsigned c_c = 0;                        // K tiles behind the tap's first one
    int l_t = 0, l_c = 0;
    int4 l_e = make_int4(0, 0, 0, 0);        // the tap's table entry, fetched a tile ahead
    if constexpr (ROW) {
        per = Cc / 8;
        if (kt0) {
            const int g = kt0 / 3, t = div_by(g, p.dKt);            // (a block's part begins with a filter row)
            c_c = (unsigned)(g - t * per);
            c_td = p.Kd > 1 ? t / p.Kh : 0;
            c_th = t - c_td * p.Kh;
        }
        run = min(per - (int)c_c, nk / 3);
    } else if (UNI) {
        per = Cc / 8;
        if (kt0) {
            const int t = div_by(kt0, p.dKt);
            c_c = (unsigned)(kt0 - t * per);
            if (MODE != MODE_DGRAD_S) {
                c_td = div_by(t, p.dKhw);
                const int r = t - c_td * nkh * nkw;
                c_th = div_by(r, p.dKw); c_tw = r - c_th * nkw;
            } else if (t > 0) {
                c_td = t / (nkh * nkw);
                const int r = t - c_td * nkh * nkw;
                c_th = r / nkw; c_tw = r - c_th * nkw;
            }
        }
        run = min(per - (int)c_c, nk);
    } else {
        const int k = kt0 * 8 + kcol;
        l_t = div_by(k, p.dCc); l_c = k - l_t * Cc;
        __syncthreads();                    // the tap table
        l_e = tab[l_t < ntap ? l_t : 0];
    }
    int left = (ROW ? nk / 3 : nk) - run;    // ... and the K tiles behind those
    int b_run = run, b_left = left;
    const int step_t = UNI ? 0 : div_by(8, p.dCc), step_c = UNI ? 0 : 8 - step_t * Cc;

    // UNI: the A offsets of the current tap, with the rows that miss the image out of range, and the wave-uniform offsets of the K
    // tile.  (They and the mask bit move on by differences: as sums of products they cost 80 ns of scalar arithmetic at every tap.)
    unsigned dA = 128, dB = BT ? (unsigned)kt_ch * p.b_pitch : 128u;                 // to the next K tile of the tap
    const unsigned tapA = tapC, tapB = BT ? (unsigned)p.Ci * p.b_pitch : tapC;       // what a tap's K tiles add up to
    unsigned a_cur[A_N], la = aoff0, lb = b0;
    if (UNI && kt0) {                        // (a part further on begins elsewhere)
        la += c_td * aD + c_th * aH + c_tw * aW + c_c * dA;
        lb += c_td * bD + c_th * bH + c_tw * bW + c_c * dB;
    }
    unsigned b_tap = tapC, b_chunk = dB - 2 * tapC;                                  // ROW: to the next tap of the row, from its last tap to the next channels' first
    unsigned bit = p.free_taps ? 1u : (1u << (24 + c_td)) | (1u << (12 + c_th)) | (1u << c_tw);
    const unsigned aWn = aW - tapA, bWn = bW - tapB;                                                          // the next tap of the row
    const unsigned aWH = aH - aW * (unsigned)(nkw - 1) - tapA, bWH = bH - bW * (unsigned)(nkw - 1) - tapB;    // past the last one
    const unsigned aHr = aH - tapA, aHDr = aD - aH * (unsigned)(nkh - 1) - tapA;                               // ROW
    const unsigned aHD = aD - aH * (unsigned)(nkh - 1) - aW * (unsigned)(nkw - 1) - tapA, bHD = bD - bH * (unsigned)(nkh - 1) - bW * (unsigned)(nkw - 1) - tapB;
    auto set_tap = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < A_N; ++i) a_cur[i] = (a_msk[i] & bit) == bit ? a_base[i] : OOB;
    };
    // The run of K tiles is over: the next tap, or none.  Then the buffers count as empty: further stages fill with zeros, the
    // number of loads in flight stays what the waits assume, and the loop below needs no special case at its end.  (The
    // wave-uniform offsets return to zero: the bounds check holds for offsets inside a buffer's length.)
    auto next_run = [&]() __attribute__((always_inline)) {
        if constexpr (ROW) {
            if (left == 0) {
                rsA.z = 0; la = 0; dA = 0;
                run = 0x7fffffff;
                return;
            }
            if (++c_th < nkh) { la += aHr; bit = ((bit & 0xfff000u) << 1) | (bit & 0xff000000u) | 1u; }
            else { c_th = 0; la += aHDr; bit = ((bit & 0xff000000u) << 1) | 0x1001u; }
            run = min(per, left);
            left -= run;
            set_tap();
            return;
        }
        if (!UNI || left == 0) {
            rsA.z = 0; rsB.z = 0;
            la = 0; lb = 0; dA = 0; dB = 0;
            run = 0x7fffffff;
            return;
        }
        if (++c_tw < nkw) { la += aWn; lb += bWn; bit += bit & 0xfffu; }
        else {
            c_tw = 0;
            if (++c_th < nkh) { la += aWH; lb += bWH; bit = ((bit & 0xfff000u) << 1) | (bit & 0xff000000u) | 1u; }
            else { c_th = 0; la += aHD; lb += bHD; bit = ((bit & 0xff000000u) << 1) | 0x1001u; }
        }
        if (p.free_taps) bit = 1u;
        run = min(per, left);
        left -= run;
        set_tap();
    };
    if (UNI) set_tap();
    // Issues the loads of the next K tile into a stage, in four parts, so that the loop below can put each behind a few matrix
    // instructions.
    // ROW: tile u of the block brings part (u + 2) % 3 of the pixels of filter row (u + 2) / 3: the last of them with the row's first tile.
    unsigned a_wr = 0;                       // A's stage being loaded
    auto issue_row = [&](int st, int u3, int part) __attribute__((always_inline)) {
        const int j = (u3 + 2) % 3;
        unsigned char* sp = lds + a_wr + wave * 1024;
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            if (i * 4 / LPT != part) continue;
            const int k = j * A_LD + i;
            const bool in = (k + 1) * RS <= A_ROWS || (k < A_N && k * RS + wave * 8 < A_ROWS);
            load_to_lds16s(rsA, in ? sp + k * RS * 128 : lds + STAGES - 1024, k < A_N && in ? a_cur[k < A_N ? k : 0] : OOB, la);
        }
        if (part == 3 && j == 2) {
            a_wr = a_wr == (NSTA - 1) * A_BYTES ? 0u : a_wr + A_BYTES;
            la += dA;
            if (--run == 0) next_run();
        }
        if (st < 0) return;                  // (ahead of the first tile: its pixels alone)
#pragma unroll
        for (int i = 0; i < B_LD; ++i)
            if ((i + A_LD) * 4 / LPT == part) load_to_lds16s(rsB, lds + B_AT + st * STAGE + (wave * 1024 + i * RS * 128), b_off[i], lb);
        if (part == 3) {
            if (u3 < 2) lb += b_tap;
            else {
                lb += b_chunk;
                if (--b_run == 0) {
                    if (b_left == 0) { rsB.z = 0; lb = 0; b_tap = 0; b_chunk = 0; b_run = 0x7fffffff; }
                    else { lb += 2 * b_tap; b_run = min(per, b_left); b_left -= b_run; }
                }
            }
        }
    };
    unsigned lbit = 0;
    bool lin = false;
    auto issue = [&](int st, int u, int part) __attribute__((always_inline)) {
        if constexpr (ROW) { issue_row(st, u % 3, part); return; }
        unsigned char* sp = lds + st * STAGE + wave * 1024;
        if (part == 0 && !UNI) {
            lin = l_t < ntap;
            lbit = (unsigned)l_e.z;
            la = (unsigned)l_e.x + (unsigned)l_c * 16u;
            lb = (unsigned)l_e.y + (unsigned)l_c * 16u;
        }
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            if (i * 4 / LPT != part) continue;
            if (UNI) load_to_lds16s(rsA, sp + i * RS * 128, a_cur[i], la);
            else load_to_lds16(rsA, sp + i * RS * 128, (lin & ((a_msk[i] & lbit) == lbit)) ? a_base[i] + la : OOB);
        }
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            if ((i + A_LD) * 4 / LPT != part) continue;
            unsigned char* d = sp + A_BYTES + i * RS * 128;
            if (UNI) load_to_lds16s(rsB, d, b_off[i], lb);
            else if (BT) {
                const bool bl = (bt_t[i] < ntap) & (b_off[i] != OOB);
                const unsigned tbb = (unsigned)tab[bt_t[i] < ntap ? bt_t[i] : 0].y;
                load_to_lds16(rsB, d, bl ? b_off[i] + tbb + (unsigned)bt_k[i] * p.b_pitch : OOB);
                bt_k[i] += kt_ch;
                while (bt_k[i] >= p.Ci) { bt_k[i] -= p.Ci; ++bt_t[i]; }
            } else load_to_lds16(rsB, d, lin ? b_off[i] + lb : OOB);
        }
        if (part == 3) {
            if (UNI) { la += dA; lb += dB; }
            else {
                l_t += step_t; l_c += step_c;
                if (l_c >= Cc) { l_c -= Cc; ++l_t; }
                l_e = tab[l_t < ntap ? l_t : 0];
            }
            if (--run == 0) next_run();
        }
    };

    // Operands of one K tile, 16 bytes per lane and step.  While the matrix cores work on one tile the next one is read from LDS,
    // and the tiles behind it are on their way there -- with one wavefront per SIMD (a launch of about one block per CU) nothing else
    // hides the LDS latency.  Two sets of them, or (TWO false) the next tile's over those of a step just multiplied: with two
    // wavefronts per SIMD, or float's longer products, the reads are covered all the same and the registers go to other streams'
    // wavefronts (float ResNet-18 2640 -> 2566 us per step, VGG-16/224 6640 -> 6575; the 64x64 tiles lose: R50 conv4_x at 64 1650 -> 1715).
    // A float data gradient reads its weights in four pieces of 4 bytes, which takes longer: two sets where a K tile lies in one tap (one / two:
    // a stage 480 -> 256 channels at 4 x 37^2 561 / 535 us, 512 -> 512 at 6 x 9^2 189 / 181, ResNet-18 at 4 / 9 / 16 samples 1.3-1.6 % less;
    // alone, a lone layer's 256 -> 256 at 16 x 14^2 loses 1 %).  In chunks across taps the second set costs a third block per CU its
    // registers: 64 -> 24 channels at 72 x 36 x 35, stride 2, 66.7 / 70.2.
    constexpr bool TWO = ES == 4 ? BT != BT_NONE && UNI : !(BM == 128 && BN == 128 && WGN == 4);
    constexpr bool DRAIN = TWO || NST < 4;
    constexpr int AHEAD = DRAIN ? NST : NST - 1;             // tiles between the one multiplied and the one being loaded
    // The first tiles are on their way before anything else is worked out: what follows, operand addresses and the epilogue's, costs as long
    // as they take to arrive.
    if (nk > 0) {
        if constexpr (ROW) {
            static_assert(!ROW || DRAIN, "A's ring is as long as that takes");
#pragma unroll
            for (int q = 0; q < 8; ++q) issue(-1, 1 + q / 4, q % 4);
        }
#pragma unroll
        for (int i = 0; i < AHEAD - 1; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) issue(i, i, q);
    }
    __builtin_amdgcn_sched_barrier(0);

    f32x16 acc[MI][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;

    const int kg = KG == 1 ? 0 : wave / (WGM * WGN), wv = wave - kg * (WGM * WGN), wm = wv / WGN, wn = wv - wm * WGN;
    // operand addresses: row lane % 32 of the wavefront's part, chunk 2*ks + lane/32 of the K tile
    const int rl = lane & 31, kh_ = lane >> 5;
    const unsigned char *opA[KSW], *opB[KSW];    // of the first stage; stages and rows further on are constants beside them
#pragma unroll
    for (int ks = 0; ks < KSW; ++ks) {
        const unsigned x = (unsigned)((((kg * KSW + ks) * 2 + kh_) ^ ((lane >> 1) & 7)) << 4);
        opA[ks] = lds + (unsigned)(wm * WTM + rl) * 128u + x;
        opB[ks] = lds + (ROW ? (unsigned)(B_AT + (wn * WTN + rl) * 128) + x : BT ? (unsigned)(A_BYTES + (wn * WTN + rl) * 4 + (kg * KSW * 2 + kh_) * 16 * BN) : (unsigned)(A_BYTES + (wn * WTN + rl) * 128) + x);
    }
    // ROW: the lane's pixel of A under each tap of the row, or the last row of the stage, which is never loaded with anything but zeros,
    // where that tap lies beside the image
    unsigned opR[3][MI], a_rd = 0;
    if constexpr (ROW) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const int at = wm * WTM + mi * 32 + rl, row = m0 + at, w = row - div_by(row, p.dWr) * p.Wr;
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                const bool out = s == 0 ? w == 0 : s == 2 ? w == p.Wr - 1 : false;
                const int r = out ? BM + 7 : at + s;
                opR[MODE == MODE_FWD ? s : 2 - s][mi] = (unsigned)(r * 128 + ((((kg * KSW) * 2 + kh_) ^ ((r >> 1) & 7)) << 4));
            }
        }
    }
    int ks_c[KS ? KSW : 1];                  // channel of the lane's chunk ks in the K tile read next
#pragma unroll
    for (int ks = 0; ks < (KS ? KSW : 0); ++ks) ks_c[ks] = (kt0 * kt_ch + ((kg * KSW + ks) * 2 + kh_) * 4) % p.Ci;
    const int ks_step = KS ? kt_ch % p.Ci : 0;

    struct Frag { uint4 a[KSW][MI], b[KSW][NI]; };
    // (tile u: its place in the filter row, where that counts)
    auto read = [&](Frag& f, int st, int u, int ks) __attribute__((always_inline)) {
        const int o = st * STAGE;
        {
            if (ROW && ks == 0 && u % 3 == 0 && u > 0) a_rd = a_rd == (NSTA - 1) * A_BYTES ? 0u : a_rd + A_BYTES;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
                f.a[ks][mi] = *reinterpret_cast<const uint4*>(ROW ? lds + ((opR[u % 3][mi] + a_rd) ^ (unsigned)(ks << 5)) : opA[ks] + o + mi * 4096);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                if (BT) {
                    const unsigned char* q = opB[ks] + o + ks * 32 * BN + ni * 128;
                    f.b[ks][ni] = make_uint4(*reinterpret_cast<const unsigned*>(q), *reinterpret_cast<const unsigned*>(q + BN * 4),
                                             *reinterpret_cast<const unsigned*>(q + 2 * BN * 4), *reinterpret_cast<const unsigned*>(q + 3 * BN * 4));
                    if constexpr (KS) {
                        const float4 k4 = *reinterpret_cast<const float4*>(ksc + ks_c[ks]);
                        uint4& b = f.b[ks][ni];
                        b = make_uint4(__float_as_uint(__uint_as_float(b.x) * k4.x), __float_as_uint(__uint_as_float(b.y) * k4.y),
                                       __float_as_uint(__uint_as_float(b.z) * k4.z), __float_as_uint(__uint_as_float(b.w) * k4.w));
                    }
                } else f.b[ks][ni] = *reinterpret_cast<const uint4*>(opB[ks] + o + ni * 4096);
            }
            if constexpr (KS) {
                ks_c[ks] += ks_step;
                if (ks_c[ks] >= p.Ci) ks_c[ks] -= p.Ci;
            }
        }
    };
    // the products of the wavefront's K steps, each with the first part of a tile that reaches it
    auto multiply = [&](const Frag& f, int part) __attribute__((always_inline)) {
        const int ks = part * KSW / 4;
        if (part * KSW % 4) return;
        if constexpr (ES == 2) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, f.b[ks][ni]), __builtin_bit_cast(bf16x8, f.a[ks][mi]), acc[mi][ni], 0, 0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) {
                        const unsigned a = j == 0 ? f.a[ks][mi].x : j == 1 ? f.a[ks][mi].y : j == 2 ? f.a[ks][mi].z : f.a[ks][mi].w;
                        const unsigned b = j == 0 ? f.b[ks][ni].x : j == 1 ? f.b[ks][ni].y : j == 2 ? f.b[ks][ni].z : f.b[ks][ni].w;
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(b), __uint_as_float(a), acc[mi][ni], 0, 0, 0);
                    }
        }
    };
    // A tile has landed once only the loads of the tiles behind it are outstanding.  DRAIN: the stage of the tile being multiplied
    // is loaded again behind the barrier, so every wavefront's operand reads are complete before it; with a stage more, the one loaded
    // again is that of the tile before, whose operands have been multiplied, and the reads under way need not be waited for.
    auto meet = [&]() __attribute__((always_inline)) {
        LPM_WAIT_VM(LPT * (AHEAD - 2));
        if (DRAIN) __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // The epilogue's operands: requested now where the accumulators leave the registers for it and this block is sure to need
    // them, so that they arrive under the main loop; a part of a split reduction leaves it to the block that comes last.
    typedef Epilogue<E, MI, NI, MODE> Ep;
    Ep ep;
    const int er0 = m0 + wm * WTM, ec0 = n0 + wn * WTN;
    constexpr bool SPLITS = BM == 64 && BN == 64 && KG == 1;      // (the plan splits no other tile)
    static_assert(!(SPLITS || KG > 1) || Ep::R <= EARLY_ROWS, "a split tile loads its operands here or with the partial sums");
    const bool early = Ep::R <= EARLY_ROWS && (!SPLITS || p.splits == 1);
    if (early && !kg) ep.load(p, er0, ec0, rows, lane, Hc, Wc, ph, pw, Dc, pd);
    if (nk > 0) {
        Frag f0;
        meet();
#pragma unroll
        for (int q = 0; q < 4; ++q) issue(AHEAD - 1, AHEAD - 1, q);
#pragma unroll
        for (int ks = 0; ks < KSW; ++ks) read(f0, 0, 0, ks);
        // The stages of a tile are constants: the loop goes round the ring (twice, where that has an odd number of stages and the
        // registers two sets) and leaves it behind the last tile.
        // A quarter of the next tile's reads and of the loads behind it go with a quarter of this one's products: the LDS,
        // the address arithmetic and the matrix cores work side by side (all reads first, and the products would wait
        // for the LDS queue to drain; all loads first, and the matrix cores would idle meanwhile).
        // (ROW: and as often as makes whole filter rows.)
        constexpr int ROUND0 = TWO && NST % 2 ? 2 * NST : NST, ROUND = ROW && ROUND0 % 3 ? 3 * ROUND0 : ROUND0;
        Frag f1;
        int it = 0;
        auto step = [&](auto index) __attribute__((always_inline)) {        // false: that was the last tile
            constexpr int u = decltype(index)::value, st = u % NST, st1 = (u + 1) % NST, ld = DRAIN ? st : (u + NST - 1) % NST;
            Frag &cur = TWO && (u & 1) ? f1 : f0, &nxt = TWO && !(u & 1) ? f1 : f0;
            meet();
            if constexpr (TWO) {
                read(nxt, st1, u + 1, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (q < 3 && (q + 1) * KSW % 4 == 0) read(nxt, st1, u + 1, (q + 1) * KSW / 4);
                    multiply(cur, q);
                    issue(ld, u + AHEAD, q);
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {     // (the next tile's operands over those just multiplied)
                    multiply(cur, q);
                    if (q * KSW % 4 == 0) read(cur, st1, u + 1, q * KSW / 4);
                    issue(ld, u + AHEAD, q);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            ++it;
            return (ROW && u % 3 != 2) || it < nk;       // (whole filter rows)
        };
        while (round_of(step, std::make_integer_sequence<int, ROUND>{})) {}
        LPM_WAIT_VM(0);
    }
    __syncthreads();                            // the stages are dead: the epilogue takes them

    // the other groups hand their sums to the first, which adds them up in order
    if constexpr (KG > 1) {
        static_assert(MI * NI == 1, "one accumulator tile per wavefront");
        float4* ex = reinterpret_cast<float4*>(lds + WGM * WGN * Epilogue<E, MI, NI, MODE>::PIECE * 4) + lane;      // (behind the first group's epilogue areas)
        if (kg) {
            float4* d = ex + ((kg - 1) * (WGM * WGN) + wv) * 256;
#pragma unroll
            for (int q = 0; q < 4; ++q) d[q * 64] = make_float4(acc[0][0][4 * q], acc[0][0][4 * q + 1], acc[0][0][4 * q + 2], acc[0][0][4 * q + 3]);
        }
        __syncthreads();
        if (kg) return;
        float4 t[KG - 1][4];
#pragma unroll
        for (int g = 0; g < KG - 1; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) t[g][q] = ex[(g * (WGM * WGN) + wv) * 256 + q * 64];
#pragma unroll
        for (int g = 0; g < KG - 1; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc[0][0][4 * q] += t[g][q].x; acc[0][0][4 * q + 1] += t[g][q].y; acc[0][0][4 * q + 2] += t[g][q].z; acc[0][0][4 * q + 3] += t[g][q].w;
            }
    }

    if constexpr (SPLITS) if (p.splits > 1) {
        // Every block of an output tile stores its partial sums (in accumulator order, 16 bytes per lane), and the one that
        // arrives last adds them in split order and carries on with the epilogue.  Stores and loads of the partials bypass the
        // XCD's own L2 (scope "agent"), so no cache is written back or invalidated: a store counted as done has reached memory.
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(p.part + (size_t)tile * p.splits * (BM * BN), 0, (unsigned)(p.splits * BM * BN * 4), 0x00020000);
        // (rows past the last one lie past the buffer's end: a fully connected layer of 4 samples would exchange 16 times what it
        // needs; VGG-16/224 6644 -> 6625 us per step)
        const unsigned mine = er0 + rl < rows ? (unsigned)(wv * (MI * NI * 1024) + lane * 4) * 4u : 0xc0000000u;
        const int me = bz;
        typedef unsigned int u4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u4 v = {__float_as_uint(acc[mi][ni][4 * q]), __float_as_uint(acc[mi][ni][4 * q + 1]),
                                  __float_as_uint(acc[mi][ni][4 * q + 2]), __float_as_uint(acc[mi][ni][4 * q + 3])};
                    __builtin_amdgcn_raw_buffer_store_b128(v, rp, mine + (unsigned)(((mi * NI + ni) * 4 + q) * 1024), (unsigned)(me * BM * BN * 4), AUX_AGENT);
                }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        int* flag = reinterpret_cast<int*>(lds);
        if (tid == 0) *flag = (int)__hip_atomic_fetch_add(p.count + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*flag != p.splits - 1) return;
        __syncthreads();                        // (flag is read before the area is written again)
        if (tid == 0) __hip_atomic_store(p.count + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // four splits' loads (and the epilogue's operands) before the first add (eight: 60 registers more, no faster)
        static_assert(MI == 1 && NI == 1, "one accumulator tile per wavefront");
        f32x16 sum;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum[i] = 0.f;
        for (int s0 = 0; s0 < p.splits; s0 += 4) {
            u4 v[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (s0 + k < p.splits) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        v[k][q] = __builtin_amdgcn_raw_buffer_load_b128(rp, mine + (unsigned)(q * 1024), (unsigned)((s0 + k) * BM * BN * 4), AUX_AGENT);
                }
            if (s0 == 0) ep.load(p, er0, ec0, rows, lane, Hc, Wc, ph, pw, Dc, pd);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (s0 + k < p.splits) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        sum[4 * q] += __uint_as_float(v[k][q].x); sum[4 * q + 1] += __uint_as_float(v[k][q].y);
                        sum[4 * q + 2] += __uint_as_float(v[k][q].z); sum[4 * q + 3] += __uint_as_float(v[k][q].w);
                    }
                }
        }
        acc[0][0] = sum;
    }

    // the wavefront's private staging area for the epilogue
    if (!SPLITS && !early) ep.load(p, er0, ec0, rows, lane, Hc, Wc, ph, pw, Dc, pd);
    float* area = reinterpret_cast<float*>(lds) + wave * MI * Ep::PIECE;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4*>(area + mi * Ep::PIECE + rl * Ep::PITCH + ni * 32 + q * 8 + kh_ * 4) =
                    make_float4(acc[mi][ni][4 * q], acc[mi][ni][4 * q + 1], acc[mi][ni][4 * q + 2], acc[mi][ni][4 * q + 3]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    ep.store(p, area, er0, ec0, rows, lane, Hc, Wc, ph, pw, Dc, pd);
    if constexpr (MODE == MODE_FWD && ES == 2) if (p.fwd_pool && p.Wr == 32) {
        __syncthreads();
        if constexpr (BM < 64) {}
        else if constexpr (MI == 1) {
            if (!(wm & 1)) ep.pool32(p, area, area + WGN * Ep::PIECE, er0, ec0, rows, lane);
        } else {
#pragma unroll
            for (int mi = 0; mi < MI; mi += 2) ep.pool32(p, area + mi * Ep::PIECE, area + (mi + 1) * Ep::PIECE, er0 + mi * 32, ec0, rows, lane);
        }
    }
}

template <typename E, int BM, int BN, int WGM, int WGN, int KG, int NST, int MODE, int KIND, int BT, int OCC>
__global__ void __launch_bounds__(WGM * WGN * KG * 64, OCC) igemm_kernel(const IgemmArgs p) {
    igemm_block<E, BM, BN, WGM, WGN, KG, NST, MODE, KIND, BT>(p, blockIdx.x, gridDim.x, blockIdx.z);
}

// Two contractions that do not read each other's results, in one launch (64x64 tiles): the blocks of the first, then those of
// the second.
struct IgemmPair { IgemmArgs p[2]; FastDiv tiles_d[2]; int tiles[2]; int second; };
template <typename E, int NST, int MODE0, int MODE1, bool UNI, int BT>
__global__ void __launch_bounds__(256, 2) igemm_pair(const IgemmPair g) {
    const int k = (int)blockIdx.x >= g.second, b = (int)blockIdx.x - (k ? g.second : 0), z = div_by(b, g.tiles_d[k]);
    if constexpr (MODE0 == MODE1) igemm_block<E, 64, 64, 2, 2, 1, NST, MODE0, UNI ? KT_TAP : KT_CHUNKS, BT>(g.p[k], b - z * g.tiles[k], g.tiles[k], z);
    else if (k == 0) igemm_block<E, 64, 64, 2, 2, 1, NST, MODE0, UNI ? KT_TAP : KT_CHUNKS, BT>(g.p[0], b - z * g.tiles[0], g.tiles[0], z);
    else igemm_block<E, 64, 64, 2, 2, 1, NST, MODE1, UNI ? KT_TAP : KT_CHUNKS, BT>(g.p[1], b - z * g.tiles[1], g.tiles[1], z);
}

// --------------------------------------------------------------------------------------------------
struct IgemmPlan { int tile, alone /* tile of a launch of its own */, splits, kt_total, kt_per; int64_t tiles; };
// Output tiles.  64x64: the launches of a few hundred blocks that small micro-batches make.  128x64, 128x128: half the
// operand traffic per product once there are enough tiles; 128x128 (eight wavefronts) with three stages where there is about one tile
// per CU, with two where there are two blocks per CU to hide each other's latencies.  256x128, eight wavefronts of 64x64 each: a
// quarter less LDS traffic per product, for what fills the card even so.  32x32, 32x64: the wavefronts of a block share the reduction (see
// plan_igemm).
enum { TILE_64 = 0, TILE_128x64, TILE_128, TILE_128_DEEP, TILE_256, TILE_32, TILE_32x64 };
static const int TILE_M[7] = {64, 128, 128, 128, 256, 32, 32}, TILE_N[7] = {64, 64, 128, 128, 128, 32, 64};
static int64_t tiles_of(int tile, int64_t M, int N) { return ((M + TILE_M[tile] - 1) / TILE_M[tile]) * ((N + TILE_N[tile] - 1) / TILE_N[tile]); }

// kt: K tiles (of the longest residue class); unit: see part_unit
static IgemmPlan plan_igemm(int es, int64_t M, int N, int kt, int unit) {
    IgemmPlan pl{};
    pl.tile = TILE_64;
    if (es == 2) {
        // Measured alone on MI355X (us, 64x64 / 128x64 / 128x128 of 4 wavefronts, which 8 have replaced / of 8 wavefronts):
        //   25088 x 256, K 2304: 51 / 46 / 39 / 43     12544 x 256, K 2304: 31 / 25 / 25 / 22      6272 x 512, K 2304: 33 / 25 / 27 / 24
        //    3136 x 512, K 4608: 26 / 29 / 47 / 34      3136 x 256, K 2304: 13 / 17 / 24 / 21     17496 x 160, K  864: 19 / 15 / 21 / 26
        // Alone, 64x64 wins up to some 384 tiles of 128x64.  Beside the other streams of a step, where the operand traffic of all of them
        // adds up, the larger tile wins from 180 on (per step, line at 384 / 250 / 180 / 120 / 90, in us: ResNet-18/CIFAR 3361 / 3312 /
        // 3308 / 3366 / 3371, VGG-16/224 6828 / 6833 / 6772 / 6778 / 6760, R50 conv4_x at 64 1746 / 1752 / 1749 / 1750 / 1870).
        const bool wide = N % 128 == 0 || N % 128 > 64;
        const int64_t n128 = tiles_of(TILE_128, M, N), t256 = tiles_of(TILE_256, M, N);
        // 128x128 of two stages / 256x128, alone: 25088 x 256, K 2304 35.4 / 32.9.  Where one block per CU covers its own latencies: from a
        // dozen K tiles on -- with fewer a block is loads and stores, one after the other, and two smaller ones take turns (R50 conv4_x,
        // two micro-batches of 36 / 48 / 64 / 96 / 128 samples, with four K tiles 1448 / 1848 / 2079 / 2977 / 3512, with twelve 1413 / 1774 /
        // 2042 / 2903 / 3488) -- and where the tiles fill 70 % of their rounds of CUs (14x14, 256 -> 512, 3x3, the three contractions:
        // 264 to 312 tiles 192-205 us, 128x128 instead 189-203; 80 % would leave out 25088 x 256, 107 us against 114).  With one column of
        // tiles both read the gathered rows once: VGG-16/224 6590 there, 6603 with 256x128.
        if (wide && N > 128 && kt >= 12 && 10 * t256 >= 7 * 256 * ((t256 + 255) / 256)) pl.tile = TILE_256;
        else if (wide && n128 >= 384) pl.tile = TILE_128;
        else if (wide && n128 >= 180) pl.tile = TILE_128_DEEP;
        else if (tiles_of(TILE_128x64, M, N) >= 180) pl.tile = TILE_128x64;
    }
    pl.kt_total = std::max(1, kt);
    pl.tiles = tiles_of(pl.tile, M, N);
    // A dozen K tiles per block (float, whose products take eight times as long: eight) while the tiles alone leave CUs idle: an
    // exchange of partial tiles costs 3 us, as long as a block's loads of ten K tiles take.  Measured with 8 / 12 / 16 per block,
    // in us: 16 x 8^2 x 256 channels, 3x3 10.4 / 9.8 / 10.3, 16 x 4^2 x 512 11.8 / 10.4 / 10.6, 16 x 16^2 x 128 (18 K tiles) 9.3 in two
    // parts, 7.3 in one.
    // No more than a block per CU: a second one on some of them delays the exchange (ResNet-18/CIFAR 3308 us per step with up to 320
    // blocks, 3275 with 256, 3315 with 224).
    int s = std::max(1, es == 2 ? pl.kt_total / 12 : (pl.kt_total + 4) / 8);
    const int64_t cap = (M <= 64 ? 1024 : 256) / pl.tiles;
    s = pl.tile == TILE_64 ? (int)std::min<int64_t>(s, std::max<int64_t>(1, cap)) : 1;
    pl.splits = std::max(1, std::min(s, pl.kt_total));
    pl.kt_per = (pl.kt_total + pl.splits * unit - 1) / (pl.splits * unit) * unit;
    pl.splits = (pl.kt_total + pl.kt_per - 1) / pl.kt_per;
    // Launched by itself, a call whose 64x64 tiles leave CUs idle goes on smaller ones instead whose reduction the wavefronts of the
    // block share: their sums meet in LDS, which takes 0.4 us where the exchange between blocks takes 3.  Alone, us, in parts / so: bf16 16 x 8^2 x 256
    // channels 3x3 9.2 / 6.7, 13 x 12^2 x 192 9.0 / 6.4, float 8 x 32^2 x 64 11.5 / 8.2, 8 x 16^2 x 128 11.9 / 8.7, 4 x 32^2 x 64 10.9 / 6.3.
    // A block reads all of K one tile after the other, and in a network, where the weights come from beyond the L2, up to 40 K tiles take less
    // than the exchange (32 x 4^2 x 512, 72 of them, 12.5 / 9.5 alone, but ResNet-18/CIFAR 2636 / 2683 us per step); rings of eight and six stages cover
    // that latency (16 images forward in parts 138.5, with four stages 139.2, with eight 134.6).  Fewer than 120 tiles leave more CUs
    // idle than the parts would.  bf16 without parts from a dozen K tiles on (16 images forward 136.2 / 133.7).  32x64 tiles fetch half
    // as many bytes again per product, which the products of float cover; bf16 in two parts on a full card stays (ResNet-18/CIFAR at 32 2719 / 2743).
    // Per step: float ResNet-18 at 4 / 8 / 16 samples 3026 / 2889, 2420 / 2376, 1705 / 1690, ResNet-18/CIFAR at 8 1991 / 1953, at 16 2135 / 2144
    // (LOCKED 1677 / 1651), of width 32 1034 / 1014, 48 2166 / 2147, VGG-16/CIFAR at 32 1172 / 1175, bottlenecks 128 wide at 8 655 / 641.
    // Beyond the upper lines for 32x64, alone, us, 64x64 / so: bf16 in two parts, 208 to 256 tiles (26 to 32 x 8^2 x 256) 9.7 / 7.3, 216 (16 x 12^2 x 192) 9.1 / 6.4,
    // which the step does not bear out; without parts, 270 (20 x 12^2 x 192) 7.2 / 9.1, 320 (40 x 8^2 x 256) 8.3 / 10.5, (20 x 16^2 x 128) 6.2 / 7.6.
    pl.alone = pl.tile;
    if (pl.tile == TILE_64 && pl.kt_total <= 40 && (pl.splits > 1 || (es == 2 && pl.kt_total >= 12))) {
        const int64_t t32 = tiles_of(TILE_32, M, N), t3264 = tiles_of(TILE_32x64, M, N);
        if (t32 >= 120 && t32 <= 256) pl.alone = TILE_32;
        else if (t3264 >= 120 && t3264 <= (es == 4 ? 320 : pl.splits > 1 ? 192 : 256)) pl.alone = TILE_32x64;
    }
    return pl;
}

static size_t plan_ws(const IgemmPlan& pl) {
    return pl.splits > 1 ? LPM_COUNT_BYTES + (size_t)pl.tiles * pl.splits * TILE_M[pl.tile] * TILE_N[pl.tile] * sizeof(float) : 0;
}

// byte offsets below 4 GiB (with the rows of a tile past the last one, and the bytes that the gathered tensor's buffer begins early:
// `halo` elements), 31-bit element counts
static bool fits(int dtype, const ConvGeom& g, int64_t halo_in, int64_t halo_out) {
    const int64_t es = dtype == LPM_BF16 ? 2 : 4, lim = ((int64_t)1 << 32) - 1, e31 = (int64_t)1 << 31;
    const int64_t in = g.rows_in() * g.Cin, out = g.rows_out() * g.Cout;
    return in < e31 && out < e31 && (in + halo_in) * es < lim && (out + halo_out) * es < lim &&
           (int64_t)(g.Cout + 256) * g.K() * es < lim && (int64_t)(g.Cin + 256) * g.taps() * g.Cout * es < lim;
}
static bool taps_fit(const ConvGeom& g, int ci, int es) {
    return g.Kd <= 8 && g.Kh <= 12 && g.Kw <= 12 && (((int64_t)ci * es) % 128 == 0 || g.taps() <= MAX_TAB);
}
static bool fwd_free(const ConvGeom& g) { return g.pad == 0 && g.pad_d == 0; }      // no tap of a forward pass leaves the image

bool mfma_fwd_ok(int dtype, const ConvGeom& g) {
    const int es = dtype == LPM_BF16 ? 2 : 4;
    if ((g.Cin * es) % 16 || !fits(dtype, g, (((int64_t)g.pad_d * g.H + g.pad) * g.W + g.pad) * g.Cin, 0)) return false;
    return taps_fit(g, g.Cin, es) || (fwd_free(g) && ((g.Cin * es) % 128 == 0 || g.taps() <= MAX_TAB));
}
// (a strided data gradient goes by residue classes of the image axes: stride^2 classes, stride^3 for a volume -- at most 16)
bool mfma_dgrad_ok(int dtype, const ConvGeom& g) {
    const int es = dtype == LPM_BF16 ? 2 : 4;
    return (g.Cout * es) % 16 == 0 && (dtype == LPM_BF16 || g.Cin % 4 == 0) && g.stride <= 4 && (g.stride <= 2 || !g.is3d()) &&
           fits(dtype, g, 0, (((int64_t)(g.Kd - 1) * g.Ho + g.Kh - 1) * g.Wo + g.Kw - 1) * g.Cout) && taps_fit(g, g.Cout, es);
}

// Whether the taps of a filter row can go one after the other, their pixels loaded once (KT_ROW).
static bool by_rows(int es, int ci, int kw, int stride, int pad) { return es == 2 && ci % 64 == 0 && kw == 3 && stride == 1 && pad == 1; }
// K tiles that every part of a split reduction has whole
static int part_unit(int es, int ci, int kw, int stride, int pad) { return by_rows(es, ci, kw, stride, pad) ? 3 : 1; }

static int k_tiles(int64_t taps, int ci, int es) { return (int)((taps * ci * es / 16 + 7) / 8); }
static IgemmPlan plan_fwd(int dtype, const ConvGeom& g) {
    const int es = dtype == LPM_BF16 ? 2 : 4;
    IgemmPlan pl = plan_igemm(es, g.rows_out(), g.Cout, k_tiles(g.taps(), g.Cin, es), part_unit(es, g.Cin, g.Kw, g.stride, g.pad));
    if (es == 2 && g.Wo == 32) pl.alone = pl.tile;      // (pooling windows of 32-wide images take two rows of 32 pixels; the plan does not know which layers pool)
    return pl;
}
// taps a residue class of a strided data gradient meets at most
static IgemmPlan plan_dgrad(int dtype, const ConvGeom& g) {
    const int es = dtype == LPM_BF16 ? 2 : 4, s = g.stride;
    const int64_t taps = (int64_t)((g.Kd + s - 1) / s) * ((g.Kh + s - 1) / s) * ((g.Kw + s - 1) / s);
    int64_t rows = g.rows_in();
    if (s > 1) rows += 128 * (g.D > 1 ? s * s * s : s * s);          // (every class ends in a ragged tile: up to 63 rows of the 64-row tiles whose
                                                                      // scratch goes by this count; for the choice of a larger tile, an estimate)
    IgemmPlan pl = plan_igemm(es, rows, g.Cin, k_tiles(taps, g.Cout, es), part_unit(es, g.Cout, g.Kw, s, g.pad));
    if (s > 1) pl.alone = pl.tile;                                    // (the 32-row kernels know no residue classes)
    return pl;
}
bool mfma_dgrad_kscale_ok(const ConvGeom& g) { return g.Cout <= MAX_KSCALE; }
size_t mfma_fwd_ws_bytes(int dtype, const ConvGeom& g) { return plan_ws(plan_fwd(dtype, g)); }
size_t mfma_dgrad_ws_bytes(int dtype, const ConvGeom& g) { return plan_ws(plan_dgrad(dtype, g)); }

// whether the forward contraction of this layer can also store the 2x2 max-pooling of its output: the windows of 32
// consecutive output pixels are whole ones, or those of 64 (two image rows;
// VGG-16/CIFAR 1827 us per step with a pass of its own over the 32x32 layer, 1808 without)
bool mfma_fwd_pools(int dtype, const ConvGeom& g) {
    return dtype == LPM_BF16 && mfma_fwd_ok(dtype, g) && !g.is3d() && !(g.Ho & 1) && (g.Wo == 2 || g.Wo == 4 || g.Wo == 8 || g.Wo == 16 || g.Wo == 32) && g.Cout % 8 == 0;
}

template <typename E, int BM, int BN, int WGM, int WGN, int KG, int NST, int MODE, int KIND, int BT, int OCC>
static hipError_t go(const IgemmArgs& a, int64_t tiles, hipStream_t st) {
    constexpr int rings = KIND == KT_ROW ? row_stages(NST) * (BM + 8) * 128 + NST * BN * 128 + 1024 : NST * (BM + BN) * 128;
    constexpr int stages = rings + (KIND != KT_CHUNKS ? 0 : MAX_TAB * 16) + (BT == BT_SCALED ? MAX_KSCALE * 4 : 0);
    constexpr int epilogue = KG * BM * WGN * (BN / WGN + 4) * 4, bytes = stages > epilogue ? stages : epilogue;
    static DeviceSet done;
    const hipError_t attr = allow_lds(igemm_kernel<E, BM, BN, WGM, WGN, KG, NST, MODE, KIND, BT, OCC>, bytes, done);
    if (attr != hipSuccess) return attr;
    launch_last(igemm_kernel<E, BM, BN, WGM, WGN, KG, NST, MODE, KIND, BT, OCC>, dim3((unsigned)tiles, 1, a.splits), dim3(WGM * WGN * KG * 64), bytes, st, a);
    return hipGetLastError();
}

template <typename E, int MODE, int KIND, int BT>
static hipError_t go_tile(const IgemmPlan& pl, const IgemmArgs& a, int64_t tiles, hipStream_t st) {
    if constexpr (sizeof(E) == 2) {
        if (pl.tile == TILE_128x64) return go<E, 128, 64, 2, 2, 1, 3, MODE, KIND, BT, 2>(a, tiles, st);
        if (pl.tile == TILE_128_DEEP) return go<E, 128, 128, 2, 4, 1, 3, MODE, KIND, BT, 2>(a, tiles, st);
        if constexpr (KIND != KT_ROW) {
            if (pl.tile == TILE_128) return go<E, 128, 128, 2, 4, 1, 2, MODE, KIND, BT, 2>(a, tiles, st);
            if (pl.tile == TILE_256) return go<E, 256, 128, 4, 2, 1, 3, MODE, KIND, BT, 2>(a, tiles, st);
        }
    }
    if constexpr (MODE != MODE_DGRAD_S) {
        if (pl.tile == TILE_32) return go<E, 32, 32, 1, 1, 4, 8, MODE, KIND, BT, 2>(a, tiles, st);
        if (pl.tile == TILE_32x64) return go<E, 32, 64, 1, 2, 2, 6, MODE, KIND, BT, 2>(a, tiles, st);
    }
    // About one block per CU: nothing but its own loads in flight keeps the memory path busy, four stages (R50 conv4_x at 64 1.81 ->
    // 1.77 ms per step).  More blocks: three, so that three of them, or other streams' kernels, share a CU (VGG-16/224 6.83 against
    // 6.95 ms with four).
    if (tiles * a.splits <= 320) return go<E, 64, 64, 2, 2, 1, 4, MODE, KIND, BT, 2>(a, tiles, st);
    return go<E, 64, 64, 2, 2, 1, 3, MODE, KIND, BT, 2>(a, tiles, st);
}
template <typename E, int MODE, int BT>
static hipError_t go_uni(const IgemmPlan& pl, const IgemmArgs& a, int64_t tiles, hipStream_t st) {
    // Filter rows: where a tap is one K tile (the order of the sums is the same), and on 64x64 and 32-row tiles up to 40 K tiles, or 24 a part (per step,
    // tap by tap / so, in us: R50 conv4_x at 64 1621 / 1590, VGG-16/CIFAR 1800 / 1769, ResNet-18/CIFAR 2706 / 2637; without the split ones VGG-16/CIFAR
    // 1794, ResNet-18/CIFAR 2683).  With two blocks of 128x128 to a CU the registers do not suffice (4 x 112^2 x 128 20.5 / 23.6).
    // Larger tiles and longer sums keep their order: 1 % per step at most, and a forward sum in another order moves masks and maxima of the
    // deep networks that make them.  Longer ones alone, tap by tap / so: 45 K tiles (16 x 14^2 x 320) 11.3 / 11.1; 54 (x 384) 18.8 / 15.8, at 16 x 16^2
    // 16.1 / 16.5; 72 (32 x 8^2 x 512) 16.0 / 15.2, at 16 x 14^2 24.4 / 24.9, in parts of 36 (64 x 4^2) 13.5 / 13.2.
    if constexpr (sizeof(E) == 2 && MODE != MODE_DGRAD_S)
        if (by_rows(2, a.Ci, a.Kw, a.stride, a.pad) && (a.Ci == 64 ? pl.tile != TILE_128 && pl.tile != TILE_256 : TILE_M[pl.tile] <= 64 && (a.kt_total <= 40 || a.kt_per_split <= 24)))
            return go_tile<E, MODE, KT_ROW, BT>(pl, a, tiles, st);
    if ((a.Ci * (int)sizeof(E)) % 128 == 0) return go_tile<E, MODE, KT_TAP, BT>(pl, a, tiles, st);
    return go_tile<E, MODE, KT_CHUNKS, BT>(pl, a, tiles, st);
}

hipError_t launch_zero_counts(void* const* heads, int n, hipStream_t st);

// Filter rows in pieces of a few channels (rows.hip): channels that make no whole K tiles.
bool rows_take(const IgemmArgs& a, bool keep_order);
hipError_t launch_rows(int mode, const IgemmArgs& a, hipStream_t st);

struct IgemmCall { int dtype, mode, tiles; bool any_order; IgemmArgs a; IgemmPlan pl; };
static_assert(sizeof(IgemmCall) <= sizeof(HeldCall::bytes), "room for a held call");

// what follows from the plan's tile
static void lay_tiles(IgemmCall& c) {
    IgemmArgs& a = c.a;
    const int bm = TILE_M[c.pl.tile], nt = (a.N + TILE_N[c.pl.tile] - 1) / TILE_N[c.pl.tile];
    int mt = (a.M + bm - 1) / bm;
    if (c.mode == MODE_DGRAD_S) {          // row tiles per residue class (d % stride, h % stride, w % stride)
        const int s = a.stride, ncls = (a.Dr > 1 ? s : 1) * s * s;
        const int64_t m = a.M / ((int64_t)a.Dr * a.Hr * a.Wr);
        mt = 0;
        for (int k = 0; k < ncls; ++k) {
            a.cls_tile0[k] = mt;
            const int pd = k / (s * s), ph = (k / s) % s, pw = k % s;
            const int64_t Dc = a.Dr > 1 ? (a.Dr - pd + s - 1) / s : 1, Hc = (a.Hr - ph + s - 1) / s, Wc = (a.Wr - pw + s - 1) / s;
            mt += (int)((m * Dc * Hc * Wc + bm - 1) / bm);
        }
        for (int k = ncls; k <= 16; ++k) a.cls_tile0[k] = mt;
        a.images = (int)m;
        a.dS = fast_div(s);
        for (int k = 0; k < 2; ++k) { a.dWc[k] = fast_div(a.Wr / s + k); a.dHc[k] = fast_div(a.Hr / s + k); a.dDc[k] = fast_div(a.Dr / s + k); }
    }
    a.dNt = fast_div(nt);
    c.tiles = mt * nt;
}

// Whether the call goes by pieces.  A reduction that blocks or wavefronts would share stays there: its sums are short, and in one walk through all of K they
// end further from the exact ones (560 calls of 3x3 and 5x5 filters, 24 to 480 channels, at most 512 tiles of 32x32: 10 % more results that are not the rounded
// exact ones, for 6 % (wavefronts) to 12 % (blocks) of the time; where one block has all of K the two kernels are equally far off, 0.5 % apart).
static bool in_pieces(const IgemmCall& c) {
    if (c.dtype != LPM_BF16 || c.mode == MODE_DGRAD_S || c.pl.splits > 1 || c.pl.alone != c.pl.tile) return false;
    return rows_take(c.a, !c.any_order);
}

static hipError_t go_call(IgemmCall c, hipStream_t st) {
    IgemmArgs& a = c.a;
    if (in_pieces(c)) return launch_rows(c.mode, a, st);
    if (c.pl.alone != c.pl.tile) {
        c.pl.tile = c.pl.alone;
        c.pl.splits = a.splits = 1;
        c.pl.kt_per = a.kt_per_split = c.pl.kt_total;
        lay_tiles(c);
    }
    const bool bf = c.dtype == LPM_BF16;
    if (c.mode == MODE_FWD) return bf ? go_uni<bf16_t, MODE_FWD, BT_NONE>(c.pl, a, c.tiles, st) : go_uni<float, MODE_FWD, BT_NONE>(c.pl, a, c.tiles, st);
    if (c.mode == MODE_UNPOOL) return go_uni<bf16_t, MODE_UNPOOL, BT_NONE>(c.pl, a, c.tiles, st);
    const bool s1 = c.mode == MODE_DGRAD;
    if (bf) return s1 ? go_uni<bf16_t, MODE_DGRAD, BT_NONE>(c.pl, a, c.tiles, st) : go_uni<bf16_t, MODE_DGRAD_S, BT_NONE>(c.pl, a, c.tiles, st);
    if (a.kscale) return s1 ? go_uni<float, MODE_DGRAD, BT_SCALED>(c.pl, a, c.tiles, st) : go_uni<float, MODE_DGRAD_S, BT_SCALED>(c.pl, a, c.tiles, st);
    return s1 ? go_uni<float, MODE_DGRAD, BT_PLAIN>(c.pl, a, c.tiles, st) : go_uni<float, MODE_DGRAD_S, BT_PLAIN>(c.pl, a, c.tiles, st);
}

template <typename E, int NST, int MODE0, int MODE1, bool UNI, int BT>
static hipError_t go_pair(const IgemmPair& g, int blocks, hipStream_t st) {
    constexpr int stages = NST * 128 * 128 + (UNI ? 0 : MAX_TAB * 16) + (BT == BT_SCALED ? MAX_KSCALE * 4 : 0);
    constexpr int epilogue = 64 * 2 * (32 + 4) * 4, bytes = stages > epilogue ? stages : epilogue;
    static DeviceSet done;
    const hipError_t attr = allow_lds(igemm_pair<E, NST, MODE0, MODE1, UNI, BT>, bytes, done);
    if (attr != hipSuccess) return attr;
    launch_last(igemm_pair<E, NST, MODE0, MODE1, UNI, BT>, dim3((unsigned)blocks), dim3(256), bytes, st, g);
    return hipGetLastError();
}
template <typename E, int MODE0, int MODE1, int BT>
static hipError_t go_pair_uni(const IgemmPair& g, bool uni, int blocks, hipStream_t st) {
    if (blocks <= 320) return uni ? go_pair<E, 4, MODE0, MODE1, true, BT>(g, blocks, st) : go_pair<E, 4, MODE0, MODE1, false, BT>(g, blocks, st);
    return uni ? go_pair<E, 3, MODE0, MODE1, true, BT>(g, blocks, st) : go_pair<E, 3, MODE0, MODE1, false, BT>(g, blocks, st);
}

static bool uni_of(const IgemmCall& c) { return (c.a.Ci * (c.dtype == LPM_BF16 ? 2 : 4)) % 128 == 0; }
// Whether x (held back) and y go in one launch.  What a launch costs beyond its K loop, 4 us, is as much as the whole of a small
// contraction, and where both leave CUs idle they run side by side (us per step, apart / together: float ResNet-18 2746 / 2588, width-48
// ResNet 2408 / 2272, 3-D ResNet 1673 / 1600, ResNet-18/CIFAR 2808 / 2750, 16 images forward 163 / 152).  Larger tiles are for launches
// that fill the card by themselves; a 128x64 plan of a few K tiles -- a projection's data gradient, mostly output -- runs
// on 64x64 here, whatever their number (volumetric at 3 and 4 volumes, 1536 and 2048 tiles: 1944 and 2236 left alone, 1915 and 2200 together; ResNets
// of width 32 to 64 at 13 to 128 samples, up to 4096 tiles, within 0.5 %).
static bool pairs(const IgemmCall& x, const IgemmCall& y) {
    if (x.dtype != y.dtype || uni_of(x) != uni_of(y) || (x.pl.splits > 1 && y.pl.splits > 1)) return false;      // (they share the scratch area)
    auto small = [](const IgemmCall& c) { return c.pl.tile == TILE_64 || (c.pl.tile == TILE_128x64 && c.pl.kt_total <= 4); };
    if (!small(x) || !small(y)) return false;
    if (x.mode == MODE_FWD) return y.mode == MODE_FWD;
    if (x.dtype == LPM_F32 && !(x.a.kscale && y.a.kscale)) return false;
    return x.mode == MODE_DGRAD && (y.mode == MODE_DGRAD || y.mode == MODE_DGRAD_S);
}

static hipError_t run_pair(IgemmCall x, IgemmCall y, hipStream_t st) {
    if (x.mode == MODE_FWD && y.pl.kt_per > x.pl.kt_per) std::swap(x, y);      // the longer blocks first
    IgemmPair g;
    IgemmCall* c[2] = {&x, &y};
    int blocks[2];
    for (int k = 0; k < 2; ++k) {
        if (c[k]->pl.tile != TILE_64) { c[k]->pl.tile = TILE_64; lay_tiles(*c[k]); }
        g.p[k] = c[k]->a;
        g.tiles[k] = c[k]->tiles;
        g.tiles_d[k] = fast_div(c[k]->tiles);
        blocks[k] = c[k]->tiles * c[k]->a.splits;
    }
    g.second = blocks[0];
    const int n = blocks[0] + blocks[1];
    const bool uni = uni_of(x);
    if (x.mode == MODE_FWD) return x.dtype == LPM_BF16 ? go_pair_uni<bf16_t, MODE_FWD, MODE_FWD, BT_NONE>(g, uni, n, st) : go_pair_uni<float, MODE_FWD, MODE_FWD, BT_NONE>(g, uni, n, st);
    if (x.dtype == LPM_BF16) return y.mode == MODE_DGRAD ? go_pair_uni<bf16_t, MODE_DGRAD, MODE_DGRAD, BT_NONE>(g, uni, n, st) : go_pair_uni<bf16_t, MODE_DGRAD, MODE_DGRAD_S, BT_NONE>(g, uni, n, st);
    return y.mode == MODE_DGRAD ? go_pair_uni<float, MODE_DGRAD, MODE_DGRAD, BT_SCALED>(g, uni, n, st) : go_pair_uni<float, MODE_DGRAD, MODE_DGRAD_S, BT_SCALED>(g, uni, n, st);
}

// hold, with: see HeldCall
static hipError_t run_igemm(int dtype, int mode, const IgemmArgs& args, const IgemmPlan& pl, void* ws, bool ws_zeroed, bool any_order, hipStream_t st, HeldCall* hold, HeldCall* with) {
    IgemmCall c{dtype, mode, 0, any_order, args, pl};
    IgemmArgs& a = c.a;
    const int es = dtype == LPM_BF16 ? 2 : 4;
    a.Di = std::max(a.Di, 1); a.Dr = std::max(a.Dr, 1); a.Kd = std::max(a.Kd, 1);
    a.dWr = fast_div(a.Wr); a.dHr = fast_div(a.Hr); a.dDr = fast_div(a.Dr); a.dCc = fast_div(a.Ci * es / 16);
    a.dKt = fast_div(a.Ci * es / 128); a.dKhw = fast_div(a.Kh * a.Kw); a.dKw = fast_div(a.Kw);
    a.kt_total = pl.kt_total; a.kt_per_split = pl.kt_per; a.splits = pl.splits;
    lay_tiles(c);
    if (pl.splits > 1) {
        if (pl.tile != TILE_64) return hipErrorInvalidValue;      // (nor does this happen)
        a.count = (unsigned*)ws;
        a.part = (float*)((char*)ws + LPM_COUNT_BYTES);
        if (c.tiles > (int64_t)(LPM_COUNT_BYTES / 4) || c.tiles > pl.tiles) return hipErrorInvalidValue;      // (the plan's cap keeps this out)
        if (!ws_zeroed && (pl.alone == pl.tile || hold || with)) {
            const hipError_t e = launch_zero_counts(&ws, 1, st);
            if (e != hipSuccess) return e;
        }
    }
    if (with && with->held) {      // (first: hold may be the same place)
        IgemmCall x;
        memcpy(&x, with->bytes, sizeof(x));
        if (pairs(x, c)) {
            with->held = false;
            return run_pair(x, c, st);
        }
        const hipError_t e = run_held(*with, st);
        if (e != hipSuccess) return e;
    }
    if (hold) {
        if (hold->held) return hipErrorInvalidValue;      // (what waits there would be lost)
        memcpy(hold->bytes, &c, sizeof(c));
        hold->held = true;
        return hipSuccess;
    }
    return go_call(c, st);
}

hipError_t run_held(HeldCall& h, hipStream_t st) {
    if (!h.held) return hipSuccess;
    h.held = false;
    IgemmCall x;
    memcpy(&x, h.bytes, sizeof(x));
    const hipEvent_t end = take_stop_event();      // (not this kernel's: the one that follows it)
    const hipError_t e = go_call(x, st);
    give_stop_event(end);
    return e;
}

hipError_t mfma_conv_fwd(int dtype, const ConvGeom& g, const void* x, const void* w, const float* scale, const float* bias,
                         const void* add, int relu, void* y, void* ws, bool ws_zeroed, hipStream_t st, void* pool_y,
                         HeldCall* hold, HeldCall* with) {
    if (pool_y && (add || !mfma_fwd_pools(dtype, g))) return hipErrorInvalidValue;
    const int es = dtype == LPM_BF16 ? 2 : 4;
    IgemmArgs a{};
    a.fwd_pool = (uint16_t*)pool_y;
    a.A = x; a.B = w; a.C = y;
    a.scale = scale; a.bias = bias; a.add = add; a.relu = relu;
    a.M = (int)g.rows_out(); a.N = g.Cout;
    a.Hi = g.H; a.Wi = g.W; a.Di = g.D; a.Ci = g.Cin; a.Hr = g.Ho; a.Wr = g.Wo; a.Dr = g.Do;
    a.Kh = g.Kh; a.Kw = g.Kw; a.Kd = g.Kd; a.stride = g.stride; a.pad = g.pad; a.pad_d = g.pad_d;
    a.free_taps = fwd_free(g);
    a.a_bytes = (unsigned)(g.rows_in() * g.Cin * es);
    a.b_pitch = (unsigned)((int64_t)g.K() * es);
    a.b_bytes = (unsigned)((int64_t)g.Cout * g.K() * es);
    return run_igemm(dtype, MODE_FWD, a, plan_fwd(dtype, g), ws, ws_zeroed, g.any_order, st, hold, with);
}

// wt: weights laid out [Cin][taps][Cout] (bf16); float layers pass w itself, [Cout][taps][Cin]
// kscale: float layers, the per-channel scale that dz does not carry, or NULL
// side (may be NULL): the gradient is the last contribution to a tensor whose producer's epilogue backward this kernel
// performs -- see DgradSide
hipError_t mfma_conv_dgrad(int dtype, const ConvGeom& g, const void* dz, const void* wt, void* dx, int accumulate, const void* mask,
                           const float* mscale, void* ws, bool ws_zeroed, hipStream_t st, const UnpoolDesc* unpool, const DgradSide* side, const float* kscale,
                           HeldCall* hold, HeldCall* with) {
    if (kscale && (dtype == LPM_BF16 || g.Cout > MAX_KSCALE)) return hipErrorInvalidValue;      // (bf16: the transposed copy carries the scale)
    if (unpool && (side || dtype != LPM_BF16 || g.stride != 1 || g.Cin % 8)) return hipErrorInvalidValue;      // (the epilogue routes whole chunks of eight channels)
    const int es = dtype == LPM_BF16 ? 2 : 4;
    IgemmArgs a{};
    a.A = dz; a.B = wt; a.C = dx;
    a.mask = mask; a.mscale = mscale; a.kscale = kscale;
    if (accumulate) {                    // dx += : its old values are the addend
        if (side) return hipErrorInvalidValue;
        a.add = dx;
    }
    if (side) { a.add = side->earlier; a.C2 = side->shortcut; a.acc2 = side->shortcut_acc; a.c2scale = side->shortcut_scale; }
    if (unpool) {
        a.C = nullptr; a.add = nullptr; a.mask = nullptr;
        a.pool_x = (const uint16_t*)unpool->pool_x; a.pool_dst = (uint16_t*)unpool->dst;
        a.pool_acc = unpool->accumulate; a.pool_mask = unpool->mask; a.mscale = unpool->mscale;
    }
    a.M = (int)g.rows_in(); a.N = g.Cin;
    a.Hi = g.Ho; a.Wi = g.Wo; a.Di = g.Do; a.Ci = g.Cout; a.Hr = g.H; a.Wr = g.W; a.Dr = g.D;
    a.Kh = g.Kh; a.Kw = g.Kw; a.Kd = g.Kd; a.stride = g.stride; a.pad = g.pad; a.pad_d = g.pad_d;
    a.a_bytes = (unsigned)(g.rows_out() * g.Cout * es);
    a.b_pitch = (unsigned)((int64_t)g.taps() * (dtype == LPM_BF16 ? g.Cout : g.Cin) * es);
    a.b_bytes = (unsigned)((int64_t)g.Cout * g.K() * es);
    return run_igemm(dtype, unpool ? MODE_UNPOOL : g.stride > 1 ? MODE_DGRAD_S : MODE_DGRAD, a, plan_dgrad(dtype, g), ws, ws_zeroed, g.any_order, st, hold, with);
}

// clears the arrival counts at the head of up to 16 scratch areas
struct ZeroArgs { unsigned* head[16]; };
__global__ void __launch_bounds__(256) zero_counts(ZeroArgs a) {
    reinterpret_cast<uint4*>(a.head[blockIdx.x])[threadIdx.x] = make_uint4(0, 0, 0, 0);
}
hipError_t launch_zero_counts(void* const* heads, int n, hipStream_t st) {
    static_assert(LPM_COUNT_BYTES == 256 * 16, "one 16-byte store per thread");
    for (int d = 0; d < n; d += 16) {
        ZeroArgs a{};
        const int k = std::min(16, n - d);
        for (int i = 0; i < k; ++i) a.head[i] = (unsigned*)heads[d + i];
        hipLaunchKernelGGL(zero_counts, dim3(k), dim3(256), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lpm
