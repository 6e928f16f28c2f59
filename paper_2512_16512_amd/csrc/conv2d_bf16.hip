// bf16 conv2d on the gfx950 matrix cores: X (NCHW) and W (OIHW) hold bf16
// bit patterns, products are exact in fp32, accumulation and Y (NCHW) are
// fp32.  The same zero-padded cross-correlation as the fp32 kernels, computed
// as an implicit GEMM with M = OC, N = batch*OH*OW, K = C*R*S in OIHW order
// (k = (ic*R + kh)*S + kw).
//
// Register-staged, double-buffered LDS tiles, as the fp32 channel-major conv
// kernel: each thread owns one output pixel of the B tile for the whole K
// loop and gathers its input values through a per-workgroup LDS table of
// k -> (input offset, kh, kw), so the gather needs no integer division; an
// input position in the padding is a zero.  The weights are the row-major
// A[OC][K] operand (16-byte loads when K is a multiple of 8 and the base is
// 16-byte aligned).  The fragments are those of the bf16 GEMM: one
// ds_read_b128 per A fragment from k-contiguous padded rows, and two gfx950
// transpose reads per B fragment from the pixel-contiguous B tile.
#include <algorithm>
#include <type_traits>

#include "fast_div.h"
#include "lds_dma.h"
#include "mfma_bf16.h"
#include "patch_geom.h"
#include "tile_map.h"
#include "xtc_internal.h"

namespace xtc {
namespace {

template <int BM, int BN, int BK, int WM, int WN, int MI, int PAD, bool VEC>
struct ConvBf16Cfg {
    static constexpr int NWM = BM / WM, NWN = BN / WN;
    static constexpr int NT = NWM * NWN * 64;
    static constexpr int TM = WM / MI, TN = WN / MI;
    typedef Bf16Mfma<MI> MF;
    static constexpr int KG = MF::KG;
    static constexpr int KCH = 8 * KG;              // k per MFMA instruction
    static constexpr int AS = BK + PAD;             // LDS row stride of the weight tile
    static constexpr int BS = BN + 32;              // LDS row stride of the pixel tile
    static constexpr int WA = VEC ? 8 : 1;          // weight elements per global load
    static constexpr int A_CPR = BK / WA;
    static constexpr int A_LOADS = BM * BK / (WA * NT);
    static constexpr int B_ROWS_PER_PASS = NT / BN; // gather: a thread owns one pixel column
    static constexpr int B_LOADS = BK / B_ROWS_PER_PASS;
    typedef typename VecU16<WA>::t vec_t;
    static_assert(BM % WM == 0 && BN % WN == 0, "wave tile must divide the block tile");
    static_assert(WM % MI == 0 && WN % MI == 0, "MFMA tile must divide the wave tile");
    static_assert(NT % BN == 0 && BK % B_ROWS_PER_PASS == 0, "gather split");
    static_assert(A_LOADS * WA * NT == BM * BK, "weight tile must split evenly");
    static_assert(BK % KCH == 0, "block_k must be a multiple of the MFMA k");
    static_assert(PAD % 8 == 0, "padding must keep 16-byte alignment");
};

template <int BM, int BN, int BK, int WM, int WN, int MI, int PAD, bool VEC>
__global__ void __launch_bounds__((BM / WM) * (BN / WN) * 64)
conv2d_bf16_kernel(ConvArgs p) {
    typedef ConvBf16Cfg<BM, BN, BK, WM, WN, MI, PAD, VEC> G;
    typedef typename G::MF MF;
    typedef typename G::vec_t vec_t;
    constexpr int WA = G::WA;

    __shared__ __attribute__((aligned(16))) unsigned short As[2][BM * G::AS];
    __shared__ __attribute__((aligned(16))) unsigned short Bs[2][BK * G::BS];
    extern __shared__ int2 ktab[];  // [K]: {ic*H*W + kh*W + kw, kh | kw << 16}

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / G::NWN, wn = wave % G::NWN;
    const int lrow = lane % MI, lgrp = lane / MI;

    const int C = p.C, H = p.H, Wd = p.W, R = p.R, S = p.S;
    const int OC = p.OC, OHW = p.OH * p.OW;
    const int M = OC, N = p.Nb * OHW, K = C * R * S;
    const int HW = H * Wd;

    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, tiles_m, tiles_n, p.raster, p.xcd_remap, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    const int RS = R * S;
    for (int k = tid; k < K; k += G::NT) {
        const int ic = k / RS, rem = k - ic * RS;
        const int kh = rem / S, kw = rem - kh * S;
        ktab[k] = make_int2(ic * HW + kh * Wd + kw, kh | (kw << 16));
    }

    const int bcol = tid % BN, brow0 = tid / BN;
    const int q = n0 + bcol;
    const bool qok = q < N;
    int xbase = 0, ih0 = 0, iw0 = 0;
    if (qok) {
        const int img = q / OHW, pix = q - img * OHW;
        const int oh = pix / p.OW, ow = pix - oh * p.OW;
        ih0 = oh * p.sh - p.ph;
        iw0 = ow * p.sw - p.pw;
        xbase = img * C * HW + ih0 * Wd + iw0;
    }

    const unsigned short *__restrict__ Wt = reinterpret_cast<const unsigned short *>(p.Wt);
    const unsigned short *__restrict__ X = reinterpret_cast<const unsigned short *>(p.X);

    vec_t ra[G::A_LOADS];
    unsigned short rb[G::B_LOADS];

    auto load_tiles = [&](int kt) {
        const int k0 = kt * BK;
#pragma unroll
        for (int i = 0; i < G::A_LOADS; ++i) {
            const int idx = tid + i * G::NT;
            const int r = idx / G::A_CPR, c = (idx % G::A_CPR) * WA;
            const int gm = m0 + r, gk = k0 + c;
            const int valid = gm < M ? K - gk : 0;
            ra[i] = load_pred_u16<WA>(Wt + (gm < M ? gm : 0) * K + (valid > 0 ? gk : 0), valid);
        }
#pragma unroll
        for (int i = 0; i < G::B_LOADS; ++i) {
            const int k = k0 + brow0 + i * G::B_ROWS_PER_PASS;
            unsigned short v = 0;
            if (qok && k < K) {
                const int2 t = ktab[k];
                const int ih = ih0 + (t.y & 0xffff), iw = iw0 + (t.y >> 16);
                if ((unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)Wd) v = X[xbase + t.x];
            }
            rb[i] = v;
        }
    };

    auto store_tiles = [&](int st) {
#pragma unroll
        for (int i = 0; i < G::A_LOADS; ++i) {
            const int idx = tid + i * G::NT;
            const int r = idx / G::A_CPR, c = (idx % G::A_CPR) * WA;
            *reinterpret_cast<vec_t *>(&As[st][r * G::AS + c]) = ra[i];
        }
#pragma unroll
        for (int i = 0; i < G::B_LOADS; ++i)
            Bs[st][(brow0 + i * G::B_ROWS_PER_PASS) * G::BS + bcol] = rb[i];
    };

    typename MF::acc_t acc[G::TM][G::TN];
#pragma unroll
    for (int i = 0; i < G::TM; ++i)
#pragma unroll
        for (int j = 0; j < G::TN; ++j)
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) acc[i][j][r] = 0.f;

    __syncthreads();  // k-offset table ready
    const int KT = (K + BK - 1) / BK;
    load_tiles(0);
    store_tiles(0);
    __syncthreads();
    for (int kt = 0; kt < KT; ++kt) {
        const int cur = kt & 1;
        const bool has_next = kt + 1 < KT;
        if (has_next) load_tiles(kt + 1);

        const unsigned short *as = &As[cur][(wm * WM + lrow) * G::AS + 8 * lgrp];
        // transpose-read base: row 8*(k-group) + (lane%16)/4, column
        // (lane%MI rounded down to 16) + 4*(lane%4)
        const unsigned short *bs =
            &Bs[cur][(8 * lgrp + ((lane & 15) >> 2)) * G::BS + wn * WN + (lrow & ~15) + 4 * (lane & 3)];
#pragma unroll
        for (int kk = 0; kk < BK; kk += G::KCH) {
            u16x8 a[G::TM], b[G::TN];
#pragma unroll
            for (int i = 0; i < G::TM; ++i)
                a[i] = *reinterpret_cast<const u16x8 *>(as + i * MI * G::AS + kk);
#pragma unroll
            for (int j = 0; j < G::TN; ++j) {
                const u16x4 lo = ds_read_tr16(bs + kk * G::BS + j * MI);
                const u16x4 hi = ds_read_tr16(bs + (kk + 4) * G::BS + j * MI);
                b[j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
#pragma unroll
            for (int i = 0; i < G::TM; ++i)
#pragma unroll
                for (int j = 0; j < G::TN; ++j) acc[i][j] = MF::mma(a[i], b[j], acc[i][j]);
        }

        if (has_next) store_tiles(cur ^ 1);
        __syncthreads();
    }

    float *__restrict__ Y = p.Y;
#pragma unroll
    for (int j = 0; j < G::TN; ++j) {
        const int col = n0 + wn * WN + j * MI + lrow;
        if (col >= N) continue;
        const int img = col / OHW, pix = col - img * OHW;
        float *ybase = Y + img * OC * OHW + pix;
#pragma unroll
        for (int i = 0; i < G::TM; ++i)
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) {
                const int oc = m0 + wm * WM + i * MI + MF::row(lane, r);
                if (oc < M) ybase[oc * OHW] = (p.relu && acc[i][j][r] < 0.f) ? 0.f : acc[i][j][r];
            }
    }
}

template <int BM, int BN, int BK, int WM, int WN, int MI, int PAD>
hipError_t launch_conv_bf16(const ConvArgs &a, hipStream_t s) {
    const int M = a.OC, N = a.Nb * a.OH * a.OW, K = a.C * a.R * a.S;
    const unsigned tiles = (unsigned)(((M + BM - 1) / BM) * ((N + BN - 1) / BN));
    const size_t dyn = (size_t)K * sizeof(int2);
    ConvArgs args = a;
    void *kargs[] = {&args};
    const bool vec = (K % 8 == 0) && ((reinterpret_cast<uintptr_t>(a.Wt) & 15) == 0);
    const void *fn =
        vec ? reinterpret_cast<const void *>(&conv2d_bf16_kernel<BM, BN, BK, WM, WN, MI, PAD, true>)
            : reinterpret_cast<const void *>(&conv2d_bf16_kernel<BM, BN, BK, WM, WN, MI, PAD, false>);
    return hipLaunchKernel(fn, dim3(tiles), dim3((BM / WM) * (BN / WN) * 64), kargs, dyn, s);
}

// ---------------------------------------------------------------------------
// Halo-tiled bf16 kernel (k_order = 2) for stride-1 3x3 convolutions of rows
// of about 56 pixels.  The gather above loads every input value once per
// tap; here a stage stages a 16-channel input patch once for all nine taps:
//  - a workgroup computes 64 output channels x 256 consecutive output pixels
//    of one image (four 64x64 waves of 32x32x16 instructions).  The pixels
//    span at most 6 output rows when OW >= 51, so their inputs fit in a patch
//    of PR = 8 input rows;
//  - the patch is stored channel-innermost, [half][row][column][8 channels],
//    16 bytes per cell: the B fragment of a lane (8 channels of one pixel at
//    one tap) is then one 16-byte read of the cell the tap points at, for
//    any column shift.  Input column iw sits at patch column iw + CO;
//    columns and rows outside the image hold zeros;
//  - bank layout: gfx950 serves a ds_read_b128 in four phases of 16 lanes
//    ({0-3, 12-15, 20-23, 24-27}, {4-11, 16-19, 28-31} and the same + 32),
//    and a 16-byte cell occupies one of 16 bank groups.  Patch row r (64
//    columns) is stored rotated by (r * OW) mod 16 cells inside a row of 80
//    cells, so the 32 pixels of a fragment stay on consecutive bank groups
//    also when they wrap to the next output row (unrotated, the wrap moved
//    them by OW - 64 groups onto other lanes' banks).  Output channel rows
//    of the weights hold their two 8-channel halves swapped when bit 3 of
//    the channel is set, which puts the rows a phase reads on distinct
//    groups.  Stores are served 8 lanes at a time over 32 banks (128
//    bytes), so a thread writes its two patch cells in an order that keeps
//    each group of 8 lanes on 8 distinct 16-byte slots;
//  - the patch is filled through registers: a thread loads one dword (two
//    neighbouring input columns) of each of the 16 channels and repacks them
//    into the two columns' cells.  NCHW rows of even width keep every pair
//    dword-aligned;
//  - the weights of a stage, W[oc][c0 .. c0+15][kh][kw], are 144 contiguous
//    values per output channel (16-byte aligned when C % 16 == 0); a thread
//    loads one 8-channel slab (72 values) and repacks it into the
//    [tap][oc][16 channels] cells of the A fragments;
//  - the reduction runs over 16-channel chunks and, inside a chunk, over the
//    taps; an instruction's two k lane groups take channels 0-7 and 8-15 of
//    the tap.
namespace halo_bf16 {
constexpr int BM = 64, BN = 256, WM = 64, WN = 64, NWAVES = 4, NT = 256;
constexpr int MI = 32, TM = WM / MI, TN = WN / MI;
constexpr int CC = 16;                        // channels per stage
constexpr int NTAP = 9;
constexpr int PR = 8;                         // patch rows
constexpr int PC = 64;                        // patch columns
constexpr int PCA = 80;                       // cells per stored patch row (PC + the rotation)
constexpr int CO = 2;                         // patch column of input column 0 (even)
constexpr int CELL = 16;                      // bytes: 8 channels of one (row, column)
constexpr int HALF = PR * PCA * CELL;         // one 8-channel half of the patch
constexpr int P_BYTES = 2 * HALF;
constexpr int W_BYTES = NTAP * BM * CC * 2;   // [tap][oc][16 channels]
constexpr int STAGE_BYTES = P_BYTES + W_BYTES;
static_assert(NT == PR * PC / 2, "one patch column pair per thread");
static_assert(2 * BM <= NT, "one weight slab per thread");
}  // namespace halo_bf16

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(halo_bf16::NT) __attribute__((amdgpu_waves_per_eu(2, 2)))
conv2d_bf16_halo_kernel(ConvArgs p) {
    using namespace halo_bf16;
    typedef Bf16Mfma<MI> MF;
    __shared__ __attribute__((aligned(16))) unsigned char smem[2 * STAGE_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int lrow = lane % MI, lgrp = lane / MI;   // lgrp: channel half of the fragments

    const int C = p.C, H = p.H, Wd = p.W;
    const int OC = p.OC, OW = p.OW, OHW = p.OH * p.OW;
    const int chunks = (OHW + BN - 1) / BN;   // per image
    const int tiles_m = (OC + BM - 1) / BM, tiles_n = p.Nb * chunks;
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, tiles_m, tiles_n, p.raster, p.xcd_remap, tm, tn);
    const int m0 = tm * BM;
    const int img = tn / chunks, p0 = (tn - img * chunks) * BN;
    const int oh0 = p0 / OW;                  // first output row of the tile
    const int ih0 = oh0 - p.ph;               // input row of patch row 0
    const int KT = C / CC;

    // Patch loads: patch row pr, column pair cp (input columns 2cp - CO, +1),
    // through a buffer resource: one offset per thread, the channel step in a
    // scalar offset, and pairs outside the image at an out-of-range offset,
    // which reads zeros.
    const int pr = tid >> 5, cp = tid & 31;
    const int prot = (pr * OW) & 15;            // rotation of this patch row
    const bool sw = (cp >> 2) & 1;              // store order of the two cells
    const int cell0 = (pr * PCA + 2 * cp + prot + (sw ? 1 : 0)) * CELL;
    const int cell1 = (pr * PCA + 2 * cp + prot + (sw ? 0 : 1)) * CELL;
    const int ih = ih0 + pr, iw = 2 * cp - CO;
    const bool pok = ih >= 0 && ih < H && iw >= 0 && iw + 1 < Wd;
    // dwords per channel plane; read into a scalar register, since the
    // compiler otherwise recomputes it on both sides of the divergent select
    // below and then holds it per lane, which turns every buffer load that
    // takes it as a scalar offset into a loop over lanes
    const int HW2 = __builtin_amdgcn_readfirstlane(H * Wd / 2);
    const int xoff = pok ? (img * C * HW2 + (ih * Wd + iw) / 2) * 4 : kOOB;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned short *>(reinterpret_cast<const unsigned short *>(p.X)), 0,
        p.Nb * C * HW2 * 4, 0x00020000);
    // Weight loads (threads 0 .. 2*BM-1): output channel m0 + woc, channels
    // 8*wh .. 8*wh+7 of the stage, all nine taps: nine 16-byte chunks.
    const int woc = tid >> 1, wh = tid & 1;
    // byte offset of this thread's 8-channel half in an output channel row
    // (halves swapped when bit 3 of the channel is set)
    const int wslot = (woc * CC + 8 * (wh ^ ((woc >> 3) & 1))) * 2;
    const bool wthr = tid < 2 * BM;
    const bool wok = wthr && m0 + woc < OC;
    const int woff = wok ? ((m0 + woc) * C + 8 * wh) * NTAP * 2 : kOOB;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned short *>(reinterpret_cast<const unsigned short *>(p.Wt)), 0,
        OC * C * NTAP * 2, 0x00020000);

    // two register sets, so that the loads of a stage are in flight for two
    // stages' worth of matrix work before they are stored
    unsigned xs[2][CC];
    u32x4_t ws[2][NTAP];
    // Loads of stage kt into set S.  Past the last stage (live false) the
    // offsets are out of range: the loads return zeros without touching
    // memory.  Loads under a branch would make the compiler's wait before
    // each store count conservatively, and wait for loads it does not need.
    auto gload = [&](auto S, int kt, bool live) __attribute__((always_inline)) {
        const int c0 = live ? kt * CC : 0;
        const int xo = live ? xoff : kOOB, wo = live ? woff : kOOB;
#pragma unroll
        for (int c = 0; c < CC; ++c)
            xs[S][c] = __builtin_amdgcn_raw_buffer_load_b32(rx, xo, (c0 + c) * HW2 * 4, 0);
        // every thread issues the weight loads (threads without a slab at an
        // out-of-range offset), so that all waves count the same loads
#pragma unroll
        for (int q = 0; q < NTAP; ++q)
            ws[S][q] = __builtin_amdgcn_raw_buffer_load_b128(rw, wo, c0 * NTAP * 2 + q * 16, 0);
    };
    // halfword e (0 .. 71) of the weight slab in set S
    auto wv = [&](auto S, int e) __attribute__((always_inline)) {
        return (ws[S][e >> 3][(e >> 1) & 3] >> (16 * (e & 1))) & 0xffffu;
    };
    auto lstore = [&](auto S) __attribute__((always_inline)) {
        unsigned char *P = smem + S * STAGE_BYTES;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4_t lo, hi;   // columns 2cp and 2cp + 1
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned a = xs[S][8 * h + 2 * j], b = xs[S][8 * h + 2 * j + 1];
                lo[j] = (a & 0xffffu) | (b << 16);
                hi[j] = (a >> 16) | (b & 0xffff0000u);
            }
            // writes are served 8 lanes at a time over 128 bytes of banks:
            // threads whose column pair has bit 2 set write their odd cell
            // first, so each group of 8 lanes covers 8 distinct 16-byte slots
            const u32x4_t c0 = sw ? hi : lo, c1 = sw ? lo : hi;
            *reinterpret_cast<u32x4_t *>(P + h * HALF + cell0) = c0;
            *reinterpret_cast<u32x4_t *>(P + h * HALF + cell1) = c1;
        }
        if (wthr) {
            unsigned char *Wl = P + P_BYTES;
#pragma unroll
            for (int t = 0; t < NTAP; ++t) {
                u32x4_t v;
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    v[d] = wv(S, 2 * d * NTAP + t) | (wv(S, (2 * d + 1) * NTAP + t) << 16);
                *reinterpret_cast<u32x4_t *>(Wl + t * BM * CC * 2 + wslot) = v;
            }
        }
    };

    // Fragment bases.  A: output channel i*32 + lrow, channels 8*lgrp .. +7
    // (halves swapped when bit 3 of the channel is set).  B: this lane's
    // pixel of column block j, one base per kernel row kh (the rotation
    // depends on the patch row); patch position (0, 0) past the image.
    const int a_base = P_BYTES + (lrow * CC + 8 * (lgrp ^ ((lrow >> 3) & 1))) * 2;
    int b_base[TN][3];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int pix = p0 + wave * WN + j * MI + lrow;
        int r = 0, c = 0;
        if (pix < OHW) {
            const int oh = pix / OW, ow = pix - oh * OW;
            r = oh - oh0;
            c = ow - p.pw + CO;
        }
#pragma unroll
        for (int kh = 0; kh < 3; ++kh)
            b_base[j][kh] = lgrp * HALF + ((r + kh) * PCA + c + (((r + kh) * OW) & 15)) * CELL;
    }

    typename MF::acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) acc[i][j][r] = 0.f;

    u16x8 af[2][TM], bfr[2][TN];
    auto load_frags = [&](int buf, int t, int fb) __attribute__((always_inline)) {
        const unsigned char *P = smem + buf * STAGE_BYTES;
        const int kh = t / 3, kw = t - 3 * kh;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            af[fb][i] = *reinterpret_cast<const u16x8 *>(P + a_base + ((t * BM + i * MI) * CC) * 2);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            bfr[fb][j] = *reinterpret_cast<const u16x8 *>(P + b_base[j][kh] + kw * CELL);
    };
    auto mfmas = [&](int fb) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = MF::mma(af[fb][i], bfr[fb][j], acc[i][j]);
    };

    // Stage kt is computed from LDS buffer kt % 2, which register set kt % 2
    // filled; that set then takes the loads of stage kt + 2, and set
    // (kt + 1) % 2, loaded a stage earlier, is stored into the other buffer
    // after the nine taps.
    const std::integral_constant<int, 0> S0;
    const std::integral_constant<int, 1> S1;
    auto stage = [&](auto S, int kt) __attribute__((always_inline)) {
        constexpr int NS = 1 - decltype(S)::value;
        gload(S, kt + 2, kt + 2 < KT);
        // keep the loads ahead of the taps (the scheduler would otherwise sink
        // them to the end of the stage, one stage before their use)
        __builtin_amdgcn_sched_barrier(0);
        load_frags(S, 0, 0);
#pragma unroll
        for (int t = 0; t < NTAP; ++t) {
            if (t + 1 < NTAP) load_frags(S, t + 1, (t + 1) & 1);
            mfmas(t & 1);
        }
        if (kt + 1 < KT) lstore(std::integral_constant<int, NS>());
        __syncthreads();
    };
    gload(S0, 0, true);
    gload(S1, 1, KT > 1);
    lstore(S0);
    __syncthreads();
    for (int kt = 0; kt < KT; kt += 2) {
        stage(S0, kt);
        if (kt + 1 < KT) stage(S1, kt + 1);
    }

    float *__restrict__ Y = p.Y + (size_t)img * OC * OHW;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int pix = p0 + wave * WN + j * MI + lrow;
        if (pix >= OHW) continue;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) {
                const int oc = m0 + i * MI + MF::row(lane, r);
                if (oc < OC)
                    __builtin_nontemporal_store((p.relu && acc[i][j][r] < 0.f) ? 0.f : acc[i][j][r],
                                                &Y[oc * OHW + pix]);
            }
    }
}

// ---------------------------------------------------------------------------
// Patch kernel (k_order = 2 outside the halo kernel's class) for 3x3
// convolutions of any stride, padding, row length, alignment and batch, with
// a channel count that is a multiple of 8.  The gather kernel above loads
// every input value once per tap, two bytes at a time, and its reduction is
// one serial chain of small steps: 32x128x28x28 -> 128 took 92.7 us (80
// TFLOP/s) and one image of it 90.7 us, both bound by that chain; this kernel
// takes 17.8 us (416 TFLOP/s; 19.0 by a kernel trace) and 9.0 us.  By counters
// a wave lives 38000 clocks there, of which the matrix cores are busy 24% and
// LDS 29% (a quarter of that conflicts); over half are waits for copies and at
// the two barriers of a chunk, with one wave per SIMD to run.  Here, as in
// the halo kernel, a stage of 16 channels stages its input patch once for
// all nine taps, without that kernel's restrictions:
//  - a workgroup computes BM output channels x BN consecutive pixels of the
//    flattened (image, output row, output column) order.  Padded input rows
//    are numbered through the batch (PH per image), so that a tile that
//    crosses into the next image still reads one contiguous run of them, and
//    small images share tiles;
//  - the input rows a tile reads are one contiguous run of bytes per image
//    and channel.  They are copied as they are, in aligned 16-byte units
//    (which never cross a page), straight into a raw LDS area, and so are the
//    288 bytes that a chunk has per output channel in the OIHW weights: about
//    nine copy instructions per wave and chunk, no registers, RD chunks ahead
//    of the matrix cores.  Loads to registers of the cells' own pieces (one
//    dword per channel and column pair, 16 bytes per weight slab at 144-byte
//    strides) took 24.2 us where this took 19.0;
//  - between two barriers the waves then turn the raw chunk into cells: 16
//    bytes hold 8 channels of one padded row and column ([8-channel
//    half][row][column], WPA columns per row), or 8 channels of one (tap,
//    output channel).  A pixel's fragment at tap (kh, kw) is the cell kh*WPA +
//    kw past its own.  Cells in the padding hold zeros from the start of the
//    kernel and are never written;
//  - KS groups of waves share one tile, group g reducing the chunks g, g +
//    KS, ... in its own LDS areas; their sums are added in group order at the
//    end.  With few tiles (a small batch or a small image) this divides the
//    serial chain of chunks by KS.
namespace patch_bf16 {
constexpr int MI = 32, CC = 16, NTAP = 9;
constexpr int W_ROW = CC * NTAP * 2;              // raw weight bytes per output channel and chunk
template <int BM_, int BN_, int WM_, int WN_, int KS_, int RD_>
struct Cfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KS = KS_, RD = RD_;
    static constexpr int NWN = BN / WN, NWAVES = (BM / WM) * NWN;   // waves per group
    static constexpr int NTG = NWAVES * 64, NT = NTG * KS;          // threads per group, in all
    static constexpr int TM = WM / MI, TN = WN / MI;
    static constexpr int NSLAB = (2 * BM + NTG - 1) / NTG;          // weight slabs per thread
    static constexpr int NBW = (BM * W_ROW / 1024 + NWAVES - 1) / NWAVES;   // weight copies per wave
    static constexpr int WRAW = NBW * NWAVES * 1024;
    static constexpr int W_BYTES = NTAP * BM * CC * 2;              // [tap][oc][16 channels]
    static constexpr int SU0 = BN >= 128 ? 64 : 32;                 // smaller of the two slot sizes compiled
    static constexpr int RED_BYTES = (KS - 1) * NWAVES * TM * TN * 4096;    // partial sums
};
constexpr int kMaxLds = 160 * 1024;
}  // namespace patch_bf16

// Launch geometry of the patch kernel (computed on the host).
struct PatchArgs {
    ConvArgs c;
    FastDiv by_ohw, by_ow, by_ppr;
    int PH;      // padded input rows an image's outputs read: (OH-1)*stride_h + R
    int WPA;     // cells per stored patch row
    int PPR;     // items per row: column pairs (PAIR) or columns
    int half;    // bytes of one 8-channel half of the patch
};

// SU: 16-byte units a channel's raw slot holds; NI: patch items (a column
// pair, PAIR, or a column, of one half) per thread.
template <typename CFG, int SU, int NI, bool PAIR>
__global__ void __launch_bounds__(CFG::NT)
conv2d_bf16_patch_kernel(PatchArgs pa) {
    using namespace patch_bf16;
    typedef Bf16Mfma<MI> MF;
    constexpr int BM = CFG::BM, BN = CFG::BN, WM = CFG::WM, WN = CFG::WN, KS = CFG::KS, RD = CFG::RD;
    constexpr int TM = CFG::TM, TN = CFG::TN, NTG = CFG::NTG, NSLAB = CFG::NSLAB, NBW = CFG::NBW;
    constexpr int NBX = CC * SU / CFG::NTG;                     // input copies per wave and chunk
    static_assert(NBX * CFG::NTG == CC * SU, "a chunk's units split evenly");
    constexpr int RAW = CFG::WRAW + NBX * CFG::NWAVES * 1024;   // raw bytes per chunk: weights, input
    static_assert((RD - 1) * (NBW + NBX) < 64, "vmcnt range");
    extern __shared__ __attribute__((aligned(1024))) unsigned char psm[];

    const ConvArgs &p = pa.c;
    const int tid = threadIdx.x;
    const int kg = __builtin_amdgcn_readfirstlane(tid / NTG);   // K group of this wave
    const int t = tid % NTG;                                    // thread inside its group
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / CFG::NWN, wn = wave % CFG::NWN;
    const int l32 = lane & 31, lgrp = lane >> 5;

    const int C = p.C, H = p.H, Wd = p.W, OC = p.OC, OH = p.OH, OW = p.OW, OHW = OH * OW;
    const int N = p.Nb * OHW;
    const int PH = pa.PH, WPA = pa.WPA, PPR = pa.PPR, HALF = pa.half;
    const int tiles_m = (OC + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, tiles_m, tiles_n, p.raster, p.xcd_remap, tm, tn);
    const int m0 = tm * BM, q0 = tn * BN;

    // the tile's pixels run from (img0, oh0) to (img1, oh1)
    const int img0 = div_by(q0, pa.by_ohw), oh0 = div_by(q0 - img0 * OHW, pa.by_ow);
    const int q1 = min(q0 + BN, N) - 1;
    const int img1 = div_by(q1, pa.by_ohw), oh1 = div_by(q1 - img1 * OHW, pa.by_ow);
    const int prow0 = oh0 * p.sh;                                  // first padded row, counted from img0
    // input rows the tile reads of image i: first and count (0: none)
    auto seg_first = [&](int i) { return max((i == img0 ? oh0 * p.sh : 0) - p.ph, 0); };
    auto seg_rows = [&](int i) {
        return max(min((i == img1 ? oh1 : OH - 1) * p.sh + 2 - p.ph, H - 1) - seg_first(i) + 1, 0);
    };
    const int area_bytes = RD * RAW + CFG::W_BYTES + 2 * HALF;
    unsigned char *const raw = psm + kg * area_bytes;              // [RD][weights | input]
    unsigned char *const cells = raw + RD * RAW;                   // weights | patch halves

    // zeros into every patch cell (the padding keeps them)
    const u32x4_t zero4 = {0u, 0u, 0u, 0u};
    for (int o = t * 16; o < 2 * HALF; o += NTG * 16)
        *reinterpret_cast<u32x4_t *>(cells + CFG::W_BYTES + o) = zero4;

    // Two tables, built once by the first threads of each group in its raw
    // area.  Per unit u of a channel's slot: {byte offset of its segment's
    // first input row in channel 0, its unit_entry}.  Per input row r: {that byte offset, position of the row in
    // the slot (before the segment's misalignment), its patch cell, -}.
    const int plane = __builtin_amdgcn_readfirstlane(H * Wd * 2);   // bytes per channel plane
    const int xmis = (int)(reinterpret_cast<unsigned long long>(p.X) & 15);
    int2 *const utab = reinterpret_cast<int2 *>(raw);               // [SU]
    int4 *const rtab = reinterpret_cast<int4 *>(raw + SU * 8);      // rows
    int nrows = 0;
    {
        int ub = 0;
        for (int i = img0; i <= img1; ++i) {
            const int n = seg_rows(i), f = seg_first(i), nu = slot_units(n * Wd * 2);
            const int start = xmis + (i * C * H + f) * Wd * 2;
            for (int u = t; u < nu; u += NTG) utab[ub + u] = make_int2(start, unit_entry(u, n * Wd * 2));
            for (int r = t; r < n; r += NTG)
                rtab[nrows + r] = make_int4(start, ub * 16 + r * Wd * 2,
                                            ((i - img0) * PH + f + r + p.ph - prow0) * WPA + p.pw, 0);
            nrows += n;
            ub += nu;
        }
        for (int u = ub + t; u < SU; u += NTG) utab[u] = make_int2(0, -1);
    }
    __syncthreads();

    // Raw copies.  Weights: unit (output channel, u < 18); input: unit
    // (channel < 16, u < SU).  Offsets are for chunk 0; a chunk adds a scalar
    // offset, a multiple of 16 bytes for both.
    int woff[NBW], xoff[NBX];
    unsigned whi = 0;                                               // bit k: unit of the upper 8 channels
#pragma unroll
    for (int k = 0; k < NBW; ++k) {
        const int v = (wave * NBW + k) * 64 + lane, oc = v / 18, u = v - oc * 18;
        woff[k] = oc < BM && m0 + oc < OC ? (m0 + oc) * C * NTAP * 2 + u * 16 : kOOB;
        whi |= (u >= 9 ? 1u : 0u) << k;
    }
    unsigned xhi = 0;
#pragma unroll
    for (int k = 0; k < NBX; ++k) {
        const int v = (wave * NBX + k) * 64 + lane, ch = v / SU;
        const int2 e = utab[v - ch * SU];
        // (unsigned: channels past the last one, masked below, may lie past 2^31)
        xoff[k] = unit_offset(e.y, (int)((unsigned)e.x + (unsigned)ch * (unsigned)plane), kOOB);
        xhi |= (ch >= 8 ? 1u : 0u) << k;
    }
    const i32x4 rw = make_rsrc(p.Wt, OC * C * NTAP * 2);
    const i32x4 rx = make_rsrc(reinterpret_cast<const unsigned char *>(p.X) - xmis,
                               (xmis + p.Nb * C * plane + 15) & ~15);
    const unsigned raw_lds = __builtin_amdgcn_readfirstlane(lds_address(raw));
    // copies of chunk kc into ring slot s (zeros past the last channel)
    auto issue = [&](int kc, int s) __attribute__((always_inline)) {
        const int c0 = kc * CC;
        const bool lo = c0 < C, hi = c0 + 8 < C;
        const int wso = lo ? c0 * NTAP * 2 : 0, xso = lo ? c0 * plane : 0;
        const unsigned base = raw_lds + s * RAW;
#pragma unroll
        for (int k = 0; k < NBW; ++k)
            dma16_so(rw, base + (wave * NBW + k) * 1024, lo && (hi || !((whi >> k) & 1)) ? woff[k] : kOOB, wso);
#pragma unroll
        for (int k = 0; k < NBX; ++k)
            dma16_so(rx, base + CFG::WRAW + (wave * NBX + k) * 1024,
                     lo && (hi || !((xhi >> k) & 1)) ? xoff[k] : kOOB, xso);
    };

    // This thread's patch items: source (raw byte of channel 0 of its half,
    // before the segment's misalignment), that misalignment's constant part
    // and the cell it fills (-1: none).
    constexpr int slot = SU * 16;
    int isrc[NI], imis[NI], idst[NI];
    const int nitems = nrows * PPR;
#pragma unroll
    for (int k = 0; k < NI; ++k) {
        const int j = t + k * NTG, h = j >= nitems ? 1 : 0, jh = j - h * nitems;
        isrc[k] = 0; imis[k] = 0; idst[k] = -1;
        if (jh < nitems) {
            const int r = div_by(jh, pa.by_ppr), iw = (jh - r * PPR) * (PAIR ? 2 : 1);
            const int4 e = rtab[r];
            isrc[k] = 8 * h * slot + e.y + iw * 2;
            imis[k] = e.x + 8 * h * plane;
            idst[k] = CFG::W_BYTES + h * HALF + (e.z + iw) * 16;
        }
    }
    auto repack = [&](int s) __attribute__((always_inline)) {
        const unsigned char *R = raw + s * RAW;
#pragma unroll
        for (int k = 0; k < NSLAB; ++k) {
            // slab j: output channel j >> 1, channels 8(j & 1) .. +7, nine taps
            const int j = t + k * NTG, oc = j >> 1, h = j & 1;
            if (j < 2 * BM) {
                u32x4_t ws[NTAP];
#pragma unroll
                for (int q = 0; q < NTAP; ++q)
                    ws[q] = *reinterpret_cast<const u32x4_t *>(R + j * (W_ROW / 2) + q * 16);
                auto wv = [&](int e) __attribute__((always_inline)) {   // halfword e = channel e / 9, tap e % 9
                    return (ws[e >> 3][(e >> 1) & 3] >> (16 * (e & 1))) & 0xffffu;
                };
                unsigned char *D = cells + (oc * CC + 8 * (h ^ ((oc >> 3) & 1))) * 2;
#pragma unroll
                for (int q = 0; q < NTAP; ++q) {
                    u32x4_t v;
#pragma unroll
                    for (int d = 0; d < 4; ++d) v[d] = wv(2 * d * NTAP + q) | (wv((2 * d + 1) * NTAP + q) << 16);
                    *reinterpret_cast<u32x4_t *>(D + q * BM * CC * 2) = v;
                }
            }
        }
        const unsigned char *X = R + CFG::WRAW;
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            if (idst[k] >= 0) {
                u32x4_t ev, od;   // the item's column (pair: its even and odd one)
                unsigned v[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const unsigned char *q = X + isrc[k] + c * slot + ((imis[k] + c * plane) & 15);
                    v[c] = PAIR ? *reinterpret_cast<const unsigned *>(q) : *reinterpret_cast<const unsigned short *>(q);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    ev[j] = (v[2 * j] & 0xffffu) | (v[2 * j + 1] << 16);
                    od[j] = (v[2 * j] >> 16) | (v[2 * j + 1] & 0xffff0000u);
                }
                *reinterpret_cast<u32x4_t *>(cells + idst[k]) = ev;
                if constexpr (PAIR) *reinterpret_cast<u32x4_t *>(cells + idst[k] + 16) = od;
            }
        }
    };

    // Fragment bases.  A (weights): output channel wm*WM + 32i + l32, the
    // lane group's 8 channels (halves swapped when bit 3 of the channel is
    // set: conflict-free).  B: the cell of this lane's pixel at tap (0, 0).
    const int a_base = ((wm * WM + l32) * CC + 8 * (lgrp ^ ((l32 >> 3) & 1))) * 2;
    int b_base[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int q = q0 + wn * WN + j * MI + l32;
        int cell = 0;
        if (q < N) {
            const int img = div_by(q, pa.by_ohw), pix = q - img * OHW;
            const int oh = div_by(pix, pa.by_ow), ow = pix - oh * OW;
            cell = ((img - img0) * PH + oh * p.sh - prow0) * WPA + ow * p.sw;
        }
        b_base[j] = CFG::W_BYTES + lgrp * HALF + cell * 16;
    }

    typename MF::acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) acc[i][j][r] = 0.f;

    auto compute = [&]() __attribute__((always_inline)) {
        u16x8 af[2][TM], bfr[2][TN];
        auto frags = [&](int tap, int fb) __attribute__((always_inline)) {
            const int kh = tap / 3, kw = tap - 3 * kh;
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[fb][i] = *reinterpret_cast<const u16x8 *>(cells + a_base + (tap * BM + i * MI) * CC * 2);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                bfr[fb][j] = *reinterpret_cast<const u16x8 *>(cells + b_base[j] + kh * WPA * 16 + kw * 16);
        };
        frags(0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tap = 0; tap < NTAP; ++tap) {
            if (tap + 1 < NTAP) frags(tap + 1, (tap + 1) & 1);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = MF::mma(af[tap & 1][i], bfr[tap & 1][j], acc[i][j]);
            // the next tap's reads between this tap's instructions (the
            // scheduler would otherwise sink each read to just before its use)
            constexpr int NM = TM * TN, ND = TM + TN, PER = (ND + NM - 1) / NM;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                  // MFMA
                if (tap + 1 < NTAP && m * PER < ND) __builtin_amdgcn_sched_group_barrier(0x100, PER, 0);  // DS read
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // Every group runs the same number of trips (chunks past the last one
    // are copied as zeros), so the barriers match.  A trip:
    // wait for this wave's copies of its chunk, barrier (every wave's have
    // landed and every wave is done with the cells), repack, barrier (cells
    // complete, raw slot read), refill the slot, compute.
    const int nchunk = (C + CC - 1) / CC;
    const int trips = (nchunk + KS - 1) / KS;
    __syncthreads();                        // the tables have been read
#pragma unroll
    for (int s = 0; s < RD; ++s) issue(kg + s * KS, s);
    for (int it = 0; it < trips; ++it) {
        const int s = RD == 1 ? 0 : it % RD;
        wait_vmcnt_and_lds<(RD - 1) * (NBW + NBX)>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        repack(s);
        asm volatile("" ::: "memory");
        wait_vmcnt_and_lds<(RD - 1) * (NBW + NBX)>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue(kg + (it + RD) * KS, s);
        compute();
    }
    wait_vmcnt<0>();  // no copy may still be writing LDS when it is reused or the workgroup ends

    if constexpr (KS > 1) {
        // groups 1 .. KS-1 leave their sums in LDS (each lane its own
        // registers, lane-contiguous); group 0 adds them in group order
        float *red = reinterpret_cast<float *>(psm);
        __syncthreads();
        if (kg > 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        red[((((kg - 1) * CFG::NWAVES + wave) * TM + i) * TN + j) * 1024 + r * 64 + lane] = acc[i][j][r];
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int g = 1; g < KS; ++g)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        acc[i][j][r] += red[((((g - 1) * CFG::NWAVES + wave) * TM + i) * TN + j) * 1024 + r * 64 + lane];
    }

    // Output: pixels and channels outside Y are stored at an out-of-range
    // offset, which drops them.
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(p.Y, 0, N * OC * 4, 0x00020000);
    auto store = [&](auto WHOLE) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int q = q0 + wn * WN + j * MI + l32;
            const int img = div_by(q, pa.by_ohw), pix = q - img * OHW;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int oc = m0 + wm * WM + i * MI + 4 * lgrp;
                const unsigned first = ((unsigned)(img * OC + oc) * (unsigned)OHW + (unsigned)pix) * 4u;
#pragma unroll
                for (int r = 0; r < MF::NACC; ++r) {
                    const int row = 8 * (r >> 2) + (r & 3);   // MF::row without the lane's part
                    const float v = (p.relu && acc[i][j][r] < 0.f) ? 0.f : acc[i][j][r];
                    const StoreOffset o = store_offset(decltype(WHOLE)::value, q < N, oc + row < OC, first,
                                                       (unsigned)row * (unsigned)OHW * 4u, kOOB);
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), ry, (int)o.lane,
                                                          (int)o.scalar, 0);
                }
            }
        }
    };
    if (m0 + BM <= OC) store(std::true_type{});
    else store(std::false_type{});
}

// Shapes whose patch kernel launch is laid out in *pa and *lds (bytes): 3x3,
// whole 8-channel cells, 16-byte aligned weights, and a patch that fits SU
// units per channel, NI items per thread and the LDS.
template <typename CFG, int SU, int NI>
bool patch_bf16_geom(const ConvArgs &a, bool pair, PatchArgs *pa, size_t *lds) {
    using namespace patch_bf16;
    if (a.R != 3 || a.S != 3 || a.C % 8 != 0) return false;
    if ((reinterpret_cast<uintptr_t>(a.Wt) & 15) != 0) return false;
    const long long OHW = (long long)a.OH * a.OW, N = a.Nb * OHW;
    // output rows a tile can touch, and image borders among them (between
    // two images the padded rows advance by 3 instead of stride_h)
    const long long span = std::min<long long>((CFG::BN - 1 + a.OW - 1) / a.OW + 1, (long long)a.Nb * a.OH);
    const long long cross = std::min<long long>((std::min<long long>(CFG::BN, N) - 1 + OHW - 1) / OHW, a.Nb - 1);
    const long long wpa = std::max<long long>((long long)(a.OW - 1) * a.sw + 3, (long long)a.pw + a.W);
    if (a.sh > 64 || wpa > 8192) return false;
    const long long rows = (span - 1) * a.sh + 3 + cross * std::max(3 - a.sh, 0);
    const long long half = (rows * wpa * 16 + 511) / 512 * 512;   // whole KiB for both halves
    const long long raw = CFG::WRAW + (long long)CC * SU * 16;
    const long long bytes = std::max<long long>(CFG::KS * (CFG::RD * raw + CFG::W_BYTES + 2 * half), CFG::RED_BYTES);
    if (bytes > kMaxLds) return false;
    const long long inrows = std::min<long long>(rows, (cross + 1) * (long long)a.H);   // rows inside the images
    const long long ppr = pair ? a.W / 2 : a.W;
    if (inrows * 2 * ppr > (long long)NI * CFG::NTG) return false;
    const long long units = inrows * a.W * 2 / 16 + 3 * (cross + 1);   // 16-byte units per channel
    if (units > SU || SU * 8 + inrows * 16 > raw) return false;        // (the tables share the raw area)
    pa->c = a;
    pa->by_ohw = fast_div(a.OH * a.OW);
    pa->by_ow = fast_div(a.OW);
    pa->by_ppr = fast_div((int)ppr);
    pa->PH = (a.OH - 1) * a.sh + 3;
    pa->WPA = (int)wpa;
    pa->PPR = (int)ppr;
    pa->half = (int)half;
    *lds = (size_t)bytes;
    return true;
}

template <typename CFG, int SU, int NI, bool PAIR>
hipError_t launch_patch(const PatchArgs &pa, size_t lds, hipStream_t s) {
    const int N = pa.c.Nb * pa.c.OH * pa.c.OW;
    const unsigned tiles = (unsigned)(((pa.c.OC + CFG::BM - 1) / CFG::BM) * ((N + CFG::BN - 1) / CFG::BN));
    PatchArgs args = pa;
    void *kargs[] = {&args};
    return hipLaunchKernel(reinterpret_cast<const void *>(&conv2d_bf16_patch_kernel<CFG, SU, NI, PAIR>),
                           dim3(tiles), dim3(CFG::NT), kargs, lds, s);
}

// Workgroups of the tile's kernel that a CU holds in the reference layer.
template <typename CFG>
hipError_t patch_bf16_occupancy(int, int *wg_per_cu) {
    const ConvArgs a = patch_reference_layer();
    PatchArgs pa;
    size_t lds;
    const void *fn = reinterpret_cast<const void *>(&conv2d_bf16_patch_kernel<CFG, CFG::SU0, 4, true>);
    if (!patch_bf16_geom<CFG, CFG::SU0, 4>(a, true, &pa, &lds)) {
        fn = reinterpret_cast<const void *>(&conv2d_bf16_patch_kernel<CFG, 2 * CFG::SU0, 9, true>);
        if (!patch_bf16_geom<CFG, 2 * CFG::SU0, 9>(a, true, &pa, &lds)) return hipErrorInvalidValue;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(wg_per_cu, fn, CFG::NT, lds);
}

// Tries the patch kernel with tile CFG (with its smaller slot and item count
// only, if `small_only`: long rows leave the others little to gain); false if
// the shape is outside it.
template <typename CFG>
bool try_patch_bf16(const ConvArgs &a, hipStream_t s, hipError_t *err, bool small_only = false) {
    const bool pair = a.W % 2 == 0 && (reinterpret_cast<uintptr_t>(a.X) & 3) == 0;
    PatchArgs pa;
    size_t lds;
    if (patch_bf16_geom<CFG, CFG::SU0, 4>(a, pair, &pa, &lds))
        *err = pair ? launch_patch<CFG, CFG::SU0, 4, true>(pa, lds, s) : launch_patch<CFG, CFG::SU0, 4, false>(pa, lds, s);
    else if (!small_only && patch_bf16_geom<CFG, 2 * CFG::SU0, 9>(a, pair, &pa, &lds))
        *err = pair ? launch_patch<CFG, 2 * CFG::SU0, 9, true>(pa, lds, s)
                    : launch_patch<CFG, 2 * CFG::SU0, 9, false>(pa, lds, s);
    else
        return false;
    return true;
}

// Outside the patch kernel's class.  A CU holds five workgroups of 64x64 tiles
// and four of 64x128 ones, fewer where the k-offset table of a long reduction
// takes their LDS (K = 3200: three and two).  A round of the large ones takes
// about 1.35 times as long (7x7 stride-2 first layers into 64 channels, 1176
// small or 588 large tiles: 17.1 and 20.7 us): small tiles within one round of
// theirs and, past one round of the large ones, up to two and a half (2156 and
// 1078: 27.4, 33.8; 3136 and 1568: 37.2, 38.3); else the large ones (1568 and
// 784: 24.1, 22.9; 3844 and 1922 of a 5x5 layer: 29.1, 27.1).  With fewer per CU
// a large round takes 1.7 times as long (K = 3136, 2813 and 1407: 575, 742; 980
// and 490 of K = 3200: 264, 251).  More than 64
// output channels: small tiles within a round, else 128x128 (K = 512, 980 small
// tiles 40.7 us, 245 large 46.2; 1568 72.5, 392 50.9; K = 3200, 784 258, 196 244;
// 1568 394, 392 269).
hipError_t launch_conv_bf16_gather(const ConvArgs &a, hipStream_t s) {
    const long long N = (long long)a.Nb * a.OH * a.OW;
    const long long small = (a.OC + 63) / 64 * ((N + 63) / 64), large = (a.OC + 63) / 64 * ((N + 127) / 128);
    auto round_of = [&](int bn, int most) {   // tiles of 64 x bn that run at once
        const int lds = 2 * 2 * (64 * (32 + 8) + 32 * (bn + 32)) + 8 * a.C * a.R * a.S;
        return 256LL * std::min(most, 160 * 1024 / lds);
    };
    const long long small_round = round_of(64, 5), large_round = round_of(128, 4);
    // pointwise layers of a stage or two move more than they compute
    // (26x64x55x55 -> 256: 24.3 us, 26.0 with 64x128 tiles, 29.2 with 128x128)
    if (a.R * a.S == 1 && a.C <= 64) return launch_conv_bf16<64, 64, 32, 32, 32, 32, 8>(a, s);
    if (a.OC > 64) {
        if (small <= small_round) return launch_conv_bf16<64, 64, 32, 32, 32, 32, 8>(a, s);
        return launch_conv_bf16<128, 128, 32, 64, 64, 32, 8>(a, s);
    }
    const bool few = small_round < 1280;
    const double small_rounds = (double)((small + small_round - 1) / small_round);
    const double large_rounds = (double)((large + large_round - 1) / large_round);
    if (small <= small_round || (few ? small_rounds < 1.7 * large_rounds : large > large_round && small <= 3200))
        return launch_conv_bf16<64, 64, 32, 32, 32, 32, 8>(a, s);
    return launch_conv_bf16<64, 128, 32, 32, 64, 32, 8>(a, s);
}

typedef patch_bf16::Cfg<64, 256, 64, 64, 1, 2> PatchL;
typedef patch_bf16::Cfg<64, 128, 32, 64, 1, 1> PatchM;
typedef patch_bf16::Cfg<64, 128, 32, 64, 2, 1> PatchM2;
typedef patch_bf16::Cfg<32, 64, 32, 32, 2, 1> PatchS2;
typedef patch_bf16::Cfg<32, 64, 32, 32, 4, 1> PatchS4;

template <typename CFG>
hipError_t launch_conv_bf16_patch(const ConvArgs &a, hipStream_t s) {
    hipError_t err;
    if (try_patch_bf16<CFG>(a, s, &err)) return err;
    return launch_conv_bf16_gather(a, s);
}

// The tile and split for a shape.  Every tile but PatchM's (and PatchS2's in
// short rows) takes the LDS of a whole CU, so its time doubles when the workgroups pass 256: the smallest
// tile, with the reduction split furthest, that stays within one round
// (128x28x28 -> 128 at batch 1, 8, 32: 32x64/4 9.0, 20.8, - us; 64x128/2
// 11.6, 12.4, 24.2; 64x256 16.3, 16.9, 19.0; 64x128 12.5, 13.5, 20.2), and
// past that 64x128 tiles, of which two fit a CU (64x57x57 -> 128 at batch 32:
// 40.1 us against 50.9 with 64x256).  The reduction is split no further than
// it has chunks of 16 channels: a group without one costs its barriers and sums
// (256x8x8x8 -> 8: 6.8 us in four groups, 5.5 in two; 8x8x56x56 -> 16: 7.6 with
// 64x128/2, 6.2 with 64x128).  A single half chunk pays for its patch only where
// that is small: 8 channels at stride 2 or in rows past 64 pixels gather
// (64x8x28x28/2 -> 16 7.4 us, 6.4; 7x8x100x100 -> 33 19.5, 12.4).
hipError_t launch_conv_bf16_patch_auto(const ConvArgs &a, hipStream_t s) {
    const long long N = (long long)a.Nb * a.OH * a.OW;
    auto tiles = [&](int bm, int bn) { return (a.OC + bm - 1) / bm * ((N + bn - 1) / bn); };
    hipError_t err;
    const int chunks = (a.C + patch_bf16::CC - 1) / patch_bf16::CC;
    if (a.C <= 8 && (a.sh > 1 || a.sw > 1 || a.OW > 64)) return launch_conv_bf16_gather(a, s);
    if (tiles(32, 64) <= 256 &&
        ((chunks > 2 && try_patch_bf16<PatchS4>(a, s, &err)) || try_patch_bf16<PatchS2>(a, s, &err)))
        return err;
    if (tiles(64, 128) <= 256 && chunks > 1 && try_patch_bf16<PatchM2>(a, s, &err)) return err;
    if (tiles(64, 128) > 256 && tiles(64, 256) <= 256 && try_patch_bf16<PatchL>(a, s, &err, true)) return err;
    if (try_patch_bf16<PatchM>(a, s, &err) || try_patch_bf16<PatchS2>(a, s, &err)) return err;
    return launch_conv_bf16_gather(a, s);
}

// Shapes the halo kernel covers; anything else runs the patch kernel (which
// itself falls back to the gather kernel).
inline bool bf16_halo_eligible(const ConvArgs &a) {
    using namespace halo_bf16;
    if (a.R != 3 || a.S != 3 || a.sh != 1 || a.sw != 1) return false;
    if (a.C % CC != 0 || a.W % 2 != 0 || a.pw > CO) return false;
    if (a.OW - a.pw + 3 > PC - 1) return false;            // last patch column used
    if ((reinterpret_cast<uintptr_t>(a.X) & 3) != 0 || (reinterpret_cast<uintptr_t>(a.Wt) & 15) != 0)
        return false;
    const int span = (BN - 1 + a.OW - 1) / a.OW + 1;      // output rows a tile can touch
    return span + 2 <= PR;
}

hipError_t launch_conv_bf16_halo(const ConvArgs &a, hipStream_t s) {
    if (!bf16_halo_eligible(a)) return launch_conv_bf16_patch_auto(a, s);
    const int OHW = a.OH * a.OW;
    const unsigned tiles = (unsigned)(((a.OC + halo_bf16::BM - 1) / halo_bf16::BM) * a.Nb *
                                      ((OHW + halo_bf16::BN - 1) / halo_bf16::BN));
    ConvArgs args = a;
    void *kargs[] = {&args};
    return hipLaunchKernel(reinterpret_cast<const void *>(&conv2d_bf16_halo_kernel), dim3(tiles),
                           dim3(halo_bf16::NT), kargs, 0, s);
}

// ---------------------------------------------------------------------------
// Row-streaming bf16 kernel (k_order = 3) for stride-1 3x3 convolutions of 64
// input channels with output rows of at most 64 pixels.  With bf16 inputs such
// a layer does about 190 FLOP per HBM byte, below the matrix cores' ridge
// (about 315), so the kernel is laid out for streaming X in and Y out at HBM
// rate rather than for matrix-core reuse:
//  - a workgroup owns 64 output channels of one image and a band of
//    consecutive output rows, and walks down the band RO = 2 output rows per
//    step, so that each input row enters LDS once per band and the output
//    of a step is written while the following rows are computed;
//  - all C*R*S = 576 weights of its 64 output channels stay in LDS for the
//    whole band (72 KiB, loaded once);
//  - input rows pass through a ring of NR = 8 LDS rows: the four rows a step
//    reads, the two the next step adds (stored at the end of the step,
//    published by the step's barrier) and two slots free for refilling; the
//    loads of the rows a step adds are issued during the step before (so
//    that the first step's own instructions cover the arrival of those
//    rows), into one of two register sets;
//  - wave w computes 32 output channels (half w & 1) x 32 pixels (half
//    w >> 1) of both output rows with 32x32x16 instructions, pixels as the
//    row operand and output channels as the column operand;
//  - one fragment of input row r (32 pixels, 8 channels, one column shift
//    kw) serves every output row of the step that reads row r, one per
//    kernel row kh: four input rows feed the 2 x 3 (output row, kh) pairs.
//    Per 16-channel k-step a wave reads 4 + 3 fragments for 6 instructions,
//    which keeps LDS below the matrix cores' rate and a group's reads within
//    the 15 the LDS counter can wait past;
//  - an input row is stored channel-innermost, one 16-byte cell of 8
//    channels per (column, 8-channel group), 64 columns with input column iw
//    at column iw + CO and zeros outside the image.  Group g of column c sits
//    at slot g ^ h(c), h(c) = ((c >> 1) ^ (c & ~3)) & 7, which keeps both the
//    fragment reads (each phase: 16 lanes of a 32-column run, one group) and
//    the staging writes (8 lanes of consecutive column pairs per phase, each
//    lane writing its two cells in an order that alternates every four
//    lanes) free of bank conflicts at every column shift;
//  - a weight cell holds 8 channels of one (tap, output channel); the eight
//    cells of output channel o sit at slots g ^ h(o), the same pattern, since
//    a weight fragment (32 output channels x two groups) is addressed like a
//    pixel fragment;
//  - each wave turns its output rows around through a 4 KiB LDS area of its
//    own before storing them, so that a store instruction writes runs of 128
//    bytes of one channel row (ring 64 KiB + weights 72 KiB + 4 x 4 KiB:
//    152 KiB, one workgroup per CU).
namespace rows_bf16 {
constexpr int NT = 256;                   // four waves
constexpr int BM = 64;                    // output channels per workgroup
constexpr int CH = 64;                    // input channels (all resident)
constexpr int NCG = CH / 8;               // 8-channel cells per column
constexpr int NKS = CH / 16;              // 16-channel instruction k-steps per tap
constexpr int NTAP = 9;
constexpr int RO = 2;                     // output rows per step
constexpr int NR = 8;                     // input rows in the ring
constexpr int PC = 64;                    // stored columns per input row
constexpr int CO = 2;                     // stored column of input column 0 (even)
constexpr int ROWB = PC * NCG * 16;       // bytes per stored input row
constexpr int RING_BYTES = NR * ROWB;
constexpr int W_BYTES = NTAP * BM * NCG * 16;
constexpr int STG_BYTES = 32 * 128;       // per wave: one output row, 32 channels x 32 pixels
constexpr int LDS_BYTES = RING_BYTES + W_BYTES + (NT / 64) * STG_BYTES;
static_assert(NT == 32 * NCG, "one (column pair, cell group) per thread");
static_assert(2 * NT == BM * NCG, "two weight slabs per thread");
static_assert(NR >= 3 * RO + 2, "ring: a step's rows, the next step's, and the slots being refilled");
// slot swizzle of the cells of one column (or output channel)
__device__ __forceinline__ int swz(int c) { return ((c >> 1) ^ (c & ~3)) & 7; }
}  // namespace rows_bf16

__global__ void __launch_bounds__(rows_bf16::NT)
conv2d_bf16_rows_kernel(ConvArgs p) {
    using namespace rows_bf16;
    typedef Bf16Mfma<32> MF;
    __shared__ __attribute__((aligned(16))) unsigned char smem[LDS_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, lg = lane >> 5;

    const int H = p.H, Wd = p.W, OC = p.OC, OH = p.OH, OW = p.OW;
    const int band_rows = p.tile_px;
    const int nbands = (OH + band_rows - 1) / band_rows;
    const int tiles_m = (OC + BM - 1) / BM, tiles_n = p.Nb * nbands;
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, tiles_m, tiles_n, p.raster, p.xcd_remap, tm, tn);
    const int m0 = tm * BM;
    const int img = tn / nbands, band = tn - img * nbands;
    const int oh_a = band * band_rows;
    const int rows = min(band_rows, OH - oh_a);   // output rows of the band
    const int nsteps = (rows + RO - 1) / RO;
    const int ih0 = oh_a - p.ph;                   // input row of band row 0
    const int nin = RO * nsteps + 2;               // input rows the band reads

    // ---- input rows: thread (q, g) loads column pair q (input columns
    // 2q - CO, +1) of channels 8g .. 8g+7, one dword per channel; rows and
    // pairs outside the image are read at an out-of-range offset (zeros).
    const int q = tid & 31, g = tid >> 5;
    const int iwp = 2 * q - CO;
    const bool colok = iwp >= 0 && iwp + 1 < Wd;
    const int plane = __builtin_amdgcn_readfirstlane(H * Wd * 2);      // bytes per channel plane
    const int xcol = ((img * CH + 8 * g) * H) * Wd * 2 + iwp * 2;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(p.X), 0, p.Nb * CH * plane, 0x00020000);
    // Two register sets.  Loads and output stores are unconditional
    // (out-of-range offsets instead of branches), so the compiler's counted
    // waits before a set is stored do not include the stores issued after
    // its loads.
    unsigned xv[2][RO][8];
    auto load_rows = [&](auto S, int r0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RO; ++i) {
            const int r = r0 + i, ih = ih0 + r;
            const bool ok = colok & (r < nin) & (ih >= 0) & (ih < H);
            const int o = ok ? xcol + ih * Wd * 2 : kOOB;
#pragma unroll
            for (int c = 0; c < 8; ++c)
                xv[S][i][c] = __builtin_amdgcn_raw_buffer_load_b32(rx, o, c * plane, 0);
        }
    };
    // the thread's two cells; lanes with bit 2 of q set write their odd
    // column first
    const bool wodd = (q >> 2) & 1;
    const int c0 = 2 * q + (wodd ? 1 : 0), c1 = 2 * q + (wodd ? 0 : 1);
    const int cell0 = c0 * (NCG * 16) + ((g ^ swz(c0)) << 4);
    const int cell1 = c1 * (NCG * 16) + ((g ^ swz(c1)) << 4);
    auto store_rows = [&](auto S, int r0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RO; ++i) {
            unsigned char *R = smem + ((r0 + i) % NR) * ROWB;
            u32x4_t ev, od;   // columns 2q and 2q + 1
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned a = xv[S][i][2 * j], b = xv[S][i][2 * j + 1];
                ev[j] = (a & 0xffffu) | (b << 16);
                od[j] = (a >> 16) | (b & 0xffff0000u);
            }
            *reinterpret_cast<u32x4_t *>(R + cell0) = wodd ? od : ev;
            *reinterpret_cast<u32x4_t *>(R + cell1) = wodd ? ev : od;
        }
    };

    // ---- weights: slab s (= tid, tid + NT) is output channel s >> 3,
    // channels 8(s & 7) .. +7, all nine taps: 72 contiguous values of the
    // OIHW row, nine 16-byte loads, repacked into one cell per tap.
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(p.Wt), 0, OC * CH * NTAP * 2, 0x00020000);
    unsigned char *const Wl = smem + RING_BYTES;
    const std::integral_constant<int, 0> S0;
    const std::integral_constant<int, 1> S1;
    // prologue: the weights first (they come from L2, and the in-order
    // memory counter would otherwise make their wait include the input
    // rows' HBM latency), then band rows 0 .. 3; rows 4, 5 (set 0), which
    // the first step stores at its end, stay in flight
    u32x4_t ws[2][NTAP];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int s = tid + h * NT;
        const int oc = s >> 3, wg = s & 7;
        const int off = m0 + oc < OC ? ((m0 + oc) * CH + 8 * wg) * NTAP * 2 : kOOB;
#pragma unroll
        for (int t = 0; t < NTAP; ++t) ws[h][t] = __builtin_amdgcn_raw_buffer_load_b128(rw, off, 16 * t, 0);
    }
    load_rows(S0, 0);
    load_rows(S1, RO);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int s = tid + h * NT;
        const int oc = s >> 3, wg = s & 7;
        auto wv = [&](int e) __attribute__((always_inline)) {   // halfword e = channel e / 9, tap e % 9
            return (ws[h][e >> 3][(e >> 1) & 3] >> (16 * (e & 1))) & 0xffffu;
        };
        const int slot = oc * (NCG * 16) + ((wg ^ swz(oc)) << 4);
#pragma unroll
        for (int t = 0; t < NTAP; ++t) {
            u32x4_t v;
#pragma unroll
            for (int d = 0; d < 4; ++d) v[d] = wv(2 * d * NTAP + t) | (wv((2 * d + 1) * NTAP + t) << 16);
            *reinterpret_cast<u32x4_t *>(Wl + t * BM * NCG * 16 + slot) = v;
        }
    }
    store_rows(S0, 0);
    store_rows(S1, RO);
    load_rows(S0, 2 * RO);
    __syncthreads();

    // ---- fragment offsets.  B (weights): output channel 32*(wave & 1) +
    // l32, group 2*kstep + lg.  A (pixels): pixel 32*(wave >> 1) + l32 of the
    // output row (lanes past OW read a valid cell and are not stored),
    // column shift kw, group 2*kstep + lg.
    const int oc_l = 32 * (wave & 1) + l32;
    // lanes past OW take the pixel 32 to the left (same banks, so the read
    // stays conflict-free), or the last pixel when there is none
    int px_l = 32 * (wave >> 1) + l32;
    if (px_l >= OW) px_l = px_l >= 32 && px_l - 32 < OW ? px_l - 32 : OW - 1;
    int b_off[NKS], a_off[3][NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        b_off[ks] = oc_l * (NCG * 16) + (((2 * ks + lg) ^ swz(oc_l)) << 4);
#pragma unroll
        for (int kw = 0; kw < 3; ++kw) {
            const int col = px_l + kw - p.pw + CO;
            a_off[kw][ks] = col * (NCG * 16) + (((2 * ks + lg) ^ swz(col)) << 4);
        }
    }

    // ---- output: lane (l32, lg) of wave w holds, per output row, pixels
    // 32*(w >> 1) + 8i + 4lg .. +3 (i = 0..3) of output channel m0 + oc_l.
    // Stored as they are, each 16-byte store instruction would write 32
    // pieces of 32 bytes (one per channel).  Instead each row goes through
    // the wave's own LDS area ([channel][8 chunks of 4 pixels], chunk slot
    // c ^ (channel & 7): conflict-free both ways) and is read back so that
    // lane j holds chunk j & 7 of channel 8s + (j >> 3): four stores per row,
    // each of 8 runs of 128 bytes.  A store whose channel, row or pixels lie
    // outside Y goes to an out-of-range offset and is dropped.
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
        p.Y, 0, p.Nb * OC * OH * OW * 4, 0x00020000);
    unsigned char *const stg = smem + RING_BYTES + W_BYTES + wave * STG_BYTES;
    const int ch_rd = lane & 7, oc_rd = lane >> 3;   // chunk and channel (within 8) read back
    const int px_rd = 32 * (wave >> 1) + 4 * ch_rd;
    // byte offset in Y of band row 0 for each of the lane's four stores of a
    // row (out of range where the channel or the pixels lie outside Y); a
    // row adds its row offset, which keeps an out-of-range offset out of
    // range (unsigned, and Y spans less than 2^31 bytes)
    unsigned soff[4];
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
        const int oc = m0 + 32 * (wave & 1) + 8 * s4 + oc_rd;
        soff[s4] = (oc < OC) & (px_rd < OW) ? (unsigned)((((img * OC + oc) * OH + oh_a) * OW + px_rd) * 4)
                                             : (unsigned)kOOB;
    }
    // relu as a lower bound (-inf: none), by the maximum that keeps a NaN (fmax
    // would give the bound); one instruction where a comparison and a select
    // took the 32x64x56x56 layer from 15.2 to 15.5 us.  Accumulators start at
    // +0, so a -0 result, which the bound would not keep, cannot occur
    const float lo = p.relu ? 0.f : -__builtin_inff();
    // A step's outputs are stored during the next step, one store per
    // k-step group, and its row loads are spread the same way: with one
    // wave per SIMD a burst of memory instructions stalls the wave at the
    // memory queue while its matrix instructions wait behind them.
    constexpr int NPART = RO * 4;               // output stores (and load pairs) per step
    f32x4 pend[NPART];
    int pend_off[NPART];
#pragma unroll
    for (int k = 0; k < NPART; ++k) pend_off[k] = kOOB;
    auto store_part = [&](int k) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, pend[k]), ry, pend_off[k], 0, 0);
    };
    // loads of band rows r0, r0 + 1 into set S, part k: row k / 4, channels
    // 2(k % 4), +1
    auto load_part = [&](auto S, int r0, int k) __attribute__((always_inline)) {
        const int i = k / 4, r = r0 + i, ih = ih0 + r;
        const bool ok = colok & (r < nin) & (ih >= 0) & (ih < H);
        const int o = ok ? xcol + ih * Wd * 2 : kOOB;
#pragma unroll
        for (int c = 2 * (k % 4); c < 2 * (k % 4) + 2; ++c)
            xv[S][i][c] = __builtin_amdgcn_raw_buffer_load_b32(rx, o, c * plane, 0);
    };

    // Fragments: the (kw, k-step) groups of a step in order, double-buffered
    // in registers.  The reads of the next group are issued between the
    // matrix instructions of the current one (a run of reads would likewise
    // stall the wave at the LDS queue), and the last group of a step reads
    // the first group of the next step.
    constexpr int NGRP = 3 * NKS;
    constexpr int NREAD = 3 + RO + 2;            // reads per group
    constexpr int NMMA = 3 * RO;                 // instructions per group
    static_assert(NGRP % 2 == 0 && NREAD >= NMMA && NGRP - 1 >= NPART, "group parity and interleave");
    u16x8 af[2][RO + 2], bf[2][3];
    auto frags = [&](int fb, int grp, int st) __attribute__((always_inline)) {
        const int kw = grp / NKS, ks = grp % NKS;
#pragma unroll
        for (int kh = 0; kh < 3; ++kh)
            bf[fb][kh] = *reinterpret_cast<const u16x8 *>(Wl + (kh * 3 + kw) * BM * NCG * 16 + b_off[ks]);
#pragma unroll
        for (int i = 0; i < RO + 2; ++i)
            af[fb][i] = *reinterpret_cast<const u16x8 *>(smem + ((RO * st + i) % NR) * ROWB + a_off[kw][ks]);
    };
    auto interleave = [&](bool mem) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NMMA; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
            if (mem && i == 1) __builtin_amdgcn_sched_group_barrier(0x040, 1, 0);   // the store
            if (mem && i == 3) __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);   // the loads
        }
        __builtin_amdgcn_sched_group_barrier(0x100, NREAD - NMMA, 0);
        __builtin_amdgcn_sched_barrier(0);
    };

    // step st: its groups load, into set SL, the rows the next step stores;
    // at its end it stores, from set SS, the rows the step after it adds
    auto step = [&](auto SL, auto SS, int st) __attribute__((always_inline)) {
        typename MF::acc_t acc[RO];
#pragma unroll
        for (int o = 0; o < RO; ++o)
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) acc[o][r] = 0.f;
        auto mmas = [&](int fb) __attribute__((always_inline)) {
#pragma unroll
            for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                for (int o = 0; o < RO; ++o) acc[o] = MF::mma(af[fb][o + kh], bf[fb][kh], acc[o]);
        };
#pragma unroll
        for (int grp = 0; grp + 1 < NGRP; ++grp) {
            frags((grp + 1) & 1, grp + 1, st);
            mmas(grp & 1);
            if (grp < NPART) {
                store_part(grp);
                load_part(SL, RO * st + 2 * RO + 2, grp);
            }
            interleave(grp < NPART);
        }
        // the next step's new rows into the ring (loaded during the previous
        // step; their slots were last read two steps ago), then a barrier:
        // every wave has stored them and finished the previous step's reads
        store_rows(SS, RO * st + RO + 2);
        __syncthreads();
        frags(0, 0, st + 1);
        mmas(1);
        interleave(false);
        // this step's outputs, through the staging area, stored during the
        // next step (write-back stores: nontemporal ones of lines that other
        // workgroups' stores complete would cost whole lines of HBM writes).
        // The wave's LDS operations run in order, so row 1 may overwrite
        // the area row 0 was read from.
#pragma unroll
        for (int o = 0; o < RO; ++o) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f32x4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = __builtin_elementwise_maximum(acc[o][4 * i + r], lo);
                *reinterpret_cast<f32x4 *>(stg + l32 * 128 + (((2 * i + lg) ^ (l32 & 7)) << 4)) = v;
            }
            const bool rok = RO * st + o < rows;   // uniform
            const unsigned roff = (unsigned)((RO * st + o) * OW * 4);
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                const int k = 4 * o + s4;
                pend[k] = *reinterpret_cast<const f32x4 *>(stg + (8 * s4 + oc_rd) * 128 + ((ch_rd ^ oc_rd) << 4));
                pend_off[k] = rok ? (int)(soff[s4] + roff) : kOOB;
            }
        }
    };
    frags(0, 0, 0);
    for (int st = 0; st < nsteps; st += 2) {
        step(S1, S0, st);
        if (st + 1 < nsteps) step(S0, S1, st + 1);
    }
#pragma unroll
    for (int k = 0; k < NPART; ++k) store_part(k);
}

// Shapes the row-streaming kernel covers; anything else runs the halo-tiled
// kernel (which itself falls back to the gather kernel).
inline bool bf16_rows_eligible(const ConvArgs &a) {
    using namespace rows_bf16;
    if (a.R != 3 || a.S != 3 || a.sh != 1 || a.sw != 1) return false;
    if (a.C != CH || a.W % 2 != 0 || a.pw > CO || a.OW % 4 != 0 || a.OW > 64) return false;
    if (a.OW + 1 - a.pw + CO > PC - 1) return false;   // last stored column a fragment reads
    if ((reinterpret_cast<uintptr_t>(a.X) & 3) != 0 || (reinterpret_cast<uintptr_t>(a.Wt) & 15) != 0 ||
        (reinterpret_cast<uintptr_t>(a.Y) & 15) != 0)
        return false;
    return true;
}

hipError_t launch_conv_bf16_rows(const ConvArgs &a, hipStream_t s) {
    if (!bf16_rows_eligible(a)) return launch_conv_bf16_halo(a, s);
    // bands sized so that the workgroups (one per CU: the LDS holds one)
    // cover the 256 CUs about once, rounded up to whole steps: a band's
    // time is its step count, so a last step with one row does the work of
    // two (32x64x56x56: 7 bands of 8 rows, 224 workgroups, against 8 bands
    // of 7: 18.9 -> 18.5 us between events)
    const int octiles = (a.OC + rows_bf16::BM - 1) / rows_bf16::BM;
    const int per_img = octiles * a.Nb;
    int nb = (256 + per_img - 1) / per_img;
    ConvArgs args = a;
    args.tile_px = (a.OH + nb - 1) / nb;   // output rows per band, whole steps
    args.tile_px = (args.tile_px + rows_bf16::RO - 1) / rows_bf16::RO * rows_bf16::RO;
    const int nbands = (a.OH + args.tile_px - 1) / args.tile_px;
    args.xcd_remap = 1;
    void *kargs[] = {&args};
    return hipLaunchKernel(reinterpret_cast<const void *>(&conv2d_bf16_rows_kernel),
                           dim3((unsigned)(per_img * nbands)), dim3(rows_bf16::NT), kargs, 0, s);
}

#define XTC_CONV_BF16_INSTANCE(BM, BN, BK, WM, WN, MI, PAD)                                   \
    ConvInstance {                                                                            \
        make_sched(BM, BN, BK, WM, WN, MI, MI, (MI == 32 ? 16 : 32), 2, PAD, 0),               \
            &launch_conv_bf16<BM, BN, BK, WM, WN, MI, PAD>,                                   \
            &occupancy_of<&conv2d_bf16_kernel<BM, BN, BK, WM, WN, MI, PAD, true>,             \
                          (BM / WM) * (BN / WN) * 64, (int)sizeof(int2)>                      \
    }

// lds_stages names the split of the reduction over groups of waves: 2 the
// smaller one of a tile (none; two groups for 32x64), 1 the larger (two; four)
#define XTC_CONV_BF16_PATCH_INSTANCE(CFG, STAGES)                                             \
    ConvInstance {                                                                            \
        make_sched(CFG::BM, CFG::BN, 16, CFG::WM, CFG::WN, 32, 32, 16, STAGES, 0, 0, 2),       \
            &launch_conv_bf16_patch<CFG>, &patch_bf16_occupancy<CFG>                          \
    }

const ConvInstance kConvBf16Instances[] = {
    ConvInstance{make_sched(64, 256, 16, 64, 64, 32, 32, 16, 2, -1, 0, 2),  // halo, 3x3 stride 1
                 &launch_conv_bf16_halo,
                 &occupancy_of<&conv2d_bf16_halo_kernel, halo_bf16::NT, 0>},
    ConvInstance{make_sched(64, 64, 16, 32, 32, 32, 32, 16, 2, -1, 0, 3),  // row streaming, 3x3 s1, C 64
                 &launch_conv_bf16_rows,
                 &occupancy_of<&conv2d_bf16_rows_kernel, rows_bf16::NT, 0>},
    XTC_CONV_BF16_PATCH_INSTANCE(PatchL, 2),
    XTC_CONV_BF16_PATCH_INSTANCE(PatchM, 2),
    XTC_CONV_BF16_PATCH_INSTANCE(PatchM2, 1),
    XTC_CONV_BF16_PATCH_INSTANCE(PatchS2, 2),
    XTC_CONV_BF16_PATCH_INSTANCE(PatchS4, 1),
    XTC_CONV_BF16_INSTANCE(64, 128, 32, 32, 64, 32, 8),   // outside the patch kernel's class
    XTC_CONV_BF16_INSTANCE(128, 128, 32, 64, 64, 32, 8),  // the same for OC > 64
    XTC_CONV_BF16_INSTANCE(64, 64, 32, 32, 32, 32, 8),    // few output pixels
    XTC_CONV_BF16_INSTANCE(64, 128, 64, 32, 64, 32, 8),
    XTC_CONV_BF16_INSTANCE(64, 128, 64, 32, 64, 16, 8),   // 16x16x32 instruction tile
};

}  // namespace

const ConvInstance *conv2d_bf16_instances(int *count) {
    *count = (int)(sizeof(kConvBf16Instances) / sizeof(kConvBf16Instances[0]));
    return kConvBf16Instances;
}

}  // namespace xtc
