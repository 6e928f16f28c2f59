// Host side of the C ABI declared in include/xtc.h: argument and schedule
// validation (before any HIP call), compiled-instance lookup, default
// schedules and the launch on the caller's stream.
#include <string.h>

#include "xtc_internal.h"

namespace {

using namespace xtc;

thread_local int32_t g_last_hip_error = 0;

// Largest operand span in bytes.  Kernels use 32-bit buffer offsets, and
// an element outside an operand is read through the offset kOOB
// (0x7FFFFFF0): the span stays 32 bytes below it, so that offset (plus a
// 16-byte chunk, plus the 16-byte alignment slack of the shifted bf16 loads)
// always lies past the operand's buffer range and reads zero.
constexpr int64_t kMaxSpan = 0x7FFFFFF0 - 32;
// Largest raster group; the kernels also clamp it to the tile rows.
constexpr int kMaxRaster = 64;
// Largest stride or padding, and padded extent, of a convolution: keeps
// every input coordinate oh*stride - pad + kh within 32-bit arithmetic.
constexpr int64_t kMaxConvExtent = int64_t(1) << 30;
constexpr int kLdsBytes = 160 * 1024;                  // LDS per CU on gfx950

// Products and sums of non-negative extents, saturated at INT64_MAX: the
// entry points take any int64 sizes, and a product that wrapped around
// would pass the span limits.
int64_t sat_mul(int64_t a, int64_t b) {
    int64_t r;
    return __builtin_mul_overflow(a, b, &r) ? INT64_MAX : r;
}
int64_t sat_add(int64_t a, int64_t b) {
    int64_t r;
    return __builtin_add_overflow(a, b, &r) ? INT64_MAX : r;
}
int64_t cdiv(int64_t a, int64_t b) { return a / b + (a % b != 0); }   // a >= 0, b > 0

// Bytes from the first to one past the last addressed element of a
// rows x cols row-major operand with row stride ld (0 if empty; saturated).
int64_t span_bytes(int64_t rows, int64_t cols, int64_t ld, int64_t elt) {
    if (rows <= 0 || cols <= 0) return 0;
    return sat_mul(sat_add(sat_mul(rows - 1, ld), cols), elt);
}

bool same_instance(const xtc_sched &a, const xtc_sched &b) {
    return a.block_m == b.block_m && a.block_n == b.block_n && a.block_k == b.block_k &&
           a.wave_m == b.wave_m && a.wave_n == b.wave_n && a.mfma_m == b.mfma_m &&
           a.mfma_n == b.mfma_n && a.mfma_k == b.mfma_k && a.lds_stages == b.lds_stages &&
           a.lds_pad == b.lds_pad && a.unroll_k == b.unroll_k && a.k_order == b.k_order &&
           a.k_split == b.k_split;
}

bool pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

// Structural legality of a schedule for op/dtype, independent of whether it
// was compiled.
xtc_status legal(xtc_op op, xtc_dtype dt, const xtc_sched &s) {
    if (s.size != (int32_t)sizeof(xtc_sched)) return XTC_ERR_BAD_SCHEDULE;
    // Tile sizes are powers of two, except the pixel dimension of the conv
    // kernels that stage an input patch (k_order 2), whose workgroups cover
    // a whole number of 16-pixel instruction blocks.
    const bool any_n = op == XTC_OP_CONV2D && s.k_order == 2 && s.block_n > 0 && s.block_n % 16 == 0 &&
                       s.wave_n > 0 && s.wave_n % 16 == 0;
    if (!pow2(s.block_m) || !pow2(s.block_k) || !pow2(s.wave_m) ||
        (!any_n && (!pow2(s.block_n) || !pow2(s.wave_n))))
        return XTC_ERR_BAD_SCHEDULE;
    if (s.block_m % s.wave_m || s.block_n % s.wave_n) return XTC_ERR_BAD_SCHEDULE;
    if (s.k_split != 1 && s.k_split != 2 && s.k_split != 4 && s.k_split != 8)
        return XTC_ERR_BAD_SCHEDULE;
    const int waves = (s.block_m / s.wave_m) * (s.block_n / s.wave_n) * s.k_split;
    if (waves < 1 || waves > 16) return XTC_ERR_BAD_SCHEDULE;  // <= 1024 threads
    // k_split > 1: either waves that each cover the whole tile with operands
    // straight to registers (lds_stages 0), or groups of waves that each run
    // the LDS-staged pipeline on their share of the K-steps (lds_stages >= 1)
    if (s.k_split > 1 && (op != XTC_OP_MATMUL ||
                          (s.lds_stages == 0 && (s.wave_m != s.block_m || s.wave_n != s.block_n))))
        return XTC_ERR_BAD_SCHEDULE;
    // instruction tiles the matrix cores offer for this dtype
    if (s.mfma_m != s.mfma_n) return XTC_ERR_BAD_SCHEDULE;
    if (dt == XTC_F32) {
        if (!((s.mfma_m == 32 && s.mfma_k == 2) || (s.mfma_m == 16 && s.mfma_k == 4)))
            return XTC_ERR_BAD_SCHEDULE;
    } else {
        if (!((s.mfma_m == 32 && s.mfma_k == 16) || (s.mfma_m == 16 && s.mfma_k == 32)))
            return XTC_ERR_BAD_SCHEDULE;
    }
    if (s.wave_m % s.mfma_m || s.wave_n % s.mfma_n) return XTC_ERR_BAD_SCHEDULE;
    // block_k: a whole number of fragment sets (fp32: 4 k per lane group);
    // for the patch-staging conv kernels it counts channels per stage, a
    // whole number of instruction k-steps
    const int kchunk = (op == XTC_OP_CONV2D && s.k_order == 2) ? s.mfma_k
                       : dt == XTC_F32 ? 4 * (64 / s.mfma_m) : s.mfma_k;
    if (s.block_k % kchunk) return XTC_ERR_BAD_SCHEDULE;
    // lds_stages 0: operands straight to registers (the k_split matmul
    // kernels and the few-output-channel conv kernel)
    const bool regs_ok = s.k_split > 1 || (op == XTC_OP_CONV2D && s.block_m == s.wave_m);
    if (s.lds_stages < (regs_ok ? 0 : 1) || s.lds_stages > 5) return XTC_ERR_BAD_SCHEDULE;
    if (s.lds_pad < -1 || s.lds_pad > 64) return XTC_ERR_BAD_SCHEDULE;
    if (s.unroll_k < 0) return XTC_ERR_BAD_SCHEDULE;
    if (s.raster < 0 || s.raster > kMaxRaster || s.xcd_remap < 0 || s.xcd_remap > 1)
        return XTC_ERR_BAD_SCHEDULE;
    if (s.k_order < 0 || s.k_order > 3 || (op == XTC_OP_MATMUL && s.k_order != 0))
        return XTC_ERR_BAD_SCHEDULE;
    // LDS budget of the staged tiles
    const int elt = dt == XTC_F32 ? 4 : 2;
    const int pad = s.lds_pad > 0 ? s.lds_pad : 0;
    // swizzled unpadded rows (lds_pad = -1) or rows padded by lds_pad (A) and 8 (B)
    const int bpad = s.lds_pad < 0 ? 0 : 8;
    int64_t lds = (int64_t)s.lds_stages * elt *
                  ((int64_t)s.block_m * (s.block_k + pad) + (int64_t)s.block_n * (s.block_k + bpad));
    if (s.k_split > 1) lds += (int64_t)s.k_split * s.block_m * s.block_n * 4;  // partial sums
    if (lds > kLdsBytes) return XTC_ERR_BAD_SCHEDULE;
    return XTC_OK;
}

const GemmInstance *find_gemm(xtc_dtype dt, const xtc_sched &s) {
    int n = 0;
    const GemmInstance *tab = dt == XTC_F32 ? gemm_f32_instances(&n) : gemm_bf16_instances(&n);
    for (int i = 0; i < n; ++i)
        if (same_instance(tab[i].sched, s)) return &tab[i];
    return nullptr;
}

const ConvInstance *find_conv(xtc_dtype dt, const xtc_sched &s) {
    int n = 0;
    const ConvInstance *tab = dt == XTC_F32 ? conv2d_f32_instances(&n) : conv2d_bf16_instances(&n);
    for (int i = 0; i < n; ++i)
        if (same_instance(tab[i].sched, s)) return &tab[i];
    return nullptr;
}

xtc_status hip_status(hipError_t e) {
    if (e == hipSuccess) return XTC_OK;
    g_last_hip_error = (int32_t)e;
    return XTC_ERR_HIP;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
bool aligned_to(const void *p, int64_t bytes) {
    return (reinterpret_cast<uintptr_t>(p) & (uintptr_t)(bytes - 1)) == 0;
}

// The default schedule of `batch` products of M x K and K x N.
void default_matmul(xtc_dtype dt, int64_t M, int64_t N, int64_t K, int64_t batch, xtc_sched *out) {
    const int64_t cus = 256;
    auto tiles = [&](int bm, int bn) { return sat_mul(sat_mul(cdiv(M, bm), cdiv(N, bn)), batch); };
    bool mid = false;
    if (dt == XTC_F32) {
        // The reduction-split kernels for long reductions with a narrow
        // operand; the direct-to-LDS tiles where they give the CUs enough
        // work; below that, the largest reduction-split tile that still gives
        // one tile per CU (measured over 16x16 .. 128x128 tiles on shapes from
        // 256^3 to 4096^3 and skinny ones such as 128x128x4096 and
        // 64x4096x1024).
        if (K >= 2048 && (M < N ? M : N) <= 32 && tiles(32, 32) >= cus) {
            // One operand has at most 32 rows (or columns) and the
            // reduction is long: the product streams the other operand from
            // HBM.  The reduction-split kernels read it straight into
            // registers, with more loads in flight per CU than the
            // direct-to-LDS ring holds (32768x16x4096: 3.2 -> 5.0 TB/s).
            // Tiles and orders as measured on 32768x16, 16x32768 and
            // 32768x32 (K = 4096).
            if (N <= 16) {
                // 32x16 tiles: each workgroup's reads of B serve 32 rows
                *out = make_sched(32, 16, 32, 32, 16, 16, 16, 4, 0, 0, 0, 0, 8);
                out->raster = 0;
            } else if (M <= 16) {
                *out = make_sched(32, 32, 32, 32, 32, 32, 32, 2, 0, 0, 0, 0, 4);
                out->raster = 0;
            } else {
                *out = make_sched(32, 32, 32, 32, 32, 32, 32, 2, 0, 0, 0, 0, 8);
                out->raster = 4;
            }
            return;
        } else if (tiles(64, 64) >= cus / 2 || (tiles(64, 32) >= 160 && (M < N ? M : N) > 32)) {
            // (narrow operands below half a 64x64 tile per CU leave half of a
            // 64x32 tile empty: 16x5120x1024 13.6 us, 8.0 with 16x16
            // register-fed tiles; 64x5200x1024 14.2 and 19.5)
            // The CU with the most tiles sets the time: ceil(tiles / 256)
            // tiles of block_m * block_n work at the rate the kernel reaches
            // with that many of its workgroups on a CU.  The rates (shares of
            // the matrix peak with 1, 2, 3 and more tiles per CU) are from
            // 20 shapes between 512x1024x768 and 4096^3; the estimate is
            // within 12% on those with K >= 1000 and picks the fastest tile
            // on all but one (5% slower).  Against the fixed thresholds used
            // before: 1536^3 76.9 -> 71.1 us, 2999^3 586 -> 478,
            // 512x1024x768 16.0 -> 12.1, 128x4096x1024 20.0 -> 16.0.
            struct Tile {
                int m, n;
                double rate[4];
            };
            static const Tile kTiles[] = {
                {256, 256, {.93, .93, .93, .93}}, {256, 128, {.84, .90, .90, .90}},
                {128, 128, {.76, .82, .82, .82}}, {128, 64, {.62, .82, .82, .82}},
                {64, 64, {.63, .74, .77, .77}},   {64, 32, {.45, .57, .65, .70}},
            };
            const Tile *best = nullptr;
            double least = 0;
            for (const Tile &t : kTiles) {
                const int64_t per_cu = cdiv(tiles(t.m, t.n), cus);
                const double cost = (double)per_cu * t.m * t.n / t.rate[per_cu < 4 ? per_cu - 1 : 3];
                if (!best || cost < least) {
                    best = &t;
                    least = cost;
                }
            }
            if (best->m == 256 && best->n == 256)        // eight 128x64 waves
                *out = make_sched(256, 256, 32, 128, 64, 32, 32, 2, 2, -1, 0);
            else if (best->m == 256)                     // eight 64x64 waves
                *out = make_sched(256, 128, 32, 64, 64, 32, 32, 2, 2, -1, 0);
            else
                *out = make_sched(best->m, best->n, 32, best->m / 2, best->n == 32 ? 32 : best->n / 2, 32, 32, 2,
                                  2, -1, 0);
            // few tiles per CU and a long reduction: two groups of four
            // waves per 64x64 tile, each on half of the K-steps, so that each
            // SIMD holds two waves (1000^3: 24.3 -> 22.2 us, 1024^3: 23.7 ->
            // 22.5 us; no gain with several tiles per CU, a loss for K = 128);
            // the 64x32 tile, two waves without it, always has them
            if (best->n == 32 || (best->n == 64 && best->m == 64 && tiles(64, 64) <= cus && K >= 512)) out->k_split = 2;
            mid = true;
        } else if (tiles(64, 32) >= cus)
            *out = make_sched(64, 32, 16, 64, 32, 32, 32, 2, 0, 0, 0, 0, 4);
        else if (tiles(32, 32) >= cus)
            *out = make_sched(32, 32, 32, 32, 32, 32, 32, 2, 0, 0, 0, 0, K >= 1024 ? 8 : 4);
        else
            *out = make_sched(16, 16, 32, 16, 16, 16, 16, 4, 0, 0, 0, 0, 4);
    } else {
        // The register-fed reduction-split kernels where their 64x32 tiles do
        // not outnumber the CUs (32x1000x2048: 29.7 us with LDS-staged tiles,
        // 5.4; 512^3: 6.7, 4.5; 512x1024x768: 8.6, 6.8; past it the staged
        // tiles win: 1024^3 10.7 against 13.1) or one operand is narrow
        // (10000x30x2000: 70.7, 13.0; 32768x16x4096: 48.2, 46.4); else the
        // direct-to-LDS tiles from 256x256 down to 64x128.
        // Of the three, the tile with the least work on the fullest CU: a
        // k-step of 16*TM rows costs TM row loads and 8 column loads,
        // about 56, 72 and 104 clocks (the order it gives matches the
        // measured one on 14 of 15 shapes, and is 17% off on the other).
        const int64_t c16 = sat_mul(cdiv(tiles(16, 32), cus), 56), c32 = sat_mul(cdiv(tiles(32, 32), cus), 72),
                      c64 = sat_mul(cdiv(tiles(64, 32), cus), 104);
        const int bm = c16 <= c32 && c16 <= c64 ? 16 : c32 <= c64 ? 32 : 64;
        // (a launch has less than 2^32 threads, 256 per tile)
        if ((tiles(64, 32) <= cus || (M < N ? M : N) <= 32) && tiles(bm, 32) < int64_t(1) << 24) {
            *out = make_sched(bm, 32, 32, bm, 32, 16, 16, 32, 0, 0, 0, 0, 4);
        } else if (tiles(256, 256) >= cus && M > 128)
            *out = make_sched(256, 256, 32, 128, 64, 32, 32, 16, 4, -1, 0);
        else if (tiles(128, 128) >= cus && M > 64)
            *out = make_sched(128, 128, 32, 64, 64, 32, 32, 16, 4, -1, 0);
        else   // (and where half of a larger tile's rows would lie past M)
            *out = make_sched(64, 128, 64, 32, 64, 32, 32, 16, 2, -1, 0);
    }
    const int64_t t = tiles(out->block_m, out->block_n);
    out->raster = mid ? 4 : (t >= 64 ? 8 : 0);
    // The register-fed reduction-split tiles: column-major order (graph
    // replays interleaved on one machine: 256^3 3.36 -> 3.25 us, 256x258x512
    // 5.77 -> 5.57 us, the 256x1024x128 matmul+relu 4.91 -> 4.78 us)
    if (out->k_split > 1 && out->lds_stages == 0) out->raster = 1;
    if (dt == XTC_BF16 && out->block_m == 256 && out->block_n == 256) {
        // Column-major tiles dealt round-robin to the XCDs: at any moment all
        // eight XCDs read the same few B column-panels, which the shared
        // last-level cache then serves once (measured on 8192^3: 2% faster
        // than grouped raster 8 with the XCD remap).
        out->raster = 1;
        out->xcd_remap = 0;
    }
}

// fp32 pointwise layers of up to 16 output channels: the tile of the product
// with each image, or false for the conv kernel.  That kernel adds two partial
// sums, or more of a short reduction, so the product needs as many not to sum
// more coarsely: four waves on 16x16 tiles from 128 channels (32x128x28x28 -> 16:
// error against 64 bits 1.11e-7, 1.48e-7 by the conv kernel and 2.04e-7 by
// 64x64 tiles; 8.7, 10.0 and 7.6 us; 12x512x28x28: 2.1e-7, 2.9e-7; 7.0, 18.3),
// but for many tiles of a reduction below 256 (12x128x55x55 -> 8 11.0, 9.6;
// 32x128x55x55 -> 16 26.3, 25.1; x256 14.0, 25.4 at batch 12); four on 64x32
// tiles, whose steps are 16 channels, from 64 (32x64x56x56: 8.4e-8, 8.4e-8;
// 22.8, 25.8), but for many tiles from about 96, whose input patch the conv
// kernel can stage (4x96x55x55 6.4, 5.7; 32x96x14x14 4.6, 19.6).  Below 64
// channels no tile's sums are as fine (32x16x56x56: 7.3e-8 with all, 6.0e-8;
// 9.4, 15.1).
bool pointwise_f32_few(int64_t N, int64_t HW, int64_t C, int64_t OC, xtc_sched *out) {
    if (C >= 128) {
        *out = make_sched(16, 16, 32, 16, 16, 16, 16, 4, 0, 0, 0, 0, 4);
        out->raster = 1;
        return C >= 256 || cdiv(HW, 16) * N <= (OC > 8 ? 4096 : 1024);
    }
    *out = make_sched(64, 32, 16, 64, 32, 32, 32, 2, 0, 0, 0, 0, 4);
    out->raster = 1;
    return C >= 64 && (C < 80 || cdiv(HW, 32) * N <= 256);
}

// Microseconds of a pointwise layer on either route, from the tiles on the
// fullest CU (fitted to 2808 layers of 16 to 2048 channels, images of 1 to 900
// pixels, batch 2 to 1448; of those with two tiles per CU 94% are within 20%).

// One product per image with schedule s: a tile costs a fixed part and its
// products, those of columns past the image's included.
double pointwise_per_image_us(xtc_dtype dt, int64_t N, int64_t HW, int64_t C, int64_t OC, const xtc_sched &s) {
    auto per_cu = [&](int64_t bm, int64_t bn) { return (double)cdiv(cdiv(OC, bm) * cdiv(HW, bn) * N, 256); };
    const double c = (double)C, area = (double)s.block_m * s.block_n, n = per_cu(s.block_m, s.block_n);
    const bool fed = s.lds_stages == 0;   // the register-fed kernels
    if (dt == XTC_F32) {
        if (fed) return area <= 512 ? 4 + n * c * area * 11.8e-6 : 3.5 + n * (.4 + c * area * 7e-6);
        if (area <= 64 * 32) return 2.3 + n * (1.19 + c * area * 4e-6);
        if (area <= 64 * 64) return 3 + n * (.745 + c * area * 3.84e-6);
        return 4.7 + n * ((area <= 128 * 64 ? 1.26 : 3) + c * area * 3.76e-6);
    }
    // register-staged 64x64 tiles, past three per CU 64x128 ones
    const double n64 = per_cu(64, 64);
    const double staged64 = n64 <= 3 ? 2.3 + n64 * (.37 + .01 * c) : 5.4 + 2.6 * per_cu(64, 128);
    if (fed) {
        if (HW % 2 && C <= (cdiv(OC, 64) * cdiv(HW, 64) * N > 256 ? 192 : 64)) return 2.3 + n64 * (.37 + .01 * c);
        const double rows = c * (.4 + .6 / 64 * s.block_m);
        return HW % 2   ? 4.4 + n * (.24 + .01015 * rows)
               : HW % 8 ? 3 + n * (.71 + .0053 * rows)
                        : 2.85 + n * (.32 + .0048 * rows);
    }
    if (HW % 8 == 0) return 3.8 + n * (.5 + area * (.91e-4 + c * 4.1e-7));
    if (s.block_m < 128) return C <= 128 ? staged64 : 1.4 + per_cu(64, 126) * (2.6 + .0079 * c);
    return 4.5 + per_cu(128, 126) * (3.8 + .0092 * c);
}

// The conv kernels on the pixels of all images in a row: their chain over the
// channels, and the rounds of their tiles.
double pointwise_flat_us(xtc_dtype dt, int64_t pixels, int64_t C, int64_t OC) {
    const double c = (double)C, f = c / 576, fixed = C < 512 ? 1 - c / 512 : 0;
    auto tiles = [&](int64_t bm, int64_t bn) { return cdiv(OC, bm) * cdiv(pixels, bn); };
    auto per_cu = [](int64_t t, const double (&us)[4], double step) {
        const int64_t n = cdiv(t, 256);
        return n <= 4 ? us[n - 1] : us[3] + (double)(n - 4) * step;
    };
    auto rounds = [](int64_t t) { return (double)cdiv(t, 256); };
    if (dt == XTC_F32) {
        if (OC > 64) {
            const int64_t t = tiles(128, 128);
            if (C % 32) return .9 + .885 * f * per_cu(t, {76, 142, 205, 270}, 65) + 8.5 * fixed * rounds(t);
            return 4.8 + .945 * f * per_cu(t, {50, 80, 145, 174}, 43) + 3.5 * fixed * rounds(t);
        }
        const int64_t t64 = tiles(64, 64), t256 = tiles(64, 256);
        if (C % 32) return 2.8 + .82 * f * per_cu(t64, {27, 38, 62, 78}, 18) + 2.05 * fixed * rounds(t64);
        if (t256 < 256) return 3 + .925 * f * per_cu(t64, {18, 28, 38, 48}, 12) + .83 * fixed * rounds(t64);
        return 3.3 + .985 * f * per_cu(t256, {60, 91, 145, 176}, 44) + 3.3 * fixed * rounds(t256);
    }
    const double n = rounds(tiles(64, 64));
    if (C <= 64) return 2.6 + .037 * c + n * (.41 + .0095 * c);
    if (n <= 5) return 2.8 + c * (.04 + .0052 * (n - 1)) + .48 * n;
    if (OC > 64) return 5.6 + (double)cdiv(tiles(128, 128), C > 1700 ? 512 : 768) * (5.2 + .081 * c);
    return 8.9 + (double)cdiv(tiles(64, 128), 1024) * .07 * c;
}

}  // namespace

extern "C" {

const char *xtc_status_str(xtc_status s) {
    switch (s) {
        case XTC_OK: return "ok";
        case XTC_ERR_NULL_POINTER: return "null pointer";
        case XTC_ERR_BAD_SHAPE: return "bad shape";
        case XTC_ERR_BAD_LEADING_DIM: return "bad leading dimension";
        case XTC_ERR_BAD_DTYPE: return "bad or unsupported dtype";
        case XTC_ERR_BAD_SCHEDULE: return "illegal schedule";
        case XTC_ERR_UNSUPPORTED_SCHEDULE: return "schedule not among the compiled instances";
        case XTC_ERR_TOO_LARGE: return "operand too large for 32-bit offsets";
        case XTC_ERR_HIP: return "HIP error";
        case XTC_ERR_MISALIGNED: return "pointer not aligned to its element size";
    }
    return "unknown status";
}

int32_t xtc_last_hip_error(void) { return g_last_hip_error; }

int64_t xtc_conv_max_k(void) { return kConvMaxK; }

int32_t xtc_version(void) { return 100; }

xtc_status xtc_default_schedule(xtc_op op, xtc_dtype dt, int64_t M, int64_t N, int64_t K,
                                xtc_sched *out) {
    if (!out) return XTC_ERR_NULL_POINTER;
    if (dt != XTC_F32 && dt != XTC_BF16) return XTC_ERR_BAD_DTYPE;
    if (op != XTC_OP_MATMUL && op != XTC_OP_CONV2D) return XTC_ERR_BAD_SHAPE;
    if (M < 0 || N < 0 || K < 0) return XTC_ERR_BAD_SHAPE;
    const int64_t cus = 256;
    auto tiles = [&](int bm, int bn) { return sat_mul(cdiv(M, bm), cdiv(N, bn)); };
    if (op == XTC_OP_CONV2D && dt == XTC_BF16) {
        // the row-streaming kernel (3x3 stride 1, 64 input channels, rows of
        // at most 64 pixels; 32x64x56x56 -> 64: 15.3 us kernel span against
        // 17 us for the halo-tiled kernel), which runs the halo-tiled kernel
        // outside its class, that one the patch kernel (any other 3x3 layer
        // of whole 8-channel groups, its tile and split chosen from the
        // layer's shape), and that one the gather kernel
        *out = make_sched(64, 64, 16, 32, 32, 32, 32, 16, 2, -1, 0, 3);
        out->raster = 0;
        return XTC_OK;
    }
    if (op == XTC_OP_CONV2D) {
        // The balanced halo-tiled kernel where the shape allows it (3x3,
        // stride 1, rows of about 56 pixels): 64 output channels x at most
        // 208 (or 416) pixels per workgroup, the pixel tile sized so that the
        // workgroups split evenly over the CUs; else the tap-major kernel's
        // 64x256 tiles of 4 waves (64x64 each) with a two-stage ring, two
        // workgroups per CU, so up to 512 tiles run in a single wave.  When
        // that leaves CUs idle (a small image batch), 64x64 tiles of four
        // 32x32 waves give four times as many workgroups.
        // (5x5 from 3 channels where 64x64 tiles nearly fill one round of four
        // per CU: 929 tiles 15.5 us, these 16.4; 743 tiles 13.0, 13.1; 1114
        // tiles 20.7, 18.0)
        const bool full_round = M > 16 && K < 128 && K % 72 != 0 && tiles(64, 64) > cus * 7 / 2 && tiles(64, 64) <= cus * 4;
        if (M <= 16 || (M <= 32 && K % 32 != 0 && K >= 48 && K <= 256 && !full_round)) {
            // up to 32 channels from a short reduction that is no multiple of
            // 32 (the first layer of an image network): two tiles of 16 (7x7
            // from 3 channels, batch 1, 4, 16: 12.8 -> 7.0, 22.9 -> 16.2,
            // 155 -> 47 us; 3x3, K = 27, is faster with 64x64 tiles)
            // few output channels (the paper's 7x7 stride-2 layer into 16
            // channels: 11.9 us with 64x64 tiles)
            *out = make_sched(16, 64, 128, 16, 16, 16, 16, 4, 0, 0, 0, 0);
            out->raster = 0;
            return XTC_OK;
        }
        if (K % 72 == 0 && (M > 64 || tiles(64, 416) < cus - cus / 8)) {
            // 3x3 layers of whole 8-channel stages, but for large ones up to
            // 64 channels (below): the patch kernels, with the largest tile that
            // stays within a workgroup per CU (each of the split ones takes
            // most of a CU's LDS), 64x112 past that (64x128 output channels x
            // pixels at 28x28, batch 1, 8, 32: 16x32 tiles 10.1, 63.9, - us;
            // 64x64 27.9, 29.7, 109; 64x112 50.4, 51.6, 77.9; the tap-major
            // kernel took 112, 113, 116)
            if (tiles(16, 32) <= cus)
                *out = make_sched(16, 32, 8, 16, 32, 16, 16, 4, 1, 0, 0, 2);
            else if (tiles(64, 32) <= cus)
                *out = make_sched(64, 32, 8, 16, 32, 16, 16, 4, 1, 0, 0, 2);
            else if (tiles(64, 64) <= cus)
                *out = make_sched(64, 64, 8, 16, 64, 16, 16, 4, 1, 0, 0, 2);
            else
                *out = make_sched(64, 112, 8, 16, 112, 16, 16, 4, 2, 0, 0, 2);
            out->raster = 0;
            return XTC_OK;
        }
        if (M <= 64 && K % 32 != 0 && K % 72 != 0) {
            // outside every staged kernel's class: the k-table kernels, whose
            // 64x256 tiles, register-staged for these K, ran a 7x7 first
            // layer into 64 channels at batch 16 in 157 us, 64x64 ones in 70
            *out = make_sched(64, 64, 32, 32, 32, 32, 32, 2, 2, -1, 0, 1);
            out->raster = 0;
            return XTC_OK;
        }
        *out = make_sched(64, 208, 8, 16, 208, 16, 16, 4, 2, -1, 0, 2);
        // two pixel halves per workgroup (one patch and one weight copy for
        // 416 pixels) once that still gives about a workgroup per CU
        // (32x64x56x56 layer: 65.6 -> 63.6 us)
        if (tiles(64, 416) >= cus - cus / 8)
            *out = make_sched(64, 416, 8, 16, 208, 16, 16, 4, 2, -1, 0, 2);
        if (M > 64)
            *out = make_sched(128, 128, 32, 64, 64, 32, 32, 2, 2, -1, 0, 1);
        else if (tiles(64, 256) < cus)
            *out = make_sched(64, 64, 32, 32, 32, 32, 32, 2, 2, -1, 0, 1);
        out->raster = 0;
        return XTC_OK;
    }
    default_matmul(dt, M, N, K, 1, out);
    return XTC_OK;
}

xtc_status xtc_sched_check(xtc_op op, xtc_dtype dt, const xtc_sched *s) {
    if (!s) return XTC_ERR_NULL_POINTER;
    if (dt != XTC_F32 && dt != XTC_BF16) return XTC_ERR_BAD_DTYPE;
    if (op != XTC_OP_MATMUL && op != XTC_OP_CONV2D) return XTC_ERR_BAD_SCHEDULE;
    const xtc_status st = legal(op, dt, *s);
    if (st != XTC_OK) return st;
    if (op == XTC_OP_MATMUL) return find_gemm(dt, *s) ? XTC_OK : XTC_ERR_UNSUPPORTED_SCHEDULE;
    return find_conv(dt, *s) ? XTC_OK : XTC_ERR_UNSUPPORTED_SCHEDULE;
}

xtc_status xtc_sched_occupancy(xtc_op op, xtc_dtype dt, int64_t K, const xtc_sched *s,
                               int32_t *wg_per_cu) {
    if (!s || !wg_per_cu) return XTC_ERR_NULL_POINTER;
    const xtc_status st = xtc_sched_check(op, dt, s);
    if (st != XTC_OK) return st;
    if (K < 0) return XTC_ERR_BAD_SHAPE;
    if (op == XTC_OP_CONV2D && K > kConvMaxK) return XTC_ERR_TOO_LARGE;
    if (K > (int64_t)1 << 30) return XTC_ERR_TOO_LARGE;
    OccupancyFn fn =
        op == XTC_OP_MATMUL ? find_gemm(dt, *s)->occupancy : find_conv(dt, *s)->occupancy;
    int n = 0;
    const xtc_status hs = hip_status(fn((int)K, &n));
    if (hs != XTC_OK) return hs;
    *wg_per_cu = n;
    return XTC_OK;
}

int32_t xtc_sched_list(xtc_op op, xtc_dtype dt, xtc_sched *out, int32_t cap) {
    int n = 0;
    if (op == XTC_OP_MATMUL && dt == XTC_F32) {
        const GemmInstance *t = gemm_f32_instances(&n);
        for (int i = 0; i < n && i < cap && out; ++i) out[i] = t[i].sched;
    } else if (op == XTC_OP_MATMUL && dt == XTC_BF16) {
        const GemmInstance *t = gemm_bf16_instances(&n);
        for (int i = 0; i < n && i < cap && out; ++i) out[i] = t[i].sched;
    } else if (op == XTC_OP_CONV2D && (dt == XTC_F32 || dt == XTC_BF16)) {
        const ConvInstance *t = dt == XTC_F32 ? conv2d_f32_instances(&n) : conv2d_bf16_instances(&n);
        for (int i = 0; i < n && i < cap && out; ++i) out[i] = t[i].sched;
    } else {
        return -1;
    }
    return n;
}

}  // extern "C"

namespace {

// Launches schedule s on checked operands: `batch` products of A with the
// matrices stride_b bytes apart from B, into those stride_c bytes apart from
// C.
xtc_status launch_matmul(const xtc_sched &s, xtc_dtype dtype, int M, int N, int K, const void *A, int lda,
                         const void *B, int ldb, float *C, int ldc, int relu, int batch, int64_t stride_b,
                         int64_t stride_c, void *stream) {
    const GemmInstance *inst = find_gemm(dtype, s);
    if (!inst) return XTC_ERR_UNSUPPORTED_SCHEDULE;
    GemmArgs a;
    a.M = M; a.N = N; a.K = K;
    // (an empty B spans nothing whatever its rows' distance: the kernels size
    // its range check as (K - 1) * ldb + N elements, which must not go below 0)
    a.A = A; a.lda = lda; a.B = B; a.ldb = K > 0 ? ldb : N; a.C = C; a.ldc = ldc;
    a.raster = s.raster; a.xcd_remap = s.xcd_remap;
    a.relu = relu;
    a.batch = batch; a.stride_b = (unsigned)stride_b; a.stride_c = (unsigned)stride_c;
    const int64_t elt = dtype == XTC_F32 ? 4 : 2, lda_b = lda * elt, ldb_b = ldb * elt, k_b = K * elt, n_b = N * elt;
    const bool a_rows = aligned16(A) && lda_b % 16 == 0;
    const bool b_rows = aligned16(B) && ldb_b % 16 == 0 && stride_b % 16 == 0;
    bool vec;
    switch (inst->vec_rule) {
        case kRowsDword:
            vec = aligned_to(A, 4) && aligned_to(B, 4) && lda_b % 4 == 0 && ldb_b % 4 == 0 && stride_b % 4 == 0;
            break;
        case kWholeK: vec = k_b % 16 == 0; break;
        case kWholeChunks: vec = K == 0 || (a_rows && b_rows && k_b % 16 == 0 && n_b % 16 == 0); break;
        default: vec = K == 0 || (a_rows && b_rows); break;
    }
    const GemmLaunch fn = vec ? inst->vec_launch : inst->any_launch;
    return hip_status(fn(a, static_cast<hipStream_t>(stream)));
}

xtc_status matmul_impl(int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B,
                       int64_t ldb, float *C, int64_t ldc, xtc_dtype dtype, const xtc_sched *sched,
                       void *stream, int relu) {
    if (dtype != XTC_F32 && dtype != XTC_BF16) return XTC_ERR_BAD_DTYPE;
    if (M < 0 || N < 0 || K < 0) return XTC_ERR_BAD_SHAPE;
    if (lda < (K > 1 ? K : 1) || ldb < (N > 1 ? N : 1) || ldc < (N > 1 ? N : 1))
        return XTC_ERR_BAD_LEADING_DIM;
    xtc_sched s;
    if (sched) {
        const xtc_status st = xtc_sched_check(XTC_OP_MATMUL, dtype, sched);
        if (st != XTC_OK) return st;
        s = *sched;
    } else {
        xtc_default_schedule(XTC_OP_MATMUL, dtype, M, N, K, &s);
    }
    if (M == 0 || N == 0) return XTC_OK;
    if (!C || (K > 0 && (!A || !B))) return XTC_ERR_NULL_POINTER;
    const int64_t elt = dtype == XTC_F32 ? 4 : 2;
    if (!aligned_to(A, elt) || !aligned_to(B, elt) || !aligned_to(C, 4)) return XTC_ERR_MISALIGNED;
    if (span_bytes(M, K, lda, elt) > kMaxSpan || span_bytes(K, N, ldb, elt) > kMaxSpan ||
        span_bytes(M, N, ldc, 4) > kMaxSpan || lda > kMaxSpan / elt || ldb > kMaxSpan / elt ||
        ldc > kMaxSpan / 4)
        return XTC_ERR_TOO_LARGE;
    return launch_matmul(s, dtype, (int)M, (int)N, (int)K, A, (int)lda, B, (int)ldb, C, (int)ldc, relu, 1, 0, 0,
                         stream);
}

xtc_status conv_impl(int64_t N, int64_t C, int64_t H, int64_t W, int64_t OC, int64_t R,
                     int64_t S, int64_t stride_h, int64_t stride_w, int64_t pad_h, int64_t pad_w,
                     const void *X, const void *Wt, float *Y, xtc_dtype dtype,
                     const xtc_sched *sched, void *stream, int relu) {
    if (dtype != XTC_F32 && dtype != XTC_BF16) return XTC_ERR_BAD_DTYPE;
    if (N < 0 || OC < 0 || C < 1 || H < 1 || W < 1 || R < 1 || S < 1 || stride_h < 1 ||
        stride_w < 1 || pad_h < 0 || pad_w < 0)
        return XTC_ERR_BAD_SHAPE;
    if (stride_h > kMaxConvExtent || stride_w > kMaxConvExtent || pad_h > kMaxConvExtent ||
        pad_w > kMaxConvExtent || H > kMaxConvExtent || W > kMaxConvExtent ||
        H + 2 * pad_h > kMaxConvExtent || W + 2 * pad_w > kMaxConvExtent)
        return XTC_ERR_TOO_LARGE;
    if (H + 2 * pad_h < R || W + 2 * pad_w < S) return XTC_ERR_BAD_SHAPE;
    const int64_t OH = (H + 2 * pad_h - R) / stride_h + 1;
    const int64_t OW = (W + 2 * pad_w - S) / stride_w + 1;
    const int64_t Mg = OC, Ng = sat_mul(sat_mul(N, OH), OW), Kg = sat_mul(sat_mul(C, R), S);
    xtc_sched s;
    if (sched) {
        const xtc_status st = xtc_sched_check(XTC_OP_CONV2D, dtype, sched);
        if (st != XTC_OK) return st;
        s = *sched;
    } else {
        xtc_default_schedule(XTC_OP_CONV2D, dtype, Mg, Ng, Kg, &s);
    }
    if (N == 0 || OC == 0) return XTC_OK;
    if (!X || !Wt || !Y) return XTC_ERR_NULL_POINTER;
    const int64_t xelt = dtype == XTC_F32 ? 4 : 2;
    if (!aligned_to(X, xelt) || !aligned_to(Wt, xelt) || !aligned_to(Y, 4)) return XTC_ERR_MISALIGNED;
    const int64_t elt = dtype == XTC_F32 ? 4 : 2;
    if (sat_mul(sat_mul(sat_mul(sat_mul(N, C), H), W), elt) > kMaxSpan ||
        sat_mul(sat_mul(OC, Kg), elt) > kMaxSpan || sat_mul(sat_mul(OC, Ng), 4) > kMaxSpan)
        return XTC_ERR_TOO_LARGE;
    if (Kg > kConvMaxK) return XTC_ERR_TOO_LARGE;
    // A pointwise layer (1x1, stride 1, no padding) is one product of the
    // weights with each image as it lies, C x H*W row-major: the matmul
    // kernels compute it without a gather (512x28x28 -> 128 at batch 1 and 32:
    // fp32 45.3 and 47.3 us with the conv kernels, 5.6 and 39.8; bf16 43.9 and
    // 45.5, 3.7 and 10.9).  bf16 layers of fewer than 32 channels stay with the
    // gather kernel, whose single small stage they fit (32x16x55x55 -> 64:
    // 10.0 us, 21.4 with 64-k steps of odd rows), and, where images do not
    // start on 16 bytes, those of up to 64 channels from two of its tiles per
    // CU on, or from fewer than 64 (26x64x55x55 -> 64: 9.9 us against 18.5;
    // 13x64x27x27 -> 64, 149 tiles: 5.8, 6.0; 4x64x27x27 -> 64: 5.5, 4.7).
    // Images smaller than a tile leave most of it empty and read all weights
    // each: from some batch on the conv kernels, which run the pixels of all
    // images in a row, are faster (2048x1x1 -> 1000 at batch 8, 64, 512: fp32
    // 15, 112, 856 us per image, 157, 172, 200 in a row; bf16 16, 82, 622, and 97,
    // 87, 88).
    const bool gather = dtype == XTC_BF16 &&
                        (C < 32 || (H * W % 8 != 0 && (C < 64 || (C == 64 && cdiv(OC, 64) * cdiv(Ng, 64) >= 512))));
    if (!sched && R == 1 && S == 1 && stride_h == 1 && stride_w == 1 && pad_h == 0 && pad_w == 0 && N <= 65535 &&
        !gather) {
        const int64_t HW = H * W;
        xtc_sched p;
        bool product;
        if (dtype == XTC_F32 && OC <= 16)
            product = pointwise_f32_few(N, HW, C, OC, &p);
        else {
            default_matmul(dtype, OC, HW, C, N, &p);
            // (below two tiles per CU the products always are the faster)
            product = cdiv(OC, p.block_m) * cdiv(HW, p.block_n) * N < 512;
        }
        if (product || (!(dtype == XTC_F32 && OC <= 16) &&
            pointwise_flat_us(dtype, N * HW, C, OC) >= .95 * pointwise_per_image_us(dtype, N, HW, C, OC, p)))
            return launch_matmul(p, dtype, (int)OC, (int)HW, (int)C, Wt, (int)C, X, (int)HW, Y, (int)HW, relu, (int)N,
                                 C * HW * elt, OC * HW * 4, stream);
    }
    const ConvInstance *inst = find_conv(dtype, s);
    if (!inst) return XTC_ERR_UNSUPPORTED_SCHEDULE;

    ConvArgs a;
    a.Nb = (int)N; a.C = (int)C; a.H = (int)H; a.W = (int)W; a.OC = (int)OC;
    a.R = (int)R; a.S = (int)S;
    a.sh = (int)stride_h; a.sw = (int)stride_w; a.ph = (int)pad_h; a.pw = (int)pad_w;
    a.OH = (int)OH; a.OW = (int)OW;
    a.X = static_cast<const float *>(X);
    a.Wt = static_cast<const float *>(Wt);
    a.Y = Y;
    a.raster = s.raster; a.xcd_remap = s.xcd_remap;
    a.relu = relu;
    a.tile_px = 0;
    const ConvLaunch fn = !sched && inst->by_shape ? inst->by_shape : inst->launch;
    return hip_status(fn(a, static_cast<hipStream_t>(stream)));
}

}  // namespace

extern "C" {

xtc_status xtc_matmul(int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B,
                      int64_t ldb, float *C, int64_t ldc, xtc_dtype dtype, const xtc_sched *sched,
                      void *stream) {
    return matmul_impl(M, N, K, A, lda, B, ldb, C, ldc, dtype, sched, stream, 0);
}

xtc_status xtc_matmul_relu(int64_t M, int64_t N, int64_t K, const void *A, int64_t lda,
                           const void *B, int64_t ldb, float *C, int64_t ldc, xtc_dtype dtype,
                           const xtc_sched *sched, void *stream) {
    return matmul_impl(M, N, K, A, lda, B, ldb, C, ldc, dtype, sched, stream, 1);
}

xtc_status xtc_conv2d_nchw(int64_t N, int64_t C, int64_t H, int64_t W, int64_t OC, int64_t R,
                           int64_t S, int64_t stride_h, int64_t stride_w, int64_t pad_h,
                           int64_t pad_w, const void *X, const void *Wt, float *Y, xtc_dtype dtype,
                           const xtc_sched *sched, void *stream) {
    return conv_impl(N, C, H, W, OC, R, S, stride_h, stride_w, pad_h, pad_w, X, Wt, Y, dtype, sched,
                     stream, 0);
}

xtc_status xtc_conv2d_nchw_relu(int64_t N, int64_t C, int64_t H, int64_t W, int64_t OC, int64_t R,
                                int64_t S, int64_t stride_h, int64_t stride_w, int64_t pad_h,
                                int64_t pad_w, const void *X, const void *Wt, float *Y,
                                xtc_dtype dtype, const xtc_sched *sched, void *stream) {
    return conv_impl(N, C, H, W, OC, R, S, stride_h, stride_w, pad_h, pad_w, X, Wt, Y, dtype, sched,
                     stream, 1);
}

}  // extern "C"
