// bf16 GEMM on the gfx950 matrix cores: C[M,N] = A[M,K] * B[K,N] with A and B
// bf16 (row-major), products exact in fp32, fp32 accumulation, fp32 C
// (overwritten).
//
// Schedule structure as in gemm_f32.hip (workgroup tile, wave tile, MFMA
// instruction tile, double-buffered padded LDS staging, predicated edges).
//
// Operand fragments.  The bf16 MFMAs (32x32x16, 16x16x32) take, per lane,
// 8 consecutive-k values of one A row (row lane%MI, k-group lane/MI) and 8
// consecutive-k values of one B column.  A is row-major (k-contiguous), so
// its fragment is one ds_read_b128 from a k-contiguous LDS row.  B is
// row-major too (n-contiguous) and is staged in LDS as it is (16-byte
// writes, rows padded by 32 elements); its fragment is gathered with two
// gfx950 transpose reads (ds_read_b64_tr_b16).  Within each group of 16
// lanes that instruction returns to lane 4u+t, as its element r, element t
// of the 8 bytes addressed by lane 4r+u of the group.  So when lane 4r+u
// addresses B[k0+r][n0+4u .. n0+4u+3], lane a of the group receives
// B[k0 .. k0+3][n0+a]: four consecutive k of its own column, which is the
// MFMA B-operand layout.  Two such reads (k0 and k0+4) give the 8 values.
#include "lds_dma.h"
#include "mfma_bf16.h"
#include "tile_map.h"
#include "xtc_internal.h"

namespace xtc {
namespace {

template <int BM, int BN, int BK, int WM, int WN, int MI, int PAD, bool VEC>
struct GemmBf16Cfg {
    static constexpr int NWM = BM / WM, NWN = BN / WN;
    static constexpr int NT = NWM * NWN * 64;
    static constexpr int TM = WM / MI, TN = WN / MI;
    typedef Bf16Mfma<MI> MF;
    static constexpr int KG = MF::KG;
    static constexpr int KCH = 8 * KG;      // k per MFMA instruction
    static constexpr int AS = BK + PAD;     // LDS row stride of the A tile (elements)
    static constexpr int BS = BN + 32;      // LDS row stride of the B tile (elements)
    static constexpr int W = 8;             // elements per global load
    static constexpr int A_CPR = BK / W;    // 16-byte chunks per tile row
    static constexpr int B_CPR = BN / W;
    static_assert(64 % A_CPR == 0 && 64 % B_CPR == 0, "a tile row's chunks stay in one wave");
    static constexpr int A_LOADS = BM * BK / (W * NT);
    static constexpr int B_LOADS = BK * BN / (W * NT);
    typedef typename VecU16<W>::t vec_t;
    static_assert(BM % WM == 0 && BN % WN == 0, "wave tile must divide the block tile");
    static_assert(WM % MI == 0 && WN % MI == 0, "MFMA tile must divide the wave tile");
    static_assert(BK % KCH == 0, "block_k must be a multiple of the MFMA k");
    static_assert(A_LOADS * W * NT == BM * BK, "A tile must split evenly over threads");
    static_assert(B_LOADS * W * NT == BK * BN, "B tile must split evenly over threads");
    static_assert(PAD % 8 == 0, "padding must keep 16-byte alignment");
};

template <int BM, int BN, int BK, int WM, int WN, int MI, int PAD, bool VEC>
__global__ void __launch_bounds__((BM / WM) * (BN / WN) * 64)
gemm_bf16_kernel(GemmArgs p) {
    typedef GemmBf16Cfg<BM, BN, BK, WM, WN, MI, PAD, VEC> G;
    typedef typename G::MF MF;
    typedef typename G::vec_t vec_t;
    constexpr int W = G::W;

    __shared__ __attribute__((aligned(16))) unsigned short As[2][BM * G::AS];
    __shared__ __attribute__((aligned(16))) unsigned short Bs[2][BK * G::BS];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / G::NWN, wn = wave % G::NWN;
    const int lrow = lane % MI, lgrp = lane / MI;

    const int M = p.M, N = p.N, K = p.K;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, tiles_m, tiles_n, p.raster, p.xcd_remap, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    const unsigned short *__restrict__ A = static_cast<const unsigned short *>(p.A);
    const unsigned short *__restrict__ B = static_cast<const unsigned short *>(p.b_of(blockIdx.y));
    const int lda = p.lda, ldb = p.ldb;

    vec_t ra[G::A_LOADS], rb[G::B_LOADS];

    // VEC: 16-byte aligned rows, read with plain 16-byte loads.  Otherwise
    // rows may start at any 2-byte boundary: 16-byte loads of the aligned
    // chunks that cover each group of eight, shifted into place.
    int a_first, b_first;
    const __amdgpu_buffer_rsrc_t rsa = aligned_rsrc(A, ((long long)(M - 1) * lda + K) * 2, 2, &a_first);
    const __amdgpu_buffer_rsrc_t rsb = aligned_rsrc(B, ((long long)(K - 1) * ldb + N) * 2, 2, &b_first);
    auto load_tiles = [&](int kt) {
        const int k0 = kt * BK;
#pragma unroll
        for (int i = 0; i < G::A_LOADS; ++i) {
            const int idx = tid + i * G::NT;
            const int r = idx / G::A_CPR, c = (idx % G::A_CPR) * W;
            const int gm = m0 + r, gk = k0 + c;
            const int valid = gm < M ? K - gk : 0;
            if constexpr (VEC) {
                ra[i] = load_pred_u16<W>(A + (valid > 0 ? gm * lda + gk : 0), valid);
            } else {
                // a run is one tile row: its lanes' chunks are consecutive,
                // also past K (those values are read but zeroed)
                const int e = gm < M ? gm * lda + gk : 0;
                ra[i] = load_shifted_u16x8(rsa, a_first + e, valid, idx % G::A_CPR == G::A_CPR - 1);
            }
        }
#pragma unroll
        for (int i = 0; i < G::B_LOADS; ++i) {
            const int idx = tid + i * G::NT;
            const int r = idx / G::B_CPR, c = (idx % G::B_CPR) * W;
            const int gk = k0 + r, gn = n0 + c;
            const int valid = gk < K ? N - gn : 0;
            if constexpr (VEC) {
                rb[i] = load_pred_u16<W>(B + (valid > 0 ? gk * ldb + gn : 0), valid);
            } else {
                const int e = gk < K ? gk * ldb + gn : 0;
                rb[i] = load_shifted_u16x8(rsb, b_first + e, valid, idx % G::B_CPR == G::B_CPR - 1);
            }
        }
    };

    auto store_tiles = [&](int st) {
#pragma unroll
        for (int i = 0; i < G::A_LOADS; ++i) {
            const int idx = tid + i * G::NT;
            const int r = idx / G::A_CPR, c = (idx % G::A_CPR) * W;
            *reinterpret_cast<vec_t *>(&As[st][r * G::AS + c]) = ra[i];
        }
#pragma unroll
        for (int i = 0; i < G::B_LOADS; ++i) {
            const int idx = tid + i * G::NT;
            const int r = idx / G::B_CPR, c = (idx % G::B_CPR) * W;
            *reinterpret_cast<vec_t *>(&Bs[st][r * G::BS + c]) = rb[i];
        }
    };

    typename MF::acc_t acc[G::TM][G::TN];
#pragma unroll
    for (int i = 0; i < G::TM; ++i)
#pragma unroll
        for (int j = 0; j < G::TN; ++j)
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) acc[i][j][r] = 0.f;

    const int KT = (K + BK - 1) / BK;
    if (KT > 0) {
        load_tiles(0);
        store_tiles(0);
        __syncthreads();
    }
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

    float *__restrict__ C = p.c_of(blockIdx.y);
    const int ldc = p.ldc;
#pragma unroll
    for (int i = 0; i < G::TM; ++i)
#pragma unroll
        for (int j = 0; j < G::TN; ++j) {
            const int col = n0 + wn * WN + j * MI + lrow;
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) {
                const int row = m0 + wm * WM + i * MI + MF::row(lane, r);
                if (row < M && col < N) C[row * ldc + col] = (p.relu && acc[i][j][r] < 0.f) ? 0.f : acc[i][j][r];
            }
        }
}

// ---------------------------------------------------------------------------
// Direct-to-LDS variant.  Global tiles are copied straight into LDS with
// buffer_load_dwordx4 ... lds (16 bytes per lane, no register staging), into
// a ring of STAGES LDS buffers, so STAGES-1 K-steps are in flight while the
// matrix cores work on the oldest one.  One such instruction writes 1 KiB of
// LDS contiguously (lane i at byte 16*i of the block), so the layout is
// chosen on the global side: each 16-byte chunk of a tile row is placed at
// slot = chunk ^ swizzle(row) of its LDS row, which keeps the fragment reads
// free of bank conflicts with unpadded rows (swz_a, swz_b below).  Out-of-range chunks (rows >= M
// or >= K, columns >= N or k >= K) are fetched through a buffer offset past
// the end of the buffer, which the hardware returns as zero: this variant
// needs K and N to be multiples of 8 and 16-byte aligned rows, and otherwise
// the kernel for rows at any 2-byte boundary below runs.

// A rows hold CA = BK/8 chunks of 16 bytes; chunk c of row m sits at slot
// c ^ swz_a(m), and an A fragment (16 bytes per lane) is one ds_read_b128.
// gfx950 serves a ds_read_b128 in four phases of 16 lanes: lanes
// {0-3, 12-15, 20-23, 24-27}, {4-11, 16-19, 28-31} and the same sets + 32
// (measured with a per-lane-pair conflict probe).  Lane l of a fragment
// read takes row l % 32, so a phase holds rows r with (r >> 2) in
// {0, 3, 5, 6} or in {1, 2, 4, 7}; the swizzles below give those rows
// distinct 16-byte bank groups (64 banks of 4 bytes), so every phase is
// conflict-free for the 32x32x16 reads, and for the 16x16x32 reads at
// block_k 64.
template <int CA>
__device__ __forceinline__ int swz_a(int row) {
    return CA == 4 ? (row >> 2) & 3 : (row >> 1) & 7;
}

// B rows (one k each) are read four consecutive rows at a time by the
// transpose reads, which gfx950 serves in two phases of 32 lanes (0-31,
// 32-63); XOR values {0, 6, 10, 12} on k % 4 spread the four rows a phase
// reads over distinct bank groups.  With the 16x16x32 instruction one phase
// also reads rows k and k + 8 (lane groups 0 and 1), which XOR 2 on bit 3
// of k separates (with the 32x32x16 instruction that term costs 0.6% on
// 8192^3 and is left out).
template <int MI>
__device__ __forceinline__ int swz_b(int k) {
    return ((k & 1) * 6) ^ ((k & 2) * 5) ^ (MI == 16 ? ((k >> 3) & 1) * 2 : 0);
}


template <int BM, int BN, int BK, int WM, int WN, int MI, int STAGES>
struct Bf16DmaCfg {
    static constexpr int NWM = BM / WM, NWN = BN / WN;
    static constexpr int NWAVES = NWM * NWN;
    static constexpr int NT = NWAVES * 64;
    static constexpr int TM = WM / MI, TN = WN / MI;
    typedef Bf16Mfma<MI> MF;
    static constexpr int KG = MF::KG;
    static constexpr int KCH = 8 * KG;                  // k per MFMA
    static constexpr int NS = BK / KCH;                 // MFMA k-steps per LDS stage
    static constexpr int RA = BK * 2, CA = BK / 8;      // A row bytes / chunks
    static constexpr int RB = BN * 2, CB = BN / 8;      // B row bytes / chunks
    static constexpr int A_BYTES = BM * RA, B_BYTES = BK * RB;
    static constexpr int A_BLOCKS = A_BYTES / 1024, B_BLOCKS = B_BYTES / 1024;
    static constexpr int A_PER_WAVE = A_BLOCKS / NWAVES, B_PER_WAVE = B_BLOCKS / NWAVES;
    static constexpr int LOADS = A_PER_WAVE + B_PER_WAVE;   // copies per wave per stage
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static_assert(A_PER_WAVE * NWAVES == A_BLOCKS && B_PER_WAVE * NWAVES == B_BLOCKS,
                  "tiles must split into whole 1 KiB blocks per wave");
    static_assert(CA == 4 || CA == 8, "block_k must be 32 or 64");
    static_assert(CB >= 16 && RB <= 1024, "block_n must be 128..512");
    static_assert(BK % KCH == 0 && NS % 2 == 0, "an even number of MFMA k-steps per stage");
    static_assert(STAGES >= 2 && STAGES * STAGE_BYTES <= 160 * 1024, "LDS budget");
    static_assert((STAGES - 1) * LOADS < 64, "vmcnt range");
};

// Main loop (per workgroup).  Iteration kt computes stage kt from slot
// kt % STAGES; for each k-step s it reads the fragments of step s+1 (two
// register sets alternate) while the MFMAs of step s run.  Barrier B(kt), in
// front of the last k-step's MFMAs, publishes stage kt+1 (each wave first
// waits for its own copies of it).  Copies only enter a slot whose reads
// every wave has completed, by one of two orders:
//   STAGES >= 3 (lagged ring): after B(kt) the copies of stage
//     kt+STAGES-1 go into slot (kt-1) % STAGES.  Every read of that slot
//     fed an MFMA of iteration kt-1, and a wave only reaches B(kt) after
//     those MFMAs have taken their operands (the register wait in front of
//     each MFMA), in the previous trip of the loop.  STAGES-2 stages are in
//     flight while one is computed.
//   STAGES == 2: the first MFMAs of the last k-step take every fragment of
//     slot kt's last read set; each wave then waits for all its LDS reads
//     (lgkmcnt 0) before B(kt), and the copies of stage kt+2 into slot kt
//     follow B(kt).
// Either way the ring's reuse is ordered by waits and the barrier, not by
// the latency of the copies.  Scheduling-group barriers interleave the LDS
// reads of the next k-step with the MFMAs of the current one.
template <int BM, int BN, int BK, int WM, int WN, int MI, int STAGES, bool BATCH = false>
__global__ void __launch_bounds__((BM / WM) * (BN / WN) * 64)
gemm_bf16_dma_kernel(GemmArgs p) {
    typedef Bf16DmaCfg<BM, BN, BK, WM, WN, MI, STAGES> G;
    typedef typename G::MF MF;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[STAGES * G::STAGE_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / G::NWN, wn = wave % G::NWN;
    const int lrow = lane % MI, lgrp = lane / MI;

    const int M = p.M, N = p.N, K = p.K;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, tiles_m, tiles_n, p.raster, p.xcd_remap, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    const i32x4 ra = make_rsrc(p.A, ((M - 1) * p.lda + K) * 2);
    const i32x4 rb = make_rsrc(BATCH ? p.b_of(blockIdx.y) : p.B, ((K - 1) * p.ldb + N) * 2);
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const unsigned smem_base = lds_address(smem);

    // Per-lane source coordinates of this wave's copy blocks (fixed over K).
    int a_row[G::A_PER_WAVE], a_col[G::A_PER_WAVE];
#pragma unroll
    for (int q = 0; q < G::A_PER_WAVE; ++q) {
        const int blk = wave * G::A_PER_WAVE + q;
        const int row = blk * (1024 / G::RA) + lane / G::CA;
        a_row[q] = row;
        a_col[q] = 8 * ((lane % G::CA) ^ swz_a<G::CA>(row));
    }
    int b_row[G::B_PER_WAVE], b_col[G::B_PER_WAVE];
#pragma unroll
    for (int q = 0; q < G::B_PER_WAVE; ++q) {
        const int blk = wave * G::B_PER_WAVE + q;
        const int row = blk * (1024 / G::RB) + lane / G::CB;
        b_row[q] = row;
        b_col[q] = 8 * ((lane % G::CB) ^ swz_b<MI>(row));
    }

    // Copies of one stage: prepare() computes the buffer offsets (out of
    // range, i.e. zero fill, for a stage past the end of K), fire() issues
    // them once the target slot is free.  Every stage index issues exactly
    // LOADS copies per wave, so the number of copies in flight is the same in
    // every iteration and one vmcnt value is exact throughout.
    int offA[G::A_PER_WAVE], offB[G::B_PER_WAVE];
    auto prepare = [&](int kt) {
        const int k0 = kt * BK;
#pragma unroll
        for (int q = 0; q < G::A_PER_WAVE; ++q) {
            const int gm = m0 + a_row[q], gk = k0 + a_col[q];
            offA[q] = (gm < M && gk < K) ? (gm * p.lda + gk) * 2 : kOOB;
        }
#pragma unroll
        for (int q = 0; q < G::B_PER_WAVE; ++q) {
            const int gk = k0 + b_row[q], gn = n0 + b_col[q];
            offB[q] = (gk < K && gn < N) ? (gk * p.ldb + gn) * 2 : kOOB;
        }
    };
    auto fire = [&](int st) {
        const unsigned base = smem_base + st * G::STAGE_BYTES;
#pragma unroll
        for (int q = 0; q < G::A_PER_WAVE; ++q)
            dma16(ra, base + (wave_u * G::A_PER_WAVE + q) * 1024, offA[q]);
#pragma unroll
        for (int q = 0; q < G::B_PER_WAVE; ++q)
            dma16(rb, base + G::A_BYTES + (wave_u * G::B_PER_WAVE + q) * 1024, offB[q]);
    };

    // Fragment addressing inside one stage (byte offsets).
    int a_off[G::TM], a_swz[G::TM];
#pragma unroll
    for (int i = 0; i < G::TM; ++i) {
        const int row = wm * WM + i * MI + lrow;
        a_off[i] = row * G::RA;
        a_swz[i] = swz_a<G::CA>(row);
    }
    const int rsub = (lane & 15) >> 2;  // transpose-read row inside the group of four
    // the rows this lane reads are kk + 8*lgrp + rsub (+ 4) with kk a multiple
    // of 16: == rsub (mod 4), with bit 3 equal to bit 0 of lgrp
    const int bsw = swz_b<MI>(8 * (lgrp & 1) + rsub);
    int b_chunk[G::TN];
#pragma unroll
    for (int j = 0; j < G::TN; ++j)
        b_chunk[j] = (((wn * WN + j * MI + (lrow & ~15) + 4 * (lane & 3)) >> 3) ^ bsw) * 16 +
                     8 * (lane & 1);

    typename MF::acc_t acc[G::TM][G::TN];
#pragma unroll
    for (int i = 0; i < G::TM; ++i)
#pragma unroll
        for (int j = 0; j < G::TN; ++j)
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) acc[i][j][r] = 0.f;

    u16x8 af[2][G::TM], bfr[2][G::TN];

    auto load_frags = [&](int st, int step, int buf) {
        const unsigned char *As = smem + st * G::STAGE_BYTES;
        const unsigned char *Bs = As + G::A_BYTES;
        const int kk = step * G::KCH;
#pragma unroll
        for (int i = 0; i < G::TM; ++i) {
            const int slot = ((kk >> 3) + lgrp) ^ a_swz[i];
            af[buf][i] = *reinterpret_cast<const u16x8 *>(As + a_off[i] + slot * 16);
        }
#pragma unroll
        for (int j = 0; j < G::TN; ++j) {
            const unsigned char *q0 = Bs + (kk + 8 * lgrp + rsub) * G::RB + b_chunk[j];
            const u16x4 lo = ds_read_tr16(reinterpret_cast<const unsigned short *>(q0));
            const u16x4 hi = ds_read_tr16(reinterpret_cast<const unsigned short *>(q0 + 4 * G::RB));
            bfr[buf][j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    };

    auto mfmas = [&](int buf) {
#pragma unroll
        for (int i = 0; i < G::TM; ++i)
#pragma unroll
            for (int j = 0; j < G::TN; ++j) acc[i][j] = MF::mma(af[buf][i], bfr[buf][j], acc[i][j]);
    };

    // The last k-step of a stage (lagged ring): its MFMAs with the copies
    // of the stage AHEAD ahead spread between them, so that the copies of
    // all waves do not queue at the texture unit at once right after the
    // barrier (which stalls the issuing waves, MFMAs included); the fences
    // keep the compiler from regrouping them.
    auto mfmas_with_copies = [&](int buf, int st) {
        const unsigned base = smem_base + st * G::STAGE_BYTES;
        constexpr int NM = G::TM * G::TN;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            acc[m / G::TN][m % G::TN] =
                MF::mma(af[buf][m / G::TN], bfr[buf][m % G::TN], acc[m / G::TN][m % G::TN]);
            const int q0 = m * G::LOADS / NM, q1 = (m + 1) * G::LOADS / NM;
            if (q1 > q0) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = q0; q < q1; ++q) {
                    if (q < G::A_PER_WAVE)
                        dma16(ra, base + (wave_u * G::A_PER_WAVE + q) * 1024, offA[q]);
                    else
                        dma16(rb, base + G::A_BYTES + (wave_u * G::B_PER_WAVE + q - G::A_PER_WAVE) * 1024,
                              offB[q - G::A_PER_WAVE]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // The last k-step of a stage in the two-slot ring, in two parts.  mfmas_head: the MFMAs of
    // the first A fragment against every B fragment.  They need the set's
    // last LDS read (the last B fragment), and LDS reads return in order, so
    // once they are issued every read of the slot being retired has
    // returned and the wave's lgkmcnt(0) wait in front of the barrier costs
    // nothing more.  mfmas_tail: the remaining MFMAs, with the copies of
    // the stage STAGES ahead spread between them, so that the copies of all
    // waves do not queue at the texture unit at once right after the
    // barrier (which stalls the issuing waves, MFMAs included); the fences
    // keep the compiler from regrouping them.
    auto mfmas_head = [&](int buf) {
#pragma unroll
        for (int j = 0; j < G::TN; ++j) acc[0][j] = MF::mma(af[buf][0], bfr[buf][j], acc[0][j]);
    };
    auto mfmas_tail = [&](int buf, int st) {
        const unsigned base = smem_base + st * G::STAGE_BYTES;
        constexpr int NM = (G::TM - 1) * G::TN;
        if constexpr (NM == 0) fire(st);  // one A fragment: the head was the whole step
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int i = 1 + m / G::TN, j = m % G::TN;
            acc[i][j] = MF::mma(af[buf][i], bfr[buf][j], acc[i][j]);
            const int q0 = m * G::LOADS / NM, q1 = (m + 1) * G::LOADS / NM;
            if (q1 > q0) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = q0; q < q1; ++q) {
                    if (q < G::A_PER_WAVE)
                        dma16(ra, base + (wave_u * G::A_PER_WAVE + q) * 1024, offA[q]);
                    else
                        dma16(rb, base + G::A_BYTES + (wave_u * G::B_PER_WAVE + q - G::A_PER_WAVE) * 1024,
                              offB[q - G::A_PER_WAVE]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // One MFMA followed by its share of the next step's LDS reads.
    auto interleave = [&]() {
        constexpr int NM = G::TM * G::TN;
        constexpr int ND = G::TM + 2 * G::TN;
        constexpr int PER = (ND + NM - 1) / NM;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
            if (m * PER < ND) __builtin_amdgcn_sched_group_barrier(0x100, PER, 0);  // DS read
        }
    };

    // The loop body is branch-free: the tail iterations copy zeros into
    // slots nobody reads any more and read fragments they do not use, which
    // keeps the compiler's LDS-wait analysis exact (no conservative waits at
    // control-flow merges in front of the last k-step's MFMAs).
    constexpr bool LAG = STAGES >= 3;
    constexpr int AHEAD = LAG ? STAGES - 1 : STAGES;   // stages copied before stage 0 is computed
    const int KT = (K + BK - 1) / BK;
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) {
        prepare(s);
        fire(s);
    }
    wait_vmcnt<(AHEAD - 1) * G::LOADS>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    load_frags(0, 0, 0);
    for (int kt = 0; kt < KT; ++kt) {
        const int st = kt % STAGES;
        prepare(kt + AHEAD);
#pragma unroll
        for (int s = 0; s + 1 < G::NS; ++s) {
            load_frags(st, s + 1, (s + 1) & 1);
            mfmas(s & 1);
            interleave();
        }
        if constexpr (LAG) {
            // stage kt+1 has landed (this wave's copies, then everyone's);
            // slot (kt-1) % STAGES was last read by iteration kt-1
            wait_vmcnt<(AHEAD - 2) * G::LOADS>();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            load_frags((kt + 1) % STAGES, 0, 0);
            mfmas_with_copies((G::NS - 1) & 1, (kt + AHEAD) % STAGES);
        } else {
            mfmas_head((G::NS - 1) & 1);
            // This wave's copies of stage kt+1 have landed and all its LDS
            // reads (the last ones of slot st) have returned; after the
            // barrier the same holds for every wave, so slot st is free and
            // stage kt+1 is visible.  The empty asm keeps every LDS read of
            // slot st in front of the wait.
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" ::: "memory");
            wait_vmcnt_and_lds<(STAGES - 2) * G::LOADS>();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            load_frags((kt + 1) % STAGES, 0, 0);
            mfmas_tail((G::NS - 1) & 1, st);
        }
    }
    wait_vmcnt<0>();  // no copy may still be writing LDS when the workgroup ends

    float *__restrict__ C = BATCH ? p.c_of(blockIdx.y) : p.C;
    const int ldc = p.ldc;
#pragma unroll
    for (int i = 0; i < G::TM; ++i)
#pragma unroll
        for (int j = 0; j < G::TN; ++j) {
            const int col = n0 + wn * WN + j * MI + lrow;
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) {
                const int row = m0 + wm * WM + i * MI + MF::row(lane, r);
                if (row < M && col < N)
                    __builtin_nontemporal_store((p.relu && acc[i][j][r] < 0.f) ? 0.f : acc[i][j][r],
                                                &C[row * ldc + col]);
            }
        }
}

// ---------------------------------------------------------------------------
// Register-fed reduction-split kernel (lds_stages = 0, k_split = KS) for
// products with few output tiles: few rows or columns, or all three extents
// small.  The LDS-staged kernels give 32x1000x2048 sixteen 64x64 tiles, each
// one serial chain of stages (29.3 us, 150 GB/s); here a 16*TM x 32 tile is
// shared by KS waves, wave g reducing the 32-k steps g, g + KS, ..., with the
// operands straight from memory to the 16x16x32 instruction's registers
// through a ring of D register buffers, so that a CU keeps KS*(D-1) steps of
// loads in flight (32x1000x2048: 5.4 us; 8 waves in place of 4 gain nothing,
// the loads of a CU being the limit).  No LDS, no barrier before the end.
//  - A: a lane's 8 consecutive k of its row, one 16-byte load;
//  - B is row-major, and the instruction wants 8 consecutive k of one column
//    per lane.  Lane c of 16 loads the dword of columns 2c, 2c + 1 of eight
//    rows (64 contiguous bytes per row), and the low halves make the fragment
//    of the even columns, the high halves that of the odd ones: two column
//    blocks per load, interleaved in C, no transpose;
//  - buffer loads need 4-byte alignment and are range-checked per dword.
//    ODD takes rows at any 2-byte boundary: A as the dwords that cover the
//    8 values, shifted by the row's parity, B as single values;
//  - A values past K (of the next row) are cleared in the fragments of the
//    last step, so that they do not multiply the zeros of B as infinities.
// The partial tiles are added through LDS in the order g = 0, 1, ..., KS-1.
template <int TM, int KS, int D, bool ODD>
__global__ void __launch_bounds__(KS * 64)
gemm_bf16_ksplit_kernel(GemmArgs p) {
    typedef Bf16Mfma<16> MF;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int BM = 16 * TM, BN = 32, BK = 32;
    constexpr int NREG = TM * 2 * 4;
    __shared__ float red[KS][NREG][64];

    const int lane = threadIdx.x & 63;
    const int g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lrow = lane & 15, lgrp = lane >> 4;
    const int M = p.M, N = p.N, K = p.K, lda = p.lda, ldb = p.ldb;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, tiles_m, tiles_n, p.raster, p.xcd_remap, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    // resources from the dword that holds the first element to the dword
    // that holds the last one
    const unsigned long long abase = reinterpret_cast<unsigned long long>(p.A);
    const unsigned long long bbase = reinterpret_cast<unsigned long long>(p.b_of(blockIdx.y));
    const int amis = ODD ? (int)(abase & 2) : 0, bmis = ODD ? (int)(bbase & 2) : 0;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void *>(abase - amis), 0, (amis + ((M - 1) * lda + K) * 2 + 3) & ~3, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void *>(bbase - bmis), 0, K > 0 ? (bmis + ((K - 1) * ldb + N) * 2 + 3) & ~3 : 0,
        0x00020000);
    unsigned aoff[TM];                 // byte offset of the lane's row (floored to a dword)
    unsigned ash[TM];                  // 2 where the row starts in the middle of a dword
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = m0 + i * 16 + lrow, o = amis + r * lda * 2;
        aoff[i] = r < M ? (unsigned)o & ~3u : (unsigned)kOOB;
        ash[i] = (unsigned)o & 2;
    }
    const int c0 = n0 + 2 * lrow;      // the lane's column pair
    const int boff = c0 < N ? bmis + c0 * 2 : kOOB;
    const int boff1 = c0 + 1 < N ? bmis + c0 * 2 + 2 : kOOB;   // (ODD)

    constexpr int NB = ODD ? 16 : 8;
    u32x4 fa[D][TM];
    unsigned fx[D][TM];                // (ODD) the dword after the 16 bytes
    unsigned fb[D][NB];
    auto load = [&](const int buf, const int kt) __attribute__((always_inline)) {
        const int kb = kt * BK + 8 * lgrp;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int off = kb < K ? (int)(aoff[i] + (unsigned)kb * 2u) : kOOB;
            fa[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(ra, off, 0, 0);
            if constexpr (ODD) fx[buf][i] = __builtin_amdgcn_raw_buffer_load_b32(ra, off, 16, 0);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            // unsigned: an out-of-range column plus a row offset stays past
            // the end (spans are below 2^31 - 48 bytes)
            const unsigned ro = (unsigned)min(kb + e, K) * (unsigned)ldb * 2u;
            if constexpr (ODD) {
                const bool ok = kb + e < K;   // the last dword may hold a value past the end
                fb[buf][2 * e] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(
                    rb, ok ? (int)(ro + (unsigned)boff) : kOOB, 0, 0);
                fb[buf][2 * e + 1] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(
                    rb, ok ? (int)(ro + (unsigned)boff1) : kOOB, 0, 0);
            } else {
                fb[buf][e] = __builtin_amdgcn_raw_buffer_load_b32(rb, (int)(ro + (unsigned)boff), 0, 0);
            }
        }
    };

    typename MF::acc_t acc[TM][2];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

    auto compute = [&](const int buf, const int kt) __attribute__((always_inline)) {
        u32x4 b[2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (ODD) {
                b[0][q] = fb[buf][4 * q] | (fb[buf][4 * q + 2] << 16);
                b[1][q] = fb[buf][4 * q + 1] | (fb[buf][4 * q + 3] << 16);
            } else {
                b[0][q] = (fb[buf][2 * q] & 0xffffu) | (fb[buf][2 * q + 1] << 16);
                b[1][q] = (fb[buf][2 * q] >> 16) | (fb[buf][2 * q + 1] & 0xffff0000u);
            }
        }
        const int left = K - (kt * BK + 8 * lgrp);          // k values left at this lane's 8
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            u32x4 a = fa[buf][i];
            if constexpr (ODD) {
                const unsigned w[5] = {a[0], a[1], a[2], a[3], fx[buf][i]};
#pragma unroll
                for (int q = 0; q < 4; ++q) a[q] = __builtin_amdgcn_alignbyte(w[q + 1], w[q], ash[i]);
            }
            if ((kt + 1) * BK > K) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    a[q] &= (2 * q < left ? 0xffffu : 0u) | (2 * q + 1 < left ? 0xffff0000u : 0u);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = MF::mma(__builtin_bit_cast(u16x8, a), __builtin_bit_cast(u16x8, b[j]), acc[i][j]);
        }
    };

    // D K-steps per iteration; steps past the end are loaded as zeros, so
    // that the wait counts stay exact, and not computed.
    const int KT = (K + BK - 1) / BK;
#pragma unroll
    for (int d = 0; d + 1 < D; ++d) load(d, g + d * KS);
    for (int base = g; base < KT; base += D * KS) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            load((d + D - 1) % D, base + (d + D - 1) * KS);
            if (d == 0 || base + d * KS < KT) compute(d, base + d * KS);
        }
    }

#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[g][(i * 4 + r) * 2 + j][lane] = acc[i][j][r];
    __syncthreads();
    float *__restrict__ C = p.c_of(blockIdx.y);
    const int ldc = p.ldc;
    for (int q = g; q < NREG / 2; q += KS) {       // register pair (i, r) of both column blocks
        float v0 = red[0][2 * q][lane], v1 = red[0][2 * q + 1][lane];
#pragma unroll
        for (int h = 1; h < KS; ++h) {
            v0 += red[h][2 * q][lane];
            v1 += red[h][2 * q + 1][lane];
        }
        const int row = m0 + (q >> 2) * 16 + 4 * lgrp + (q & 3);
        if (row < M) {
            float *c = C + row * ldc + c0;
            if (c0 < N) c[0] = (p.relu && v0 < 0.f) ? 0.f : v0;
            if (c0 + 1 < N) c[1] = (p.relu && v1 < 0.f) ? 0.f : v1;
        }
    }
}

template <int TM, int KS, int D, bool ODD>
hipError_t launch_bf16_ksplit(const GemmArgs &a, hipStream_t s) {
    const unsigned tiles = (unsigned)(((a.M + 16 * TM - 1) / (16 * TM)) * ((a.N + 31) / 32));
    GemmArgs args = a;
    void *kargs[] = {&args};
    return hipLaunchKernel(reinterpret_cast<const void *>(&gemm_bf16_ksplit_kernel<TM, KS, D, ODD>), dim3(tiles, (unsigned)a.batch),
                           dim3(KS * 64), kargs, 0, s);
}

template <int BM, int BN, int BK, int WM, int WN, int MI, int STAGES>
hipError_t launch_bf16_dma(const GemmArgs &a, hipStream_t s) {
    typedef Bf16DmaCfg<BM, BN, BK, WM, WN, MI, STAGES> G;
    const unsigned tiles = (unsigned)(((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN));
    GemmArgs args = a;
    void *kargs[] = {&args};
    // the batched form apart: in the plain one the two address products in
    // front of the main loop cost 8192^3 0.9% (850 -> 858 us)
    const void *fn = a.batch > 1
                         ? reinterpret_cast<const void *>(&gemm_bf16_dma_kernel<BM, BN, BK, WM, WN, MI, STAGES, true>)
                         : reinterpret_cast<const void *>(&gemm_bf16_dma_kernel<BM, BN, BK, WM, WN, MI, STAGES, false>);
    return hipLaunchKernel(fn, dim3(tiles, (unsigned)a.batch), dim3(G::NT), kargs, 0, s);
}

// ---------------------------------------------------------------------------
// Direct-to-LDS kernel for rows at any 2-byte boundary (odd row strides or
// bases).  Copies straight into LDS move whole dwords, so a row that starts in
// the middle of one lands one element late.  Fixing that on the way, through
// registers (two 16-byte loads, four lane shuffles and 15 selects and shifts
// per chunk), ran 2047x3001x1999 at 275 TFLOP/s (89.4 us); here both operands
// are copied as they lie, from the dword that holds their first element, and
// the shift is undone where it costs least (48.2 us; 1531x1021x2047 with 64-row
// tiles: 78.0 -> 24.0):
//  - A rows: a lane's row has one parity for the whole reduction; its 16
//    elements of a 32-k step are read with the dword after them and shifted
//    by v_alignbyte.  Rows hold a ninth 16-byte chunk per 64 k for that
//    dword; the 144-byte rows keep the fragment reads free of bank conflicts
//    without a swizzle (144/16 is odd);
//  - B rows: with an odd row stride the even and the odd k lie one column
//    apart.  The reduction keeps them apart instead: each instruction takes
//    either 16 even or 16 odd k (the fragments of a 32-k step are split by
//    parity with v_perm, the transpose reads step over every second row) and
//    has accumulators of its own.  The two sums of an element, one column
//    apart where their parities differ, meet at the end through LDS.  The
//    column that the shift costs is the tile's: 126 columns of output per
//    128 stored.
// Twice the accumulators of the aligned kernel, the same matrix instructions
// per FLOP.  Two LDS slots; barriers on both sides of a stage's reads, hidden by
// the CU's second workgroup where it has one: 2047x3001x1999 has 384 tiles for
// 256 CUs, and its counters show the matrix cores busy 19% of the launch, LDS
// 16%, and of a wave's life 26% vector instructions (shifts and permutes), 34%
// waits to issue and the rest waits for copies and at barriers.
template <int BM, int WM>
struct Bf16OddCfg {
    static constexpr int BN = 128, WN = 64, BK = 64, MI = 32, NOUT = BN - 2;
    static constexpr int NWN = BN / WN, NWAVES = (BM / WM) * NWN, NT = NWAVES * 64;
    static constexpr int TM = WM / MI, TN = WN / MI;
    static constexpr int RA = BK * 2 + 16, RB = BN * 2;             // LDS row bytes
    static constexpr int NA = (BM * RA / 1024 + NWAVES - 1) / NWAVES, NBC = BK * RB / 1024 / NWAVES;
    static constexpr int A_BYTES = NA * NWAVES * 1024, B_BYTES = BK * RB;
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES, LOADS = NA + NBC;
    static constexpr int LDS_BYTES = 2 * STAGE_BYTES > BM * BN * 4 ? 2 * STAGE_BYTES : BM * BN * 4;
    static_assert(BM * RA % 1024 == 0 && NBC * NWAVES * 1024 == B_BYTES, "whole copy blocks");
};

template <int BM, int WM>
__global__ void __launch_bounds__((BM / WM) * 128)
gemm_bf16_odd_kernel(GemmArgs p) {
    typedef Bf16OddCfg<BM, WM> G;
    typedef Bf16Mfma<32> MF;
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int TM = G::TM, TN = G::TN, BK = G::BK;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[G::LDS_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / G::NWN, wn = wave % G::NWN;
    const int l32 = lane & 31, lgrp = lane >> 5;
    const int M = p.M, N = p.N, K = p.K, lda = p.lda, ldb = p.ldb;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + G::NOUT - 1) / G::NOUT;
    int tm, tn;
    tile_coords(blockIdx.x, gridDim.x, tiles_m, tiles_n, p.raster, p.xcd_remap, tm, tn);
    const int m0 = tm * BM, n0 = tn * G::NOUT;   // n0 is even

    // resources from the dword that holds the first element to the one that
    // holds the last
    const unsigned long long abase = reinterpret_cast<unsigned long long>(p.A);
    const unsigned long long bbase = reinterpret_cast<unsigned long long>(p.b_of(blockIdx.y));
    const int amis = (int)(abase & 2), bmis = (int)(bbase & 2);
    const i32x4 ra = make_rsrc(reinterpret_cast<const void *>(abase - amis),
                               (amis + ((M - 1) * lda + K) * 2 + 3) & ~3);
    const i32x4 rb = make_rsrc(reinterpret_cast<const void *>(bbase - bmis),
                               K > 0 ? (bmis + ((K - 1) * ldb + N) * 2 + 3) & ~3 : 0);
    const unsigned smem_base = lds_address(smem);

    // copies: A unit v is row v / 9, chunk v % 9; B unit v is row v / 16,
    // LDS slot v % 16, holding chunk slot ^ swz(row)
    int aoff[G::NA], ak[G::NA];
#pragma unroll
    for (int q = 0; q < G::NA; ++q) {
        const int v = (wave * G::NA + q) * 64 + lane, row = v / 9, c = v - row * 9;
        ak[q] = 8 * c - 1;                        // first k the chunk can hold, less than K if any does
        aoff[q] = row < BM && m0 + row < M ? ((amis + (m0 + row) * lda * 2) & ~3) + 16 * c : kOOB;
    }
    int brow[G::NBC], bcol[G::NBC];
#pragma unroll
    for (int q = 0; q < G::NBC; ++q) {
        const int v = (wave * G::NBC + q) * 64 + lane;
        brow[q] = v >> 4;
        bcol[q] = bmis + (n0 + 8 * ((v & 15) ^ swz_b<32>(brow[q] >> 1))) * 2;
    }
    auto fire = [&](int kt, int st) __attribute__((always_inline)) {
        const unsigned base = smem_base + st * G::STAGE_BYTES;
        const int k0 = kt * BK;
#pragma unroll
        for (int q = 0; q < G::NA; ++q)
            dma16(ra, base + (wave * G::NA + q) * 1024, aoff[q] != kOOB && k0 + ak[q] < K ? aoff[q] + k0 * 2 : kOOB);
#pragma unroll
        for (int q = 0; q < G::NBC; ++q) {
            const int k = k0 + brow[q];
            // the dword of the chunk's first element; a chunk past column N
            // may read the next row (columns that are not stored)
            dma16(rb, base + G::A_BYTES + (wave * G::NBC + q) * 1024,
                  k < K ? (k * ldb * 2 + bcol[q]) & ~3 : kOOB);
        }
    };

    // fragment addresses
    int a_base[TM];
    unsigned ash[TM];                             // 2: the row starts in the middle of a dword
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int row = wm * WM + i * 32 + l32;
        a_base[i] = row * G::RA + 32 * lgrp;
        ash[i] = (unsigned)(amis + (m0 + row) * lda * 2) & 2;
    }
    const int rsub = (lane & 15) >> 2;
    int b_base[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = wn * G::WN + j * 32 + (l32 & ~15) + 4 * (lane & 3);
        b_base[j] = G::A_BYTES + (16 * lgrp + 2 * rsub) * G::RB + (((col >> 3) ^ swz_b<32>(rsub)) << 4) + 8 * (lane & 1);
    }

    typename MF::acc_t acc[2][TM][TN];            // even k, odd k
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < MF::NACC; ++r) acc[o][i][j][r] = 0.f;

    u32x4 aw[2][TM][2];
    unsigned ax[2][TM];
    u16x8 bf[2][2][TN];
    auto frags = [&](int st, int ds, int fb) __attribute__((always_inline)) {
        const unsigned char *S = smem + st * G::STAGE_BYTES;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const unsigned char *q = S + a_base[i] + ds * 64;
            aw[fb][i][0] = *reinterpret_cast<const u32x4 *>(q);
            aw[fb][i][1] = *reinterpret_cast<const u32x4 *>(q + 16);
            ax[fb][i] = *reinterpret_cast<const unsigned *>(q + 32);
        }
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const unsigned char *q = S + b_base[j] + (32 * ds + o) * G::RB;
                const u16x4 lo = ds_read_tr16(reinterpret_cast<const unsigned short *>(q));
                const u16x4 hi = ds_read_tr16(reinterpret_cast<const unsigned short *>(q + 8 * G::RB));
                bf[fb][o][j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
    };
    auto mfmas = [&](int fb, int left) __attribute__((always_inline)) {
        // left: k values left at this lane's 16
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            unsigned x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const unsigned lo = aw[fb][i][e >> 2][e & 3];
                const unsigned hi = e < 7 ? aw[fb][i][(e + 1) >> 2][(e + 1) & 3] : ax[fb][i];
                x[e] = __builtin_amdgcn_alignbyte(hi, lo, ash[i]);
            }
            if (__builtin_expect(left < 16, 0)) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    x[e] &= (2 * e < left ? 0xffffu : 0u) | (2 * e + 1 < left ? 0xffff0000u : 0u);
            }
            u32x4 ev, od;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                ev[q] = __builtin_amdgcn_perm(x[2 * q + 1], x[2 * q], 0x05040100u);
                od[q] = __builtin_amdgcn_perm(x[2 * q + 1], x[2 * q], 0x07060302u);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[0][i][j] = MF::mma(__builtin_bit_cast(u16x8, ev), bf[fb][0][j], acc[0][i][j]);
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[1][i][j] = MF::mma(__builtin_bit_cast(u16x8, od), bf[fb][1][j], acc[1][i][j]);
        }
    };

    const int KT = (K + BK - 1) / BK;
    fire(0, 0);
    fire(1, 1);
    for (int kt = 0; kt < KT; ++kt) {
        const int st = kt & 1;
        wait_vmcnt<G::LOADS>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int left = K - kt * BK - 16 * lgrp;
        frags(st, 0, 0);
        frags(st, 1, 1);
        mfmas(0, left);
        mfmas(1, left - 32);
        // every read of the slot has fed an instruction of this wave; after
        // the barrier that holds for all waves
        asm volatile("" ::: "memory");
        wait_vmcnt_and_lds<G::LOADS>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        fire(kt + 2, st);
    }
    wait_vmcnt<0>();  // no copy may still be writing LDS when it is reused or the workgroup ends
    __syncthreads();

    // position c of an even (odd) k row holds column n0 + c - pe (po)
    const int pe = (bmis >> 1) & 1, po = ((bmis >> 1) + ldb) & 1;
    float *red = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r)
                red[(wm * WM + i * 32 + MF::row(lane, r)) * G::BN + wn * G::WN + j * 32 + l32] = acc[1][i][j][r];
    __syncthreads();
    float *__restrict__ C = p.c_of(blockIdx.y);
    const int ldc = p.ldc;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int c = wn * G::WN + j * 32 + l32 - pe, col = n0 + c;
            const bool ok = c >= 0 && c < G::NOUT && col < N;
#pragma unroll
            for (int r = 0; r < MF::NACC; ++r) {
                const int lr = wm * WM + i * 32 + MF::row(lane, r), row = m0 + lr;
                if (ok && row < M) {
                    const float v = acc[0][i][j][r] + red[lr * G::BN + c + po];
                    C[row * ldc + col] = (p.relu && v < 0.f) ? 0.f : v;
                }
            }
        }
}

template <int BM, int WM>
hipError_t launch_bf16_odd(const GemmArgs &a, hipStream_t s) {
    typedef Bf16OddCfg<BM, WM> G;
    const unsigned tiles = (unsigned)(((a.M + BM - 1) / BM) * ((a.N + G::NOUT - 1) / G::NOUT));
    GemmArgs args = a;
    void *kargs[] = {&args};
    return hipLaunchKernel(reinterpret_cast<const void *>(&gemm_bf16_odd_kernel<BM, WM>), dim3(tiles, (unsigned)a.batch), dim3(G::NT),
                           kargs, 0, s);
}

template <int BM, int BN, int BK, int WM, int WN, int MI, int PAD, bool VEC>
hipError_t launch_bf16(const GemmArgs &a, hipStream_t s) {
    typedef GemmBf16Cfg<BM, BN, BK, WM, WN, MI, PAD, VEC> G;
    const unsigned tiles = (unsigned)(((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN));
    GemmArgs args = a;
    void *kargs[] = {&args};
    return hipLaunchKernel(
        reinterpret_cast<const void *>(&gemm_bf16_kernel<BM, BN, BK, WM, WN, MI, PAD, VEC>),
        dim3(tiles, (unsigned)a.batch), dim3(G::NT), kargs, 0, s);
}

// Rows at any 2-byte boundary, for the direct-to-LDS instances.  The odd-row
// kernel reduces faster, but its tiles of 126 columns write C in pieces of
// lines, and 17 of them cover what 16 of 128 columns do: short reductions stay
// with the register-staged kernel of the same tile.  Both times in us, from
// rounds of 256 tiles (28 shapes from 777x1500 to 8192^2, K = 1 to 1025; within
// 15%): 4096x4096x1 28.4 with the odd-row kernel, 14.3; x65 31.6, 18.1; x1025
// 75.6, 75.7; 2048x2047x129 15.0, 12.0; x513 21.3, 24.6; 1531x1021x65 7.3, 6.1;
// x257 8.8, 9.8.
template <int BM>
hipError_t launch_bf16_unaligned(const GemmArgs &a, hipStream_t s) {
    auto rounds = [&](int bm, int bn) {
        const long long t = (long long)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn) * a.batch;
        return (double)((t + 255) / 256);
    };
    if constexpr (BM == 64) {
        // (of the register-staged tiles the small one up to three per CU:
        // 1001x3003x1 6.4 us, 7.0 with 64x128; 1900x2040x1 8.0, 7.2; two of the
        // others share a CU, so the 126 columns cost a round where they need a
        // third: 3000x1280x129 14.1, 11.3; x385 18.7, 19.1)
        const bool third = rounds(64, 126) > 2 && rounds(64, 128) <= 2;
        if (a.K > (third ? 320 : 128)) return launch_bf16_odd<64, 32>(a, s);
        return rounds(64, 64) <= 3 ? launch_bf16<64, 64, 64, 32, 32, 32, 8, false>(a, s)
                                   : launch_bf16<64, 128, 64, 32, 64, 32, 8, false>(a, s);
    } else {
        const double n = rounds(128, 126), r = rounds(BM, BM);
        const double odd = n == 1 ? 10.5 + .0135 * a.K : 3 + n * (5 + .009 * a.K);
        if constexpr (BM == 256) {
            if (1 + r * (11 + .0605 * a.K) < odd) return launch_bf16<256, 256, 32, 128, 64, 32, 8, false>(a, s);
        } else {
            if (4 + 3 * r + a.K * (r <= 2 ? .04 : r == 3 ? .053 : .021 * r) < odd)
                return launch_bf16<128, 128, 32, 64, 64, 32, 8, false>(a, s);
        }
        return launch_bf16_odd<128, 64>(a, s);
    }
}

// The same for the register-fed instances: 2-byte loads of B against two
// 64-k steps of the register-staged kernel (101x203x33 4.3 us, 3.8; x65 4.3,
// 4.6), or three where its tiles outnumber the CUs (40000x3x129 11.1, 8.1;
// 31x20000x257 9.2, 9.2; 1000000x1x16 128, 58).
template <int TM, int KS, int D>
hipError_t launch_bf16_ksplit_odd(const GemmArgs &a, hipStream_t s) {
    const long long tiles = (long long)((a.M + 63) / 64) * ((a.N + 63) / 64) * a.batch;
    if (a.K <= (tiles > 256 ? 192 : 64)) return launch_bf16<64, 64, 64, 32, 32, 32, 8, false>(a, s);
    return launch_bf16_ksplit<TM, KS, D, true>(a, s);
}

#define XTC_BF16_INSTANCE(BM, BN, BK, WM, WN, MI, PAD)                                        \
    GemmInstance {                                                                            \
        make_sched(BM, BN, BK, WM, WN, MI, MI, (MI == 32 ? 16 : 32), 2, PAD, 0),               \
            &launch_bf16<BM, BN, BK, WM, WN, MI, PAD, true>,                                  \
            &launch_bf16<BM, BN, BK, WM, WN, MI, PAD, false>, kRowsAligned,                   \
            &occupancy_of<&gemm_bf16_kernel<BM, BN, BK, WM, WN, MI, PAD, true>,               \
                          (BM / WM) * (BN / WN) * 64, 0>                                      \
    }

// Direct-to-LDS ring (lds_pad = -1: swizzled, unpadded LDS rows), b128 A
// reads, MFMA / LDS-read interleaving.  Unaligned or non-16-byte-granular
// operands run the kernel for rows at any 2-byte boundary, with 128- or
// 64-row tiles, or for short reductions the register-staged one.
#define XTC_BF16_DMA_INSTANCE(BM, BN, BK, WM, WN, MI, STAGES)                                 \
    GemmInstance {                                                                            \
        make_sched(BM, BN, BK, WM, WN, MI, MI, (MI == 32 ? 16 : 32), STAGES, -1, 0),           \
            &launch_bf16_dma<BM, BN, BK, WM, WN, MI, STAGES>,                                 \
            &launch_bf16_unaligned<BM>, kWholeChunks,                                         \
            &occupancy_of<&gemm_bf16_dma_kernel<BM, BN, BK, WM, WN, MI, STAGES>,              \
                          (BM / WM) * (BN / WN) * 64, 0>                                      \
    }

// Register-fed reduction split: KS waves per 16*TM x 32 tile, D steps in
// flight; the ODD form for rows off a 4-byte boundary.
#define XTC_BF16_KSPLIT_INSTANCE(TM, KS, D)                                                   \
    GemmInstance {                                                                            \
        make_sched(16 * TM, 32, 32, 16 * TM, 32, 16, 16, 32, 0, 0, 0, 0, KS),                  \
            &launch_bf16_ksplit<TM, KS, D, false>, &launch_bf16_ksplit_odd<TM, KS, D>,        \
            kRowsDword, &occupancy_of<&gemm_bf16_ksplit_kernel<TM, KS, D, false>, KS * 64, 0> \
    }

const GemmInstance kBf16Instances[] = {
    XTC_BF16_DMA_INSTANCE(256, 256, 32, 128, 64, 32, 4),  // default for large problems
    XTC_BF16_DMA_INSTANCE(256, 256, 64, 128, 64, 32, 2),
    XTC_BF16_DMA_INSTANCE(256, 256, 64, 128, 128, 32, 2), // 4 waves of 128x128
    XTC_BF16_DMA_INSTANCE(256, 128, 32, 128, 64, 32, 4),
    XTC_BF16_DMA_INSTANCE(128, 128, 32, 64, 64, 32, 4),   // medium problems
    XTC_BF16_DMA_INSTANCE(64, 128, 32, 32, 64, 32, 4),
    XTC_BF16_DMA_INSTANCE(64, 128, 64, 32, 64, 32, 2),
    XTC_BF16_DMA_INSTANCE(128, 128, 64, 64, 64, 16, 2),
    XTC_BF16_KSPLIT_INSTANCE(1, 4, 3),   // 16x32 tiles: few rows
    XTC_BF16_KSPLIT_INSTANCE(2, 4, 3),   // 32x32 tiles
    XTC_BF16_KSPLIT_INSTANCE(4, 4, 3),   // 64x32 tiles
    XTC_BF16_INSTANCE(256, 256, 64, 128, 64, 32, 8),
    XTC_BF16_INSTANCE(128, 128, 64, 64, 64, 32, 8),
    XTC_BF16_INSTANCE(64, 64, 64, 32, 32, 32, 8),         // small problems
    XTC_BF16_INSTANCE(128, 128, 64, 64, 64, 16, 8),       // 16x16x32 instruction tile
};

}  // namespace

const GemmInstance *gemm_bf16_instances(int *count) {
    *count = (int)(sizeof(kBf16Instances) / sizeof(kBf16Instances[0]));
    return kBf16Instances;
}

}  // namespace xtc
