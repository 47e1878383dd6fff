// rom_contract_planes.hip -- the dense kernels' contraction S = sigma_s (P^T Psi') + q on the row-scan
// sweep's layout: a plane of ld cells per ordinate for the source, S[N][ld]; for the weighted angular flux
// Psi'[K / 4][ld][4] in BF16 or Psi'[K][ld] in FP64.  P^T comes in pieces of 16 bytes, [K / 8][N][8] in
// BF16 and [K / 2][N][2] in FP64, so a K step reads it contiguously (rows of K ordinates, K a power of
// two, put every row's piece on the same two L2 channels: 226 us at 65536 cells and 1024 ordinates).
// N and K are multiples of 32 (padding: zero rows and columns of P^T, zero planes of Psi').
//
// P^T is the left operand, so a lane's results of one matrix instruction are one cell of several
// ordinates and 32 (BF16) or 16 (FP64) lanes store consecutive cells of a plane.  Both operands go
// through LDS, two buffers deep: at the top of K step k the registers holding step k + 1 are written
// to the other buffer and the loads of step k + 2 issued; one barrier per step.
#include "rom_common.h"

namespace rom {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef double f64x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));

// Tile of block `blk`: the N tiles of one cell run are consecutive, and in single launches each XCD
// (workgroups go round-robin over the 8) owns a contiguous run of tiles, so a run of Psi' is read from
// memory once and P^T stays in every XCD's L2.
__device__ __forceinline__ int2 plane_tile(const ContractArgs& A, int BN, int blk, int nb)
{
    const int nn = (A.N + BN - 1) / BN;
    const int lb = nb % 8 == 0 ? (blk % 8) * (nb / 8) + blk / 8 : blk;
    return make_int2(lb / nn, lb % nn);
}

constexpr int kPM = 128;   // cells of a BF16 tile
constexpr int kPK = 32;    // its K step

// 256 threads = 4 waves as WN x (4 / WN); BN x 128 tile of 32x32x16 BF16 matrix instructions.
// Sources that the 256 MB cache cannot keep for the sweep anyway are stored past it (STREAM):
// 65536 cells x 1024 ordinates 210 -> 168 us (818 TFLOP/s; 256 x 256 tiles on row-major operands 172);
// with 512 ordinates, which it keeps, 48 us against 53.
template <int BN, int WN, bool STREAM>
__device__ __forceinline__ void planes_bf16_tile(const ContractArgs& A, const int blk, const int nb)
{
    if (A.sysctl && A.sysctl[A.sys_index].state != 0) return;
    constexpr int WM = 4 / WN, TN = BN / WN / 32, TM = kPM / WM / 32;
    constexpr int HB = BN * kPK / 8 / 256, HP = kPM * kPK / 8 / 256;   // 16-byte pieces per thread
    __shared__ u32x4_t Bs[2][kPK / 8][BN];
    __shared__ __attribute__((aligned(16))) uint2 Ps[2][kPK / 4][kPM];
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int wn = wave / WM, wm = wave % WM, half = lane / 32, l32 = lane % 32;
    const int2 tile = plane_tile(A, BN, blk, nb);
    const int m0 = tile.x * kPM, n0 = tile.y * BN;
    const int M = A.M, N = A.N, K = A.K, ld = A.ld;

    f32x16_t acc[TN][TM];
#pragma unroll
    for (int x = 0; x < TN; ++x)
#pragma unroll
        for (int y = 0; y < TM; ++y)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.0f;

    // rows past N and cells past M read the last one; their results are not stored.  A piece of Psi' is
    // two cells, the second possibly one past the plane (its padding, or the pool's).
    const u32x4_t* pb[HB];
    const uint2* pp[HP];
#pragma unroll
    for (int h = 0; h < HB; ++h) {
        const int e = tid + 256 * h;
        pb[h] = (const u32x4_t*)A.bt + (int64_t)(e / BN) * N + min(n0 + e % BN, N - 1);
    }
#pragma unroll
    for (int h = 0; h < HP; ++h) {
        const int e = tid + 256 * h;
        pp[h] = (const uint2*)A.a + (int64_t)(e / (kPM / 2)) * ld + min(m0 + e % (kPM / 2) * 2, M - 1);
    }
    u32x4_t rb0[HB], rb1[HB], rp0[HP], rp1[HP];   // even and odd K steps
    auto load = [&](u32x4_t (&rb)[HB], u32x4_t (&rp)[HP]) {
#pragma unroll
        for (int h = 0; h < HB; ++h) {
            rb[h] = *pb[h];
            pb[h] += (int64_t)(kPK / 8) * N;
        }
#pragma unroll
        for (int h = 0; h < HP; ++h) {
            rp[h] = *(const u32x4_a8*)pp[h];
            pp[h] += (int64_t)(kPK / 4) * ld;
        }
    };
    auto stage = [&](const int buf, const u32x4_t (&rb)[HB], const u32x4_t (&rp)[HP]) {
#pragma unroll
        for (int h = 0; h < HB; ++h) {
            const int e = tid + 256 * h;
            Bs[buf][e / BN][e % BN] = rb[h];
        }
#pragma unroll
        for (int h = 0; h < HP; ++h) {
            const int e = tid + 256 * h;
            *(u32x4_t*)&Ps[buf][e / (kPM / 2)][e % (kPM / 2) * 2] = rp[h];
        }
    };
    const int nk = K / kPK;
    // step ks: the operands of step ks + 1 into LDS, the loads of step ks + 3, the matrix work
    auto step = [&](const int ks, const int cur, u32x4_t (&rb)[HB], u32x4_t (&rp)[HP]) {
        if (ks + 1 < nk) {
            stage(cur ^ 1, rb, rp);
            if (ks + 3 < nk) load(rb, rp);
        }
#pragma unroll
        for (int kk = 0; kk < kPK / 16; ++kk) {
            bf16x8_t a[TN], b[TM];
#pragma unroll
            for (int x = 0; x < TN; ++x) a[x] = __builtin_bit_cast(bf16x8_t, Bs[cur][kk * 2 + half][(wn * TN + x) * 32 + l32]);
#pragma unroll
            for (int y = 0; y < TM; ++y) {
                const uint2 lo = Ps[cur][kk * 4 + half * 2][(wm * TM + y) * 32 + l32];
                const uint2 hi = Ps[cur][kk * 4 + half * 2 + 1][(wm * TM + y) * 32 + l32];
                b[y] = __builtin_bit_cast(bf16x8_t, (u32x4_t){lo.x, lo.y, hi.x, hi.y});
            }
#pragma unroll
            for (int x = 0; x < TN; ++x)
#pragma unroll
                for (int y = 0; y < TM; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[x], b[y], acc[x][y], 0, 0, 0);
        }
        __syncthreads();
    };
    load(rb0, rp0);
    stage(0, rb0, rp0);
    if (nk > 1) load(rb1, rp1);
    if (nk > 2) load(rb0, rp0);
    __syncthreads();
    for (int ks = 0; ks < nk; ks += 2) {
        step(ks, 0, rb1, rp1);
        if (ks + 1 < nk) step(ks + 1, 1, rb0, rp0);
    }
    // a lane holds column lane % 32 and rows 8 (e / 4) + 4 (lane / 32) + e % 4 of each 32 x 32 tile
#pragma unroll
    for (int y = 0; y < TM; ++y) {
        const int m = m0 + (wm * TM + y) * 32 + l32;
        if (m < M) {
            const float ss = ((const float*)A.sigma_s)[m], q = ((const float*)A.q)[m];
#pragma unroll
            for (int x = 0; x < TN; ++x) {
                const int n = n0 + (wn * TN + x) * 32;
                if (n < N) {
                    float* const out = (float*)A.out + (int64_t)(n + 4 * half) * ld + m;
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        float* const to = out + (int64_t)(8 * (e / 4) + e % 4) * ld;
                        const float v = fmaf(ss, acc[x][y][e], q);
                        if constexpr (STREAM) __builtin_nontemporal_store(v, to);
                        else *to = v;
                    }
                }
            }
        }
    }
}

// FP64: 64 x 64 tile, K step 16, 4 waves of 32 x 32 = 2 x 2 16x16x4 FP64 matrix instructions (7680 cells x
// 144 ordinates: 20 us, where the kernel without matrix instructions, on 256 padded ones, took 88; x 512:
// 78 us, 51 TFLOP/s, where a large FP64 product reaches 69).
constexpr int kDT = 64, kDK = 16, kDP = 80;   // LDS rows of 640 bytes: two rows of K on different bank halves
__device__ __forceinline__ void planes_f64_tile(const ContractArgs& A, const int blk, const int nb)
{
    if (A.sysctl && A.sysctl[A.sys_index].state != 0) return;
    __shared__ __attribute__((aligned(16))) double Bs[2][kDK][kDP];
    __shared__ __attribute__((aligned(16))) double Ps[2][kDK][kDP];
    typedef double D2 __attribute__((ext_vector_type(2)));
    typedef double D2u __attribute__((ext_vector_type(2), aligned(8)));
    constexpr int H = kDT * kDK / 2 / 256;
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const int wn = wave / 2, wm = wave % 2, l16 = lane % 16, l4 = lane / 16;
    const int2 tile = plane_tile(A, kDT, blk, nb);
    const int m0 = tile.x * kDT, n0 = tile.y * kDT;
    const int M = A.M, N = A.N, K = A.K, ld = A.ld;
    f64x4_t acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    const double *pb[H], *pp[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        const int e = tid + 256 * h;
        pb[h] = (const double*)A.bt + ((int64_t)(e / kDT) * N + min(n0 + e % kDT, N - 1)) * 2;
        pp[h] = (const double*)A.a + (int64_t)(e / (kDT / 2)) * ld + min(m0 + e % (kDT / 2) * 2, M - 1);
    }
    const int64_t kstep = (int64_t)kDK * ld;
    D2 rb0[H], rp0[H], rb1[H], rp1[H];   // odd and even K steps
    auto load = [&](D2 (&rb)[H], D2 (&rp)[H]) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            rb[h] = *(const D2*)pb[h];
            pb[h] += (int64_t)kDK * N;
            rp[h] = *(const D2u*)pp[h];
            pp[h] += kstep;
        }
    };
    auto stage = [&](const int buf, const D2 (&rb)[H], const D2 (&rp)[H]) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const int e = tid + 256 * h;
            Bs[buf][e / kDT * 2][e % kDT] = rb[h][0];
            Bs[buf][e / kDT * 2 + 1][e % kDT] = rb[h][1];
            *(D2*)&Ps[buf][e / (kDT / 2)][e % (kDT / 2) * 2] = rp[h];
        }
    };
    const int nk = K / kDK;
    load(rb0, rp0);
    stage(0, rb0, rp0);
    if (nk > 1) load(rb1, rp1);
    if (nk > 2) load(rb0, rp0);
    __syncthreads();
    auto step = [&](const int ks, const int cur, D2 (&rb)[H], D2 (&rp)[H]) {
        if (ks + 1 < nk) {
            stage(cur ^ 1, rb, rp);
            if (ks + 3 < nk) load(rb, rp);
        }
#pragma unroll
        for (int k = 0; k < kDK; k += 4) {
            double a[2], b[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                a[x] = Bs[cur][k + l4][wn * 32 + x * 16 + l16];
                b[x] = Ps[cur][k + l4][wm * 32 + x * 16 + l16];
            }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], b[y], acc[x][y], 0, 0, 0);
        }
        __syncthreads();
    };
    for (int ks = 0; ks < nk; ks += 2) {
        step(ks, 0, rb1, rp1);
        if (ks + 1 < nk) step(ks + 1, 1, rb0, rp0);
    }
    // a lane holds column lane % 16 and rows lane / 16 + 4 e of each 16 x 16 tile
#pragma unroll
    for (int y = 0; y < 2; ++y) {
        const int m = m0 + wm * 32 + y * 16 + l16;
        if (m < M) {
            const double ss = ((const double*)A.sigma_s)[m], q = ((const double*)A.q)[m];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int n = n0 + wn * 32 + x * 16 + l4 + 4 * e;
                    if (n < N) ((double*)A.out)[(int64_t)n * ld + m] = fma(ss, acc[x][y][e], q);
                }
            }
        }
    }
}

template <int KIND>
__device__ __forceinline__ void planes_tile(const ContractArgs& A, const int blk, const int nb)
{
    constexpr bool S = KIND >= kContractStream;
    if constexpr (KIND % kContractStream == kContractPlanes64) planes_bf16_tile<64, 1, S>(A, blk, nb);
    else if constexpr (KIND % kContractStream == kContractPlanes128) planes_bf16_tile<128, 2, S>(A, blk, nb);
    else if constexpr (KIND % kContractStream == kContractPlanes256) planes_bf16_tile<256, 2, S>(A, blk, nb);
    else planes_f64_tile(A, blk, nb);
}

// The contraction precedes a sweep and clears its start mark: the sweep is timed from itself.
template <int KIND>
__global__ __launch_bounds__(256, 2) void planes_kernel(ContractArgs A, Ctl* ctl)
{
    if (ctl && ctl->active == 0) return;
    if (ctl && blockIdx.x == 0 && threadIdx.x == 0) ctl->t_mark = ~0ull;
    planes_tile<KIND>(A, blockIdx.x, gridDim.x);
}

// Several systems in one launch: block b computes tile map[b].y of contraction map[b].x.
template <int KIND>
__global__ __launch_bounds__(256, 2) void planes_batch_kernel(const ContractArgs* __restrict__ items, const int2* __restrict__ map, Ctl* ctl)
{
    if (ctl && ctl->active == 0) return;
    if (ctl && blockIdx.x == 0 && threadIdx.x == 0) ctl->t_mark = ~0ull;
    const int2 m = map[blockIdx.x];
    planes_tile<KIND>(items[m.x], m.y, 1);
}

}  // namespace

int planes_blocks(const ContractArgs& a, int kind)
{
    if (a.M < 1 || a.N < 1 || a.ld < a.M || a.N % kPK != 0 || a.K % kPK != 0) return -1;
    const int tile = kind % kContractStream, bn = tile == kContractPlanes128 ? 128 : tile == kContractPlanes256 ? 256 : 64;
    const int bm = kind == kContractPlanesF64 ? kDT : kPM;
    return ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn);
}

#define ROM_PLANES_CASE(KIND, KERNEL, BLOCKS, ...) \
    case KIND: hipLaunchKernelGGL(KERNEL<KIND>, dim3(BLOCKS), dim3(256), 0, s, __VA_ARGS__); break;
#define ROM_PLANES(KERNEL, BLOCKS, ...)                                               \
    switch (kind) {                                                                   \
        ROM_PLANES_CASE(kContractPlanes64, KERNEL, BLOCKS, __VA_ARGS__)               \
        ROM_PLANES_CASE(kContractPlanes128, KERNEL, BLOCKS, __VA_ARGS__)              \
        ROM_PLANES_CASE(kContractPlanes256, KERNEL, BLOCKS, __VA_ARGS__)              \
        ROM_PLANES_CASE(kContractPlanesF64, KERNEL, BLOCKS, __VA_ARGS__)              \
        ROM_PLANES_CASE(kContractPlanes64 + kContractStream, KERNEL, BLOCKS, __VA_ARGS__)  \
        ROM_PLANES_CASE(kContractPlanes128 + kContractStream, KERNEL, BLOCKS, __VA_ARGS__) \
        ROM_PLANES_CASE(kContractPlanes256 + kContractStream, KERNEL, BLOCKS, __VA_ARGS__) \
    default: return hipErrorInvalidValue;                                             \
    }                                                                                 \
    return hipGetLastError();

hipError_t launch_planes(const ContractArgs& a, int kind, hipStream_t s, Ctl* ctl)
{
    const int nb = planes_blocks(a, kind);
    if (nb < 1) return hipErrorInvalidValue;
    ROM_PLANES(planes_kernel, nb, a, ctl)
}

hipError_t launch_planes_batch(const ContractArgs* items, const int2* map, int nblocks, int kind, hipStream_t s, Ctl* ctl)
{
    if (nblocks < 1) return hipErrorInvalidValue;
    ROM_PLANES(planes_batch_kernel, nblocks, items, map, ctl)
}

}  // namespace rom
