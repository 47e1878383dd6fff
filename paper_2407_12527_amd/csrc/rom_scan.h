// rom_scan.h -- the row-scan transport-sweep kernel of librom.
//
// Along one row of cells, with the y-face inflow of the row known, the upwind balance of one
// ordinate is a first-order linear recurrence,
//   psi_i = A_i psi_{i-1} + t_i,   A_i = a r_i,  t_i = r_i (S_i + b y_i),  r_i = 1 / (sigma_t + a + b)
// (diamond difference: x_{i+1} = (2 A_i - 1) x_i + 2 t_i for the x-face value), so a whole row is a
// prefix scan instead of nx dependent steps.  A lane group of G = 16, 32 or 64 lanes holds one row,
// C consecutive cells per lane (nx <= G C): each lane composes its C cells, the lane totals are
// scanned across the group in log2(G) DPP steps (row_shr 1, 2, 4, 8, row_bcast 15, 31, one fused
// multiply-add each), the exclusive result is the lane's x-face inflow, and a second pass over its
// C cells gives psi.  Rows follow one another inside the wavefront, which keeps the row's psi (the
// next row's y-face inflow) in registers: no hand-off between wavefronts, no dependency wait, no
// pipeline to fill, where the other sweeps pay for all three.
//
// The multipliers (r, A and the scan's products of A) depend on sigma_t and the ordinate only, so
// they are kept in registers and rebuilt only at rows whose sigma_t differs from the row before
// (a host-built list, exact for any medium); the next such row's sigma_t is already loaded.  A
// cell-ordinate update is then 5 vector operations: S + b y, times r, compose, final, and the
// weighted flux sum (the strip sweep: 7.2 and 3.9 scalar ones, measured on 512^2).
//
// A wavefront carries 64 / G groups of K ordinates each, all of one quadrant of one system; the
// scalar flux is summed over the workgroup's ordinates through LDS, U rows at a time in a fixed
// order, so one partial plane is written per workgroup (deterministic, no float atomics).  With one
// ordinate per group (RAW) psi itself is exchanged and weighted as it is summed, which also forms
// every moment plane of the linear kernel from one exchange; with several, their weighted sum, over
// the lane groups too by permlane swaps.  Source rows are loaded U rows ahead.  Lanes past the row's
// end compute on clamped addresses; nothing flows back from them or into another lane group.
//
// Dense kernels (MODE 2) keep a plane of cells per ordinate, so a wavefront's source rows are as
// contiguous as an isotropic source's; the weighted angular flux leaves from the exchange, where all of a
// workgroup's ordinates of a cell meet.  Bound by memory: 256^2, 1024 ordinates, FP32, reads 256 MB and
// writes 192 MB in 78 us (5.7 TB/s; the row-lane sweep on ordinate blocks took 293 us, eight wavefronts
// per workgroup, on half the CUs, 128 us); FP64 96 x 80, 20 us (strip sweep 232).
#pragma once
#include "rom_common.h"

namespace rom {

// ------------------------------------------------------------------------------------ lane moves
// `v` moved by the DPP control; lanes without a source get `old` (zero when BOUND)
template <int CTRL, bool BOUND>
__device__ __forceinline__ float dpp_move(float old, float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, 0xF, 0xF, BOUND));
}

template <int CTRL, bool BOUND>
__device__ __forceinline__ double dpp_move(double old, double v)
{
    const int2 o = __builtin_bit_cast(int2, old);
    const int2 x = __builtin_bit_cast(int2, v);
    int2 y;
    y.x = __builtin_amdgcn_update_dpp(o.x, x.x, CTRL, 0xF, 0xF, BOUND);
    y.y = __builtin_amdgcn_update_dpp(o.y, x.y, CTRL, 0xF, 0xF, BOUND);
    return __builtin_bit_cast(double, y);
}

// Scan stage controls: row_shr 1, 2, 4, 8, row_bcast 15 (lane 15 of each 16 to the next 16),
// row_bcast 31 (lane 31 to the upper 32).  The FP32 broadcasts write the rows that they are for only (masks
// 0xa and 0xc): with G = 32, lane 31 may lie past its row's end, on another system's values, and its
// broadcast reaches the other group, where a factor of zero does not hold back an infinity or a NaN.
template <int S>
constexpr int scan_ctrl() { return S == 0 ? 0x111 : S == 1 ? 0x112 : S == 2 ? 0x114 : S == 3 ? 0x118 : S == 4 ? 0x142 : 0x143; }

template <int G>
constexpr int scan_stages() { return G == 16 ? 4 : G == 32 ? 5 : 6; }

// Multipliers of the scan's stages from the lane products p (lane position `pos` in its group):
// stage s adds m[s] times the value moved in.  Lanes that receive nothing in stage s have m[s] = 0
// in the broadcast stages and are given zero by the move in the others.
template <typename T, int G, int S = 0>
__device__ __forceinline__ void scan_multipliers(T p, int lane, T (&m)[scan_stages<G>()])
{
    if constexpr (S < scan_stages<G>()) {
        if constexpr (S < 4) {
            m[S] = p;
            p *= dpp_move<scan_ctrl<S>(), false>(T(1), p);
        } else {
            const bool in = S == 4 ? (lane & 16) != 0 : (lane & 32) != 0;
            m[S] = in ? p : T(0);
            const T q = dpp_move<scan_ctrl<S>(), false>(T(1), p);
            p = in ? p * q : p;
        }
        scan_multipliers<T, G, S + 1>(p, lane, m);
    }
}

// x0 moved up one lane: the value of the lane below in the group; the group's first lane keeps x0.
template <typename T, int G>
__device__ __forceinline__ T scan_shift(T v, T x0, int pos)
{
    if constexpr (G == 16) {
        return dpp_move<0x111, false>(x0, v);   // row_shr:1
    } else if constexpr (G == 64) {
        return dpp_move<0x138, false>(x0, v);   // wave_shr:1
    } else {
        const T u = dpp_move<0x138, false>(x0, v);
        return pos == 0 ? x0 : u;
    }
}

// x[k] becomes the x-face inflow of each lane's first cell: the inclusive scan of the lane totals
// b[k] over the group, moved up one lane (the group's first lane keeps x[k]).
template <int G, int K>
__device__ __forceinline__ void scan_lanes(double (&b)[K], const double (&m)[K][scan_stages<G>()], double (&x)[K], int pos)
{
    static_assert(G != 32, "the broadcasts write every row of 16 lanes");
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double v = b[k];
        v = fma(m[k][0], dpp_move<0x111, true>(0.0, v), v);
        v = fma(m[k][1], dpp_move<0x112, true>(0.0, v), v);
        v = fma(m[k][2], dpp_move<0x114, true>(0.0, v), v);
        v = fma(m[k][3], dpp_move<0x118, true>(0.0, v), v);
        if constexpr (G >= 32) v = fma(m[k][4], dpp_move<0x142, true>(0.0, v), v);
        if constexpr (G == 64) v = fma(m[k][5], dpp_move<0x143, true>(0.0, v), v);
        x[k] = scan_shift<double, G>(v, x[k], pos);
    }
}

// FP32: each stage is one v_fmac_f32 with its moved operand (the compiler keeps a separate move).
// A DPP read needs two wait states after the write of its register: the other ordinates' stages
// and the s_nop give them.  The last instruction moves the result up one lane into x.
#define ROM_ROWS(CTRL, ROWS) CTRL " row_mask:" ROWS " bank_mask:0xf"
#define ROM_DPP(CTRL) ROM_ROWS(CTRL, "0xf")
#define ROM_FMAC_ROWS(B, M, CTRL, ROWS) "v_fmac_f32_dpp " B ", " B ", " M " " ROM_ROWS(CTRL, ROWS) " bound_ctrl:0\n\t"
#define ROM_FMAC(B, M, CTRL) ROM_FMAC_ROWS(B, M, CTRL, "0xf")
template <int G, int K>
__device__ __forceinline__ void scan_lanes(float (&b)[K], const float (&m)[K][scan_stages<G>()], float (&x)[K], int pos)
{
    constexpr int NS = scan_stages<G>();
    if constexpr (K >= 2) {
        // two ordinates at a time
#pragma unroll
        for (int k = 0; k + 1 < K; k += 2) {
#define ROM_STAGE2(S, CTRL, ROWS)                                                                        \
    asm("s_nop 1\n\t" ROM_FMAC_ROWS("%0", "%2", CTRL, ROWS) ROM_FMAC_ROWS("%1", "%3", CTRL, ROWS)        \
        : "+v"(b[k]), "+v"(b[k + 1]) : "v"(m[k][S]), "v"(m[k + 1][S]))
            asm("s_nop 1\n\t"
                ROM_FMAC("%0", "%2", "row_shr:1") ROM_FMAC("%1", "%3", "row_shr:1") "s_nop 0\n\t"
                ROM_FMAC("%0", "%4", "row_shr:2") ROM_FMAC("%1", "%5", "row_shr:2") "s_nop 0\n\t"
                ROM_FMAC("%0", "%6", "row_shr:4") ROM_FMAC("%1", "%7", "row_shr:4") "s_nop 0\n\t"
                ROM_FMAC("%0", "%8", "row_shr:8") ROM_FMAC("%1", "%9", "row_shr:8") "s_nop 1"
                : "+v"(b[k]), "+v"(b[k + 1])
                : "v"(m[k][0]), "v"(m[k + 1][0]), "v"(m[k][1]), "v"(m[k + 1][1]), "v"(m[k][2]), "v"(m[k + 1][2]),
                  "v"(m[k][3]), "v"(m[k + 1][3]));
            if constexpr (NS >= 5) ROM_STAGE2(4, "row_bcast:15", "0xa");
            if constexpr (NS >= 6) ROM_STAGE2(5, "row_bcast:31", "0xc");
#undef ROM_STAGE2
            if constexpr (G == 16)
                asm("s_nop 1\n\tv_mov_b32_dpp %0, %2 " ROM_DPP("row_shr:1") "\n\tv_mov_b32_dpp %1, %3 " ROM_DPP("row_shr:1")
                    : "+v"(x[k]), "+v"(x[k + 1]) : "v"(b[k]), "v"(b[k + 1]));
            else if constexpr (G == 64)
                asm("s_nop 1\n\tv_mov_b32_dpp %0, %2 " ROM_DPP("wave_shr:1") "\n\tv_mov_b32_dpp %1, %3 " ROM_DPP("wave_shr:1")
                    : "+v"(x[k]), "+v"(x[k + 1]) : "v"(b[k]), "v"(b[k + 1]));
        }
    }
    if constexpr (K % 2 == 1) {
        constexpr int k = K - 1;
#define ROM_STAGE1(S, CTRL, ROWS) \
    asm("s_nop 1\n\t" ROM_FMAC_ROWS("%0", "%1", CTRL, ROWS) : "+v"(b[k]) : "v"(m[k][S]))
        asm("s_nop 1\n\t"
            ROM_FMAC("%0", "%1", "row_shr:1") "s_nop 1\n\t"
            ROM_FMAC("%0", "%2", "row_shr:2") "s_nop 1\n\t"
            ROM_FMAC("%0", "%3", "row_shr:4") "s_nop 1\n\t"
            ROM_FMAC("%0", "%4", "row_shr:8") "s_nop 1"
            : "+v"(b[k]) : "v"(m[k][0]), "v"(m[k][1]), "v"(m[k][2]), "v"(m[k][3]));
        if constexpr (NS >= 5) ROM_STAGE1(4, "row_bcast:15", "0xa");
        if constexpr (NS >= 6) ROM_STAGE1(5, "row_bcast:31", "0xc");
#undef ROM_STAGE1
        if constexpr (G == 16)
            asm("s_nop 1\n\tv_mov_b32_dpp %0, %1 " ROM_DPP("row_shr:1") : "+v"(x[k]) : "v"(b[k]));
        else if constexpr (G == 64)
            asm("s_nop 1\n\tv_mov_b32_dpp %0, %1 " ROM_DPP("wave_shr:1") : "+v"(x[k]) : "v"(b[k]));
    }
    if constexpr (G == 32) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float u = x[k];
            asm("s_nop 1\n\tv_mov_b32_dpp %0, %1 " ROM_DPP("wave_shr:1") : "+v"(u) : "v"(b[k]));
            x[k] = pos == 0 ? x[k] : u;
        }
    }
}
#undef ROM_ROWS
#undef ROM_DPP
#undef ROM_FMAC_ROWS
#undef ROM_FMAC

// One stage of a transposing sum over lane halves D = 32 or 16: lanes without bit D get
// x(l) + x(l ^ D), lanes with bit D get y(l ^ D) + y(l) (the lower lane's value always first).
template <int D>
__device__ __forceinline__ float swap_sum(float x, float y)
{
    if constexpr (D == 32) {
        auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(p[0]) + __uint_as_float(p[1]);
    } else {
        auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
}

template <int D>
__device__ __forceinline__ double swap_sum(double x, double y)
{
    const uint2 a = __builtin_bit_cast(uint2, x), b = __builtin_bit_cast(uint2, y);
    uint2 u, v;
    if constexpr (D == 32) {
        auto lo = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false);
        auto hi = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
        u = make_uint2(lo[0], hi[0]);
        v = make_uint2(lo[1], hi[1]);
    } else {
        auto lo = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);
        auto hi = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
        u = make_uint2(lo[0], hi[0]);
        v = make_uint2(lo[1], hi[1]);
    }
    return __builtin_bit_cast(double, u) + __builtin_bit_cast(double, v);
}

// Sum C per-cell values over the 64 / G lane groups of a wavefront: lane (g, pos) ends with the
// totals of cells g * RC .. g * RC + RC - 1 of position pos, RC = C G / 64.
template <typename T, int G, int C>
__device__ __forceinline__ void group_sums(const T (&v)[C], T (&out)[C * G / 64])
{
    if constexpr (G == 64) {
#pragma unroll
        for (int c = 0; c < C; ++c) out[c] = v[c];
    } else if constexpr (G == 32) {
#pragma unroll
        for (int c = 0; c < C / 2; ++c) out[c] = swap_sum<32>(v[c], v[c + C / 2]);
    } else {
        T h[C / 2];
#pragma unroll
        for (int c = 0; c < C / 2; ++c) h[c] = swap_sum<32>(v[c], v[c + C / 2]);
#pragma unroll
        for (int c = 0; c < C / 4; ++c) out[c] = swap_sum<16>(h[c], h[c + C / 4]);
    }
}

// 1 / (sg + a + b) for kap = a + b, klo the rounding error of that sum.  In an optically thin cell the
// update is psi = A x + ..., A near 1, and an error of r moves 1 - A, the cell's attenuation, by as
// much times 1 / (1 - A), the same way in every cell of a medium.  FP32 therefore carries the sum's
// rounding errors (two-sum) into one Newton step: half an ulp of the exact reciprocal, where the sum
// and the hardware reciprocal alone are up to two off (a row of 1023 thin cells: 1.0e-5 of max phi
// without, 3e-6 with it).
__device__ __forceinline__ float scan_rcp(float sg, float kap, float klo)
{
    const float d = sg + kap, v = d - sg;
    const float lo = ((sg - (d - v)) + (kap - v)) + klo;
    const float r = rcp_fast(d);
    return fma(fma(-lo, r, fma(-d, r, 1.0f)), r, r);
}

// Multipliers of a cell: r, A = a r and, for diamond difference, X = 2 A - 1.  In a uniform medium every
// cell has the same ones, and with them the same rounding errors, which add up along a flight path.  FP32
// evens them out in both directions:
//   * along a row, A and X are rounded with a dither that runs evenly through +- half an ulp over the
//     cells (u), so that their mean over a row is the exact value to a fraction of that;
//   * from row to row the flux goes by b r in one column, which a dither over columns would leave with
//     one error for good (one ordinate along 1000 rows: 6.9e-5 of phi; row-lane sweep 2.2e-5).  r is
//     rounded to nearest, and b takes one of two neighbouring values by rows, so that its mean makes
//     up for r (1.7e-6; scan_even).  Neighbouring lanes take them in different rows, so that a flux across
//     columns does not meet the same share of them in each.
// The steps' own roundings remain.  `rho` is the relative rounding error of r, 1 / (r d) - 1.
__device__ __forceinline__ float ulp_of(float x) { return __uint_as_float(__float_as_uint(x) & 0x7f800000u) * 0x1p-23f; }
template <bool DD>
__device__ __forceinline__ void scan_coefficients(float sg, float kap, float klo, float a, float, float u, float& r, float& A, float& X, float& rho)
{
    sg = fminf(sg, 0x1.fffffep127f);   // a sigma_t beyond FP32 came as infinite, whose error terms are NaN
    const float d = sg + kap, v = d - sg;
    const float lo = ((sg - (d - v)) + (kap - v)) + klo;
    const float r0 = scan_rcp(sg, kap, klo);
    const float rl = fma(-lo, r0, fma(-d, r0, 1.0f)) * r0;      // r0 + rl is 1 / (sg + a + b) to twice FP32
    const float ah = a * r0, al = fma(a, rl, fma(a, r0, -ah));
    r = r0 + rl;
    rho = ((r0 - r) + rl) * d;
    A = ah + fma(u, ulp_of(ah), al);
    if constexpr (DD) {
        const float ah2 = ah + ah, xh = ah2 - 1.0f, xl = ah2 - (xh + 1.0f);
        X = xh + fma(u, ulp_of(xh), fma(2.0f, al, xl));
    }
}
template <bool DD>
__device__ __forceinline__ void scan_coefficients(double sg, double kap, double, double a, double b, double, double& r, double& A, double& X, double& rho)
{
    r = rcp_fast(sg + kap);
    A = a * r;
    if constexpr (DD) X = r > 0.0 ? ((a - b) - sg) * r : -1.0;
    rho = 0.0;
}

// The two values of an ordinate's b in a lane: `lo`, and the next one up in a fraction `part` / 2^32 of
// the rows, with the mean b (1 + rho).  The lowest bit of `part` keeps which of the two b itself is.
// A medium of kScanEven rows or fewer has one value anyway and takes b itself (24 x 200 cells with a change
// in every row: a step of 64 us, 80 with the work for two values).
constexpr int kScanEven = 4;   // rows that share a value of b
struct ScanB {
    uint32_t lo, part;
    __device__ __forceinline__ float own() const { return __uint_as_float(lo + (part & 1)); }
    __device__ __forceinline__ float at(uint32_t phase) const { return __uint_as_float(lo + (phase < part ? 1u : 0u)); }
};
__device__ __forceinline__ ScanB scan_even(float b, float rho)
{
    const uint32_t bits = __float_as_uint(b);
    // rho in ulps of b, whose significand is a whole number of them; |rho| is at most half an ulp of r
    float up = rho * (float)((bits & 0x7fffffu) | 0x800000u);
    up = b > 0.0f ? fminf(fmaxf(up, -0x1.fffffep-1f), 0x1.fffffep-1f) : 0.0f;
    const bool below = up < 0.0f;
    if (below) up = fminf(up + 1.0f, 0x1.fffffep-1f);
    return ScanB{bits - (below ? 1u : 0u), ((uint32_t)(up * 0x1p32f) & ~1u) | (below ? 1u : 0u)};
}

// ------------------------------------------------------------------------------------ row runs
// N cells of a row in vector accesses of up to 16 bytes that need element alignment only: a uniform
// base pointer and the lane's byte offset.  The N cells come in storage order.
template <typename T, int N>
__device__ __forceinline__ void run_load(const T* base, uint32_t off, T (&v)[N])
{
    constexpr int W = 16 / sizeof(T);
    typedef T VU __attribute__((ext_vector_type(W), aligned(sizeof(T))));
    typedef T V2 __attribute__((ext_vector_type(2), aligned(sizeof(T))));
    const T* p = (const T*)((const char*)base + off);
    constexpr int full = N / W * W;
#pragma unroll
    for (int q = 0; q < full; q += W) {
        const VU x = *reinterpret_cast<const VU*>(p + q);
#pragma unroll
        for (int m = 0; m < W; ++m) v[q + m] = x[m];
    }
    if constexpr (N - full >= 2) {
        const V2 x = *reinterpret_cast<const V2*>(p + full);
        v[full] = x[0];
        v[full + 1] = x[1];
    }
    if constexpr ((N - full) % 2 == 1) v[N - 1] = p[N - 1];
}

// Read-only tables through the scalar cache.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* scalar_ptr(const T* p)
{
    return (const __attribute__((address_space(4))) T*)p;
}

// Everything one task needs (uniform values).
template <typename T>
struct ScanTask {
    int nx, ny, nw;
    bool ypos;
    const T* st;          // sigma_t of the problem (pool padded by kPoolPad elements on both sides)
    const T* S;           // source of the system (same padding); linear kernel: three planes
    T* part;              // partial-flux slot (linear kernel: consecutive planes)
    const int32_t* next;  // per sweep-order row: the next row whose sigma_t differs from the row before it
    int64_t sstride;      // dense kernels: elements between the source planes of a wavefront's lane groups
    char* psi;            // dense kernels: the task's weighted angular flux, planes of four ordinates in BF16
                          // (FP32 sweeps) or of one in FP64, 8 bytes per cell
    int64_t ld;           // dense kernels: cells from one plane to the next
    const LaneDev* ords;  // the task's ordinates
    const T* xin;         // entry x-face inflow [ny + padding][NO] of this wavefront's ordinates
    bool has_xin;         // vacuum without (xin then holds NO other values)
    int64_t plane;        // cells
};

// All wavefronts of the workgroup arrive; LDS written before is visible after.  Outstanding
// global loads and stores are left in flight (a __syncthreads would drain them).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One task: the rows of the grid in sweep order, for this wavefront's ordinates.
//   MODE 0: isotropic source; 1: linear kernel (three source planes, np = 3 or 4 moment planes);
//   2: dense kernels (a source plane per ordinate, and the weighted angular flux written back)
//   INF: boundary inflow tables may be present
//   SPLIT = 2 (G = 64): a row is two strips of 64 C cells, one wavefront each.  The second strip's
//   wavefront works one batch of rows behind the first's, whose outgoing x-face values it takes from
//   LDS: the barrier of every batch orders the hand-off, no wait is needed.
template <typename T, int G, int C, int K, int U, int W, int SPLIT, int MODE, bool DD, bool INF, int DIR>
__device__ __forceinline__ void scan_rows(const ScanTask<T>& D, T* lds, const int wave, const LaneDev* __restrict__ ords,
                                          const T* __restrict__ yin, const int np_, const bool stopped)
{
    constexpr int NS = scan_stages<G>();
    constexpr bool RAW = K == 1 && SPLIT == 1;   // psi is exchanged, weighted as it is summed
    constexpr int RC = RAW ? C : C * G / 64;     // values a lane exchanges per row
    constexpr int EG = RAW ? 64 / G : 1;         // entries of a wavefront's row in the exchange
    constexpr int GC = G * C;                    // values of an entry
    constexpr int V = 16 / sizeof(T);        // cells per 16 bytes, the unit of the flux exchange
    constexpr int NPL = MODE == 1 ? 4 : 1;   // most moment planes
    constexpr int NSRC = MODE == 1 ? 3 : 1;
    constexpr int NO = (64 / G) * K;
    constexpr int KM = MODE == 1 ? K : 1;
    constexpr int KI = INF ? K : 1;
    constexpr int WE = W / SPLIT;            // wavefronts that share a strip
    constexpr int NE = WE * EG;              // entries summed per strip
    static_assert(MODE == 0 || RAW, "moment planes and angular fluxes are formed from the exchanged psi");
    static_assert(MODE != 2 || sizeof(T) == 8 || NE % 4 == 0, "BF16 angular fluxes are kept in planes of four ordinates");
    static_assert(SPLIT == 1 || (G == 64 && W % SPLIT == 0), "strips are whole wavefronts");
    const int np = MODE == 1 ? np_ : 1;      // moment planes formed
    const int lane = threadIdx.x & (kWave - 1);
    const int g = lane / G, pos = lane % G;
    const int nx = D.nx, ny = D.ny;
    const int strip = wave % SPLIT, entry = wave / SPLIT;
    const bool live = entry < D.nw;          // a wavefront without ordinates only helps to sum
    // Byte offset of this lane's cells in sweep row 0: its first cell in sweep order, clamped into
    // the row (a run then reaches at most C - 1 elements past either end of the row).  Rows are
    // fetched U ahead of a last batch that may itself reach U - 1 rows past the grid, so up to
    // 2 U - 1 rows past the last one: the pools carry that much padding.  The base pointers sit
    // `guard` elements early, so every offset is non-negative.
    const int ii0 = min((strip * G + pos) * C, nx - 1);
    const int guard = 2 * U * nx + C;
    const int64_t step = D.ypos ? nx : -(int64_t)nx;   // one row on
    const uint32_t off0 = sizeof(T) * (uint32_t)(guard + (D.ypos ? 0 : (ny - 1) * nx) + (DIR > 0 ? ii0 : nx - C - ii0));
    const uint32_t dstep = sizeof(T) * (uint32_t)step;
    // cell c of a run sits at storage position c (DIR > 0) or C - 1 - c
    constexpr auto at = [](int c) { return DIR > 0 ? c : C - 1 - c; };

    T a[K], b[K], w[K], lc[KM], ls[KM];
    ScanB even[sizeof(T) == 4 ? K : 1];   // FP32: b[k] is the current rows' value
    uint32_t phase = (uint32_t)(strip * 64 + lane) * 0xc13fa9a9u;   // neighbours in a row are out of step
    T y[K][C], rr[K][C], A[K][C], m[K][NS];
    T X[DD ? K : 1][DD ? C : 1];   // diamond difference: the x-face multiplier 2 A - 1, without its cancellation
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const LaneDev& o = ords[g * K + k];
        a[k] = to_T<T>(DD ? 2.0 * o.a : o.a);
        b[k] = to_T<T>(DD ? 2.0 * o.b : o.b);
        if constexpr (sizeof(T) == 4) even[k] = scan_even(b[k], 0.0f);
        w[k] = to_T<T>(o.w);
        if constexpr (MODE == 1) {
            lc[k] = to_T<T>(o.c);
            ls[k] = to_T<T>(o.s);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) y[k][c] = (INF && yin) ? yin[((g * K + k) * SPLIT + strip) * (G * C) + pos * C + c] : T(0);
    }
    // multipliers of a row from its sigma_t, which `rows` rows have
    auto coefficients = [&](const T (&sg)[C], const int rows) {
        const bool whole = (strip * G + pos + 1) * C <= nx;   // no cell past the row's end
#pragma unroll
        for (int k = 0; k < K; ++k) {
            T bk = b[k];
            if constexpr (sizeof(T) == 4) bk = even[k].own();
            const T kap = a[k] + bk, kv = kap - a[k], klo = (a[k] - (kap - kv)) + (bk - kv);
            T p = T(1), err = T(0), err0 = T(0);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                // a low-discrepancy dither by cell
                const int cell = (strip * G + pos) * C + c;
                const T u = T((((unsigned)cell * 0x9e3779b9u) >> 8) * 0x1p-24f - 0.5f);
                T rho, Xc;
                scan_coefficients<DD>(sg[at(c)], kap, klo, a[k], bk, u, rr[k][c], A[k][c], Xc, rho);
                if constexpr (DD) X[k][c] = Xc;
                p *= DD ? Xc : A[k][c];
                if (c == 0) err0 = rho;
                err += rho;
            }
            if constexpr (sizeof(T) == 4) {
                even[k] = ScanB{__float_as_uint(bk), 0};
                if (rows > kScanEven) even[k] = scan_even(bk, whole ? err * (1.0f / C) : err0);   // the lane's cells in the mean
                b[k] = even[k].at(phase);
            }
            scan_multipliers<T, G>(p, lane, m[k]);
        }
    };
    // A lone wavefront keeps the next changed row's sigma_t loaded ahead; where several share a SIMD
    // the registers are worth more and the row is loaded when it is needed.
    constexpr bool AHEAD = K == 1 && C <= 8;
    T sg[AHEAD ? C : 1];
    T S[U][NSRC][C];
    T x0[INF ? U : 1][KI];   // x-face inflow of the row (used by the group's first lane)
    const T* const sbase = D.S - guard;
    const T* const stbase = D.st - guard;
    // x-face inflow: vector loads (a scalar load's result is waited for with the LDS ones, every row) and
    // no branch: a vacuum face reads its first row over and over and keeps zero (300 x 517, inflow on two
    // sides, 100 ordinates: 148 us per step before, 129 so)
    const bool first = INF && pos == 0 && D.has_xin;
    uint32_t xoff = sizeof(T) * (uint32_t)(g * K);
    if constexpr (INF) asm volatile("" : "+v"(xoff));
    const uint32_t xstep = D.has_xin ? sizeof(T) * NO : 0;
    uint32_t off = off0 + (MODE == 2 ? (uint32_t)(sizeof(T) * g * D.sstride) : 0);
    auto fetch = [&](const int u) {
#pragma unroll
        for (int q = 0; q < NSRC; ++q) run_load<T, C>(sbase + q * D.plane, off, S[u][q]);
        off += dstep;
        if constexpr (INF) {
            run_load<T, KI>(D.xin, xoff, x0[u]);
            xoff += xstep;
        }
    };
    int nc = 0;   // next row whose multipliers differ (row 0 first), in FP32 also the one after it
    int nn = 0;
    if constexpr (sizeof(T) == 4) nn = scalar_ptr(D.next)[0];
    if constexpr (AHEAD) run_load<T, C>(stbase, off0, sg);
#pragma unroll
    for (int u = 0; u < U; ++u) fetch(u);

    if (stopped) return;   // checked here, behind the loads: one memory round trip less at the start

    // Flux exchange in LDS: [2 buffers][U rows][strips][NE entries][GC values], the values in groups of
    // V: group-major over the lanes where a lane holds whole groups (conflict-free 16-byte writes),
    // plain cell order elsewhere.
    typedef T VV __attribute__((ext_vector_type(V)));
    constexpr bool GROUPS = RC % V == 0;
    constexpr int VW = GROUPS ? V : RC % 2 == 0 ? 2 : 1;   // values per write
    constexpr int LE = 64 / EG;                            // lanes of an entry
    typedef T VX __attribute__((ext_vector_type(VW)));
    constexpr int ROW = SPLIT * NE * GC;
    T* const hand = lds + 2 * U * ROW;       // x-face values between strips: [2 buffers][U rows][WE][K]
    const int mine = (strip * NE + (RAW ? entry * EG + g : entry)) * GC + (GROUPS ? (lane % LE) * V : pos * C + (RAW ? 0 : g * RC));
    if (!live)   // a wavefront without ordinates adds zeros
        for (int i = lane; i < 2 * U * EG * GC; i += 64)
            lds[i / (EG * GC) * ROW + (strip * NE + entry * EG) * GC + i % (EG * GC)] = T(0);
    // weights of the entries in each plane (RAW; zero for those without ordinates)
    T wt[RAW ? NPL : 1][RAW ? NE : 1];
    if constexpr (RAW) {
        const auto to = scalar_ptr(D.ords);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int o = min(e, D.nw * EG - 1);
            const double we = e < D.nw * EG ? to[o].w : 0.0;
            wt[0][e] = to_T<T>(we);
            if constexpr (MODE == 1) {
                wt[1][e] = to_T<T>(we * to[o].m1);
                wt[2][e] = to_T<T>(we * to[o].m2);
                wt[3][e] = to_T<T>(we * to[o].m3);
            }
        }
    }
    // The flux sum in chunks of V consecutive cells of a row, one per lane and piece: this wavefront's
    // piece n is e = n W + wave (coalesced stores).  A chunk's place in the plane is a fixed byte
    // offset from the batch's lowest row.
    constexpr int CPR = SPLIT * GC / V;              // chunks per row
    constexpr int CHUNKS = U * CPR;
    constexpr int PER = (CHUNKS + 64 * W - 1) / (64 * W);
    constexpr bool EVEN = CHUNKS % (64 * W) == 0;
    // a lone wavefront per SIMD finishes a batch's sum after the next batch's first row, behind which
    // its LDS reads return; elsewhere the other wavefronts hide them
    constexpr bool DEFER = RAW && PER * NE * V * sizeof(T) <= 512;
    int pu[PER], pl[PER];          // row of the chunk (from the first strip's batch), place in the exchange buffer
    uint32_t po[PER];              // byte offset of its first cell
    int pc[PER];                   // first cell (past nx: nothing to store)
#pragma unroll
    for (int n = 0; n < PER; ++n) {
        const int e = (n * W + wave) * 64 + lane;
        const int u = min(e, CHUNKS - 1) / CPR, x = (e % CPR) * V, sp = x / GC, xs = x % GC;
        pu[n] = u - sp * U;
        if constexpr (CPR % 64 == 0 && SPLIT == 1) pu[n] = uniform(pu[n]);
        pc[n] = e < CHUNKS ? x : nx;
        const int c = xs % C, l = (RAW ? 0 : (c / RC) * G) + xs / C;   // the lane of the entry that holds it
        pl[n] = u * ROW + sp * NE * GC + (GROUPS ? ((c % RC) / V * LE + l) * V : xs);
        const int up = D.ypos ? pu[n] + (SPLIT - 1) * U : U - 1 - pu[n];   // rows above the batch's lowest
        po[n] = sizeof(T) * (uint32_t)(up * nx + (DIR > 0 ? x : nx - 1 - min(x, nx - 1)));
    }
    T* pbase = D.part + (D.ypos ? -(int64_t)(SPLIT - 1) * U * nx : (int64_t)(ny - U) * nx);   // lowest row of the batch
    // one finished piece: rows past the grid and cells past the row are not stored
    auto piece_store = [&](const int n, const int jb, const int q, const VV& sum) {
        const bool in = pu[n] < ny - jb && (SPLIT == 1 || jb + pu[n] >= 0);
        T* const at = (T*)((char*)(pbase + (MODE == 1 ? q * D.plane : 0)) + po[n]);
        if (in && pc[n] + V <= nx) {
            typedef T VU __attribute__((ext_vector_type(V), aligned(sizeof(T))));
            VU out;
#pragma unroll
            for (int i = 0; i < V; ++i) out[i] = sum[DIR > 0 ? i : V - 1 - i];
            *reinterpret_cast<VU*>(DIR > 0 ? at : at - (V - 1)) = out;
        }
        if (V > 1 && __builtin_expect(nx % V != 0, 0)) {   // uniform
            if (in && pc[n] < nx && pc[n] + V > nx) {      // the lane with the row's last cells
#pragma unroll
                for (int i = 0; i + 1 < V; ++i)
                    if (pc[n] + i < nx) at[DIR * i] = sum[i];
            }
        }
    };
    // a finished piece's weighted angular flux: the cells of a plane contiguous
    auto piece_psi = [&](const int n, const int jb, const VV (&r)[NE]) {
        constexpr int PL = sizeof(T) == 8 ? 1 : 4;   // ordinates of a plane
        constexpr int PW = 2;                        // 4-byte words per cell
        typedef uint32_t UP __attribute__((ext_vector_type(PW), aligned(8)));
        const bool in = pu[n] < ny - jb;
        char* at = D.psi + (pbase - D.part) * (4 * PW) + (int64_t)(po[n] * (4 * PW / sizeof(T)));
#pragma unroll
        for (int p = 0; p < NE / PL; ++p) {
            if (p * PL < D.nw * EG) {   // uniform
                UP v[V];
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    if constexpr (sizeof(T) == 8) {
                        v[i] = __builtin_bit_cast(UP, wt[0][p] * r[p][i]);
                    } else {
#pragma unroll
                        for (int h = 0; h < PW; ++h)
                            v[i][h] = bf16_pack(wt[0][p * PL + 2 * h] * r[p * PL + 2 * h][i],
                                                wt[0][p * PL + 2 * h + 1] * r[p * PL + 2 * h + 1][i]);
                    }
                }
                if (in && pc[n] + V <= nx) {
                    UP* const to = (UP*)at - (DIR > 0 ? 0 : V - 1);
#pragma unroll
                    for (int i = 0; i < V; ++i) to[i] = v[DIR > 0 ? i : V - 1 - i];
                }
                if (__builtin_expect(nx % V != 0, 0)) {   // uniform
                    if (in && pc[n] < nx && pc[n] + V > nx) {
#pragma unroll
                        for (int i = 0; i + 1 < V; ++i)
                            if (pc[n] + i < nx) ((UP*)at)[DIR * i] = v[i];
                    }
                }
            }
            at += D.ld * (4 * PW);
        }
    };
    // the entries of a piece, in order
    auto piece_sums = [&](const int n, const int jb, const VV (&r)[NE]) {
        if constexpr (MODE == 2) piece_psi(n, jb, r);
        if constexpr (RAW) {
#pragma unroll
            for (int q = 0; q < NPL; ++q) {
                if (q < np) {
                    VV sum;
#pragma unroll
                    for (int i = 0; i < V; ++i) sum[i] = wt[q][0] * r[0][i];
#pragma unroll
                    for (int e = 1; e < NE; ++e)
#pragma unroll
                        for (int i = 0; i < V; ++i) sum[i] = fma(wt[q][e], r[e][i], sum[i]);
                    piece_store(n, jb, q, sum);
                }
            }
        }
    };
    VV r[DEFER ? PER : 1][DEFER ? NE : 1];
    auto sum_reads = [&](const T* buf) {
#pragma unroll
        for (int n = 0; n < PER; ++n)
#pragma unroll
            for (int e = 0; e < NE; ++e) r[n][e] = *reinterpret_cast<const VV*>(buf + pl[n] + e * GC);
    };
    auto sum_store = [&](const int jb) {
        if constexpr (DEFER) {
#pragma unroll
            for (int n = 0; n < PER; ++n) piece_sums(n, jb, r[n]);
        }
        pbase += U * step;
    };
    auto sum_now = [&](const T* buf, const int jb) {
#pragma unroll
        for (int n = 0; n < PER; ++n) {
            if (!EVEN && (n * W + wave) * 64 >= CHUNKS) continue;
            const T* src = buf + pl[n];
            if constexpr (RAW) {
                VV now[NE];
#pragma unroll
                for (int e = 0; e < NE; ++e) now[e] = *reinterpret_cast<const VV*>(src + e * GC);
                piece_sums(n, jb, now);
            } else {   // four wavefronts at a time
                VV sum{};
#pragma unroll
                for (int v = 0; v < NE; v += 4) {
                    VV q[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) q[i] = v + i < NE ? *reinterpret_cast<const VV*>(src + (v + i) * GC) : VV{};
                    const VV four = (q[0] + q[1]) + (q[2] + q[3]);
                    sum = v == 0 ? four : sum + four;
                }
                piece_store(n, jb, 0, sum);
            }
        }
        pbase += U * step;
    };
    if constexpr (sizeof(T) == 4) asm volatile("" : : "s"(nn));
    const int batches = (ny + U - 1) / U + SPLIT - 1;
    for (int bi = 0, jb = 0; bi < batches; ++bi, jb += U) {
        T* const buf = lds + (bi & 1) * U * ROW;
        T xs[SPLIT > 1 ? U : 1][SPLIT > 1 ? K : 1];
        if constexpr (SPLIT > 1) {
            if (strip > 0) {
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < K; ++k) xs[u][k] = hand[((((bi & 1) ^ 1) * U + u) * WE + entry) * K + k];
            }
        }
        const int js = jb - strip * U;       // first row of this wavefront's batch
        if (live && (SPLIT == 1 || (js >= 0 && js < ny))) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if constexpr (DEFER) {
                    if (u == 1 && jb > 0) sum_store(jb - U);
                }
                // rows past the last one (a ragged last batch) compute on padding and are not summed
                const int jj = js + u;
                if constexpr (sizeof(T) == 4) {
                    // (in a golden-ratio sequence every run of rows has its share)
                    if (u % kScanEven == 0 && (U >= kScanEven || bi % (kScanEven / U) == 0)) {
                        phase += 0x9e3779b9u;
#pragma unroll
                        for (int k = 0; k < K; ++k) b[k] = even[k].at(phase);
                    }
                }
                if (__builtin_expect(jj == nc, 0)) {
                    if constexpr (AHEAD) {
                        coefficients(sg, nn - jj);
                    } else {
                        T now[C];
                        run_load<T, C>(stbase, off0 + (uint32_t)jj * dstep, now);
                        coefficients(now, nn - jj);
                    }
                    if constexpr (sizeof(T) == 4) nc = nn;
                    else nc = scalar_ptr(D.next)[jj];
                    if constexpr (AHEAD) run_load<T, C>(stbase, off0 + (uint32_t)min(nc, ny - 1) * dstep, sg);
                    if constexpr (sizeof(T) == 4) {
                        nn = scalar_ptr(D.next)[min(nc, ny - 1)];
                        asm volatile("" : : "s"(nn));   // waited for here: outstanding, it would be so at every LDS wait
                    }
                }
                T t[K][C], bt[K], x[K];
#pragma unroll
                for (int k = 0; k < K; ++k) {
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        T s = S[u][0][at(c)];
                        if constexpr (MODE == 1) s = fma(ls[k], S[u][2][at(c)], fma(lc[k], S[u][1][at(c)], s));
                        t[k][c] = fma(b[k], y[k][c], s) * rr[k][c];
                    }
                    // lane totals, the group's inflow entering its first lane
                    if constexpr (SPLIT > 1) x[k] = pos != 0 ? T(0) : strip > 0 ? xs[u][k] : first ? x0[INF ? u : 0][INF ? k : 0] : T(0);
                    else x[k] = first ? x0[INF ? u : 0][INF ? k : 0] : T(0);   // the other lanes get theirs from the scan
                    T f = x[k];
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        if (!INF && SPLIT == 1 && c == 0) f = DD ? T(2) * t[k][0] : t[k][0];
                        else if constexpr (DD) f = fma(X[k][c], f, T(2) * t[k][c]);
                        else f = fma(A[k][c], f, t[k][c]);
                    }
                    bt[k] = f;
                }
                fetch(u);
                scan_lanes<G, K>(bt, m, x, pos);
                T acc[C];   // what the lane exchanges, before the sum over lane groups
#pragma unroll
                for (int k = 0; k < K; ++k) {
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const T v = fma(A[k][c], x[k], t[k][c]);
                        if constexpr (DD) {
                            x[k] = fma(X[k][c], x[k], T(2) * t[k][c]);
                            y[k][c] = fma(T(2), v, -y[k][c]);
                        } else {
                            x[k] = v;
                            y[k][c] = v;
                        }
                        if constexpr (RAW) acc[c] = v;
                        else acc[c] = k == 0 ? w[k] * v : fma(w[k], v, acc[c]);
                    }
                }
                if constexpr (SPLIT > 1) {   // the strip's outgoing x-face values
                    if (strip + 1 < SPLIT && lane == 63) {
#pragma unroll
                        for (int k = 0; k < K; ++k) hand[(((bi & 1) * U + u) * WE + entry) * K + k] = x[k];
                    }
                }
                T out[RC];
                if constexpr (RAW) {
#pragma unroll
                    for (int c = 0; c < C; ++c) out[c] = acc[c];
                } else {
                    group_sums<T, G, C>(acc, out);
                }
                T* const to = buf + u * ROW + mine;
#pragma unroll
                for (int h = 0; h < RC / VW; ++h) {
                    VX v;
#pragma unroll
                    for (int e = 0; e < VW; ++e) v[e] = out[h * VW + e];
                    *reinterpret_cast<VX*>(to + (GROUPS ? h * LE * V : h * VW)) = v;
                }
            }
        }
        if constexpr (DEFER) {
            if ((U == 1 || !live) && jb > 0) sum_store(jb - U);
        }
        lds_barrier();
        // The buffer is written again two batches on, after the next barrier, which every wavefront
        // reaches only after its reads here.
        if constexpr (DEFER) sum_reads(buf);
        else sum_now(buf, jb);
    }
    if constexpr (DEFER) sum_store((ny - 1) / U * U);
}

// Everything of one workgroup: W wavefronts for the task of its block, no dependency between
// workgroups.
template <typename T, int G, int C, int K, int U, int W, int SPLIT, int MODE, bool DD, bool INF>
__device__ __forceinline__ void scan_group(const ScanArgs& A, const __attribute__((address_space(4))) ScanTaskDev& TK, T* lds)
{
    constexpr int NO = (64 / G) * K;
    const int wave = uniform(threadIdx.x >> 6);
    const int sys = TK.sys, quad = TK.quad;
    const bool stopped = !A.mode_all && (scalar_ptr(A.ctl)->active == 0 || scalar_ptr(A.sysctl + sys)->state != 0);
    if (blockIdx.x == 0 && threadIdx.x == 0) A.ctl->t_first = wall_clock64();
    ScanTask<T> D;
    D.nx = TK.nx;
    D.ny = TK.ny;
    D.nw = TK.nw;
    D.ypos = quad < 2;
    D.plane = (int64_t)D.nx * D.ny;
    D.st = (const T*)A.sigma_t + TK.field_off;
    D.S = (const T*)A.src + TK.src_off;
    if constexpr (MODE == 2) {
        // the first iteration's source is the same for every ordinate
        D.ld = ang_plane(D.plane);
        D.sstride = A.ang_iso ? 0 : D.ld;
        if (!A.ang_iso) D.S = (const T*)A.ang + TK.ang_off + min(wave / SPLIT, TK.nw - 1) * NO * D.ld;
        D.psi = (char*)A.psi + TK.ang_off * (sizeof(T) == 8 ? 8 : 2);
    }
    D.part = (T*)A.part + TK.part_off;
    D.next = A.next + TK.next_off;
    const int wv = min(wave / SPLIT, D.nw - 1);
    D.ords = A.ords + TK.ord_off;
    const LaneDev* ords = D.ords + wv * NO;
    // inflow tables: x-face [group][ny + padding][NO], y-face [group][NO][SPLIT G C], sweep order
    D.has_xin = INF && TK.xin_off >= 0;
    D.xin = (const T*)A.inflow + (D.has_xin ? TK.xin_off + (int64_t)wv * (D.ny + 2 * kScanAhead) * NO : 0);
    const T* yin = INF && TK.yin_off >= 0 ? (const T*)A.inflow + TK.yin_off + (int64_t)wv * NO * (SPLIT * G * C) : nullptr;
    const int np = A.mom_r ? 4 : 3;
    if (quad == 0 || quad == 3)
        scan_rows<T, G, C, K, U, W, SPLIT, MODE, DD, INF, 1>(D, lds, wave, ords, yin, np, stopped);
    else
        scan_rows<T, G, C, K, U, W, SPLIT, MODE, DD, INF, -1>(D, lds, wave, ords, yin, np, stopped);
}

// Single-ordinate form: every problem of the plan in one shape.
template <typename T, int G, int C, int U, int W, int MODE, bool DD, bool INF>
__global__ __launch_bounds__(64 * W) void scan_kernel(ScanArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    scan_group<T, G, C, 1, U, W, 1, MODE, DD, INF>(A, *scalar_ptr(A.tasks + blockIdx.x), (T*)smem);
}

// Rows fetched ahead and summed per batch of the single-ordinate form, which serves latency-bound
// solves with one wavefront per SIMD: enough rows that a source row from beyond the L2 arrives in
// time (256 x 256, 256 ordinates: 63 us per sweep with 4 rows, 58 with 8 or 16).
template <typename T, int C, int MODE>
constexpr int scan_ahead()
{
    constexpr int words = C * (int)sizeof(T) / 4 * (MODE == 1 ? 3 : 1);
    return words <= 8 ? 8 : words <= 16 ? 4 : words <= 32 && MODE != 1 ? 2 : 1;
}

template <typename T, int G, int C, int W, int MODE, bool DD, bool INF>
hipError_t launch_scan_w(const ScanArgs& a, int ntasks, hipStream_t s)
{
    constexpr int U = scan_ahead<T, C, MODE>();
    static_assert(U <= kScanAhead, "pools and tables are padded for kScanAhead rows");
    if (ntasks < 1) return hipErrorInvalidValue;
    constexpr size_t lds = sizeof(T) * 2 * U * W * (size_t)(C * 64);
    static_assert(lds <= 160 * 1024, "LDS");
    auto kern = scan_kernel<T, G, C, U, W, MODE, DD, INF>;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(ntasks), dim3(64 * W), lds, s, a);
    return hipGetLastError();
}

template <typename T, int G, int C, int W, int MODE, bool DD>
hipError_t launch_scan_t(const ScanArgs& a, int ntasks, bool inf, hipStream_t s)
{
    return inf ? launch_scan_w<T, G, C, W, MODE, DD, true>(a, ntasks, s) : launch_scan_w<T, G, C, W, MODE, DD, false>(a, ntasks, s);
}

}  // namespace rom
