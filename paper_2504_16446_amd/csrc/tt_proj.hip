// Forward model and adjoint kernels for gfx950.
//
// Forward (Eq. forward_model, evaluated in the order the paper writes it):
//   1. map:    M_s[v][u] = sum_i B_{s,u,i} c_{v,i}       (MFMA, one pass over c
//              serves a batch of projections; u runs over the unique segments
//              only -- for even orders segments c and c + n_seg/2 coincide)
//   2. march:  I_{s,j,k,c} = step * sum_n sum_{8 corners} T(x_n - x_v) M_s[v][c mod U]
//              (one thread per ray, float64 sample positions, float32 sums)
// Adjoint (transpose, voxel-driven so no atomics are needed):
//   yf[s][j][k][u] = step * sum_{c mod U = u} y[s][j][k][c]
//   g_v = sum_s B_s^T Q_s(v),  Q_s(v)[u] = sum_{(j,k,n)} T(x_n - x_v) yf[s][j][k][u]
//   Each thread owns one voxel and enumerates the rays within the L1 radius of
//   its detector position and the samples of each ray inside its tent support;
//   each wave then contracts its 64 voxels' Q_s with B_s on MFMA, accumulating
//   g in registers over all projections.
#include "tt_device.h"
#include "tt_internal.h"

namespace tt {

typedef float f4 __attribute__((ext_vector_type(4)));

// MFMA 16x16x4 fp32 operand layout (one wave):
//   A[16][4]: lane l supplies A[l % 16][l / 16]
//   B[4][16]: lane l supplies B[l / 16][l % 16]
//   D[16][16]: lane l holds D[4 (l / 16) + r][l % 16], r = 0..3
__device__ __forceinline__ f4 mfma16x16x4(float a, float b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

typedef short s4 __attribute__((ext_vector_type(4)));  // four bf16 bit patterns

// bf16 MFMA 16x16x16 (fp32 accumulate) operand layout (one wave):
//   A[16][16]: lane l supplies A[l % 16][4 (l / 16) + q], q = 0..3
//   B[16][16]: lane l supplies B[4 (l / 16) + q][l % 16]
//   D as for the fp32 16x16x4 instruction.
__device__ __forceinline__ f4 mfma16x16x16bf16(s4 a, s4 b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// gfx950 bf16 MFMA 16x16x32: lane l supplies A[l % 16][8 (l / 16) + q] and
// B[8 (l / 16) + q][l % 16], q = 0..7; D as above.
typedef short s8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f4 mfma16x16x32bf16(s8 a, s8 b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0,
                                                   0);
}

// float -> bf16 bit pattern, round to nearest even (finite inputs).
__device__ __forceinline__ short f2bf(float x)
{
    unsigned u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}

__device__ __forceinline__ float bf16_value(float x) { return __uint_as_float((unsigned)(unsigned short)f2bf(x) << 16); }

__device__ __forceinline__ long long pad_index(int v, int ny, int nz)
{
    int iz = v % nz;
    int t = v / nz;
    int iy = t % ny;
    int ix = t / ny;
    return ((long long)(ix + 1) * (ny + 2) + (iy + 1)) * (nz + 2) + (iz + 1);
}

// ---------------------------------------------------------------------------
// map (fp32 MFMA).  Block = 64 voxels x 256 rows (row = p * UP + u), four
// waves each owning 64 rows (4 row tiles) and all 4 voxel tiles, i.e. 16
// independent 16x16 accumulators.  The c tile is staged transposed in LDS;
// the B operands come from a copy of Bu pre-swizzled into MFMA lane order
// (Bsw[(row_tile * Cp/4 + ks) * 64 + lane] = Bu[16 row_tile + lane % 16][4 ks + lane / 16]),
// so every operand load is one coalesced 256-byte read.
// ---------------------------------------------------------------------------
constexpr int kCtStride = 80;  // padded voxel stride of the transposed c tile in LDS

template <int UP>
__global__ __launch_bounds__(256) void k_map_fp32(const float *__restrict__ c, const float *__restrict__ Bsw,
                                                  int V, int C, int Cp, int ny, int nz, int s0, int np,
                                                  long long vol_pad, float *__restrict__ M)
{
    extern __shared__ float cT[];  // [Cp][kCtStride]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int v0 = blockIdx.x * 64;
    const int nv = min(64, V - v0);
    const float *cb = c + (long long)v0 * C;
    for (int e = tid; e < 64 * Cp; e += 256) cT[(e >> 6) * kCtStride + (e & 63)] = 0.0f;
    __syncthreads();
    const float invC = 1.0f / (float)C;
    for (int e = tid; e < nv * C; e += 256) {
        int v = (int)(((float)e + 0.5f) * invC);
        int k = e - v * C;
        cT[k * kCtStride + v] = cb[e];
    }
    __syncthreads();

    const int KS = Cp / 4;
    const int rt0 = (s0 * UP) / 16 + blockIdx.y * 16 + wave * 4;  // first row tile of this wave
    const int kq = lane >> 4;
    f4 acc[4][4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = f4{0.f, 0.f, 0.f, 0.f};
    for (int kc = 0; kc < KS / 4; ++kc) {
        float a[4][4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) a[mt][kk] = Bsw[((long long)(rt0 + mt) * KS + kc * 4 + kk) * 64 + lane];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const float b = cT[(kc * 16 + kk * 4 + kq) * kCtStride + nt * 16 + (lane & 15)];
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = mfma16x16x4(a[mt][kk], b, acc[nt][mt]);
            }
        }
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int v = v0 + nt * 16 + (lane & 15);
        if (v >= V) continue;
        const long long vp = pad_index(v, ny, nz);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const int row = blockIdx.y * 256 + wave * 64 + mt * 16 + 4 * kq;  // within the batch
            const int p = row / UP, u0 = row % UP;
            if (p < np) *reinterpret_cast<f4 *>(M + (long long)p * vol_pad * UP + vp * UP + u0) = acc[nt][mt];
        }
    }
}

// Register-resident variant for Cp <= 64 (ell_max <= 8): each wave keeps
// its B operands for every k-step in registers, and the block walks a range
// of consecutive voxel tiles, prefetching the next tile's coefficients
// into registers while the current tile's MFMAs run, so coefficient loads,
// MFMAs and the M stores of consecutive tiles overlap.  A block of NW waves
// covers the same 256 rows, each wave 16 / NW row tiles: eight waves of two
// row tiles (120 registers, four waves per SIMD) measured 2-3% faster than
// four waves of four (216 registers, two waves per SIMD).
constexpr int kCtStrideRb = 81;  // odd: the transposed tile writes hit distinct banks
constexpr int kMapWaves = 8;

template <int UP, int KS, int NW>
__global__ __launch_bounds__(64 * NW) void k_map_fp32_rb(const float *__restrict__ c, const float *__restrict__ Bsw,
                                                          int V, int C, int ny, int nz, int s0, int np,
                                                          long long vol_pad, float *__restrict__ M)
{
    constexpr int Cp = 4 * KS;
    constexpr int NT = 64 * NW;                 // threads of the block
    constexpr int MW = 16 / NW;                 // row tiles per wave (256 rows per block)
    constexpr int NPF = (16 * Cp + NT - 1) / NT;  // float4 per thread covering a 64 x C tile (C <= Cp)
    __shared__ float cT[Cp * kCtStrideRb];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kq = lane >> 4;
    const int rt0 = (s0 * UP) / 16 + blockIdx.y * 16 + wave * MW;
    float a[MW][KS];
#pragma unroll
    for (int mt = 0; mt < MW; ++mt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) a[mt][ks] = Bsw[((long long)(rt0 + mt) * KS + ks) * 64 + lane];
    // padding coefficients C..Cp-1 stay zero for every tile
    for (int e = tid; e < (Cp - C) * 64; e += NT) cT[(C + e / 64) * kCtStrideRb + (e & 63)] = 0.0f;
    const int ntiles = (V + 63) / 64;
    const int n4 = 16 * C;  // float4 in a full tile
    const float invC = 1.0f / (float)C;
    f4 pf[NPF];
    auto prefetch = [&](int t) {
        const int nvals = min(64, V - t * 64) * C;
        const f4 *src = reinterpret_cast<const f4 *>(c + (long long)t * 64 * C);  // 256 C bytes per tile: aligned
        const float *srcf = c + (long long)t * 64 * C;
#pragma unroll
        for (int i = 0; i < NPF; ++i) {
            const int e4 = tid + NT * i;
            pf[i] = f4{0.f, 0.f, 0.f, 0.f};
            if (4 * e4 + 3 < nvals) {
                pf[i] = src[e4];
            } else if (4 * e4 < nvals) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (4 * e4 + q < nvals) pf[i][q] = srcf[4 * e4 + q];
            }
        }
    };
    // each block walks a contiguous range of tiles, so that its stores into
    // every projection's M are one sequential stream (scattered 1 KiB pieces
    // stall on DRAM write credits)
    const int per = (ntiles + (int)gridDim.x - 1) / (int)gridDim.x;
    const int tend = min(ntiles, (int)blockIdx.x * per + per);
    int tile = blockIdx.x * per;
    if (tile < tend) prefetch(tile);
    for (; tile < tend; ++tile) {
        __syncthreads();  // the previous tile's LDS reads are done
#pragma unroll
        for (int i = 0; i < NPF; ++i) {
            const int e4 = tid + NT * i;
            if (e4 < n4) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int e = 4 * e4 + q;
                    const int v = (int)(((float)e + 0.5f) * invC);
                    cT[(e - v * C) * kCtStrideRb + v] = pf[i][q];
                }
            }
        }
        __syncthreads();
        if (tile + 1 < tend) prefetch(tile + 1);  // in flight during the MFMAs
        f4 acc[4][MW];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int mt = 0; mt < MW; ++mt) acc[nt][mt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const float b = cT[(ks * 4 + kq) * kCtStrideRb + nt * 16 + (lane & 15)];
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) acc[nt][mt] = mfma16x16x4(a[mt][ks], b, acc[nt][mt]);
            }
        }
        const int v0 = tile * 64;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int v = v0 + nt * 16 + (lane & 15);
            if (v >= V) continue;
            const long long vp = pad_index(v, ny, nz);
#pragma unroll
            for (int mt = 0; mt < MW; ++mt) {
                const int row = blockIdx.y * 256 + wave * 16 * MW + mt * 16 + 4 * kq;  // within the batch
                const int p = row / UP, u0 = row % UP;
                if (p < np) *reinterpret_cast<f4 *>(M + (long long)p * vol_pad * UP + vp * UP + u0) = acc[nt][mt];
            }
        }
    }
}

template <int UP, int KS>
static hipError_t map_fp32_rb_t(const Dims &d, const float *c, const float *Bsw, int s0, int np, float *M,
                                hipStream_t st)
{
    const int V = d.nx * d.ny * d.nz;
    const long long vol_pad = (long long)(d.nx + 2) * (d.ny + 2) * (d.nz + 2);
    const int gy = (np * UP + 255) / 256, ntiles = (V + 63) / 64;
    // one resident round of blocks over all row groups (measured 3% faster
    // than four rounds: fewer concurrent M store streams)
    static const int resident = [] {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_map_fp32_rb<UP, KS, kMapWaves>, 64 * kMapWaves,
                                                         0) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 512;
        return std::max(1, per_cu * cus);
    }();
    const int gx = std::max(1, std::min(ntiles, resident / gy));
    hipLaunchKernelGGL((k_map_fp32_rb<UP, KS, kMapWaves>), dim3(gx, gy), dim3(64 * kMapWaves), 0, st, c, Bsw, V, d.C,
                       d.ny, d.nz, s0, np, vol_pad, M);
    return hipGetLastError();
}

template <int UP>
static hipError_t map_fp32_t(const Dims &d, const float *c, const float *Bsw, int s0, int np, float *M,
                             hipStream_t st)
{
    const bool aligned = reinterpret_cast<uintptr_t>(c) % 16 == 0;  // float4 tile loads
    switch (aligned ? d.Cp : 0) {
    case 16: return map_fp32_rb_t<UP, 4>(d, c, Bsw, s0, np, M, st);
    case 32: return map_fp32_rb_t<UP, 8>(d, c, Bsw, s0, np, M, st);
    case 48: return map_fp32_rb_t<UP, 12>(d, c, Bsw, s0, np, M, st);
    case 64: return map_fp32_rb_t<UP, 16>(d, c, Bsw, s0, np, M, st);
    default: break;  // larger orders: B operands streamed from memory
    }
    const int V = d.nx * d.ny * d.nz;
    const long long vol_pad = (long long)(d.nx + 2) * (d.ny + 2) * (d.nz + 2);
    dim3 grid((V + 63) / 64, (np * UP + 255) / 256);
    size_t lds = (size_t)d.Cp * kCtStride * sizeof(float);
    hipLaunchKernelGGL(k_map_fp32<UP>, grid, dim3(256), lds, st, c, Bsw, V, d.C, d.Cp, d.ny, d.nz, s0, np,
                       vol_pad, M);
    return hipGetLastError();
}

hipError_t launch_map_fp32(const Dims &d, const float *c, const float *Bsw, int s0, int np, float *M,
                           hipStream_t st)
{
    if ((s0 * d.Up) % 16) return hipErrorInvalidValue;  // batches start on a row tile
    switch (d.Up) {
    case 4: return map_fp32_t<4>(d, c, Bsw, s0, np, M, st);
    case 8: return map_fp32_t<8>(d, c, Bsw, s0, np, M, st);
    case 16: return map_fp32_t<16>(d, c, Bsw, s0, np, M, st);
    default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// map, bf16 tier: c is rounded to bf16 while it is staged in LDS, B comes as
// bf16 in MFMA lane order, products accumulate in fp32.  K = Cp runs in
// 32-coefficient steps on the 16x16x32 instruction, the last one filled up with
// zeros when Cp / 16 is odd.  (It must not end in a 16x16x16 step: that
// instruction right behind a 16x16x32 one on the same accumulator took the
// accumulator's first two registers before they were written, in a few tiles of a
// million, so that repeated forwards differed by 1e-3.)  Row tile rt of Bsw16 holds
// for step kp and lane l the eight values Bu[16 rt + l % 16][32 kp + 8 (l / 16) + q]
// at ((rt KP + kp) 64 + l) 8, KP = ceil(Cp / 32).  Same tiling as the fp32 kernel.
// ---------------------------------------------------------------------------
template <int UP>
__global__ __launch_bounds__(256) void k_map_bf16(const float *__restrict__ c, const short *__restrict__ Bsw16,
                                                  int V, int C, int Cp, int ny, int nz, int s0, int np,
                                                  long long vol_pad, float *__restrict__ M)
{
    extern __shared__ short cb[];  // [64][32 KP + 8] bf16, row = voxel (16-byte rows)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int KP = (Cp + 31) / 32, ld = 32 * KP + 8;
    const int v0 = blockIdx.x * 64;
    const int nv = min(64, V - v0);
    const float *cg = c + (long long)v0 * C;
    for (int e = tid; e < 64 * ld; e += 256) cb[e] = 0;
    __syncthreads();
    const float invC = 1.0f / (float)C;
    for (int e = tid; e < nv * C; e += 256) {
        int v = (int)(((float)e + 0.5f) * invC);
        int k = e - v * C;
        cb[v * ld + k] = f2bf(cg[e]);
    }
    __syncthreads();

    const int rt0 = (s0 * UP) / 16 + blockIdx.y * 16 + wave * 4;
    const int kq = lane >> 4;
    f4 acc[4][4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = f4{0.f, 0.f, 0.f, 0.f};
    for (int kp = 0; kp < KP; ++kp) {
        s8 a[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
            a[mt] = *reinterpret_cast<const s8 *>(Bsw16 + ((long long)(rt0 + mt) * KP + kp) * 512 + lane * 8);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const s8 b = *reinterpret_cast<const s8 *>(cb + (nt * 16 + (lane & 15)) * ld + kp * 32 + 8 * kq);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) acc[nt][mt] = mfma16x16x32bf16(a[mt], b, acc[nt][mt]);
        }
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int v = v0 + nt * 16 + (lane & 15);
        if (v >= V) continue;
        const long long vp = pad_index(v, ny, nz);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const int row = blockIdx.y * 256 + wave * 64 + mt * 16 + 4 * kq;
            const int p = row / UP, u0 = row % UP;
            if (p < np) *reinterpret_cast<f4 *>(M + (long long)p * vol_pad * UP + vp * UP + u0) = acc[nt][mt];
        }
    }
}

// Register-resident bf16 variant for Cp <= 64, organised as k_map_fp32_rb: a
// block of kMapWaves waves covers 256 rows, each wave 16 / NW row tiles with
// its A operands for every k-step in registers; the block walks a contiguous
// range of 64-voxel tiles (sequential M store streams), prefetching the next
// tile's coefficients into registers during the MFMAs, and rounds them to
// bf16 while staging them in LDS.  Same rounding points and MFMA order as
// k_map_bf16, hence the same results.
template <int UP, int CPT, int NW>
__global__ __launch_bounds__(64 * NW) void k_map_bf16_rb(const float *__restrict__ c, const short *__restrict__ Bsw16,
                                                         int V, int C, int ny, int nz, int s0, int np,
                                                         long long vol_pad, float *__restrict__ M)
{
    constexpr int Cp = 16 * CPT, KP = (CPT + 1) / 2;
    constexpr int ld = 32 * KP + 8;             // LDS row of one voxel, in shorts (16-byte multiple)
    constexpr int NT = 64 * NW;                 // threads of the block
    constexpr int MW = 16 / NW;                 // row tiles per wave (256 rows per block)
    constexpr int NPF = (16 * Cp + NT - 1) / NT;  // float4 per thread covering a 64 x C tile (C <= Cp)
    __shared__ short cb[64 * ld];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kq = lane >> 4;
    const int rt0 = (s0 * UP) / 16 + blockIdx.y * 16 + wave * MW;
    s8 a8[MW][KP];
#pragma unroll
    for (int mt = 0; mt < MW; ++mt)
#pragma unroll
        for (int kp = 0; kp < KP; ++kp)
            a8[mt][kp] = *reinterpret_cast<const s8 *>(Bsw16 + ((long long)(rt0 + mt) * KP + kp) * 512 + lane * 8);
    // coefficients C..ld-1 of every voxel row stay zero for every tile
    for (int e = tid; e < 64 * (ld - C); e += NT) cb[(e / (ld - C)) * ld + C + e % (ld - C)] = 0;
    const int ntiles = (V + 63) / 64;
    const int n4 = 16 * C;  // float4 in a full tile
    const float invC = 1.0f / (float)C;
    f4 pf[NPF];
    auto prefetch = [&](int t) {
        const int nvals = min(64, V - t * 64) * C;
        const f4 *src = reinterpret_cast<const f4 *>(c + (long long)t * 64 * C);  // 256 C bytes per tile: aligned
        const float *srcf = c + (long long)t * 64 * C;
#pragma unroll
        for (int i = 0; i < NPF; ++i) {
            const int e4 = tid + NT * i;
            pf[i] = f4{0.f, 0.f, 0.f, 0.f};
            if (4 * e4 + 3 < nvals) {
                pf[i] = src[e4];
            } else if (4 * e4 < nvals) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (4 * e4 + q < nvals) pf[i][q] = srcf[4 * e4 + q];
            }
        }
    };
    const int per = (ntiles + (int)gridDim.x - 1) / (int)gridDim.x;
    const int tend = min(ntiles, (int)blockIdx.x * per + per);
    int tile = blockIdx.x * per;
    if (tile < tend) prefetch(tile);
    for (; tile < tend; ++tile) {
        __syncthreads();  // the previous tile's LDS reads are done
#pragma unroll
        for (int i = 0; i < NPF; ++i) {
            const int e4 = tid + NT * i;
            if (e4 < n4) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int e = 4 * e4 + q;
                    const int v = (int)(((float)e + 0.5f) * invC);
                    cb[v * ld + (e - v * C)] = f2bf(pf[i][q]);
                }
            }
        }
        __syncthreads();
        if (tile + 1 < tend) prefetch(tile + 1);  // in flight during the MFMAs
        f4 acc[4][MW];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int mt = 0; mt < MW; ++mt) acc[nt][mt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kp = 0; kp < KP; ++kp) {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const s8 b = *reinterpret_cast<const s8 *>(cb + (nt * 16 + (lane & 15)) * ld + kp * 32 + 8 * kq);
#pragma unroll
                for (int mt = 0; mt < MW; ++mt) acc[nt][mt] = mfma16x16x32bf16(a8[mt][kp], b, acc[nt][mt]);
            }
        }
        const int v0 = tile * 64;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int v = v0 + nt * 16 + (lane & 15);
            if (v >= V) continue;
            const long long vp = pad_index(v, ny, nz);
#pragma unroll
            for (int mt = 0; mt < MW; ++mt) {
                const int row = blockIdx.y * 256 + wave * 16 * MW + mt * 16 + 4 * kq;  // within the batch
                const int p = row / UP, u0 = row % UP;
                if (p < np) *reinterpret_cast<f4 *>(M + (long long)p * vol_pad * UP + vp * UP + u0) = acc[nt][mt];
            }
        }
    }
}

template <int UP, int CPT>
static hipError_t map_bf16_rb_t(const Dims &d, const float *c, const uint16_t *Bsw16, int s0, int np, float *M,
                                hipStream_t st)
{
    const int V = d.nx * d.ny * d.nz;
    const long long vol_pad = (long long)(d.nx + 2) * (d.ny + 2) * (d.nz + 2);
    const int gy = (np * UP + 255) / 256, ntiles = (V + 63) / 64;
    static const int resident = [] {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_map_bf16_rb<UP, CPT, kMapWaves>, 64 * kMapWaves,
                                                         0) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 512;
        return std::max(1, per_cu * cus);
    }();
    const int gx = std::max(1, std::min(ntiles, resident / gy));
    hipLaunchKernelGGL((k_map_bf16_rb<UP, CPT, kMapWaves>), dim3(gx, gy), dim3(64 * kMapWaves), 0, st, c,
                       reinterpret_cast<const short *>(Bsw16), V, d.C, d.ny, d.nz, s0, np, vol_pad, M);
    return hipGetLastError();
}

template <int UP>
static hipError_t map_bf16_t(const Dims &d, const float *c, const uint16_t *Bsw16, int s0, int np, float *M,
                             hipStream_t st)
{
    const bool aligned = reinterpret_cast<uintptr_t>(c) % 16 == 0;  // float4 tile loads
    switch (aligned ? d.Cp : 0) {
    case 16: return map_bf16_rb_t<UP, 1>(d, c, Bsw16, s0, np, M, st);
    case 32: return map_bf16_rb_t<UP, 2>(d, c, Bsw16, s0, np, M, st);
    case 48: return map_bf16_rb_t<UP, 3>(d, c, Bsw16, s0, np, M, st);
    case 64: return map_bf16_rb_t<UP, 4>(d, c, Bsw16, s0, np, M, st);
    default: break;  // larger orders: one tile per block, A operands loaded per step
    }
    const int V = d.nx * d.ny * d.nz;
    const long long vol_pad = (long long)(d.nx + 2) * (d.ny + 2) * (d.nz + 2);
    dim3 grid((V + 63) / 64, (np * UP + 255) / 256);
    size_t lds = (size_t)64 * ((d.Cp + 31) / 32 * 32 + 8) * sizeof(short);
    hipLaunchKernelGGL(k_map_bf16<UP>, grid, dim3(256), lds, st, c, reinterpret_cast<const short *>(Bsw16), V, d.C,
                       d.Cp, d.ny, d.nz, s0, np, vol_pad, M);
    return hipGetLastError();
}

hipError_t launch_map_bf16(const Dims &d, const float *c, const uint16_t *Bsw16, int s0, int np, float *M,
                           hipStream_t st)
{
    if ((s0 * d.Up) % 16) return hipErrorInvalidValue;
    switch (d.Up) {
    case 4: return map_bf16_t<4>(d, c, Bsw16, s0, np, M, st);
    case 8: return map_bf16_t<8>(d, c, Bsw16, s0, np, M, st);
    case 16: return map_bf16_t<16>(d, c, Bsw16, s0, np, M, st);
    default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// march: one thread per ray; block = 16 (j) x 16 (k) rays of one projection.
// Ray positions are set up in float64 in padded index coordinates (voxel ix
// sits at ix + 1, borders of M are zero), so no bounds test is needed inside
// the loop.  The staged path computes each slab's sample count and first
// position in float64 and steps its samples in float32 relative to the
// staged box; the global path steps in float64.
//
// The tile's rays are marched slab by slab: a slab is W planes of the
// horizontal axis A most aligned with the rays.  Before each slab the block
// stages the box of M that holds every corner its samples touch into LDS
// (rows along z, coalesced), then each thread walks its own samples in that
// slab and gathers the 8 corners from LDS.  The box size comes from the
// per-projection slab plan; projections without a plan (steep rays) gather
// straight from global memory.
// ---------------------------------------------------------------------------

// Ray setup shared by both paths: index-space base point b and step ds of the
// ray through pixel (j, k), and its sample range [n0, n1] (empty if n0 > n1).
// Joseph's method (jos): the samples are the ray's cuts with the voxel-centre
// planes of its dominant axis A, so the base point is moved to the cut with
// plane A = 0 and the spacing is d / |d_A|: sample n lies on plane
// n sign(d_A), and the same box constraints keep the planes 1..n_A and the
// cuts whose in-plane coordinates stay inside (0, n + 1).
__device__ __forceinline__ void ray_setup(const ProjFrame &f, int j, int k, int nx, int ny, int nz, float step,
                                          double b[3], double ds[3], int &n0, int &n1, bool jos = false)
{
    const double n3[3] = {(double)nx, (double)ny, (double)nz};
    double tlo = -1e300, thi = 1e300;
    double scale = (double)step;
#pragma unroll
    for (int a = 0; a < 3; ++a) b[a] = f.o[a] + j * f.ej[a] + k * f.ek[a] + 0.5 * (n3[a] + 1.0);
    if (jos) {
        const int A = f.jos_a;
        const double t0 = -b[A] * f.inv_d[A];
#pragma unroll
        for (int a = 0; a < 3; ++a) b[a] = a == A ? 0.0 : fma(t0, f.d[a], b[a]);
        scale = fabs(f.inv_d[A]);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        ds[a] = (jos && a == f.jos_a) ? (f.d[a] > 0.0 ? 1.0 : -1.0) : scale * f.d[a];
        if (f.inv_d[a] != 0.0) {
            // index coordinate b + n ds must stay inside (0, n + 1)
            double ia = (jos && a == f.jos_a) ? ds[a] : f.inv_d[a] / scale;
            double t1 = -b[a] * ia, t2 = (n3[a] + 1.0 - b[a]) * ia;
            tlo = fmax(tlo, fmin(t1, t2));
            thi = fmin(thi, fmax(t1, t2));
        } else if (!(b[a] > 0.0 && b[a] < n3[a] + 1.0)) {
            thi = -1e300;
        }
    }
    n0 = 0;
    n1 = -1;
    if (tlo < thi) {
        n0 = (int)ceil(tlo);
        n1 = (int)floor(thi);
    }
}

template <int UP>
__device__ __forceinline__ void march_global(const float *__restrict__ Mp, const double b[3], const double ds[3], int n0,
                                             int n1, int nx, int ny, int nz, float acc[UP])
{
    const long long sz = UP, sy = (long long)(nz + 2) * UP, sx = (long long)(ny + 2) * sy;
    for (int n = n0; n <= n1; ++n) {
        double px = fma((double)n, ds[0], b[0]);
        double py = fma((double)n, ds[1], b[1]);
        double pz = fma((double)n, ds[2], b[2]);
        int ix = min(max((int)floor(px), 0), nx);
        int iy = min(max((int)floor(py), 0), ny);
        int iz = min(max((int)floor(pz), 0), nz);
        float fx = (float)(px - ix), fy = (float)(py - iy), fz = (float)(pz - iz);
        float gx = 1.0f - fx, gy = 1.0f - fy, gz = 1.0f - fz;
        float w00 = gx * gy, w01 = gx * fy, w10 = fx * gy, w11 = fx * fy;
        const float *q = Mp + ix * sx + iy * sy + iz * sz;
        float w[8] = {w00 * gz, w00 * fz, w01 * gz, w01 * fz, w10 * gz, w10 * fz, w11 * gz, w11 * fz};
        const long long off[8] = {0, sz, sy, sy + sz, sx, sx + sz, sx + sy, sx + sy + sz};
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) {
#pragma unroll
            for (int u4 = 0; u4 < UP; u4 += 4) {
                f4 m = *reinterpret_cast<const f4 *>(q + off[cc] + u4);
                acc[u4 + 0] = fmaf(w[cc], m.x, acc[u4 + 0]);
                acc[u4 + 1] = fmaf(w[cc], m.y, acc[u4 + 1]);
                acc[u4 + 2] = fmaf(w[cc], m.z, acc[u4 + 2]);
                acc[u4 + 3] = fmaf(w[cc], m.w, acc[u4 + 3]);
            }
        }
    }
}

// Global-memory march of the fused sparse forward: at every sample the 8
// corner voxels' coefficients are mapped to the unique segments with the
// projection's sparse map (tab[u * kk + t] = (basis index, constant)).
template <int UP>
__device__ __forceinline__ void march_global_fused(const float *__restrict__ cv, const int2 *tab, int kk, int C,
                                                   const double b[3], const double ds[3], int n0, int n1, int nx,
                                                   int ny, int nz, int U, float acc[UP])
{
    for (int n = n0; n <= n1; ++n) {
        const double px = fma((double)n, ds[0], b[0]);
        const double py = fma((double)n, ds[1], b[1]);
        const double pz = fma((double)n, ds[2], b[2]);
        // padded cell [i, i + 1] holds voxels i - 1 and i along each axis
        const int ix = min(max((int)floor(px), 0), nx);
        const int iy = min(max((int)floor(py), 0), ny);
        const int iz = min(max((int)floor(pz), 0), nz);
        const float fx = (float)(px - ix), fy = (float)(py - iy), fz = (float)(pz - iz);
        const float gx = 1.0f - fx, gy = 1.0f - fy, gz = 1.0f - fz;
        for (int cc = 0; cc < 8; ++cc) {
            const int x = ix - 1 + (cc >> 2), y = iy - 1 + ((cc >> 1) & 1), z = iz - 1 + (cc & 1);
            if ((unsigned)x >= (unsigned)nx || (unsigned)y >= (unsigned)ny || (unsigned)z >= (unsigned)nz) continue;
            const float wc = ((cc & 4) ? fx : gx) * ((cc & 2) ? fy : gy) * ((cc & 1) ? fz : gz);
            const float *src = cv + ((long long)(x * ny + y) * nz + z) * C;
#pragma unroll
            for (int u = 0; u < UP; ++u) {
                if (u < U) {
                    float v = 0.0f;
                    for (int t = 0; t < kk; ++t) {
                        const int2 e = tab[u * kk + t];
                        v = fmaf(__int_as_float(e.y), src[e.x], v);
                    }
                    acc[u] = fmaf(wc, v, acc[u]);
                }
            }
        }
    }
}

// With 4 unique segments (32 KiB boxes) five blocks fit a CU's LDS; asking
// for five waves per SIMD (a small spill of setup values) measured 4% faster
// than the four that 116 VGPRs allow.  Larger UP keep their registers: their
// spills were much larger and slower.
//
// FUSED: the sparse variant of the forward (sect. "Pipelines": the
// reciprocal-space map applied inside the ray-sum kernel, so no mapped volume
// is stored).  M is then the coefficient volume c[nx][ny][nz][C] itself, the
// grid covers all projections (s0 = 0), and each staged box voxel's unique
// segment values are formed while staging, m_u = sum_t tab[u][t].w *
// c[v][tab[u][t].i] over the kk kept basis functions of (s, u); one thread
// stages one (voxel, segment) pair.  The gather from the box is the same.
template <int UP, bool FUSED, int NCM = 8>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((UP == 4 && !FUSED) ? 5 : 1))) void k_march(const float *__restrict__ M, const ProjFrame *__restrict__ frames,
                                               int s0, int nx, int ny, int nz, int nj, int nk, int nseg, int U,
                                               float step, long long vol_pad, float *__restrict__ I,
                                               const int2 *__restrict__ sp, int kk, int C,
                                               const float *__restrict__ cT, const int *__restrict__ gtab, int ng,
                                               int jos, int rings)
{
    constexpr int Q = UP / 4;      // float4 per staged voxel
    // FUSED: the map table int2[UP][kk] (global-memory gathers), the channel
    // list int[ng] and its constants float[ng][UP] (staging), then the box
    extern __shared__ f4 lds[];
    __shared__ int arange[2];
    const int tab_f4 = FUSED ? (UP * kk * 8 + 15) / 16 + (ng * (UP + 1) * 4 + 15) / 16 : 0;
    f4 *box = lds + tab_f4;        // [Q][W + 1][eb][ez]
    const int ntj = (nj + kMarchTile - 1) / kMarchTile, ntk = (nk + kMarchTile - 1) / kMarchTile;
    const int lb = blockIdx.x;
    const int p = lb / (ntj * ntk), s = s0 + p;
    const int tj = (lb / ntk) % ntj, tk = lb % ntk;
    const int j = tj * kMarchTile + (threadIdx.x % kMarchTile);
    const int k = tk * kMarchTile + (threadIdx.x / kMarchTile);
    const bool live = j < nj && k < nk;
    const ProjFrame &f = frames[s];
    if (!FUSED && rings && f.ring_r[kRingOne] > 0) return;  // this projection runs in k_march_ring
    const float *Mp = FUSED ? M : M + (long long)p * vol_pad * UP;
    int2 *tab = reinterpret_cast<int2 *>(lds);
    int *gch = reinterpret_cast<int *>(lds + (UP * kk * 8 + 15) / 16);  // [ng] channels, then [ng][UP] constants
    const float *gw = reinterpret_cast<const float *>(gch + ng);
    if constexpr (FUSED) {
        const int2 *src = sp + (long long)s * UP * kk;
        for (int i = threadIdx.x; i < UP * kk; i += 256) tab[i] = src[i];
        const int *gsrc = gtab + (long long)s * ng * (UP + 1);
        for (int i = threadIdx.x; i < ng * (UP + 1); i += 256) gch[i] = gsrc[i];
        __syncthreads();
    }
    double b[3], ds[3];
    int n0 = 0, n1 = -1;
    if (live) ray_setup(f, j, k, nx, ny, nz, step, b, ds, n0, n1, jos != 0);
    float acc[UP];
#pragma unroll
    for (int u = 0; u < UP; ++u) acc[u] = 0.0f;

    const int W = f.slab_w;
    if (W == 0) {
        if (n0 <= n1) {
            if constexpr (FUSED)
                march_global_fused<UP>(M, tab, kk, C, b, ds, n0, n1, nx, ny, nz, U, acc);
            else
                march_global<UP>(Mp, b, ds, n0, n1, nx, ny, nz, acc);
        }
    } else {
        const int A = f.slab_a, B = 1 - A, EB = f.slab_eb, EZ = f.slab_ez;
        // samples are visited in increasing index coordinate along A
        const bool fwd = f.d[A] > 0.0;
        const int count = n1 - n0 + 1;
        if (threadIdx.x == 0) {
            arange[0] = INT_MAX;
            arange[1] = INT_MIN;
        }
        __syncthreads();
        if (count > 0) {
            const int nf = fwd ? n0 : n1, nl = fwd ? n1 : n0;
            atomicMin(&arange[0], (int)floor(fma((double)nf, ds[A], b[A])));
            atomicMax(&arange[1], (int)floor(fma((double)nl, ds[A], b[A])));
        }
        __syncthreads();
        const int amin = arange[0], amax = arange[1];
        // Staged box origin of slab A0: the lowest corner, along B and z, of the
        // tile's rays between planes A0 and A0 + W.  Each vertex coordinate is
        // affine in A0 with the common slope d_B / d_A (resp. d_z / d_A), so the
        // minimum over the 8 vertices is kb + A0 rB (resp. kz + A0 rZ).
        const double n3[3] = {(double)nx, (double)ny, (double)nz};
        double b00[3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
            b00[a] = f.o[a] + (tj * kMarchTile) * f.ej[a] + (tk * kMarchTile) * f.ek[a] + 0.5 * (n3[a] + 1.0);
        const double rB = f.d[B] * f.inv_d[A], rZ = f.d[2] * f.inv_d[A];
        const double T = kMarchTile - 1;
        double kb = 1e300, kz = 1e300;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const double J = (v & 1) ? T : 0.0, K = (v & 2) ? T : 0.0, P = (v & 4) ? (double)W : 0.0;
            const double t = P - (b00[A] + J * f.ej[A] + K * f.ek[A]);
            kb = fmin(kb, b00[B] + J * f.ej[B] + K * f.ek[B] + t * rB);
            kz = fmin(kz, b00[2] + J * f.ej[2] + K * f.ek[2] + t * rZ);
        }
        const int plane = EB * EZ, nbox = (W + 1) * plane;
        const int nbs = (nbox + 63) & ~63;  // LDS stride of one float4 component array of the box
        // M strides (in voxels) of the box axes A and B; z is contiguous
        const int sy = nz + 2, sx = (ny + 2) * sy;
        const int sA = A == 0 ? sx : sy, sB = A == 0 ? sy : sx;
        const unsigned nAp = (A == 0 ? nx : ny) + 1, nBp = (A == 0 ? ny : nx) + 1, nZp = nz + 1;
        // LDS layout box[q][e]: the q-th float4 of all staged voxels, then the next
        const int da = plane, db = EZ, dz = 1;
        // Staging walk: thread t stages box elements e = t + 256 i.  Its first
        // element's (plane, row, z) and the step of 256 elements are decoded
        // once; every later element follows by adds and two carries, and its M
        // offset from the slab origin (in voxels, 32-bit) likewise.
        const int e_pl = threadIdx.x / plane, e_r = threadIdx.x - e_pl * plane;
        const int e_ib = e_r / EZ, e_iz = e_r - e_ib * EZ;
        const int s_pl = 256 / plane, s_r = 256 - s_pl * plane;
        const int s_ib = s_r / EZ, s_iz = s_r - s_ib * EZ;
        const int s_off = s_pl * sA + s_ib * sB + s_iz;  // M offset of one step without carries
        const int cz_off = sB - EZ, cb_off = sA - EB * sB;  // extra M offset of a z / row carry
        // Samples in sample order m have index position q0 + m dq with dq_A > 0.
        const int nstart = fwd ? n0 : n1;
        double q0[3], dq[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            q0[a] = fma((double)nstart, ds[a], b[a]);
            dq[a] = fwd ? ds[a] : -ds[a];
        }
        const double inv_dqA = 1.0 / dq[A];  // |d_A| >= 1/4 for a planned projection
        const float dqA = (float)dq[A], dqB = (float)dq[B], dqZ = (float)dq[2];
        const float wmax = (float)(W - 1), bmax = (float)(EB - 2), zmax = (float)(EZ - 2);
        int m = 0;
        for (int A0 = amin; A0 <= amax; A0 += W) {
            const int B0 = (int)floor(fma((double)A0, rB, kb)) - 1, Z0 = (int)floor(fma((double)A0, rZ, kz)) - 1;
            __syncthreads();  // the previous slab's gathers are done
            if constexpr (FUSED) {
              if (cT) {
                // thread t stages box elements e = t + 256 i (the walk of the
                // copying path), EPI of them per pass: the ng selected channels of
                // each voxel come from the channel-major copy cT[i][voxel], so a
                // wave's loads of one channel are 64 consecutive z voxels; the
                // unique segment values m_u = sum_g w[g][u] cT[g] are written as
                // Q float4s
                const long long V = (long long)nx * ny * nz;
                const int nA = A == 0 ? nx : ny, nB = A == 0 ? ny : nx;
                int pl = e_pl, ib = e_ib, iz = e_iz;
                auto voxel = [&](int e, long long &vox) {
                    const int a = A0 + pl - 1, bq = B0 + ib - 1, z = Z0 + iz - 1;
                    const bool in = e < nbox && (unsigned)a < (unsigned)nA && (unsigned)bq < (unsigned)nB &&
                                    (unsigned)z < (unsigned)nz;
                    const int x = A == 0 ? a : bq, y = A == 0 ? bq : a;
                    vox = in ? ((long long)x * ny + y) * nz + z : 0LL;
                    pl += s_pl;
                    ib += s_ib;
                    iz += s_iz;
                    if (iz >= EZ) {
                        iz -= EZ;
                        ++ib;
                    }
                    if (ib >= EB) {
                        ib -= EB;
                        ++pl;
                    }
                    return in;
                };
                // EPI voxels per thread and pass (e = t, t + 256, ...), all
                // their (ng <= NCM) channel loads in flight together, then the
                // weighted sums
                constexpr int EPI = NCM <= 16 ? 4 : 2;
                for (int e0 = threadIdx.x; e0 < nbox; e0 += 256 * EPI) {
                    long long vv[EPI];
                    bool in[EPI];
#pragma unroll
                    for (int i = 0; i < EPI; ++i) in[i] = voxel(e0 + 256 * i, vv[i]);
                    float x[EPI][NCM];
#pragma unroll
                    for (int g = 0; g < NCM; ++g) {
#pragma unroll
                        for (int i = 0; i < EPI; ++i) x[i][g] = 0.0f;
                        if (g < ng) {
                            const float *ch = cT + (long long)gch[g] * V;
#pragma unroll
                            for (int i = 0; i < EPI; ++i) x[i][g] = ch[vv[i]];
                        }
                    }
                    float m[EPI][UP];
#pragma unroll
                    for (int i = 0; i < EPI; ++i)
#pragma unroll
                        for (int u = 0; u < UP; ++u) m[i][u] = 0.0f;
#pragma unroll
                    for (int g = 0; g < NCM; ++g) {
                        if (g < ng) {
#pragma unroll
                            for (int u = 0; u < UP; ++u) {
                                const float wv = gw[g * UP + u];
#pragma unroll
                                for (int i = 0; i < EPI; ++i) m[i][u] = fmaf(wv, x[i][g], m[i][u]);
                            }
                        }
                    }
#pragma unroll
                    for (int q = 0; q < Q; ++q)
#pragma unroll
                        for (int i = 0; i < EPI; ++i)
                            if (e0 + 256 * i < nbox)
                                box[q * nbs + e0 + 256 * i] =
                                    in[i] ? f4{m[i][4 * q], m[i][4 * q + 1], m[i][4 * q + 2], m[i][4 * q + 3]}
                                          : f4{0.f, 0.f, 0.f, 0.f};
                }
              } else {
                // work item (box voxel e, segment u = thread mod UP), VS voxels per
                // pass; EF items per thread have their loads in flight together
                // (an item outside the volume reads c's first voxel and stores 0)
                constexpr int VS = 256 / UP, EF = 4;
                const int u = threadIdx.x & (UP - 1);
                float *boxf = reinterpret_cast<float *>(box) + (long long)(u >> 2) * nbs * 4 + (u & 3);
                const int2 *tu = tab + u * kk;
                const int v0 = threadIdx.x / UP;
                int pl = v0 / plane, ib = (v0 - pl * plane) / EZ, iz = v0 - pl * plane - ib * EZ;
                const int t_pl = VS / plane, t_r = VS - t_pl * plane, t_ib = t_r / EZ, t_iz = t_r - t_ib * EZ;
                const int nA = A == 0 ? nx : ny, nB = A == 0 ? ny : nx;
                for (int e0 = v0; e0 < nbox; e0 += VS * EF) {
                    const float *src[EF];
                    bool ok[EF];
#pragma unroll
                    for (int i = 0; i < EF; ++i) {
                        const int a = A0 + pl - 1, bq = B0 + ib - 1, z = Z0 + iz - 1;
                        ok[i] = u < U && e0 + VS * i < nbox && (unsigned)a < (unsigned)nA &&
                                (unsigned)bq < (unsigned)nB && (unsigned)z < (unsigned)nz;
                        const int x = A == 0 ? a : bq, y = A == 0 ? bq : a;
                        src[i] = M + (ok[i] ? ((long long)(x * ny + y) * nz + z) * C : 0LL);
                        pl += t_pl;
                        ib += t_ib;
                        iz += t_iz;
                        if (iz >= EZ) {
                            iz -= EZ;
                            ++ib;
                        }
                        if (ib >= EB) {
                            ib -= EB;
                            ++pl;
                        }
                    }
                    float v[EF];
#pragma unroll
                    for (int i = 0; i < EF; ++i) v[i] = 0.0f;
#pragma unroll 2
                    for (int t = 0; t < kk; ++t) {
                        const int2 te = tu[t];
                        const float wt = __int_as_float(te.y);
#pragma unroll
                        for (int i = 0; i < EF; ++i) v[i] = fmaf(wt, src[i][te.x], v[i]);
                    }
#pragma unroll
                    for (int i = 0; i < EF; ++i)
                        if (e0 + VS * i < nbox) boxf[(e0 + VS * i) * 4] = ok[i] ? v[i] : 0.0f;
                }
              }
            } else {
            // direct global -> LDS copies (gfx950 global_load_lds, 16 bytes a
            // lane): wave w copies elements e = 256 i + 64 w + lane of every
            // float4 component array, all in flight together; elements outside
            // the padded volume and the tail up to the 64-element stride copy
            // the zero border voxel at padded index 0
            const f4 *src0 = reinterpret_cast<const f4 *>(Mp) + ((long long)A0 * sA + (long long)B0 * sB + Z0) * Q;
            const f4 *zsrc = reinterpret_cast<const f4 *>(Mp);
            const int wb = threadIdx.x & ~63, lane = threadIdx.x & 63;
            int pl = e_pl, ib = e_ib, iz = e_iz, off = e_pl * sA + e_ib * sB + e_iz;
            for (int eb = wb; eb < nbox; eb += 256) {
                const bool in = eb + lane < nbox && (unsigned)(A0 + pl) <= nAp && (unsigned)(B0 + ib) <= nBp &&
                                (unsigned)(Z0 + iz) <= nZp;
                const f4 *gsrc = in ? src0 + (long long)off * Q : zsrc;
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gsrc + q),
                                                     (__attribute__((address_space(3))) void *)(box + q * nbs + eb),
                                                     16, 0, 0);
                // advance by 256 elements
                pl += s_pl;
                ib += s_ib;
                iz += s_iz;
                off += s_off;
                if (iz >= EZ) {
                    iz -= EZ;
                    ++ib;
                    off += cz_off;
                }
                if (ib >= EB) {
                    ib -= EB;
                    ++pl;
                    off += cb_off;
                }
            }
            __builtin_amdgcn_s_waitcnt(0);
            }
            __syncthreads();
            // samples of this slab: index position along A below A0 + W
            int m_end = m;
            if (m < count) m_end = min(count, max(m, (int)ceil((A0 + W - q0[A]) * inv_dqA)));
            // positions relative to the box origin, in float32 (magnitudes of a
            // few tens); the cell is clamped into the box and the fractions are
            // taken against the clamped cell, so a sample that rounding puts
            // on the far side of a slab face still interpolates correctly
            const float ra = (float)(fma((double)m, dq[A], q0[A]) - A0);
            const float rb = (float)(fma((double)m, dq[B], q0[B]) - B0);
            const float rz = (float)(fma((double)m, dq[2], q0[2]) - Z0);
            float mm = 0.0f;
            for (; m < m_end; ++m, mm += 1.0f) {
                const float pa = fmaf(mm, dqA, ra), pb = fmaf(mm, dqB, rb), pz = fmaf(mm, dqZ, rz);
                const float la = fminf(fmaxf(floorf(pa), 0.0f), wmax);
                const float lbb = fminf(fmaxf(floorf(pb), 0.0f), bmax);
                const float lz = fminf(fmaxf(floorf(pz), 0.0f), zmax);
                const float fa = pa - la, fb = pb - lbb, fz = pz - lz;
                const float ga_ = 1.0f - fa, gb_ = 1.0f - fb, gz_ = 1.0f - fz;
                const float w00 = ga_ * gb_, w01 = ga_ * fb, w10 = fa * gb_, w11 = fa * fb;
                const float w[8] = {w00 * gz_, w00 * fz, w01 * gz_, w01 * fz, w10 * gz_, w10 * fz, w11 * gz_, w11 * fz};
                const int off8[8] = {0, dz, db, db + dz, da, da + dz, da + db, da + db + dz};
                const int base = __umul24(__umul24((int)la, EB) + (int)lbb, EZ) + (int)lz;
#pragma unroll
                for (int cc = 0; cc < 8; ++cc) {
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        const f4 mv = box[q * nbs + base + off8[cc]];
                        acc[4 * q + 0] = fmaf(w[cc], mv.x, acc[4 * q + 0]);
                        acc[4 * q + 1] = fmaf(w[cc], mv.y, acc[4 * q + 1]);
                        acc[4 * q + 2] = fmaf(w[cc], mv.z, acc[4 * q + 2]);
                        acc[4 * q + 3] = fmaf(w[cc], mv.w, acc[4 * q + 3]);
                    }
                }
            }
        }
    }
    if (!live) return;
    const float wgt = jos ? f.jos_w : step;  // Joseph: each cut weighs 1 / |d_A|
    float *out = I + (((long long)s * nj + j) * nk + k) * nseg;
#pragma unroll
    for (int u = 0; u < UP; ++u) {
        if (u < U) {
            for (int cseg = u; cseg < nseg; cseg += U) out[cseg] = wgt * acc[u];
        }
    }
}

// ---------------------------------------------------------------------------
// march over a ring of staged planes (four or eight unique segments): one thread
// per ray, block = 16 x 16 rays of one projection, as k_march, with one plane of the
// slab axis A staged per step instead of a slab of them.
//
// Plane a holds the voxels that the tile's samples with index position in
// [a - 1, a + 1) along A touch, from its own origin; a sample in [a, a + 1) reads
// planes a and a + 1.  The ring keeps R planes: while the rays gather from a and
// a + 1, the copies of a + 2 .. a + R - 1 are in flight, so a step waits only for a copy
// issued R - 2 steps before.  One barrier per step: it ends the reads of plane a - 1,
// whose slot then takes plane a + R - 1.
//
// What bounded the slab march: every slab waited for its own copies with nothing in
// flight beside them (32^3, one block per compute unit: 47 of 59 us), and its staging
// took about as many VALU instructions as the samples.  Here a thread's elements of a
// plane are the same for all planes, so inside the volume a copy is one add.  March in ms,
// slabs -> rings: 32^3 x 4 unique segments 0.062 -> 0.043, 100^3 x 4 1.59 -> 1.37,
// 128^3 x 8 7.71 -> 6.38, 256^3 x 8 73.1 -> 62.1.  What bounds it now is latency: at 128^3
// VALU issue takes 52% of the cycles and the LDS 50% (half of that bank conflicts of the
// corner reads, 16 bytes per corner and four segments), and the two blocks that fit a
// compute unit (1.9 waves per SIMD) do not cover one with the other.
//
// A plane's float4 halves (eight segments) lie one after the other, so that neighbouring
// voxels are 16 bytes apart and a wave's reads spread over all banks (interleaved by
// voxel: 256^3 63.2, 128^3 6.46 ms).
//
// The copies are written in assembly, because the compiler otherwise waits for all of
// them before any LDS read (it cannot tell the slots apart); they have no register
// output.  wait_copies is the only wait for them.
// ---------------------------------------------------------------------------
constexpr int kRingCopies = 8;  // copies of 64 float4 per wave and plane (at most)

__device__ __forceinline__ void copy_to_lds(const void *base, unsigned off, unsigned lds_byte)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_byte), "v"(off), "s"(base)
                 : "memory", "m0");
}

// x in 32.32 fixed point, in scalar registers
__device__ __forceinline__ long long fixed32(double x)
{
    const double hi = floor(x);
    const int h = __builtin_amdgcn_readfirstlane((int)hi);
    const unsigned l = __builtin_amdgcn_readfirstlane((unsigned)((x - hi) * 4294967296.0));
    return (long long)(((unsigned long long)(unsigned)h << 32) | l);
}

// waits until at most n of this wave's copies are outstanding (n uniform; more than
// 24 as 24), and for its LDS reads
__device__ __forceinline__ void wait_copies(int n)
{
    switch (n) {
#define TT_WAIT(k) \
    case k: asm volatile("s_waitcnt vmcnt(" #k ") lgkmcnt(0)" ::: "memory"); break;
        TT_WAIT(0) TT_WAIT(1) TT_WAIT(2) TT_WAIT(3) TT_WAIT(4) TT_WAIT(5) TT_WAIT(6) TT_WAIT(7) TT_WAIT(8)
        TT_WAIT(9) TT_WAIT(10) TT_WAIT(11) TT_WAIT(12) TT_WAIT(13) TT_WAIT(14) TT_WAIT(15) TT_WAIT(16)
        TT_WAIT(17) TT_WAIT(18) TT_WAIT(19) TT_WAIT(20) TT_WAIT(21) TT_WAIT(22) TT_WAIT(23)
#undef TT_WAIT
    default: asm volatile("s_waitcnt vmcnt(24) lgkmcnt(0)" ::: "memory"); break;
    }
}

template <int UP>
__global__ __launch_bounds__(256) void k_march_ring(const float *__restrict__ M, const ProjFrame *__restrict__ frames,
                                                    int s0, int nx, int ny, int nz, int nj, int nk, int nseg, int U,
                                                    float step, long long vol_pad, float *__restrict__ I, int jos,
                                                    int kind)
{
    constexpr int Q = UP / 4;
    extern __shared__ f4 ring[];  // [R][Q][plane voxel]
    __shared__ int arange[2];
    const int ntj = (nj + kMarchTile - 1) / kMarchTile, ntk = (nk + kMarchTile - 1) / kMarchTile;
    const int lb = blockIdx.x;
    const int p = lb / (ntj * ntk), s = s0 + p;
    const ProjFrame &f = frames[s];
    const int R = f.ring_r[kind];
    if (R == 0) return;  // this projection runs in another launch
    const int tj = (lb / ntk) % ntj, tk = lb % ntk;
    const int j = tj * kMarchTile + (threadIdx.x % kMarchTile);
    const int k = tk * kMarchTile + (threadIdx.x / kMarchTile);
    const bool live = j < nj && k < nk;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    double b[3], ds[3];
    int n0 = 0, n1 = -1;
    if (live) ray_setup(f, j, k, nx, ny, nz, step, b, ds, n0, n1, jos != 0);
    float acc[UP];
#pragma unroll
    for (int u = 0; u < UP; ++u) acc[u] = 0.0f;

    const int A = f.slab_a, B = 1 - A, EB = f.ring_eb, EZ = f.ring_ez;
    const bool fwd = f.d[A] > 0.0;  // samples are visited in increasing index coordinate along A
    int left = n1 - n0 + 1;         // samples still to visit
    if (threadIdx.x == 0) {
        arange[0] = INT_MAX;
        arange[1] = INT_MIN;
    }
    __syncthreads();
    if (left > 0) {
        const int nf = fwd ? n0 : n1, nl = fwd ? n1 : n0;
        atomicMin(&arange[0], (int)floor(fma((double)nf, A ? ds[1] : ds[0], A ? b[1] : b[0])));
        atomicMax(&arange[1], (int)floor(fma((double)nl, A ? ds[1] : ds[0], A ? b[1] : b[0])));
    }
    __syncthreads();
    const int amin = __builtin_amdgcn_readfirstlane(arange[0]), amax = __builtin_amdgcn_readfirstlane(arange[1]);
    if (amin <= amax) {
        // Origin of plane a: the lowest position along B and z of the tile's rays
        // between planes a - 1 and a + 1, kb + a rB and kz + a rZ (affine in a)
        const double n3[3] = {(double)nx, (double)ny, (double)nz};
        double b00[3];
#pragma unroll
        for (int q = 0; q < 3; ++q)
            b00[q] = f.o[q] + (tj * kMarchTile) * f.ej[q] + (tk * kMarchTile) * f.ek[q] + 0.5 * (n3[q] + 1.0);
        const double rB = f.d[B] * f.inv_d[A], rZ = f.d[2] * f.inv_d[A];
        double kb = 1e300, kz = 1e300;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const double J = (v & 1) ? kMarchTile - 1 : 0.0, K = (v & 2) ? kMarchTile - 1 : 0.0, P = (v & 4) ? 1.0 : -1.0;
            const double t = P - (b00[A] + J * f.ej[A] + K * f.ek[A]);
            kb = fmin(kb, b00[B] + J * f.ej[B] + K * f.ek[B] + t * rB);
            kz = fmin(kz, b00[2] + J * f.ej[2] + K * f.ek[2] + t * rZ);
        }
        // in fixed point, stepped from plane to plane by scalar adds (off by 2^-32 per
        // plane at most, within the 1e-6 that the origin is lowered by)
        const long long rBf = fixed32(rB), rZf = fixed32(rZ);
        long long gB = fixed32(fma((double)amin, rB, kb - 1e-6)), gZ = fixed32(fma((double)amin, rZ, kz - 1e-6));
        long long tB = gB, tZ = gZ;  // of the next plane to stage; gB, gZ of the plane gathered from
        // M strides (in voxels) of the plane's axes; z is contiguous
        const int sy = nz + 2, sx = (ny + 2) * sy;
        const int sA = A == 0 ? sx : sy, sB = A == 0 ? sy : sx;
        const int nAp = (A == 0 ? nx : ny) + 1, nBp = (A == 0 ? ny : nx) + 1, nZp = nz + 1;
        // this lane's elements of a plane: wave w copies elements 256 i + 64 w + lane;
        // byte offset from the plane's origin, and (row, z) for planes that leave the volume
        const int nel = EB * EZ * Q, nch = (nel + 63) >> 6, slot_bytes = nch * 1024;
        const int ncp = (nch - wave + 3) >> 2;  // copies of this wave per plane
        unsigned off[kRingCopies], rz[kRingCopies];
#pragma unroll
        for (int i = 0; i < kRingCopies; ++i) {
            const int e = min(256 * i + 64 * wave + lane, nel - 1);
            const int qe = Q == 2 && e >= EB * EZ ? 1 : 0, vox = e - qe * EB * EZ;
            const int ib = vox / EZ, iz = vox - ib * EZ;
            off[i] = (unsigned)((ib * sB + iz) * Q + qe) * 16u;
            rz[i] = (unsigned)(ib << 16 | iz << 4 | qe);
        }
        const char *Mp = reinterpret_cast<const char *>(M) + (long long)p * vol_pad * UP * 4;
        const unsigned ring0 = __builtin_amdgcn_readfirstlane(
            (unsigned)(uintptr_t)(__attribute__((address_space(3))) char *)ring + wave * 1024);
        auto stage = [&](int a, int slot) {
            const int B0 = (int)(tB >> 32), Z0 = (int)(tZ >> 32);
            tB += rBf;
            tZ += rZf;
            const unsigned dst = ring0 + slot * slot_bytes;
            if (a >= 0 && a <= nAp && B0 >= 0 && B0 + EB - 1 <= nBp && Z0 >= 0 && Z0 + EZ - 1 <= nZp) {
                const char *src = Mp + ((long long)a * sA + (long long)B0 * sB + Z0) * (Q * 16);
#pragma unroll
                for (int i = 0; i < kRingCopies; ++i)
                    if (i < ncp) copy_to_lds(src, off[i], dst + i * 4096);
            } else {  // voxels outside the padded volume copy one of its border, which is zero
                const char *src = Mp + (long long)min(max(a, 0), nAp) * sA * (Q * 16);
#pragma unroll
                for (int i = 0; i < kRingCopies; ++i)
                    if (i < ncp) {
                        const int vb = min(max(B0 + (int)(rz[i] >> 16), 0), nBp);
                        const int vz = min(max(Z0 + (int)(rz[i] >> 4 & 0xfff), 0), nZp);
                        copy_to_lds(src, (unsigned)((vb * sB + vz) * Q + (int)(rz[i] & 15)) * 16u, dst + i * 4096);
                    }
            }
        };
        // current sample's index position (float64: sums of up to the ray's length)
        double pA, pB, pZ;
        const double dA = fwd ? (A ? ds[1] : ds[0]) : -(A ? ds[1] : ds[0]);
        const double dB = fwd ? (A ? ds[0] : ds[1]) : -(A ? ds[0] : ds[1]), dZ = fwd ? ds[2] : -ds[2];
        {
            const double m0 = (double)(fwd ? n0 : n1);
            pA = fma(m0, A ? ds[1] : ds[0], A ? b[1] : b[0]);
            pB = fma(m0, A ? ds[0] : ds[1], A ? b[0] : b[1]);
            pZ = fma(m0, ds[2], b[2]);
        }
        const float bmax = (float)(EB - 2), zmax = (float)(EZ - 2);
        const int row_bytes = EZ * 16, q_f4 = EB * EZ;

        const int last = amax + 1;  // last plane needed
        int issued = amin - 1;      // last plane whose copies are issued
        for (int i = 0; i < R - 1 && issued < last; ++i) {
            ++issued;
            stage(issued, i);
        }
        int slot = 0;
        for (int a = amin; a <= amax; ++a) {
            wait_copies(max(0, issued - (a + 1)) * ncp);
            __builtin_amdgcn_s_barrier();  // planes a, a + 1 are staged; plane a - 1 is read
            asm volatile("" ::: "memory");
            const int nslot = slot + 1 == R ? 0 : slot + 1;
            if (issued < last) {
                ++issued;
                stage(issued, slot == 0 ? R - 1 : slot - 1);
            }
            const int B0 = (int)(gB >> 32), Z0 = (int)(gZ >> 32);
            gB += rBf;
            gZ += rZf;
            const int B1 = (int)(gB >> 32), Z1 = (int)(gZ >> 32);
            // bytes from a voxel of plane a to the same (B, z) in plane a + 1
            const int up = (nslot - slot) * slot_bytes + ((B0 - B1) * EZ + Z0 - Z1) * 16;
            const char *pl = reinterpret_cast<const char *>(ring) + slot * slot_bytes;
            // (the last step takes what is left, also where the summed position of a
            // last sample is rounded to the far side of its plane)
            const double aend = a == amax ? 1e300 : (double)(a + 1);
            while (left > 0 && pA < aend) {
                // the cell is clamped into the plane's box and the fractions are taken
                // against the clamped cell (float32 may round a position up to a face)
                const float fa = (float)(pA - (double)a), pb = (float)(pB - (double)B0), pz = (float)(pZ - (double)Z0);
                const float lbb = fminf(fmaxf(floorf(pb), 0.0f), bmax), lz = fminf(fmaxf(floorf(pz), 0.0f), zmax);
                const float fb = pb - lbb, fz = pz - lz;
                const float ga_ = 1.0f - fa, gb_ = 1.0f - fb, gz_ = 1.0f - fz;
                const float w00 = ga_ * gb_, w01 = ga_ * fb, w10 = fa * gb_, w11 = fa * fb;
                const float w[8] = {w00 * gz_, w00 * fz, w01 * gz_, w01 * fz, w10 * gz_, w10 * fz, w11 * gz_, w11 * fz};
                const char *c0 = pl + (__umul24((int)lbb, EZ) + (int)lz) * 16;
                const f4 *cell[4] = {reinterpret_cast<const f4 *>(c0), reinterpret_cast<const f4 *>(c0 + row_bytes),
                                     reinterpret_cast<const f4 *>(c0 + up),
                                     reinterpret_cast<const f4 *>(c0 + up + row_bytes)};
#pragma unroll
                for (int cc = 0; cc < 8; ++cc) {
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        const f4 mv = cell[cc >> 1][(cc & 1) + q * q_f4];
                        acc[4 * q + 0] = fmaf(w[cc], mv.x, acc[4 * q + 0]);
                        acc[4 * q + 1] = fmaf(w[cc], mv.y, acc[4 * q + 1]);
                        acc[4 * q + 2] = fmaf(w[cc], mv.z, acc[4 * q + 2]);
                        acc[4 * q + 3] = fmaf(w[cc], mv.w, acc[4 * q + 3]);
                    }
                }
                pA += dA;
                pB += dB;
                pZ += dZ;
                --left;
            }
            slot = nslot;
        }
    }
    if (!live) return;
    const float wgt = jos ? f.jos_w : step;  // Joseph: each cut weighs 1 / |d_A|
    float *out = I + (((long long)s * nj + j) * nk + k) * nseg;
#pragma unroll
    for (int u = 0; u < UP; ++u) {
        if (u < U) {
            for (int cseg = u; cseg < nseg; cseg += U) out[cseg] = wgt * acc[u];
        }
    }
}

// Which projections run on rings is the geometry's (plan_rings), so that the forward batch
// changes no result; in how many launches they do is the batch's.  Two, by LDS size, need
// blocks enough that the second one's length is less than what the smaller rings gain.
// March of all batches in ms, rings in one launch and in two, beside a launch of slabs in
// batches that have a projection without a ring (in brackets, projections in random order,
// so that every batch has all kinds):
//                            blocks    one          two          slabs only
//   128^3 x 8 / 300 projections 512    9.28 (13.4)  12.1 (19.3)  10.5 (12.3)
//                              2048    8.18 (9.73)  8.69 (10.4)  8.79 (9.06)
//                              4096    7.58 (8.39)  7.41 (8.26)  8.14 (8.35)
//                              6144    7.32 (8.04)  7.17 (7.74)  8.02 (8.14)
//   200^3 x 8 / 120            2704    11.0 (11.9)  11.1 (12.1)  11.7 (11.7)
//                              5408    10.2 (10.4)  9.72 (10.0)  11.0 (11.0)
//   100^3 x 4 / 240             784    2.12 (2.25)  2.45 (3.12)  2.49 (2.65)
//                              3136    1.73 (1.72)  1.76 (1.96)  1.92 (1.91)
//                             11760    1.46 (1.49)  1.37 (1.37)  1.60 (1.63)
//   200^3 x 4 / 120            5408    5.08 (5.09)  4.81 (4.91)  5.58 (5.54)
//   90^3 x 4 / 240             8640    1.08 (1.09)  1.02 (1.03)  1.18 (1.21)
// (With four segments from 4096 blocks on only where a batch has one kind of projection,
// which then is one launch.)
template <int UP>
static hipError_t march_t(const Dims &d, const ProjFrame *frames, const float *M, int s0, int np, float *I,
                          hipStream_t st)
{
    const long long vol_pad = (long long)(d.nx + 2) * (d.ny + 2) * (d.nz + 2);
    dim3 grid(((d.nk + kMarchTile - 1) / kMarchTile) * ((d.nj + kMarchTile - 1) / kMarchTile) * np);
    bool rings = false;  // projections that have a ring run on it
    if constexpr (UP <= 8) {
        auto in = [&](int kind) {  // projections of this batch in a launch
            const int *sum = d.ring_sums + (size_t)kind * (d.S + 1);
            return sum[s0 + np] - sum[s0];
        };
        auto launch = [&](int kind) {
            hipLaunchKernelGGL((k_march_ring<UP>), grid, dim3(kMarchTile * kMarchTile), d.ring_lds[kind], st, M, frames, s0,
                               d.nx, d.ny, d.nz, d.nj, d.nk, d.nseg, d.U, d.step, vol_pad, I, d.joseph, kind);
            return hipGetLastError();
        };
        const int all = in(kRingOne), kinds = (in(kRingSmall) > 0) + (in(kRingLarge) > 0) + (all < np);
        if (in(kRingWhole) == np) return launch(kRingWhole);
        const bool two = grid.x >= (UP == 8 || kinds == 1 ? 4096 : 8192);
        rings = all > 0;
        for (const int kind : {kRingOne, kRingSmall, kRingLarge})
            if (two == (kind != kRingOne) && in(kind) > 0)
                if (hipError_t e = launch(kind); e != hipSuccess) return e;
        if (all == np) return hipSuccess;
    }
    hipLaunchKernelGGL((k_march<UP, false>), grid, dim3(kMarchTile * kMarchTile), d.march_lds, st, M, frames, s0,
                       d.nx, d.ny, d.nz, d.nj, d.nk, d.nseg, d.U, d.step, vol_pad, I, nullptr, 0, 0, nullptr, nullptr, 0,
                       d.joseph, (int)rings);
    return hipGetLastError();
}

template <int UP>
static hipError_t march_fused_t(const Dims &d, const ProjFrame *frames, const float *c, const int2 *sp,
                                const float *cT, const int *gtab, float *I, hipStream_t st)
{
    dim3 grid(((d.nk + kMarchTile - 1) / kMarchTile) * ((d.nj + kMarchTile - 1) / kMarchTile) * d.S);
    const int lds = (UP * d.sparse_k * 8 + 15) / 16 * 16 + (d.sparse_ng * (UP + 1) * 4 + 15) / 16 * 16 + d.march_lds;
    // channel-major staging unrolled for up to 8, 16 or kFusedCmChannels
    // channels (the wider forms cost registers that narrow lists do not need)
    static_assert(kFusedCmChannels == 32, "the widths below");
    if (cT && d.sparse_ng > kFusedCmChannels) return hipErrorInvalidValue;
    if (cT && d.sparse_ng > 16)
        hipLaunchKernelGGL((k_march<UP, true, 32>), grid, dim3(kMarchTile * kMarchTile), lds, st, c, frames, 0, d.nx,
                           d.ny, d.nz, d.nj, d.nk, d.nseg, d.U, d.step, 0LL, I, sp, d.sparse_k, d.C, cT, gtab,
                           d.sparse_ng, d.joseph, 0);
    else if (cT && d.sparse_ng > 8)
        hipLaunchKernelGGL((k_march<UP, true, 16>), grid, dim3(kMarchTile * kMarchTile), lds, st, c, frames, 0, d.nx,
                           d.ny, d.nz, d.nj, d.nk, d.nseg, d.U, d.step, 0LL, I, sp, d.sparse_k, d.C, cT, gtab,
                           d.sparse_ng, d.joseph, 0);
    else
        hipLaunchKernelGGL((k_march<UP, true, 8>), grid, dim3(kMarchTile * kMarchTile), lds, st, c, frames, 0, d.nx,
                           d.ny, d.nz, d.nj, d.nk, d.nseg, d.U, d.step, 0LL, I, sp, d.sparse_k, d.C, cT, gtab,
                           d.sparse_ng, d.joseph, 0);
    return hipGetLastError();
}

// cT[i][v] = c[v][i]: 64 voxels per block step, staged in LDS (odd row stride)
__global__ __launch_bounds__(256) void k_channel_major(const float *__restrict__ c, long long V, int C,
                                                       float *__restrict__ cT)
{
    extern __shared__ float tile[];  // [64][C + 1]
    const int ld = C + 1;
    for (long long v0 = (long long)blockIdx.x * 64; v0 < V; v0 += (long long)gridDim.x * 64) {
        const int nv = (int)min(64LL, V - v0);
        __syncthreads();
        for (int e = threadIdx.x; e < nv * C; e += 256) {
            const int v = e / C, i = e - v * C;
            tile[v * ld + i] = c[v0 * C + e];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < 64 * C; e += 256) {
            const int i = e >> 6, v = e & 63;
            if (v < nv) cT[(long long)i * V + v0 + v] = tile[v * ld + i];
        }
    }
}

hipError_t launch_march_fused(const Dims &d, const ProjFrame *frames, const float *c, const int2 *sp,
                              const int *gtab, float *cT, float *I, hipStream_t st)
{
    if (d.sparse_k < 1) return hipErrorInvalidValue;
    const long long V = (long long)d.nx * d.ny * d.nz;
    if (d.sparse_cm) {
        hipLaunchKernelGGL(k_channel_major, dim3((unsigned)std::min<long long>((V + 63) / 64, 4096)), dim3(256),
                           64 * (d.C + 1) * sizeof(float), st, c, V, d.C, cT);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    } else {
        cT = nullptr;  // stage from the coefficient records
    }
    switch (d.Up) {
    case 4: return march_fused_t<4>(d, frames, c, sp, cT, gtab, I, st);
    case 8: return march_fused_t<8>(d, frames, c, sp, cT, gtab, I, st);
    case 16: return march_fused_t<16>(d, frames, c, sp, cT, gtab, I, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_march(const Dims &d, const ProjFrame *frames, const float *M, int s0, int np, float *I,
                        hipStream_t st)
{
    switch (d.Up) {
    case 4: return march_t<4>(d, frames, M, s0, np, I, st);
    case 8: return march_t<8>(d, frames, M, s0, np, I, st);
    case 16: return march_t<16>(d, frames, M, s0, np, I, st);
    default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// fold: yf = scale * antipodal fold of y (zero beyond U).
// ---------------------------------------------------------------------------
template <int UP>
__global__ __launch_bounds__(256) void k_fold(const float *__restrict__ y, long long npix, int nseg, int U,
                                              float scale, float *__restrict__ yf)
{
    for (long long px = blockIdx.x * 256LL + threadIdx.x; px < npix; px += (long long)gridDim.x * 256) {
        const float *yr = y + px * nseg;
        float acc[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) acc[u] = 0.0f;
#pragma unroll
        for (int u = 0; u < UP; ++u)
            if (u < U)
                for (int cseg = u; cseg < nseg; cseg += U) acc[u] += yr[cseg];
        f4 *o = reinterpret_cast<f4 *>(yf + px * UP);
#pragma unroll
        for (int u4 = 0; u4 < UP; u4 += 4)
            o[u4 / 4] = f4{scale * acc[u4], scale * acc[u4 + 1], scale * acc[u4 + 2], scale * acc[u4 + 3]};
    }
}

static int grid_for(long long n) { return (int)min((n + 255) / 256, 4096LL); }

hipError_t launch_fold(const Dims &d, const float *y, float scale, float *yf, hipStream_t st)
{
    const long long npix = (long long)d.S * d.nj * d.nk;
    const int g = grid_for(npix);
    switch (d.Up) {
    case 4: hipLaunchKernelGGL(k_fold<4>, dim3(g), dim3(256), 0, st, y, npix, d.nseg, d.U, scale, yf); break;
    case 8: hipLaunchKernelGGL(k_fold<8>, dim3(g), dim3(256), 0, st, y, npix, d.nseg, d.U, scale, yf); break;
    case 16: hipLaunchKernelGGL(k_fold<16>, dim3(g), dim3(256), 0, st, y, npix, d.nseg, d.U, scale, yf); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// r = Ip - data; yf = step * fold(2 w r); partial sums of w r^2 per block.
template <int UP>
__global__ __launch_bounds__(256) void k_residual_fold(const float *__restrict__ Ip, const float *__restrict__ data,
                                                       const float *__restrict__ w, float *r, long long npix,
                                                       int nseg, int U, float step, float *__restrict__ yf,
                                                       double *__restrict__ partials)
{
    __shared__ double ws[4];
    double loss = 0.0;
    for (long long px = blockIdx.x * 256LL + threadIdx.x; px < npix; px += (long long)gridDim.x * 256) {
        float acc[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) acc[u] = 0.0f;
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            if (u < U) {
                for (int cseg = u; cseg < nseg; cseg += U) {
                    long long e = px * nseg + cseg;
                    float rv = Ip[e] - data[e];
                    float wv = w ? w[e] : 1.0f;
                    if (r) r[e] = rv;
                    loss += (double)wv * (double)rv * (double)rv;
                    acc[u] += 2.0f * wv * rv;
                }
            }
        }
        f4 *o = reinterpret_cast<f4 *>(yf + px * UP);
#pragma unroll
        for (int u4 = 0; u4 < UP; u4 += 4)
            o[u4 / 4] = f4{step * acc[u4], step * acc[u4 + 1], step * acc[u4 + 2], step * acc[u4 + 3]};
    }
    double tot = block_sum(loss, ws);
    if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

hipError_t launch_residual_fold(const Dims &d, const float *Ip, const float *data, const float *w, float *r,
                                float *yf, double *partials, int nblocks, hipStream_t st)
{
    const long long npix = (long long)d.S * d.nj * d.nk;
    switch (d.Up) {
    case 4:
        hipLaunchKernelGGL(k_residual_fold<4>, dim3(nblocks), dim3(256), 0, st, Ip, data, w, r, npix, d.nseg, d.U,
                           d.step, yf, partials);
        break;
    case 8:
        hipLaunchKernelGGL(k_residual_fold<8>, dim3(nblocks), dim3(256), 0, st, Ip, data, w, r, npix, d.nseg, d.U,
                           d.step, yf, partials);
        break;
    case 16:
        hipLaunchKernelGGL(k_residual_fold<16>, dim3(nblocks), dim3(256), 0, st, Ip, data, w, r, npix, d.nseg,
                           d.U, d.step, yf, partials);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// backproject (sixteen unique segments): block = brick of 4 (x) x 8 (y) x 8 (z) voxels; wave w owns the
// x-slice w (64 voxels = 4 column tiles of 16).  Loops over all projections.
// ---------------------------------------------------------------------------
// Q tile entry (u = 4 ks + lane / 16) of voxel column 16 nt + lane % 16 (row stride UP + 1)
template <int UP>
__device__ __forceinline__ float qw_at(const float *Qw, int nt, int ks, int lane)
{
    return Qw[(nt * 16 + (lane & 15)) * (UP + 1) + ks * 4 + (lane >> 4)];
}

// Samples of one ray inside the cube of a voxel.  The dominant axis of d comes
// first in the frame's float vectors: |P_0 + tau d_0| < 1 bounds tau to an
// interval of length 2 / |d_0| that holds at most n_tau samples, and the tent
// factors, clamped at 0, drop those outside the cube along the other axes.
// So every ray evaluates the same n_tau samples (three, or four for steep
// diagonals, at step 1) without a branch; kept as a range per ray over all
// three axes, a loop and its exec masks, the adjoint's lanes waited for the
// ray with the most samples at every step.  (Also at small steps, where the range is
// shorter: 64^3 / 120 projections / 4 unique segments at step 0.1 1136 us with a
// range, 1068 with the fixed number, 870 with its loop unrolled by four.)
struct TentRay {
    float d[3], sd[3];  // ray direction, and the sample spacing along each axis
    float ca, cb;       // first sample: n = ceil(ca P_0 + cb)
    float step, off;    // tau = step n + off
    int more;           // samples beyond three (uniform over the projection)
};

__device__ __forceinline__ TentRay tent_ray(const ProjFrame &f, float tr, float step, float inv_step)
{
    TentRay t;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        t.d[a] = f.df[a];
        t.sd[a] = step * f.df[a];
    }
    t.ca = -f.inv_d0 * inv_step;
    t.cb = tr - fabsf(f.inv_d0) * inv_step;
    t.step = step;
    t.off = -tr * step;
    t.more = f.n_tau - 3;
    return t;
}

// max(0, 1 - |x|), one instruction (clamp modifier)
__device__ __forceinline__ float tent1(float x) { return __builtin_amdgcn_fmed3f(1.0f - fabsf(x), 0.0f, 1.0f); }

template <bool MANY>
__device__ __forceinline__ float ray_weight(const float P[3], const TentRay &t)
{
    const float tau = fmaf(ceilf(fmaf(t.ca, P[0], t.cb)), t.step, t.off);
    float x = fmaf(tau, t.d[0], P[0]), y = fmaf(tau, t.d[1], P[1]), z = fmaf(tau, t.d[2], P[2]);
    float w = tent1(x) * tent1(y) * tent1(z);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        x += t.sd[0];
        y += t.sd[1];
        z += t.sd[2];
        w = fmaf(tent1(x) * tent1(y), tent1(z), w);
    }
    const int fours = MANY ? t.more & ~3 : 0;
    for (int n = 0; n < fours; n += 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x += t.sd[0];
            y += t.sd[1];
            z += t.sd[2];
            w = fmaf(tent1(x) * tent1(y), tent1(z), w);
        }
    }
    for (int i = fours; i < t.more; ++i) {
        x += t.sd[0];
        y += t.sd[1];
        z += t.sd[2];
        w = fmaf(tent1(x) * tent1(y), tent1(z), w);
    }
    return w;
}

template <int UP, int MT, bool BF16, bool JOS>
__global__ __launch_bounds__(256) void k_backproject(const float *__restrict__ yf, const ProjFrame *__restrict__ frames,
                                                     const float *__restrict__ Bu, const s4 *__restrict__ BuT16, int S, int nx, int ny, int nz,
                                                     int nj, int nk, int C, int Cp, float step,
                                                     float *__restrict__ g, float beta, const float *__restrict__ c,
                                                     double *__restrict__ partials)
{
    __shared__ float Qs[4][64 * (UP + 1)];
    __shared__ double ws[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nbx = (nx + 3) / 4, nby = (ny + 7) / 8;
    const int bid = xcd_block(blockIdx.x, gridDim.x);
    const int bx = bid % nbx, by = (bid / nbx) % nby, bz = bid / (nbx * nby);
    const int ix = bx * 4 + wave, iy = by * 8 + (lane >> 3), iz = bz * 8 + (lane & 7);
    const bool valid = ix < nx && iy < ny && iz < nz;
    const double xv[3] = {ix - 0.5 * (nx - 1), iy - 0.5 * (ny - 1), iz - 0.5 * (nz - 1)};
    const double inv_step = 1.0 / (double)step;
    const float stepf = step, inv_stepf = (float)inv_step;

    f4 acc[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = f4{0.f, 0.f, 0.f, 0.f};

    // float32 trilinear path with 8+ unique segments: the last KD of the KS
    // k-steps of projection s's MFMA chain run at the top of projection s + 1,
    // beside that projection's set-up arithmetic, so that no wave issues the
    // whole chain at once (Q_s is still in the wave's LDS tile then)
    constexpr int KS = UP / 4, KD = (BF16 || JOS) ? 0 : KS / 2, KE = KS - KD;
    float pend[KD > 0 ? KD : 1][MT];
    auto deferred_mfma = [&]() {
#pragma unroll
        for (int kd = 0; kd < KD; ++kd) {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const float bv = qw_at<UP>(Qs[wave], nt, KE + kd, lane);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = mfma16x16x4(pend[kd][mt], bv, acc[mt][nt]);
            }
        }
    };
    float *Qw = Qs[wave];
    for (int s = 0; s < S; ++s) {
        const ProjFrame &f = frames[s];
        // this projection's B_s^T operands, loaded now so that the gather below
        // hides their latency (they are only read by the MFMAs at its end)
        s4 avb[MT];
        float avf[UP / 4][MT];
        if constexpr (BF16) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                avb[mt] = BuT16[((long long)s * Cp + mt * 16 + (lane & 15)) * 4 + (lane >> 4)];
        } else {
            const float *Bs = Bu + (long long)s * UP * Cp;
#pragma unroll
            for (int ks = 0; ks < UP / 4; ++ks)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) avf[ks][mt] = Bs[(ks * 4 + (lane >> 4)) * Cp + mt * 16 + (lane & 15)];
        }
        float q[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) q[u] = 0.0f;
        if (JOS && valid) {
            // Joseph's method: the rays whose cut with the voxel's own layer
            // (normal to the dominant axis) lies within one voxel along the two
            // in-plane axes; weight (1 - |Delta_B|)(1 - |Delta_C|) / |d_A|.
            const double w0 = xv[0] - f.o[0], w1 = xv[1] - f.o[1], w2 = xv[2] - f.o[2];
            const double a = w0 * f.ej[0] + w1 * f.ej[1] + w2 * f.ej[2];
            const double bb = w0 * f.ek[0] + w1 * f.ek[1] + w2 * f.ek[2];
            const double af = floor(a), bf = floor(bb);
            const int ai = (int)af, bi = (int)bf;
            const float ar = (float)(a - af), br = (float)(bb - bf);
            const float gjB = f.jos_gj[0], gjC = f.jos_gj[1], gkB = f.jos_gk[0], gkC = f.jos_gk[1];
            const int jlo = max(0, ai + (int)ceilf(ar - f.jos_rj)), jhi = min(nj - 1, ai + (int)floorf(ar + f.jos_rj));
            for (int j = jlo; j <= jhi; ++j) {
                const float dj = (float)(j - ai) - ar;
                const float eB = dj * gjB, eC = dj * gjC;
                // dk range with |dk gk + e| < 1 on both in-plane axes, branch-free: a
                // flat axis (kFlatInv) gives all dk or none, and the other axis is
                // never flat, so a non-empty range is finite
                const float xB1 = (-1.0f - eB) * f.jos_igk[0], xB2 = (1.0f - eB) * f.jos_igk[0];
                const float xC1 = (-1.0f - eC) * f.jos_igk[1], xC2 = (1.0f - eC) * f.jos_igk[1];
                const float lo = fmaxf(fminf(xB1, xB2), fminf(xC1, xC2));
                const float hi = fminf(fmaxf(xB1, xB2), fmaxf(xC1, xC2));
                if (!(lo < hi)) continue;
                const int klo = max(0, bi + (int)ceilf(br + lo - 1e-4f));
                const int khi = min(nk - 1, bi + (int)floorf(br + hi + 1e-4f));
                const f4 *yrow = reinterpret_cast<const f4 *>(yf + ((long long)s * nj + j) * nk * UP);
                for (int k = klo; k <= khi; ++k) {
                    f4 yv[UP / 4];
#pragma unroll
                    for (int u4 = 0; u4 < UP / 4; ++u4) yv[u4] = yrow[k * (UP / 4) + u4];
                    const float dk = (float)(k - bi) - br;
                    const float wB = fmaxf(0.0f, 1.0f - fabsf(fmaf(dk, gkB, eB)));
                    const float wC = fmaxf(0.0f, 1.0f - fabsf(fmaf(dk, gkC, eC)));
                    const float wt = wB * wC * f.jos_w;
#pragma unroll
                    for (int u4 = 0; u4 < UP; u4 += 4) {
                        q[u4 + 0] = fmaf(wt, yv[u4 / 4].x, q[u4 + 0]);
                        q[u4 + 1] = fmaf(wt, yv[u4 / 4].y, q[u4 + 1]);
                        q[u4 + 2] = fmaf(wt, yv[u4 / 4].z, q[u4 + 2]);
                        q[u4 + 3] = fmaf(wt, yv[u4 / 4].w, q[u4 + 3]);
                    }
                }
            }
        }
        if (!JOS && (KD > 0 || valid)) {
            // (with deferred MFMAs evaluated for every lane, so that they share
            // this block; lanes outside the volume visit no rows)
            // Voxel centre in the ray frame: detector coordinates (a, bb) and
            // the along-ray coordinate t / step, in float64 (magnitudes up to
            // the volume size), each split into an integer and a fraction in
            // [0, 1) so that every offset below is a small float32 number.
            const double w0 = xv[0] - f.o[0], w1 = xv[1] - f.o[1], w2 = xv[2] - f.o[2];
            const double a = w0 * f.ej[0] + w1 * f.ej[1] + w2 * f.ej[2];
            const double bb = w0 * f.ek[0] + w1 * f.ek[1] + w2 * f.ek[2];
            const double ts = (w0 * f.d[0] + w1 * f.d[1] + w2 * f.d[2]) * inv_step;
            const double af = floor(a), bf = floor(bb), tf = floor(ts);
            const int ai = (int)af, bi = (int)bf, ti = (int)tf;
            const float ar = (float)(a - af), br = (float)(bb - bf), tr = (float)(ts - tf);
            const TentRay tent = tent_ray(f, tr, stepf, inv_stepf);
            const float ljf = (float)f.lj;
            const int jlo = max(0, ai + (int)ceilf(ar - ljf));
            const int jhi = valid ? min(nj - 1, ai + (int)floorf(ar + ljf)) : jlo - 1;
            if constexpr (KD > 0) {
                if (s > 0) deferred_mfma();
            }
            // hull intercepts shifted by this voxel's fraction br and the 1e-4 slack
            const float cu[3] = {f.hull[1] + (br + 1e-4f), f.hull[3] + (br + 1e-4f), f.hull[5] + (br + 1e-4f)};
            const float cl[3] = {f.hull[7] + (br - 1e-4f), f.hull[9] + (br - 1e-4f), f.hull[11] + (br - 1e-4f)};
            const f4 *ys = reinterpret_cast<const f4 *>(yf + (long long)s * nj * nk * UP);
            for (int j = jlo; j <= jhi; ++j) {
                // rays of this row that can meet the open cube around the voxel
                const float dj = (float)(j - ai) - ar;
                const float zmax = fminf(fminf(fmaf(f.hull[0], dj, cu[0]), fmaf(f.hull[2], dj, cu[1])),
                                         fmaf(f.hull[4], dj, cu[2]));
                const float zmin = fmaxf(fmaxf(fmaf(f.hull[6], dj, cl[0]), fmaf(f.hull[8], dj, cl[1])),
                                         fmaf(f.hull[10], dj, cl[2]));
                const int klo = max(0, bi + (int)ceilf(zmin));
                const int khi = min(nk - 1, bi + (int)floorf(zmax));
                const float pj0 = dj * f.ejf[0], pj1 = dj * f.ejf[1], pj2 = dj * f.ejf[2];
                const f4 *yrow = ys + __umul24(j, nk * (UP / 4));  // row offsets stay below 2^24 float4
                float dk = (float)(klo - bi) - br;
                for (int k = klo; k <= khi; ++k, dk += 1.0f) {
                    f4 yv[UP / 4];
#pragma unroll
                    for (int u4 = 0; u4 < UP / 4; ++u4) yv[u4] = yrow[k * (UP / 4) + u4];  // in flight meanwhile
                    const float P[3] = {fmaf(dk, f.ekf[0], pj0), fmaf(dk, f.ekf[1], pj1), fmaf(dk, f.ekf[2], pj2)};
                    const float wsum = ray_weight<false>(P, tent);
#pragma unroll
                    for (int u4 = 0; u4 < UP; u4 += 4) {
                        q[u4 + 0] = fmaf(wsum, yv[u4 / 4].x, q[u4 + 0]);
                        q[u4 + 1] = fmaf(wsum, yv[u4 / 4].y, q[u4 + 1]);
                        q[u4 + 2] = fmaf(wsum, yv[u4 / 4].z, q[u4 + 2]);
                        q[u4 + 3] = fmaf(wsum, yv[u4 / 4].w, q[u4 + 3]);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < UP; ++u) Qw[lane * (UP + 1) + u] = q[u];
        // Qw is private to this wave, whose LDS accesses complete in program
        // order: only compiler reordering has to be fenced.
        __builtin_amdgcn_wave_barrier();
        // g tile += B_s^T (coefficients x u) * Q^T (u x voxels)
        if constexpr (BF16) {
            // K = 16 (u padded with zeros): A from BuT16[s][coefficient][u], B = Q rounded to bf16
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const float *qv = Qw + (nt * 16 + (lane & 15)) * (UP + 1);
                const int u0 = 4 * (lane >> 4);
                s4 bv;
                bv.x = u0 + 0 < UP ? f2bf(qv[min(u0 + 0, UP - 1)]) : (short)0;
                bv.y = u0 + 1 < UP ? f2bf(qv[min(u0 + 1, UP - 1)]) : (short)0;
                bv.z = u0 + 2 < UP ? f2bf(qv[min(u0 + 2, UP - 1)]) : (short)0;
                bv.w = u0 + 3 < UP ? f2bf(qv[min(u0 + 3, UP - 1)]) : (short)0;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = mfma16x16x16bf16(avb[mt], bv, acc[mt][nt]);
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < KE; ++ks) {
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) {
                    const float bv = qw_at<UP>(Qw, nt, ks, lane);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = mfma16x16x4(avf[ks][mt], bv, acc[mt][nt]);
                }
            }
#pragma unroll
            for (int kd = 0; kd < KD; ++kd)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) pend[kd][mt] = avf[KE + kd][mt];
        }
        __builtin_amdgcn_wave_barrier();
    }
    if constexpr (KD > 0) {
        if (S > 0) deferred_mfma();
    }

    // epilogue: lane holds rows (coefficients) 16 mt + 4 (lane/16) + r of voxel column 16 nt + lane % 16
    double c2 = 0.0;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int lv = nt * 16 + (lane & 15);
        const int vy = by * 8 + (lv >> 3), vz = bz * 8 + (lv & 7);
        if (ix < nx && vy < ny && vz < nz) {
            const long long base = (((long long)ix * ny + vy) * nz + vz) * C;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = mt * 16 + 4 * (lane >> 4) + r;
                    if (i < C) {
                        float val = acc[mt][nt][r];
                        if (c) {
                            float cv = c[base + i];
                            val += beta * cv;
                            c2 += (double)cv * (double)cv;
                        }
                        g[base + i] = val;
                    }
                }
            }
        }
    }
    if (partials) {
        double tot = block_sum(c2, ws);
        if (tid == 0) partials[bid] = tot;
    }
}


// ---------------------------------------------------------------------------
// backproject with LDS-staged residual windows (four or eight unique segments).
//
// A block owns bricks of 64-voxel cubes (4 x 4 x 4, one per wave) and walks the
// projections two at a time.  Per pair it stages two detector windows (the
// brick's shadow widened by one voxel's reach) with gfx950's direct
// global-to-LDS copies, every lane enumerates the rays of its voxel from LDS,
// and each wave contracts its voxels' Q of both projections with B^T on MFMA,
// accumulating g in registers over all projections.
//
// PAIR (no detector offsets, even nx): the sample lattice
// o + j e_j + k e_k + n step d with o = -((nj-1)/2 e_j + (nk-1)/2 e_k) is
// symmetric under x -> -x with (j, k, n) -> (nj-1-j, nk-1-k, -n), and so are
// the voxel grid, the tent and Joseph's cuts.  So the weight of ray (j, k) at
// voxel v is that of ray (nj-1-j, nk-1-k) at the inverted voxel v', and one
// enumeration serves both.  Waves 0, 1 own two cubes of the lower half
// (ix < nx / 2), waves 2, 3 their inverses lane by lane; the lower group
// enumerates s0, the upper s0 + 1, from a window that holds each ray's own and
// reflected residual side by side, and hands the inverse's Q to the partner
// wave.  Without PAIR every wave enumerates both projections.
//
// What bounds it: VALU issue, which the MFMAs share.  Counters of the kernel
// this one replaced (128^3, 300 projections, eight unique segments): 718 VALU
// instructions (4 cycles each) and 48 fp32 MFMAs (32 cycles each) per wave and
// pair, together 90% of the SIMD cycles.  Hence:
//  - the contraction runs on 16x16x32 bf16 MFMA with B and Q in three bf16 pieces
//    each (x = x0 + x1 + x2 to 2^-27): the six products b0q0 b0q1 b1q0 b1q1 b0q2
//    b2q0 of two projections fill K = 32 three times (eight segments: 36 MFMAs of
//    16 cycles per pair instead of 48 of 32).  The dropped products are below
//    2^-26 of the result, under the rounding of an fp32 sum;
//  - windows have one size for all projections, so a lane's place in a window and
//    its source offset from the window origin are computed once, and a copy is
//    one add and one instruction;
//  - window origins (the same for all lanes) are worked out by one lane per
//    projection, 64 pairs at a time;
//  - the tent samples of a ray are a fixed number without branches (ray_weight).
// Adjoint, before -> now: 256^3 / 400 projections / 8 unique segments 118.1 -> 76.3 ms;
// 128^3 / 300 / 8 11.3 -> 7.3; 100^3 / 240 / 4 2.89 -> 2.22 (Joseph 1.95 -> 1.61);
// 97 x 89 x 107 / 220 / 8 with detector offsets (unpaired) 4.79 -> 3.39; relative
// error against float64 4.7e-7 -> 1.3e-7 (100^3), 7.2e-7 -> 3.9e-7 (128^3, with the
// forward's).  Now bound by VALU issue: 95% of the cycles at 128^3, with 84% of the lanes.
// ---------------------------------------------------------------------------
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));

// x0 + x1 + x2 = x to 2^-27 relative, two values per word (bf16, nearest even)
__device__ __forceinline__ void split_bf16(float a, float b, unsigned &h, unsigned &m, unsigned &l)
{
    h = __builtin_bit_cast(unsigned, __builtin_convertvector((f2{a, b}), bf2));
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = __builtin_bit_cast(unsigned, __builtin_convertvector((f2{a, b}), bf2));
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xffff0000u);
    l = __builtin_bit_cast(unsigned, __builtin_convertvector((f2{a, b}), bf2));
}

// Operand tiles of Q in LDS, 16 bytes per voxel: with eight segments one tile per
// piece; with four [q0 | q1] and [q2 | q0] (bf16 tier: [q0 | 0]).  K = 32 then holds
// one product of four projections, so two pairs share a contraction.
// It pays from 48 padded coefficients on (fewer MFMAs and adds); below, the smaller
// tiles leave room for more blocks.
template <int UP, int MT>
constexpr int kPairs = UP == 4 && MT >= 3 ? 2 : 1;
template <int UP, bool BF16>
constexpr int kQTiles = BF16 ? 1 : (UP == 8 ? 3 : 2);

template <int UP, bool BF16>
__device__ __forceinline__ void put_q(const float *q, uint4 *t, int stride)
{
    unsigned h[UP / 2], m[UP / 2], l[UP / 2];
#pragma unroll
    for (int i = 0; i < UP / 2; ++i) split_bf16(q[2 * i], q[2 * i + 1], h[i], m[i], l[i]);
    if constexpr (UP == 8) {
        t[0] = make_uint4(h[0], h[1], h[2], h[3]);
        if constexpr (!BF16) {
            t[stride] = make_uint4(m[0], m[1], m[2], m[3]);
            t[2 * stride] = make_uint4(l[0], l[1], l[2], l[3]);
        }
    } else if constexpr (BF16) {
        t[0] = make_uint4(h[0], h[1], 0u, 0u);
    } else {
        t[0] = make_uint4(h[0], h[1], m[0], m[1]);
        t[stride] = make_uint4(l[0], l[1], h[0], h[1]);
    }
}

// Waves per SIMD that the registers have to leave room for.
//  - Two from 64 padded coefficients on: left alone, the kernels of four segments take 272
//    to 312 registers (accumulators in accumulation registers and moves between), which is
//    one wave per SIMD.  72^3 / 120 projections / 4 unique segments / 91 coefficients, one
//    wave -> two: 1161 -> 642 us, unpaired 1916 -> 1172, Joseph 929 -> 522 and 1511 -> 879;
//    bf16 tier, 66 coefficients: 1013 -> 498.  (Unpaired trilinear float32 with 66 stays
//    below 256 by itself, and is 4% faster so.)
//  - Five or six (unpaired: smaller windows) for Joseph's method with up to 16
//    coefficients, the least arithmetic per barrier: 101 x 100 x 100 / 240 projections
//    unpaired 1787 -> 1559 us (gathering from memory, without barriers: 1592); paired
//    100^3 / 240 1204 -> 1090, 128 x 127 x 127 / 300 2757 -> 2546 (72^3 / 160, whose last
//    blocks then run alone, 331 -> 345).
//  - Three otherwise; four (DEEP) with four segments and 48 coefficients, unpaired, where
//    four blocks per compute unit at a time save a round, or in many rounds: three waves
//    -> four, 120 projections with detector offsets, by blocks per unit: 64^3 (4) 534 -> 415
//    us, Joseph 387 -> 277; 80^3 (8) 821 -> 809, 585 -> 538; 128^3 / 300 (32) 7720 -> 7470,
//    5375 -> 4927; but 48^3 (2) 274 -> 303, 72^3 (6) 621 -> 675.  The third piece of Q then
//    has a tile of half the size, as four blocks have 40 KiB of LDS each.  Paired kernels
//    spill more there and take it only with many samples per ray and a round to save.
template <int UP, int MT, bool BF16, bool JOS, bool PAIR, bool DEEP>
constexpr int kAdjointWaves = MT >= 4 ? (UP == 4 && MT == 5 && !BF16 && !JOS && !PAIR ? 1 : 2)
                                      : UP == 4 && MT == 1 && JOS ? (PAIR ? 5 : 6) : DEEP ? 4 : 3;

// Q for a packed contraction (DEEP): [q0 | q1] and q2
__device__ __forceinline__ void put_q_packed(const float *q, uint4 *t, uint2 *t2)
{
    unsigned h[2], m[2], l[2];
    split_bf16(q[0], q[1], h[0], m[0], l[0]);
    split_bf16(q[2], q[3], h[1], m[1], l[1]);
    *t = make_uint4(h[0], h[1], m[0], m[1]);
    *t2 = make_uint2(l[0], l[1]);
}

// sum over projections s0 .. s1 - 1 of B^T Q at one voxel (centred position x, y, z) in
// float32, four coefficients per 16 of them (Bu: from the first).  For the few sums that
// k_backproject_win cannot take: all rays in reach of the voxel, from memory.
template <int UP, int MT, bool BF16, bool JOS>
__device__ __forceinline__ void sum_in_f32(const float *yf, const ProjFrame *frames, const float *Bu, int s0, int s1,
                                           int nj, int nk, int Cp, float step, double x, double y, double z, f4 *sum)
{
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) sum[mt] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int s = s0; s < s1; ++s) {
        const ProjFrame &f = frames[s];
        const double w0 = x - f.o[0], w1 = y - f.o[1], w2 = z - f.o[2];
        const double a = w0 * f.ej[0] + w1 * f.ej[1] + w2 * f.ej[2];
        const double b = w0 * f.ek[0] + w1 * f.ek[1] + w2 * f.ek[2];
        const double ts = (w0 * f.d[0] + w1 * f.d[1] + w2 * f.d[2]) / (double)step;
        const int ai = (int)floor(a), bi = (int)floor(b);
        const float ar = (float)(a - floor(a)), br = (float)(b - floor(b));
        const float rj = JOS ? f.jos_rj : (float)f.lj, rk = JOS ? f.jos_rk : (float)f.lk;
        const int j1 = min(nj - 1, ai + (int)floorf(ar + rj)), k0 = max(0, bi + (int)ceilf(br - rk));
        const int k1 = min(nk - 1, bi + (int)floorf(br + rk));
        const TentRay tent = tent_ray(f, (float)(ts - floor(ts)), step, 1.0f / step);
        float q[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) q[u] = 0.0f;
#pragma unroll 1
        for (int j = max(0, ai + (int)ceilf(ar - rj)); j <= j1; ++j)
#pragma unroll 1
            for (int k = k0; k <= k1; ++k) {
                const float dj = (float)(j - ai) - ar, dk = (float)(k - bi) - br;
                float wt;
                if constexpr (JOS) {
                    wt = tent1(fmaf(dk, f.jos_gk[0], dj * f.jos_gj[0])) *
                         tent1(fmaf(dk, f.jos_gk[1], dj * f.jos_gj[1])) * f.jos_w;
                } else {
                    const float P[3] = {fmaf(dk, f.ekf[0], dj * f.ejf[0]), fmaf(dk, f.ekf[1], dj * f.ejf[1]),
                                        fmaf(dk, f.ekf[2], dj * f.ejf[2])};
                    wt = ray_weight<false>(P, tent);
                }
                if (!(wt > 0.0f)) continue;
                const float *ray = yf + (((long long)s * nj + j) * nk + k) * UP;
#pragma unroll
                for (int u = 0; u < UP; ++u) q[u] = fmaf(wt, ray[u], q[u]);
            }
#pragma unroll
        for (int u = 0; u < UP; ++u)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const float *row = Bu + ((long long)s * UP + u) * Cp + mt * 16;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    sum[mt][r] = BF16 ? fmaf(bf16_value(row[r]), bf16_value(q[u]), sum[mt][r])
                                      : fmaf(row[r], q[u], sum[mt][r]);
            }
    }
}

// Copies of 128 float4 per window and pair (at most; window_lds has the sizes)
template <int UP, bool PAIR>
constexpr int kWinCopies = UP == 4 ? (PAIR ? 4 : 2) : (PAIR ? 6 : 4);

template <int UP, int MT, bool BF16, bool JOS, bool PAIR, bool DEEP = false, bool MANY = false>
__global__ __launch_bounds__(256, (kAdjointWaves<UP, MT, BF16, JOS, PAIR, DEEP>)) void k_backproject_win(const float *__restrict__ yf,
                                                         const ProjFrame *__restrict__ frames,
                                                         const uint4 *__restrict__ Bop, const float *__restrict__ Bu,
                                                         int S, int nx, int ny, int nz,
                                                         int nj, int nk, int C, int Cp, float step,
                                                         float *__restrict__ g, float beta, const float *__restrict__ c,
                                                         double *__restrict__ partials, int WR, int WC, int s_per,
                                                         float *__restrict__ split)
{
    // blockIdx.y > 0: the projections are split over blocks, each of which writes
    // its own sum to split[blockIdx.y][V C] (added in order by k_add_splits)
    const int s_begin = blockIdx.y * s_per, s_end = min(S, s_begin + s_per);
    constexpr int Q = UP / 4;               // float4 per ray
    constexpr int RW = PAIR ? 2 * Q : Q;    // float4 per staged ray: own, then reflected
    constexpr int QT = kQTiles<UP, BF16>;
    extern __shared__ f4 wins[];            // [2][WR * WC * RW rounded up to 128]
    constexpr int PB = kPairs<UP, MT>;      // pairs per contraction
    constexpr int QS = 2 * PB * 64;         // stride of the operand tiles
    constexpr bool PACK = DEEP && !BF16;
    static_assert(!DEEP || (UP == 4 && MT == 3), "");
    __shared__ uint4 Qt[4][PACK ? 1 : QT][2 * PB][64];  // [wave][tile][projection][voxel]
    __shared__ uint2 Q2[PACK ? 4 : 1][PACK ? 2 * PB : 1][64];
    __shared__ int2 wtab[2][64];            // window origins of the next 64 pairs
    __shared__ double ws[4];
    const int tid = threadIdx.x, lane = tid & 63;
    // wave-uniform (scalar) wave index: frames and windows stay in scalar registers
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 1;              // PAIR: lower / upper voxel group; also the window this wave stages
    const bool upper = PAIR && grp == 1;
    const int nxh = PAIR ? nx >> 1 : nx;
    const int nbx = (nxh + 3) / 4, nby = PAIR ? (ny + 3) / 4 : (ny + 7) / 8;
    const int bid = xcd_block(blockIdx.x, gridDim.x);
    const int bx = bid % nbx, by = (bid / nbx) % nby, bz = bid / (nbx * nby);
    const int x0 = 4 * bx, y0 = PAIR ? 4 * by : 8 * by + 4 * (wave >> 1), z0 = 8 * bz + 4 * (wave & 1);
    // this lane's voxel (PAIR: the lower voxel of its pair, then its own)
    const int px = x0 + (lane >> 4), py = y0 + ((lane >> 2) & 3), pz = z0 + (lane & 3);
    const bool valid = px < nxh && py < ny && pz < nz;
    const int ix = upper ? nx - 1 - px : px, iy = upper ? ny - 1 - py : py, iz = upper ? nz - 1 - pz : pz;
    const double xv[3] = {ix - 0.5 * (nx - 1), iy - 0.5 * (ny - 1), iz - 0.5 * (nz - 1)};
    const double inv_step = 1.0 / (double)step;

    // window origin of projection s: the first row and column that a voxel of the
    // box can reach (one more for rounding), moved so that WR x WC rays fit the detector
    auto origin = [&](int s, bool inverted) {
        const ProjFrame &f = frames[s];
        const double lo0[3] = {4 * bx - 0.5 * (nx - 1), (PAIR ? 4 : 8) * by - 0.5 * (ny - 1), 8 * bz - 0.5 * (nz - 1)};
        const double hi0[3] = {min(nxh, 4 * bx + 4) - 1 - 0.5 * (nx - 1),
                               min(ny, (PAIR ? 4 : 8) * (by + 1)) - 1 - 0.5 * (ny - 1),
                               min(nz, 8 * bz + 8) - 1 - 0.5 * (nz - 1)};
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const double lo = inverted ? -hi0[q] : lo0[q], hi = inverted ? -lo0[q] : hi0[q];
            a += ((f.ej[q] >= 0.0 ? lo : hi) - f.o[q]) * f.ej[q];
            b += ((f.ek[q] >= 0.0 ? lo : hi) - f.o[q]) * f.ek[q];
        }
        const double rj = JOS ? (double)f.jos_rj : f.lj, rk = JOS ? (double)f.jos_rk : f.lk;
        return make_int2(max(0, min(nj - WR, (int)ceil(a - rj) - 1)), max(0, min(nk - WC, (int)ceil(b - rk) - 1)));
    };
    // origins of both windows of 64 pairs from s0 on (waves 0 and 1); the table is
    // read only between a pair's second barrier and the next pair's first
    auto fill_origins = [&](int s0) {
        if (wave < 2 && s0 + 2 * lane + wave < s_end) wtab[wave][lane] = origin(s0 + 2 * lane + wave, PAIR && wave == 1);
    };
    int wj[2] = {0, 0}, wk[2] = {0, 0};
    auto take_origins = [&](int s0) {
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const int2 o = wtab[w][((s0 - s_begin) >> 1) & 63];
            wj[w] = __builtin_amdgcn_readfirstlane(o.x);
            wk[w] = __builtin_amdgcn_readfirstlane(o.y);
        }
    };

    // The two waves of a group stage window grp.  Copy i moves elements
    // (2 i + wave % 2) 64 + lane; a lane always copies the same part of a ray
    // (64 is a multiple of RW), so its source byte offset from the projection's
    // residual is a constant plus (own part) or minus (reflected part) the offset
    // of the window origin.  Elements past the window repeat its last ray.
    const int nel = WR * WC * RW, wsz = (nel + 127) & ~127;
    const bool refl = PAIR && (lane & (RW - 1)) >= Q;
    unsigned soff[kWinCopies<UP, PAIR>];
#pragma unroll
    for (int i = 0; i < kWinCopies<UP, PAIR>; ++i) {
        const int e = (2 * i + (wave & 1)) * 64 + lane;
        const int ray = min(e / RW, WR * WC - 1), part = lane & (RW - 1);
        const int r = ray / WC, rel = r * nk + (ray - r * WC);
        soff[i] = 16u * (unsigned)(refl ? (nj * nk - 1 - rel) * Q + part - Q : rel * Q + part);
    }
    auto stage = [&](int s) {
        const char *src = reinterpret_cast<const char *>(yf) + (long long)s * nj * nk * Q * 16;
        const int o = ((grp ? wj[1] : wj[0]) * nk + (grp ? wk[1] : wk[0])) * Q * 16;
        const unsigned d = refl ? -(unsigned)o : (unsigned)o;
        f4 *dst = wins + grp * wsz + (wave & 1) * 64;
#pragma unroll
        for (int i = 0; i < kWinCopies<UP, PAIR>; ++i)
            if (i * 128 < nel)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + (soff[i] + d)),
                                                 (__attribute__((address_space(3))) void *)(dst + i * 128), 16, 0, 0);
    };

    f4 acc[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = f4{0.f, 0.f, 0.f, 0.f};

    fill_origins(s_begin);
    __syncthreads();
    take_origins(s_begin);
    if (s_begin + grp < s_end) stage(s_begin + grp);
    for (int s0 = s_begin; s0 < s_end; s0 += 2) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();  // this pair's windows are staged
#pragma unroll 1
        for (int h = 0; h < (PAIR ? 1 : 2); ++h) {
            const int w = PAIR ? grp : h, s = s0 + w;  // window and projection enumerated
            float q[UP], qm[UP];
#pragma unroll
            for (int u = 0; u < UP; ++u) q[u] = qm[u] = 0.0f;
            if (s < s_end && valid) {
                const ProjFrame &f = frames[s];
                const int j0 = w ? wj[1] : wj[0], k0 = w ? wk[1] : wk[0];
                // voxel centre in the ray frame (float64), split into integer + fraction
                const double w0 = xv[0] - f.o[0], w1 = xv[1] - f.o[1], w2 = xv[2] - f.o[2];
                const double a = w0 * f.ej[0] + w1 * f.ej[1] + w2 * f.ej[2];
                const double bb = w0 * f.ek[0] + w1 * f.ek[1] + w2 * f.ek[2];
                const double af = floor(a), bf = floor(bb);
                const int ai = (int)af, bi = (int)bf;
                const float ar = (float)(a - af), br = (float)(bb - bf);
                const float rj = JOS ? f.jos_rj : (float)f.lj;
                const int jlo = max(j0 - ai, (int)ceilf(ar - rj)), jhi = min(j0 + WR - 1 - ai, (int)floorf(ar + rj));
                const float kmin = (float)(k0 - bi), kmax = (float)(k0 + WC - 1 - bi);
                const f4 *row = wins + w * wsz + ((jlo + ai - j0) * WC + (bi - k0)) * RW;
                const float fjhi = (float)jhi;
                // a ray's residual (and the mirrored ray's), read before its weight is
                // worked out, then added with that weight
                f4 y[RW];
                auto load_ray = [&](const f4 *p) {
#pragma unroll
                    for (int i = 0; i < RW; ++i) y[i] = p[i];
                };
                auto add_ray = [&](float wt) {
#pragma unroll
                    for (int i = 0; i < RW; ++i) {
                        float *t = i < Q ? q + 4 * i : qm + 4 * (i - Q);
#pragma unroll
                        for (int e = 0; e < 4; ++e) t[e] = fmaf(wt, y[i][e], t[e]);
                    }
                };
                if constexpr (JOS) {
                    // Joseph's method: the rays whose cut with the voxel's layer lies
                    // within one voxel in-plane, weight (1 - |Delta_B|)(1 - |Delta_C|) /
                    // |d_A|; the inverse voxel's cut of the mirrored ray is the negated
                    // cut point, so the same weight serves both voxels of a pair
                    for (float fj = (float)jlo; fj <= fjhi; fj += 1.0f, row += WC * RW) {
                        const float dj = fj - ar;
                        const float eB = dj * f.jos_gj[0], eC = dj * f.jos_gj[1];
                        // dk range with |dk gk + e| < 1 on both in-plane axes (a flat
                        // axis gives all dk or none; the other one is never flat)
                        const float xB1 = (-1.0f - eB) * f.jos_igk[0], xB2 = (1.0f - eB) * f.jos_igk[0];
                        const float xC1 = (-1.0f - eC) * f.jos_igk[1], xC2 = (1.0f - eC) * f.jos_igk[1];
                        const float lo = fmaxf(fminf(xB1, xB2), fminf(xC1, xC2));
                        const float hi = fminf(fmaxf(xB1, xB2), fmaxf(xC1, xC2));
                        if (!(lo < hi)) continue;
                        const float kf = fmaxf(kmin, ceilf(br + lo - 1e-4f));
                        const float ke = fminf(kmax, floorf(br + hi + 1e-4f));
                        const f4 *ray = row + (int)kf * RW;
                        for (float fk = kf; fk <= ke; fk += 1.0f, ray += RW) {
                            load_ray(ray);
                            const float dk = fk - br;
                            const float wB = tent1(fmaf(dk, f.jos_gk[0], eB));
                            const float wC = tent1(fmaf(dk, f.jos_gk[1], eC));
                            add_ray(wB * wC * f.jos_w);
                        }
                    }
                } else {
                    const double ts = (w0 * f.d[0] + w1 * f.d[1] + w2 * f.d[2]) * inv_step;
                    const TentRay tent = tent_ray(f, (float)(ts - floor(ts)), step, (float)inv_step);
                    // hull intercepts shifted by this voxel's fraction br and the 1e-4 slack
                    const float cu[3] = {f.hull[1] + (br + 1e-4f), f.hull[3] + (br + 1e-4f), f.hull[5] + (br + 1e-4f)};
                    const float cl[3] = {f.hull[7] + (br - 1e-4f), f.hull[9] + (br - 1e-4f), f.hull[11] + (br - 1e-4f)};
                    for (float fj = (float)jlo; fj <= fjhi; fj += 1.0f, row += WC * RW) {
                        // rays of this row that can meet the open cube around the voxel
                        const float dj = fj - ar;
                        const float zmax = fminf(fminf(fmaf(f.hull[0], dj, cu[0]), fmaf(f.hull[2], dj, cu[1])),
                                                 fmaf(f.hull[4], dj, cu[2]));
                        const float zmin = fmaxf(fmaxf(fmaf(f.hull[6], dj, cl[0]), fmaf(f.hull[8], dj, cl[1])),
                                                 fmaf(f.hull[10], dj, cl[2]));
                        const float kf = fmaxf(kmin, ceilf(zmin)), ke = fminf(kmax, floorf(zmax));
                        const float pj0 = dj * f.ejf[0], pj1 = dj * f.ejf[1], pj2 = dj * f.ejf[2];
                        const f4 *ray = row + (int)kf * RW;
                        for (float fk = kf; fk <= ke; fk += 1.0f, ray += RW) {
                            load_ray(ray);
                            const float dk = fk - br;
                            const float P[3] = {fmaf(dk, f.ekf[0], pj0), fmaf(dk, f.ekf[1], pj1),
                                                fmaf(dk, f.ekf[2], pj2)};
                            add_ray(ray_weight<MANY>(P, tent));
                        }
                    }
                }
            }
            // own Q to this wave's tile, the inverse's to the partner's
            const int slot = PB == 2 ? (s0 & 2) + w : w;
            if constexpr (PACK) {
                put_q_packed(q, &Qt[wave][0][slot][lane], &Q2[wave][slot][lane]);
                if constexpr (PAIR) put_q_packed(qm, &Qt[wave ^ 2][0][slot][lane], &Q2[wave ^ 2][slot][lane]);
            } else {
                put_q<UP, BF16>(q, &Qt[wave][0][slot][lane], QS);
                if constexpr (PAIR) put_q<UP, BF16>(qm, &Qt[wave ^ 2][0][slot][lane], QS);
            }
        }
        const bool last = s0 + 2 >= s_end, contract = PB == 1 || (s0 & 2) || last;
        if (PB == 2 && last && !(s0 & 2)) {  // a lone last pair: nothing in the other two slots
#pragma unroll
            for (int t = 0; t < (PACK ? 1 : QT); ++t) Qt[wave][t][2][lane] = Qt[wave][t][3][lane] = make_uint4(0, 0, 0, 0);
            if constexpr (PACK) Q2[wave][2][lane] = Q2[wave][3][lane] = make_uint2(0, 0);
        }
        // B^T operands (tables in operand order; a projection past the last one has
        // Q = 0).  Lane group kq serves projection kq / 2 of the pair and product set
        // kq % 2, or, with two pairs per contraction, projection kq of the four.
        const int kq = lane >> 4, sel = PB == 2 ? 0 : kq & 1, sl = PB == 2 ? kq : kq >> 1, n = lane & 15;
        constexpr int NA = BF16 ? 1 : (PB == 2 ? 3 : 2);
        uint4 A[NA][MT];
        if (contract) {
            int set[NA];
            if constexpr (BF16)
                set[0] = UP == 8 ? 4 + sel : (sel ? 4 : 3);
            else if constexpr (PB == 2)
                set[0] = 0, set[1] = 1, set[2] = 2;
            else if constexpr (UP == 8)
                set[0] = sel, set[1] = 2 + sel;
            else
                set[0] = sel, set[1] = sel ? 4 : 2;
            const uint4 *bp = Bop + (long long)min((PB == 2 ? s0 & ~3 : s0) + sl, s_end - 1) * 6 * Cp + n;
#pragma unroll
            for (int i = 0; i < NA; ++i)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) A[i][mt] = bp[set[i] * Cp + mt * 16];
        }
        if (((s0 + 2 - s_begin) & 127) == 0) fill_origins(s0 + 2);
        __syncthreads();  // Q is complete; the windows are free
        // copies for the next pair run during this pair's MFMAs; the operands are
        // waited for first, as the copies share their counter
        __builtin_amdgcn_s_waitcnt(0);
        if (!last) {
            take_origins(s0 + 2);
            if (s0 + 2 + grp < s_end) stage(s0 + 2 + grp);
        }
        if (!contract) continue;
        // g tile += B^T (coefficients x (projection, piece, u)) * Q, the smallest
        // products first.  The bf16 MFMA cuts off what it shifts out of its
        // accumulator, always towards zero: with the sum over all projections kept
        // there, the relative error grew with their number (1.1e-6 at 240, 2.1e-6 at
        // 300, against 4.7e-7 and 7.2e-7), so a pair's products start from zero and
        // are added to g with a rounded float32 add.
        const uint4 *qb = &Qt[wave][0][sl][n];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const s8 b0 = __builtin_bit_cast(s8, qb[nt * 16]);
            if constexpr (BF16) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[mt][nt] = mfma16x16x32bf16(__builtin_bit_cast(s8, A[0][mt]), b0, acc[mt][nt]);
            } else {
                // eight: (b0 q2, b2 q0), (b0 q1, b1 q1), (b0 q0, b1 q0); four: (b0 q2 + b2 q0),
                // then (b0 q0 + b0 q1) and (b1 q0 + b1 q1), together or (two pairs) in turn
                s8 b2;
                if constexpr (PACK) {
                    const uint2 l = Q2[wave][sl][nt * 16 + n];
                    const uint4 h = __builtin_bit_cast(uint4, b0);
                    b2 = __builtin_bit_cast(s8, make_uint4(l.x, l.y, h.x, h.y));
                } else {
                    b2 = __builtin_bit_cast(s8, qb[(UP == 4 ? QS : sel ? 0 : 2 * QS) + nt * 16]);
                }
                f4 t[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    t[mt] = mfma16x16x32bf16(__builtin_bit_cast(s8, A[NA - 1][mt]), b2, f4{0.f, 0.f, 0.f, 0.f});
                if constexpr (UP == 8 || PB == 2) {
                    const s8 b1 = UP == 8 ? __builtin_bit_cast(s8, qb[QS + nt * 16]) : b0;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        t[mt] = mfma16x16x32bf16(__builtin_bit_cast(s8, A[UP == 8 ? 0 : 1][mt]), b1, t[mt]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    t[mt] = mfma16x16x32bf16(__builtin_bit_cast(s8, A[0][mt]), b0, t[mt]);
                    acc[mt][nt] += t[mt];
                }
            }
        }
    }

    // What the pieces cannot hold: from the largest bf16 on the first one is infinite and
    // the next NaN (in the bf16 tier, an infinite Q times the operands' padding), and below
    // 2^-110 the third one loses bits (relative error at residuals around 2^-116 2e-6,
    // around 2^-124 5e-4).  Sums that are NaN, or so small that each of their up to 2^12 terms
    // may be, are taken again in float32: an infinite residual gives an infinite gradient,
    // and no sum is less exact than in float32.
    // (By voxel, as a NaN is in all its coefficients; but with 48 of them and four segments
    // the maximum costs the trilinear kernel a spill, 2.22 -> 2.35 ms at 100^3 / 240.)
    constexpr bool by_element = MT >= 3 && !JOS;
    unsigned again = 0;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        float most = 0.0f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = acc[mt][nt][r];
                if constexpr (by_element) {
                    if (v != v || (!BF16 && v != 0.0f && fabsf(v) < 0x1p-98f)) again |= 1u << nt;
                } else {
                    most = fmaxf(most, fabsf(v));
                }
            }
        const float first = acc[0][nt][0];
        if (!by_element && (first != first || (!BF16 && most > 0.0f && most < 0x1p-98f))) again |= 1u << nt;
    }
    if (__builtin_expect(__any(again != 0), 0)) {
#pragma unroll 1
        for (int nt = 0; nt < 4; ++nt) {
            if (!(again >> nt & 1)) continue;
            const int qx = x0 + nt, qy = y0 + ((lane >> 2) & 3), qz = z0 + (lane & 3);
            f4 sum[MT];
            sum_in_f32<UP, MT, BF16, JOS>(yf, frames, Bu + 4 * (lane >> 4), s_begin, s_end, nj, nk, Cp, step,
                                          (upper ? nx - 1 - qx : qx) - 0.5 * (nx - 1),
                                          (upper ? ny - 1 - qy : qy) - 0.5 * (ny - 1),
                                          (upper ? nz - 1 - qz : qz) - 0.5 * (nz - 1), sum);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[mt][t] = t == nt ? sum[mt] : acc[mt][t];
        }
    }

    if (split) {
        g = split + (long long)blockIdx.y * nx * ny * nz * C;
        c = nullptr;
        partials = nullptr;
    }
    // epilogue: lane holds rows (coefficients) 16 mt + 4 (lane/16) + r of voxel column 16 nt + lane % 16
    double c2 = 0.0;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int qx = x0 + nt, qy = y0 + ((lane >> 2) & 3), qz = z0 + (lane & 3);
        if (qx < nxh && qy < ny && qz < nz) {
            const int vx = upper ? nx - 1 - qx : qx, vy = upper ? ny - 1 - qy : qy, vz = upper ? nz - 1 - qz : qz;
            const long long base = (((long long)vx * ny + vy) * nz + vz) * C;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = mt * 16 + 4 * (lane >> 4) + r;
                    if (i < C) {
                        float val = acc[mt][nt][r];
                        if (c) {
                            float cv = c[base + i];
                            val += beta * cv;
                            c2 += (double)cv * (double)cv;
                        }
                        g[base + i] = val;
                    }
                }
            }
        }
    }
    if (partials) {
        double tot = block_sum(c2, ws);
        if (tid == 0) partials[bid] = tot;
    }
}

// g = sum over the splits (in order) + beta c, with the float64 partials of sum c^2
__global__ __launch_bounds__(256) void k_add_splits(const float *__restrict__ split, int ns, long long n,
                                                    float *__restrict__ g, float beta, const float *__restrict__ c,
                                                    double *__restrict__ partials)
{
    __shared__ double ws[4];
    double c2 = 0.0;
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        float v = split[e];
        for (int i = 1; i < ns; ++i) v += split[i * n + e];
        if (c) {
            const float cv = c[e];
            v += beta * cv;
            c2 += (double)cv * (double)cv;
        }
        g[e] = v;
    }
    if (partials) {
        const double tot = block_sum(c2, ws);
        if (threadIdx.x == 0) partials[blockIdx.x] = tot;
    }
}

// Splits of the projections over blocks, so that a small volume fills the chip.  A
// compute unit works off n = ceil(blocks splits / units) blocks, three at a time; one
// or two left over run alone, at about half and four fifths of the rate of three
// (one or two waves per SIMD do not hide the LDS and scalar latencies).  Every split
// writes and reads a coefficient volume, at about 4 TB/s, against about 1.2 us per
// block and pair of projections.  Adjoint with its fold, unsplit -> split: 32^3 / 60
// projections / 15 coefficients (128 blocks, six splits) 81 -> 52 us, 48^3 / 120 / 28
// (432 blocks, three) 180 -> 172 us.  Over 60 random shapes of 10^3 to 76^3 the choice is
// 1.00 to 6.4 times as fast as no split, but for one with 66 coefficients, whose kernels run
// two blocks at a time (62^3 / 312 projections, unpaired: 1657 -> 1688 us).
static int adjoint_splits(const Dims &d, int blocks, int units, double &gain)
{
    const double vol_us = 4.0 * d.nx * d.ny * d.nz * d.C / 4e6;
    int best = 1;
    double best_t = 1e300, whole_t = 0.0;
    for (int ns = 1; ns <= kMaxSplits && (ns == 1 || 8 * ns <= d.S); ++ns) {
        const int n = (int)(((long long)blocks * ns + units - 1) / units), r = n % 3;
        const double work = 3 * (n / 3) + (r == 0 ? 0.0 : r == 1 ? 2.0 : 2.5);
        const double t = 1.2 * 0.5 * d.S / ns * work + (ns > 1 ? 5.0 + (2 * ns + 1) * vol_us : 0.0);
        if (ns == 1) whole_t = t;
        if (t < 0.97 * best_t) {
            best_t = t;
            best = ns;
        }
    }
    gain = whole_t - best_t;
    return best;
}

// Windows of the staged adjoint for a block's voxel box: rows and columns that hold
// every ray of its voxels in any projection (centre span . |e| + 2 reach + 3 for
// rounding), at most the detector; returns the dynamic LDS bytes of the two
// windows, or 0 where they take more copies than the kernel keeps offsets for or
// leave fewer than three blocks per CU.  Without pairs they always fit: e_j and e_k are
// unit vectors and 2 reach <= 2 |e|_1, so 5 |e_x| + 9 |e_y| + 9 |e_z| + 3 <= 16.7, that is
// 16 x 16 rays, four of six copies and 42 KiB at most.
static int window_lds(const std::vector<ProjFrame> &frames, const Dims &d, bool pair, bool jos, int &wr, int &wc)
{
    wr = wc = 0;
    const double sx = 3.0, sy = pair ? 3.0 : 7.0, sz = 7.0;
    for (const ProjFrame &f : frames) {
        const double rj = jos ? (double)f.jos_rj : f.lj, rk = jos ? (double)f.jos_rk : f.lk;
        const double sj = sx * fabs(f.ej[0]) + sy * fabs(f.ej[1]) + sz * fabs(f.ej[2]) + 2 * rj;
        const double sk = sx * fabs(f.ek[0]) + sy * fabs(f.ek[1]) + sz * fabs(f.ek[2]) + 2 * rk;
        wr = std::max(wr, (int)floor(sj) + 3);
        wc = std::max(wc, (int)floor(sk) + 3);
    }
    wr = std::min(wr, d.nj);
    wc = std::min(wc, d.nk);
    if (d.Up > 8) return 0;
    const int nel = (wr * wc * (d.Up / 4) * (pair ? 2 : 1) + 127) & ~127;
    const int fixed = (d.Up == 8 ? 3 : d.Cp >= 48 ? 4 : 2) * 8192 + 2048;
    const int copies = d.Up == 4 ? (pair ? kWinCopies<4, true> : kWinCopies<4, false>)
                                 : (pair ? kWinCopies<8, true> : kWinCopies<8, false>);
    return nel <= copies * 128 && 2 * nel * 16 + fixed <= 53 * 1024 ? 2 * nel * 16 : 0;
}

static int win_blocks(const Dims &d, bool pair)
{
    return pair ? ((d.nx / 2 + 3) / 4) * ((d.ny + 3) / 4) * ((d.nz + 7) / 8)
                : ((d.nx + 3) / 4) * ((d.ny + 7) / 8) * ((d.nz + 7) / 8);
}

// Samples of a ray above which the loop over those beyond the first three is unrolled by
// four (steps below about 0.45).  One sample at a time -> by fours, 64^3 / 120 projections /
// 45 coefficients, at steps 0.5, 0.4, 0.25, 0.1 (in brackets the kernels before the staged
// one, with a range per ray):
//   4 segments  445 -> 471  486 -> 426  602 -> 487  1072 ->  763 us  (464 474 512  766)
//   unpaired    664 -> 513  731 -> 546  921 -> 669  1698 -> 1171     (595 641 781 1340)
//   8 segments  542 -> 542  585 -> 565  713 -> 639  1236 ->  938     (803 842 957 1434)
//   unpaired    722 -> 738  792 -> 760  995 -> 886  1822 -> 1438     (790 833 966 1501)
// (4 segments from 0.4 on with four waves per SIMD).
constexpr int kFewSamples = 7;

void plan_adjoint(const std::vector<ProjFrame> &frames, Dims &d)
{
    int dev = 0, units = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || units < 1)
        units = 256;
    for (int jos = 0; jos < 2; ++jos) {
        AdjointPlan &p = d.adj[jos];
        p.pair = d.inv_pair;
        p.lds = window_lds(frames, d, p.pair != 0, jos != 0, p.wr, p.wc);
        if (p.lds == 0 && p.pair) {  // a paired window is twice as large per ray
            p.pair = 0;
            p.lds = window_lds(frames, d, false, jos != 0, p.wr, p.wc);
        }
        p.split_gain = 0.0;
        p.splits = p.lds > 0 ? adjoint_splits(d, win_blocks(d, p.pair != 0), units, p.split_gain) : 1;
        p.many = 0;
        for (const ProjFrame &f : frames)
            if (f.n_tau > kFewSamples) p.many = 1;
        // blocks per unit: four at a time where that saves a round, or in many rounds
        const long long n = ((long long)win_blocks(d, p.pair != 0) * p.splits + units - 1) / units;
        p.deep = n >= 10 ? 2 : (n + 2) / 3 > (n + 3) / 4 ? 1 : 0;
    }
}

int backproject_blocks(const Dims &d)
{
    const AdjointPlan &p = d.adj[d.joseph];
    return win_blocks(d, p.lds > 0 && p.pair);
}
int backproject_blocks_max(const Dims &d) { return std::max(win_blocks(d, true), win_blocks(d, false)); }

template <int UP, int MT, bool BF16, bool JOS>
static hipError_t bp_launch(const Dims &d, const ProjFrame *frames, const float *yf, const AdjointTables &t,
                            float *split, float *g, float beta, const float *c, double *partials, hipStream_t st)
{
    const AdjointPlan &p = d.adj[JOS];
    const int nb = backproject_blocks(d);
    if constexpr (UP > 8) {
        hipLaunchKernelGGL((k_backproject<UP, MT, BF16, JOS>), dim3(nb), dim3(256), 0, st, yf, frames, t.Bu,
                           reinterpret_cast<const s4 *>(t.BuT16), d.S, d.nx, d.ny, d.nz, d.nj, d.nk, d.C, d.Cp, d.step,
                           g, beta, c, partials);
        return hipGetLastError();
    } else {
        if (p.lds == 0) return hipErrorInvalidValue;  // (cannot be: see window_lds)
        const uint4 *bop = reinterpret_cast<const uint4 *>(t.Bop);
        const int ns = split ? p.splits : 1;
        const int s_per = ns > 1 ? (d.S + 4 * ns - 1) / (4 * ns) * 4 : d.S;  // whole double pairs
        const dim3 grid(nb, (d.S + s_per - 1) / s_per);
        float *sp = grid.y > 1 ? split : nullptr;
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(256), p.lds, st, yf, frames, bop, t.Bu, d.S, d.nx, d.ny, d.nz, d.nj,
                               d.nk, d.C, d.Cp, d.step, g, beta, c, partials, p.wr, p.wc, s_per, sp);
        };
        constexpr bool deep = UP == 4 && MT == 3 && !(BF16 && JOS);  // (that one fits four waves by itself)
        const bool many = !JOS && p.many;
        if constexpr (!JOS) {
            if (many && p.pair && p.deep == 1)
                launch(k_backproject_win<UP, MT, BF16, false, true, deep, true>);
            else if (many && p.pair)
                launch(k_backproject_win<UP, MT, BF16, false, true, false, true>);
            else if (many && p.deep)
                launch(k_backproject_win<UP, MT, BF16, false, false, deep, true>);
            else if (many)
                launch(k_backproject_win<UP, MT, BF16, false, false, false, true>);
        }
        if (!many && p.pair)
            launch(k_backproject_win<UP, MT, BF16, JOS, true>);
        else if (!many && p.deep)
            launch(k_backproject_win<UP, MT, BF16, JOS, false, deep>);
        else if (!many)
            launch(k_backproject_win<UP, MT, BF16, JOS, false>);
        // (the sum must not run over scratch that was not written)
        if (hipError_t e = hipGetLastError(); e != hipSuccess || !sp) return e;
        hipLaunchKernelGGL(k_add_splits, dim3(nb), dim3(256), 0, st, sp, (int)grid.y,
                           (long long)d.nx * d.ny * d.nz * d.C, g, beta, c, partials);
        return hipGetLastError();
    }
}

template <int UP, int MT>
static hipError_t bp_t(const Dims &d, const ProjFrame *frames, const float *yf, const AdjointTables &t, float *split, int bf16,
                       float *g, float beta, const float *c, double *partials, hipStream_t st)
{
    if (bf16 && d.joseph) return bp_launch<UP, MT, true, true>(d, frames, yf, t, split, g, beta, c, partials, st);
    if (bf16) return bp_launch<UP, MT, true, false>(d, frames, yf, t, split, g, beta, c, partials, st);
    if (d.joseph) return bp_launch<UP, MT, false, true>(d, frames, yf, t, split, g, beta, c, partials, st);
    return bp_launch<UP, MT, false, false>(d, frames, yf, t, split, g, beta, c, partials, st);
}

template <int UP>
static hipError_t bp_mt(const Dims &d, const ProjFrame *frames, const float *yf, const AdjointTables &t, float *split, int bf16,
                        float *g, float beta, const float *c, double *partials, hipStream_t st)
{
    switch (d.Cp / 16) {
    case 1: return bp_t<UP, 1>(d, frames, yf, t, split, bf16, g, beta, c, partials, st);
    case 2: return bp_t<UP, 2>(d, frames, yf, t, split, bf16, g, beta, c, partials, st);
    case 3: return bp_t<UP, 3>(d, frames, yf, t, split, bf16, g, beta, c, partials, st);
    case 4: return bp_t<UP, 4>(d, frames, yf, t, split, bf16, g, beta, c, partials, st);
    case 5: return bp_t<UP, 5>(d, frames, yf, t, split, bf16, g, beta, c, partials, st);
    case 6: return bp_t<UP, 6>(d, frames, yf, t, split, bf16, g, beta, c, partials, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_backproject(const Dims &d, const ProjFrame *frames, const float *yf, const AdjointTables &t,
                              float *split, int bf16, float *g, float beta, const float *c, double *partials, hipStream_t st)
{
    switch (d.Up) {
    case 4: return bp_mt<4>(d, frames, yf, t, split, bf16, g, beta, c, partials, st);
    case 8: return bp_mt<8>(d, frames, yf, t, split, bf16, g, beta, c, partials, st);
    case 16: return bp_mt<16>(d, frames, yf, t, split, bf16, g, beta, c, partials, st);
    default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// out[0] (+)= scale * sum(partials[0..n))
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_sum_partials(const double *__restrict__ partials, int n, double *out,
                                                      double scale, int accumulate)
{
    __shared__ double ws[4];
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) v += partials[i];
    double tot = block_sum(v, ws);
    if (threadIdx.x == 0) out[0] = (accumulate ? out[0] : 0.0) + scale * tot;
}

hipError_t launch_sum_partials(const double *partials, int n, double *out, double scale, int accumulate,
                               hipStream_t st)
{
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, st, partials, n, out, scale, accumulate);
    return hipGetLastError();
}

}  // namespace tt
