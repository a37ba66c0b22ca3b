// Warm-start network layers on gfx950: 3x3x3 convolutions (stride 1, zero
// padding 1) in channels-last layout as implicit GEMMs on bf16 MFMA with fp32
// accumulation, their gradients, Adam, the MSE loss and layout packing.
//
//   forward  y[v, co] = b[co] + sum_d sum_ci x[v + d - 1, ci] w[d, ci, co]
//   dgrad    gx[v, ci] = sum_d sum_co gy[v - d + 1, co] w[d, ci, co]
//            = the forward with w'[d][co][ci] = w[2 - d][ci][co]
//   wgrad    gw[d, ci, co] = sum_v x[v + d - 1, ci] gy[v, co]
//
// Channel counts are 32 or 64 (the network pads 28 to 32).  Tap index
// d = (dx * 3 + dy) * 3 + dz.  Activations are bf16, weights fp32 masters
// with bf16 MFMA-ordered copies.
#include "tt_device.h"
#include "tt_internal.h"

namespace tt {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));    // eight bf16 bit patterns
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16;

// gfx950 v_mfma_f32_16x16x32_bf16: D[16x16] += A[16x32] B[32x16].  Lane l
// supplies row (A) / column (B) l % 16 and eight consecutive k of the group
// l / 16; D as for the 16x16x16 forms (lane holds rows 4 (l / 16) + r of
// column l % 16).  A and B take the same k order, so the per-lane k
// assignment inside a group does not change the sum.
__device__ __forceinline__ f4 mfma_bf16(s8 a, s8 b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0,
                                                   0);
}

__device__ __forceinline__ u16 f2bf(float x)
{
    unsigned u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}

__device__ __forceinline__ float bf2f(u16 h) { return __uint_as_float((unsigned)h << 16); }

enum { EPI_RELU_BF16 = 0, EPI_BIAS_F32 = 1, EPI_MASK_BF16 = 2 };

// ---------------------------------------------------------------------------
// Convolution as implicit GEMM: rows = CO, columns = the block's voxels, K = 27
// taps x CI.  Tile: 4 (x) x TY (y) x 8 (z) voxels, wave w owning the x-slice w.  The
// (tile + 1)-halo of the input is staged in LDS once, as it is in memory; each tap
// reads it at a shifted position.  The 16-byte octets of a voxel are rotated by the
// voxel's index (octet ^ (p mod 8 or 4)), which spreads the reads of one octet of
// 16 voxels over the banks without padding.
//
// What bounded the kernel it replaces (batch 8 x 48^3, 64 -> 64: 280 us, MFMAs busy
// 29%): each wave read a weight fragment right before its use, from L2 (all fragments
// are 27 CI CO shorts, more than L1 holds), the halo's loads were waited for one by
// one, and its stores were two bytes a lane.  Now the weights come two steps ahead, a
// fragment serves VT = TY / 2 column tiles (64 voxels a wave instead of 32), ten halo
// loads of a thread are in flight together, and a lane stores four channels.  TY = 8
// where there are blocks enough to fill the chip, TY = 4 for smaller volumes.
// Forward / input gradient, batch 8 x 48^3, before -> now: 64 -> 64 280 -> 235 / 319 ->
// 242 us (834 / 808 TFLOP/s; a large bf16 matrix product reaches 1130 here), 32 -> 64
// 149 -> 116 / 210 -> 144, 64 -> 32 191 -> 141 / 165 -> 138, 32 -> 32 84 -> 63 / 92 -> 73;
// batch 1, 64 -> 64 48 -> 35 / 55 -> 37.
// ---------------------------------------------------------------------------
template <int CI, int CO, int EPI, int TY>
__global__ __launch_bounds__(256, 2) void k_conv(const u16 *__restrict__ x, const s8 *__restrict__ wsw,
                                              const float *__restrict__ bias, const u16 *__restrict__ mask,
                                              void *__restrict__ y, int X, int Y, int Z)
{
    constexpr int TX = 4, TZ = 8, HY = TY + 2, HZ = TZ + 2, HV = (TX + 2) * HY * HZ;
    constexpr int CH = CI / 8;                   // 16-byte octets per voxel
    constexpr int VT = TY / 2, NT = CO / 16, CB = CI / 32;
    __shared__ uint4 halo[HV * CH];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nbz = (Z + TZ - 1) / TZ, nby = (Y + TY - 1) / TY, nbx = (X + TX - 1) / TX;
    int b = blockIdx.x;
    const int bz = b % nbz;
    b /= nbz;
    const int by = b % nby;
    b /= nby;
    const int bx = b % nbx;
    const int n = b / nbx;
    const int x0 = bx * TX - 1, y0 = by * TY - 1, z0 = bz * TZ - 1;
    const long long vol = (long long)X * Y * Z;
    const u16 *xn = x + (long long)n * vol * CI;
    // the halo's octets, ten loads of a thread in flight together (outside the volume
    // they read the image's first voxel and store zero)
    constexpr int NH = (HV * CH + 255) / 256;
#pragma unroll
    for (int i0 = 0; i0 < NH; i0 += 10) {
        uint4 r[10];
#pragma unroll
        for (int i = i0; i < min(i0 + 10, NH); ++i) {
            const int e = min(tid + 256 * i, HV * CH - 1), p = e / CH;
            const int hz = p % HZ, hy = (p / HZ) % HY, hx = p / (HZ * HY);
            const int gx = x0 + hx, gy = y0 + hy, gz = z0 + hz;
            const bool in = (unsigned)gx < (unsigned)X && (unsigned)gy < (unsigned)Y && (unsigned)gz < (unsigned)Z;
            const uint4 v = *reinterpret_cast<const uint4 *>(
                xn + (in ? (((long long)gx * Y + gy) * Z + gz) * CI + e % CH * 8 : 0LL));
            r[i - i0] = in ? v : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = i0; i < min(i0 + 10, NH); ++i) {
            const int e = tid + 256 * i, p = e / CH;
            if (e < HV * CH) halo[p * CH + ((e % CH) ^ (p & (CH - 1)))] = r[i - i0];
        }
    }
    // weight fragments of step (tap, cb), two steps ahead of the MFMAs
    const int kq = lane >> 4, m = lane & 15;
    const s8 *wp = wsw + lane;
    s8 wv[3][NT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) wv[i][nt] = wp[(i * NT + nt) * 64];
    __syncthreads();

    f4 acc[VT][NT];
#pragma unroll
    for (int vt = 0; vt < VT; ++vt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[vt][nt] = f4{0.f, 0.f, 0.f, 0.f};
    // the voxel this lane supplies to column tile vt: y = 2 vt + m / 8, z = m % 8 of slice `wave`
    int row = (wave * HY + (m >> 3)) * HZ + (m & 7);
    constexpr int STEPS = 27 * CB;
    for (int xy = 0; xy < 9; ++xy) {
#pragma unroll
        for (int i = 0; i < 3 * CB; ++i) {  // dz, cb
            const int dz = i / CB, cb = i % CB;
            const int ahead = min(xy * 3 * CB + i + 2, STEPS - 1);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) wv[(i + 2) % 3][nt] = wp[(ahead * NT + nt) * 64];
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) {
                const int p = row + dz + vt * 2 * HZ;
                const s8 xv = __builtin_bit_cast(s8, halo[p * CH + ((cb * 4 + kq) ^ (p & (CH - 1)))]);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[vt][nt] = mfma_bf16(wv[i % 3][nt], xv, acc[vt][nt]);
            }
        }
        row += xy % 3 == 2 ? (HY - 2) * HZ : HZ;  // the next (dx, dy)
    }
    // epilogue: lane holds channels 16 nt + 4 kq + r of voxel column m: four channels a store
    const int gx = x0 + 1 + wave, gz = z0 + 1 + (m & 7);
#pragma unroll
    for (int vt = 0; vt < VT; ++vt) {
        const int gy = y0 + 1 + 2 * vt + (m >> 3);
        if (gx >= X || gy >= Y || gz >= Z) continue;
        const long long vi = (long long)n * vol + ((long long)gx * Y + gy) * Z + gz;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int co = nt * 16 + 4 * kq;
            f4 v = acc[vt][nt];
            if (EPI == EPI_MASK_BF16) {
                const uint2 k = *reinterpret_cast<const uint2 *>(mask + vi * CO + co);
                v[0] = __uint_as_float(k.x << 16) > 0.0f ? v[0] : 0.0f;
                v[1] = __uint_as_float(k.x & 0xffff0000u) > 0.0f ? v[1] : 0.0f;
                v[2] = __uint_as_float(k.y << 16) > 0.0f ? v[2] : 0.0f;
                v[3] = __uint_as_float(k.y & 0xffff0000u) > 0.0f ? v[3] : 0.0f;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] += bias[co + r];
            }
            if (EPI == EPI_BIAS_F32) {
                *reinterpret_cast<f4 *>(reinterpret_cast<float *>(y) + vi * CO + co) = v;
            } else {
                if (EPI == EPI_RELU_BF16) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.0f);
                }
                const unsigned lo = f2bf(v[0]) | (unsigned)f2bf(v[1]) << 16, hi = f2bf(v[2]) | (unsigned)f2bf(v[3]) << 16;
                *reinterpret_cast<uint2 *>(reinterpret_cast<u16 *>(y) + vi * CO + co) = make_uint2(lo, hi);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Weight gradient gw[d][ci][co] = sum_v x[v + d - 1, ci] gy[v, co] as a GEMM with
// K = voxels.  Block (dx, chunk) accumulates the nine taps (dx, *, *) over the voxel
// tiles t = chunk, chunk + nchunks, ... in registers (each wave a quarter of the
// CI x CO outputs of every tap) and writes its partials; a second kernel sums them
// in chunk order.
//
// The tile (2 x 8 x 8 voxels) of gy and its halo of x (x shifted by dx - 1, one
// voxel more in y and z) are staged channels-last, as they are in memory.  The
// operands need eight consecutive voxels of one channel per lane, so they are read
// with gfx950's transposing LDS loads (a group of 16 lanes reads 4 voxels x 16
// channels and each lane gets one channel's 4 voxels); a tap is a shifted read.
// K = 32 takes the z-rows y = j, j + 2, j + 4, j + 6 (lane group kq: y = j + 2 kq), so
// that the operand of tap dy at j is that of row offset j + dy - 1 in the same lanes:
// 12 x fragments per x-slice serve 18 (j, tap) products.  The next tile's loads are
// in flight during the MFMAs.
//
// What bounded the kernel it replaces (one tap per block): 27 reads of x and gy and
// an 8 x 8 register transpose per staged octet, MFMAs 4-8% of the time.  Layer
// 64 -> 64 at batch 8 x 48^3: 829 -> 214 us.
//
// gb: each tile's gy is summed, as it is staged, by one of its three blocks.
// ---------------------------------------------------------------------------
constexpr int WX = 2, WY = 8, WZ = 8, WV = WX * WY * WZ;      // tile
constexpr int WHY = WY + 2, WHZ = WZ + 2, WHV = WX * WHY * WHZ;  // x halo (x extent WX)

typedef short s4 __attribute__((ext_vector_type(4)));

// eight voxels (two groups of four, `step` shorts apart) of one channel per lane
__device__ __forceinline__ s8 read_tr(const u16 *p, int step)
{
    typedef __attribute__((address_space(3))) s4 *lp;
    const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p));
    const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + step));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

template <int CI, int CO>
__global__ __launch_bounds__(256, 2) void k_wgrad(const u16 *__restrict__ x, const u16 *__restrict__ gy, int N, int X,
                                                  int Y, int Z, int nchunks, float *__restrict__ part,
                                                  float *__restrict__ bpart)
{
    constexpr int LX = CI + 8, LG = CO + 8;     // padded voxel strides (shorts): spread over the banks
    constexpr int CX = CI / 8, CG = CO / 8;     // 16-byte octets per voxel
    constexpr int NX = (WHV * CX + 255) / 256, NG = WV * CG / 256;  // staged octets per thread
    constexpr int WM = CI == CO ? 2 : (CI < CO ? 1 : 4), WN = 4 / WM;  // waves over ci and co
    constexpr int MT = CI / 16 / WM, NT = CO / 16 / WN;
    __shared__ __attribute__((aligned(16))) u16 xs[WHV * LX];
    __shared__ __attribute__((aligned(16))) u16 gs[WV * LG];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the three blocks of a chunk run on one XCD (blocks go round the eight XCDs)
    const int i8 = blockIdx.x >> 3, chunk = (i8 / 3) * 8 + (blockIdx.x & 7), dxi = i8 % 3;
    if (chunk >= nchunks) return;
    const int nbz = (Z + WZ - 1) / WZ, nby = (Y + WY - 1) / WY, nbx = (X + WX - 1) / WX;
    const int ntiles = N * nbx * nby * nbz;
    const long long vol = (long long)X * Y * Z;

    uint4 rx[NX], rg[NG];
    auto load = [&](int t) {
#pragma unroll
        for (int i = 0; i < NX; ++i) rx[i] = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < NG; ++i) rg[i] = make_uint4(0, 0, 0, 0);
        if (t >= ntiles) return;
        int b = t;
        const int z0 = b % nbz * WZ;
        b /= nbz;
        const int y0 = b % nby * WY;
        b /= nby;
        const int x0 = b % nbx * WX, n = b / nbx;
        const u16 *xn = x + (long long)n * vol * CI, *gn = gy + (long long)n * vol * CO;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int e = tid + 256 * i, p = e / CX;
            const int gx = x0 + p / (WHY * WHZ) + dxi - 1, gyy = y0 + p / WHZ % WHY - 1, gz = z0 + p % WHZ - 1;
            if (e < WHV * CX && (unsigned)gx < (unsigned)X && (unsigned)gyy < (unsigned)Y && (unsigned)gz < (unsigned)Z)
                rx[i] = *reinterpret_cast<const uint4 *>(xn + (((long long)gx * Y + gyy) * Z + gz) * CI + e % CX * 8);
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int e = tid + 256 * i, p = e / CG;
            const int gx = x0 + p / (WY * WZ), gyy = y0 + p / WZ % WY, gz = z0 + p % WZ;
            if (gx < X && gyy < Y && gz < Z)
                rg[i] = *reinterpret_cast<const uint4 *>(gn + (((long long)gx * Y + gyy) * Z + gz) * CO + e % CG * 8);
        }
    };

    f4 acc[9][MT][NT];
#pragma unroll
    for (int a = 0; a < 9; ++a)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[a][mt][nt] = f4{0.f, 0.f, 0.f, 0.f};
    float bs[8];  // sums of this thread's octet of gy channels
#pragma unroll
    for (int q = 0; q < 8; ++q) bs[q] = 0.0f;
    // this lane's place in a transposing read: voxel row lane % 16 / 4, four channels
    const int kq = lane >> 4, m = lane & 15;
    const int wm = wave % WM, wn = wave / WM;
    const u16 *xa = xs + (2 * kq * WHZ + (m >> 2)) * LX + wm * MT * 16 + (m & 3) * 4;
    const u16 *ga = gs + (2 * kq * WZ + (m >> 2)) * LG + wn * NT * 16 + (m & 3) * 4;

    load(chunk);
    for (int t = chunk, it = 0; t < ntiles; t += nchunks, ++it) {
        __syncthreads();  // the previous tile's reads are done
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int e = tid + 256 * i;
            if (e < WHV * CX) *reinterpret_cast<uint4 *>(xs + e / CX * LX + e % CX * 8) = rx[i];
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int e = tid + 256 * i;
            *reinterpret_cast<uint4 *>(gs + e / CG * LG + e % CG * 8) = rg[i];
        }
        if (bpart && it % 3 == dxi) {
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                const unsigned w[4] = {rg[i].x, rg[i].y, rg[i].z, rg[i].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    bs[2 * q] += __uint_as_float(w[q] << 16);
                    bs[2 * q + 1] += __uint_as_float(w[q] & 0xffff0000u);
                }
            }
        }
        __syncthreads();
        load(t + nchunks);  // next tile in flight during the MFMAs
#pragma unroll 1
        for (int xi = 0; xi < WX; ++xi) {
            s8 bv[2][NT];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    bv[j][nt] = read_tr(ga + (xi * WY + j) * WZ * LG + nt * 16, 4 * LG);
#pragma unroll
            for (int r = 0; r < 4; ++r) {  // halo row offset: y = r - 1 + 2 kq
#pragma unroll
                for (int dz = 0; dz < 3; ++dz) {
                    s8 av[MT];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        av[mt] = read_tr(xa + ((xi * WHY + r) * WHZ + dz) * LX + mt * 16, 4 * LX);
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy) {
                        const int j = r - dy;
                        if (j < 0 || j > 1) continue;
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt)
                                acc[dy * 3 + dz][mt][nt] = mfma_bf16(av[mt], bv[j][nt], acc[dy * 3 + dz][mt][nt]);
                    }
                }
            }
        }
    }
    // partial[chunk][tap][ci][co]; lane holds rows ci = 16 mt + 4 kq + r, column co = 16 nt + lane % 16
    float *pp = part + ((long long)chunk * 27 + dxi * 9) * CI * CO;
#pragma unroll
    for (int a = 0; a < 9; ++a)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    pp[(a * CI + (wm * MT + mt) * 16 + 4 * kq + r) * CO + (wn * NT + nt) * 16 + m] = acc[a][mt][nt][r];
    if (bpart) {  // thread t holds channels 8 (t % CG) .. + 7
        float *red = reinterpret_cast<float *>(xs);
        static_assert(sizeof(xs) >= 256 * 8 * sizeof(float), "room for the sums");
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 8; ++q) red[tid * 8 + q] = bs[q];
        __syncthreads();
        if (tid < CO) {
            float s = 0.0f;
            for (int i = tid / 8; i < 256; i += CG) s += red[i * 8 + tid % 8];
            bpart[((long long)chunk * 3 + dxi) * CO + tid] = s;
        }
    }
}

__global__ __launch_bounds__(256) void k_wgrad_reduce(const float *__restrict__ part, int nchunks, int n,
                                                      float *__restrict__ gw)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    float s = 0.0f;
#pragma unroll 8
    for (int c = 0; c < nchunks; ++c) s += part[(long long)c * n + e];
    gw[e] = s;
}

// bias gradient: gb[co] = sum over blocks, one block per channel: thread t
// adds partials t, t + 256, ... in order, then a fixed-shape tree in LDS
__global__ __launch_bounds__(256) void k_bias_reduce(const float *__restrict__ partial, int nblk, int CO, float *gb)
{
    __shared__ float sh[256];
    const int c = blockIdx.x, t = threadIdx.x;
    float s = 0.0f;
    for (int b = t; b < nblk; b += 256) s += partial[(long long)b * CO + c];
    sh[t] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) sh[t] += sh[t + w];
        __syncthreads();
    }
    if (t == 0) gb[c] = sh[0];
}

// MFMA-ordered bf16 copies of w[27][ci][co]: forward (B[k = ci][n = co]) and
// dgrad (w'[d][co][ci] = w[26 - d][ci][co], B[k = co][n = ci]), eight k per lane.
__global__ __launch_bounds__(256) void k_swizzle(const float *__restrict__ w, int CI, int CO, s8 *__restrict__ wf,
                                                 s8 *__restrict__ wd)
{
    const int total = 27 * (CI / 32) * (CO / 16) * 64;  // = 27 (CO / 32) (CI / 16) 64
    for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
        const int l = e % 64;
        int r = e / 64;
        // forward: e = ((tap * CB + cb) * NT + nt) * 64 + l with CB = CI/32, NT = CO/16
        {
            const int nt = r % (CO / 16), cb = (r / (CO / 16)) % (CI / 32), tap = r / ((CO / 16) * (CI / 32));
            const int co = nt * 16 + l % 16, ci0 = cb * 32 + 8 * (l / 16);
            s8 v;
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = (short)f2bf(w[((long long)tap * CI + ci0 + q) * CO + co]);
            wf[e] = v;
        }
        // dgrad: input channels CO, output channels CI: e = ((tap * (CO/32) + cb) * (CI/16) + nt) * 64 + l
        {
            const int nt = r % (CI / 16), cb = (r / (CI / 16)) % (CO / 32), tap = r / ((CI / 16) * (CO / 32));
            const int src = 26 - tap;
            const int ci = nt * 16 + l % 16, co0 = cb * 32 + 8 * (l / 16);
            s8 v;
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = (short)f2bf(w[((long long)src * CI + ci) * CO + co0 + q]);
            wd[e] = v;
        }
    }
}

__global__ __launch_bounds__(256) void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                                              float *__restrict__ v, long long n, float lr, float b1, float b2,
                                              float eps, float c1, float c2)
{
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const float ge = g[e];
        const float me = b1 * m[e] + (1.0f - b1) * ge;
        const float ve = b2 * v[e] + (1.0f - b2) * ge * ge;
        m[e] = me;
        v[e] = ve;
        w[e] -= lr * (me / c1) / (sqrtf(ve / c2) + eps);
    }
}

// gy = scale (y - t) on the first creal of cpad channels (0 elsewhere), in bf16;
// partials of sum (y - t)^2 in float64.
__global__ __launch_bounds__(256) void k_mse(const float *__restrict__ y, const float *__restrict__ t, long long nvox,
                                             int cpad, int creal, float scale, u16 *__restrict__ gy,
                                             double *__restrict__ partials)
{
    __shared__ double ws[4];
    double s = 0.0;
    const long long n = nvox * cpad;
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const long long v = e / cpad;
        const int c = (int)(e % cpad);
        float d = 0.0f;
        if (c < creal) {
            d = y[e] - t[v * creal + c];
            s += (double)d * d;
        }
        if (gy) gy[e] = f2bf(scale * d);
    }
    s = block_sum(s, ws);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// out[v][c] = bf16(scale[c] * (x[v][c] - shift[c])) for c < cin, 0 for cin <= c < cpad
__global__ __launch_bounds__(256) void k_pack(const float *__restrict__ x, long long nvox, int cin, int cpad,
                                              float pre, const float *__restrict__ shift,
                                              const float *__restrict__ scale, u16 *__restrict__ out)
{
    const long long n = nvox * cpad;
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const long long v = e / cpad;
        const int c = (int)(e % cpad);
        float val = 0.0f;
        if (c < cin) {
            val = pre * x[v * cin + c];
            if (shift) val -= shift[c];
            if (scale) val *= scale[c];
        }
        out[e] = f2bf(val);
    }
}

// Patchwise inference.  Tiles of T^3 voxels at per-axis origins ox[], oy[], oz[]
// (tile t = (i nx_t + j) ny_t... in x-major order).
// gather: out[t][T^3][cpad] = bf16(scale[c] (pre vol[o_t + u][c] - shift[c])) for c < cin.
__global__ __launch_bounds__(256) void k_tile_gather(const float *__restrict__ vol, int X, int Y, int Z, int cv, int cin,
                                                     int cpad, const int *__restrict__ ox, int ntx,
                                                     const int *__restrict__ oy, int nty, const int *__restrict__ oz,
                                                     int ntz, int T, float pre, const float *__restrict__ shift,
                                                     const float *__restrict__ scale, int t0, int nt,
                                                     u16 *__restrict__ out)
{
    const long long per = (long long)T * T * T * cpad;
    const long long n = per * nt;
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const int t = t0 + (int)(e / per);
        long long r = e % per;
        const int c = (int)(r % cpad);
        r /= cpad;
        const int uz = (int)(r % T), uy = (int)((r / T) % T), ux = (int)(r / ((long long)T * T));
        const int iz = t % ntz, iy = (t / ntz) % nty, ix = t / (ntz * nty);
        const int gx = ox[ix] + ux, gy = oy[iy] + uy, gz = oz[iz] + uz;
        float v = 0.0f;
        if (c < cin && gx < X && gy < Y && gz < Z) {
            v = pre * vol[(((long long)gx * Y + gy) * Z + gz) * cv + c];
            if (shift) v -= shift[c];
            if (scale) v *= scale[c];
        }
        out[e] = f2bf(v);
    }
}

// Separable blending weight of position u in a tile starting at o along an
// axis of length n: a linear ramp over `ramp` voxels on sides that overlap
// another tile, 1 on sides at the volume boundary.
__device__ __forceinline__ float ramp_w(int u, int o, int T, int n, int ramp)
{
    float w = 1.0f;
    if (o > 0) w = fminf(w, (u + 0.5f) / ramp);
    if (o + T < n) w = fminf(w, (T - u - 0.5f) / ramp);
    return w;
}

// blend: out[v][c] = sum_t w_t(v) y_t[v - o_t][c] / sum_t w_t(v) for c < creal,
// 0 for creal <= c < cout.  One thread per (voxel, channel); fixed tile order.
__global__ __launch_bounds__(256) void k_tile_blend(const float *__restrict__ y, int cy, int creal, int X, int Y, int Z,
                                                    const int *__restrict__ ox, int ntx, const int *__restrict__ oy,
                                                    int nty, const int *__restrict__ oz, int ntz, int T, int ramp,
                                                    int cout, float *__restrict__ out)
{
    const long long n = (long long)X * Y * Z * cout;
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const int c = (int)(e % cout);
        const long long v = e / cout;
        const int gz = (int)(v % Z), gy = (int)((v / Z) % Y), gx = (int)(v / ((long long)Y * Z));
        float num = 0.0f, den = 0.0f;
        if (c < creal) {
            for (int ix = 0; ix < ntx; ++ix) {
                const int ux = gx - ox[ix];
                if (ux < 0 || ux >= T) continue;
                const float wx = ramp_w(ux, ox[ix], T, X, ramp);
                for (int iy = 0; iy < nty; ++iy) {
                    const int uy = gy - oy[iy];
                    if (uy < 0 || uy >= T) continue;
                    const float wy = ramp_w(uy, oy[iy], T, Y, ramp);
                    for (int iz = 0; iz < ntz; ++iz) {
                        const int uz = gz - oz[iz];
                        if (uz < 0 || uz >= T) continue;
                        const float w = wx * wy * ramp_w(uz, oz[iz], T, Z, ramp);
                        const long long t = ((long long)ix * nty + iy) * ntz + iz;
                        num += w * y[((t * T + ux) * T + uy) * (long long)T * cy + (long long)uz * cy + c];
                        den += w;
                    }
                }
            }
        }
        out[e] = den > 0.0f ? num / den : 0.0f;
    }
}

int grid_for(long long n) { return (int)min((n + 255) / 256, 8192LL); }

// Blocks of the 4 x 8 x 8-voxel tile below which the 4 x 4 x 8 one is used: it has about
// twice as many, of which three fit a compute unit at once (768), and saves nothing once
// they need a second round.  Narrow against wide tile, forward 64 -> 64: 54 blocks 12.0 and
// 18.6 us, 128 12.6 and 19.0, 225 19.3 and 19.3, 396 27.3 and 28.2, 432 36.4 and 32.0, 500
// 40.0 and 33.1, 1728 121 and 112; 64 -> 32: 225 11.2 and 13.0, 396 16.2 and 17.0, 432 23.1
// and 18.5; 32 -> 32: 336 9.2 and 10.1, 450 11.6 and 10.5.
constexpr int kConvWideBlocks = 400;

template <int CI, int CO, int EPI>
hipError_t conv_t(const u16 *x, const void *wsw, const float *bias, const u16 *mask, void *y, int N, int X, int Y, int Z,
                  hipStream_t st)
{
    auto blocks = [&](int ty) { return N * ((X + 3) / 4) * ((Y + ty - 1) / ty) * ((Z + 7) / 8); };
    const s8 *w = reinterpret_cast<const s8 *>(wsw);
    if (blocks(8) >= kConvWideBlocks)
        hipLaunchKernelGGL((k_conv<CI, CO, EPI, 8>), dim3(blocks(8)), dim3(256), 0, st, x, w, bias, mask, y, X, Y, Z);
    else
        hipLaunchKernelGGL((k_conv<CI, CO, EPI, 4>), dim3(blocks(4)), dim3(256), 0, st, x, w, bias, mask, y, X, Y, Z);
    return hipGetLastError();
}

template <int EPI>
hipError_t conv_dispatch(int ci, int co, const u16 *x, const void *wsw, const float *bias, const u16 *mask, void *y,
                         int N, int X, int Y, int Z, hipStream_t st)
{
    if (ci == 32 && co == 32) return conv_t<32, 32, EPI>(x, wsw, bias, mask, y, N, X, Y, Z, st);
    if (ci == 32 && co == 64) return conv_t<32, 64, EPI>(x, wsw, bias, mask, y, N, X, Y, Z, st);
    if (ci == 64 && co == 32) return conv_t<64, 32, EPI>(x, wsw, bias, mask, y, N, X, Y, Z, st);
    if (ci == 64 && co == 64) return conv_t<64, 64, EPI>(x, wsw, bias, mask, y, N, X, Y, Z, st);
    return hipErrorInvalidValue;
}

template <int CI, int CO>
hipError_t wgrad_t(const u16 *x, const u16 *gy, int N, int X, int Y, int Z, int nchunks, float *part, float *bpart,
                   float *gw, hipStream_t st)
{
    hipLaunchKernelGGL((k_wgrad<CI, CO>), dim3(3 * 8 * ((nchunks + 7) / 8)), dim3(256), 0, st, x, gy, N, X, Y, Z, nchunks,
                       part, bpart);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((27 * CI * CO + 255) / 256), dim3(256), 0, st, part, nchunks, 27 * CI * CO,
                       gw);
    return hipGetLastError();
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers used by the C ABI
// ---------------------------------------------------------------------------
hipError_t net_conv(int epi, int ci, int co, const uint16_t *x, const void *wsw, const float *bias,
                    const uint16_t *mask, void *y, int N, int X, int Y, int Z, hipStream_t st)
{
    switch (epi) {
    case EPI_RELU_BF16: return conv_dispatch<EPI_RELU_BF16>(ci, co, x, wsw, bias, mask, y, N, X, Y, Z, st);
    case EPI_BIAS_F32: return conv_dispatch<EPI_BIAS_F32>(ci, co, x, wsw, bias, mask, y, N, X, Y, Z, st);
    case EPI_MASK_BF16: return conv_dispatch<EPI_MASK_BF16>(ci, co, x, wsw, bias, mask, y, N, X, Y, Z, st);
    default: return hipErrorInvalidValue;
    }
}

// Chunks of voxel tiles: three blocks each, so that 168 chunks are the 504 blocks that
// fit the chip at once (two per compute unit); at least two tiles per chunk, as each
// writes 27 CI CO partials.
int net_wgrad_chunks(int N, int X, int Y, int Z)
{
    const long long ntiles = (long long)N * ((X + WX - 1) / WX) * ((Y + WY - 1) / WY) * ((Z + WZ - 1) / WZ);
    return (int)std::max(1LL, std::min(168LL, (ntiles + 1) / 2));
}

size_t net_wgrad_work_bytes(int ci, int co, int N, int X, int Y, int Z)
{
    return (size_t)net_wgrad_chunks(N, X, Y, Z) * (27 * ci * co + 3 * co) * sizeof(float);
}

hipError_t net_wgrad(int ci, int co, const uint16_t *x, const uint16_t *gy, int N, int X, int Y, int Z, float *work,
                     float *gw, float *gb, hipStream_t st)
{
    const int nch = net_wgrad_chunks(N, X, Y, Z);
    float *bp = gb ? work + (size_t)27 * nch * ci * co : nullptr;
    hipError_t e;
    if (ci == 32 && co == 32) e = wgrad_t<32, 32>(x, gy, N, X, Y, Z, nch, work, bp, gw, st);
    else if (ci == 32 && co == 64) e = wgrad_t<32, 64>(x, gy, N, X, Y, Z, nch, work, bp, gw, st);
    else if (ci == 64 && co == 32) e = wgrad_t<64, 32>(x, gy, N, X, Y, Z, nch, work, bp, gw, st);
    else if (ci == 64 && co == 64) e = wgrad_t<64, 64>(x, gy, N, X, Y, Z, nch, work, bp, gw, st);
    else return hipErrorInvalidValue;
    if (e != hipSuccess || !gb) return e;
    hipLaunchKernelGGL(k_bias_reduce, dim3(co), dim3(256), 0, st, bp, 3 * nch, co, gb);
    return hipGetLastError();
}

hipError_t net_swizzle(const float *w, int ci, int co, void *wf, void *wd, hipStream_t st)
{
    const int total = 27 * (ci / 32) * (co / 16) * 64;
    hipLaunchKernelGGL(k_swizzle, dim3((total + 255) / 256), dim3(256), 0, st, w, ci, co, reinterpret_cast<s8 *>(wf),
                       reinterpret_cast<s8 *>(wd));
    return hipGetLastError();
}

hipError_t net_adam(float *w, const float *g, float *m, float *v, long long n, int t, float lr, float b1, float b2,
                    float eps, hipStream_t st)
{
    const float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3(grid_for(n)), dim3(256), 0, st, w, g, m, v, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t net_mse(const float *y, const float *t, long long nvox, int cpad, int creal, float scale, uint16_t *gy,
                   double *partials, int nblocks, double *loss, hipStream_t st)
{
    hipLaunchKernelGGL(k_mse, dim3(nblocks), dim3(256), 0, st, y, t, nvox, cpad, creal, scale, gy, partials);
    return launch_sum_partials(partials, nblocks, loss, 1.0, 0, st);
}

hipError_t net_tile_gather(const float *vol, int X, int Y, int Z, int cv, int cin, int cpad, const int *ox, int ntx,
                           const int *oy, int nty, const int *oz, int ntz, int T, float pre, const float *shift,
                           const float *scale, int t0, int nt, uint16_t *out, hipStream_t st)
{
    const long long n = (long long)T * T * T * cpad * nt;
    hipLaunchKernelGGL(k_tile_gather, dim3(grid_for(n)), dim3(256), 0, st, vol, X, Y, Z, cv, cin, cpad, ox, ntx, oy, nty,
                       oz, ntz, T, pre, shift, scale, t0, nt, out);
    return hipGetLastError();
}

hipError_t net_tile_blend(const float *y, int cy, int creal, int X, int Y, int Z, const int *ox, int ntx, const int *oy,
                          int nty, const int *oz, int ntz, int T, int ramp, int cout, float *out, hipStream_t st)
{
    const long long n = (long long)X * Y * Z * cout;
    hipLaunchKernelGGL(k_tile_blend, dim3(grid_for(n)), dim3(256), 0, st, y, cy, creal, X, Y, Z, ox, ntx, oy, nty, oz,
                       ntz, T, ramp, cout, out);
    return hipGetLastError();
}

hipError_t net_pack(const float *x, long long nvox, int cin, int cpad, float pre, const float *shift,
                    const float *scale, uint16_t *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_pack, dim3(grid_for(nvox * cpad)), dim3(256), 0, st, x, nvox, cin, cpad, pre, shift, scale,
                       out);
    return hipGetLastError();
}

}  // namespace tt
