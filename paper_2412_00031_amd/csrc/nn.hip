// nn.hip -- kernels and C ABI (include/nn.h) of the warm-start 3-D U-Net.
//
// The network predicts the factor tau of T = T0 * tau (multiplicative
// factorisation, Sec. 3.1) from the model so that the sweeps of Eq. (4) start
// near their fixed point.  3^3 convolutions run on the matrix cores
// (v_mfma_f32_16x16x16_bf16: bf16 operands, fp32 accumulation) as implicit
// GEMMs over channels-last activations; pooling, transposed up-sampling, the
// 1x1 head, the loss and Adam are plain vector kernels.  Every reduction runs
// in a fixed order, so results are bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#include "nn.h"
#include "tt_internal.h"

namespace {

using tt::fail;

#define NN_HIP(call)                                                                          \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess) return fail(TT_EHIP, "%s: %s", #call, hipGetErrorString(e_));   \
    } while (0)

#define NN_LAUNCHED() NN_HIP(hipGetLastError())

typedef short s4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

constexpr int kMB = 4;  // 16-position blocks of one wave in the convolution

__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;  // NaN
    u += 0x7fffu + ((u >> 16) & 1u);                      // round to nearest even
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

unsigned blocks_of(long long n, int per) { return (unsigned)((n + per - 1) / per); }

hipStream_t S(void* st) { return reinterpret_cast<hipStream_t>(st); }

// ------------------------------------------------------------------ casts
__global__ void k_to_bf16(const float* __restrict__ x, long long n, uint16_t* __restrict__ y) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        y[i] = f2bf(x[i]);
}

__global__ void k_from_bf16(const uint16_t* __restrict__ x, long long n, float* __restrict__ y) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        y[i] = bf2f(x[i]);
}

unsigned grid_stride_blocks(long long n) {
    long long b = (n + 255) / 256;
    return (unsigned)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

// ------------------------------------------------------- weight fragments
// Operand-B fragment of the 16x16x16 bf16 MFMA: lane l holds B[4(l/16)+v][l%16],
// v = 0..3.  The packed index is (((t*KB + kb)*NB + nb)*64 + lane)*4 + v.
// flip = 0: B[k][n] = W[t][kb*16+k][nb*16+n] (rows >= cin are zero).
// flip = 1: data-gradient weights W'[t][o][i] = W[26-t][i][o].
__global__ void k_conv3_pack(const float* __restrict__ W, int cin, int cout, int KB, int NB, int flip,
                             uint16_t* __restrict__ frag) {
    const long long total = 27LL * KB * NB * 256;
    for (long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x; idx < total;
         idx += (long long)gridDim.x * blockDim.x) {
        const int v = (int)(idx & 3), lane = (int)((idx >> 2) & 63);
        long long rest = idx >> 8;
        const int nb = (int)(rest % NB);
        rest /= NB;
        const int kb = (int)(rest % KB);
        const int t = (int)(rest / KB);
        const int kr = kb * 16 + 4 * (lane >> 4) + v;
        const int nc = nb * 16 + (lane & 15);
        float w;
        if (!flip)
            w = kr < cin ? W[((long long)t * cin + kr) * cout + nc] : 0.0f;
        else
            w = W[((long long)(26 - t) * cin + nc) * cout + kr];
        frag[idx] = f2bf(w);
    }
}

// ---------------------------------------------------------- conv forward
// One wave computes 64 consecutive positions (4 blocks of 16) x all NB*16
// output channels; K runs over 27 taps x cin.  Operand A (lane l: position
// p0 + 16 mb + l%16, channels 4(l/16)..+3 of the k-block) is one 8-byte load
// from the channels-last input; out-of-range neighbours read a clamped
// address and are zeroed.  Result layout: lane l holds rows 4(l/16)+r, col l%16.
template <int NB>
__global__ __launch_bounds__(256) void k_conv3_fwd(const uint16_t* __restrict__ x, int D, int H, int W,
                                                   long long npos, int cxt, int cxo, int KB,
                                                   const uint16_t* __restrict__ frag,
                                                   const float* __restrict__ bias, int relu,
                                                   uint16_t* __restrict__ y, int cyt, int cyo) {
    const int lane = threadIdx.x & 63;
    const long long wave = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const long long p0 = wave * (16 * kMB);
    if (p0 >= npos) return;
    const int li = lane & 15, g = lane >> 4;
    int pz[kMB], py[kMB], px[kMB];
    long long pc[kMB];
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb) {
        long long p = p0 + 16 * mb + li;
        if (p >= npos) p = npos - 1;
        pc[mb] = p;
        px[mb] = (int)(p % W);
        long long q = p / W;
        py[mb] = (int)(q % H);
        pz[mb] = (int)((q / H) % D);
    }
    f4_t acc[kMB][NB];
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f4_t{0.f, 0.f, 0.f, 0.f};
    const s4_t* fr = reinterpret_cast<const s4_t*>(frag) + lane;
    const uint16_t* xb = x + cxo + 4 * g;
    for (int t = 0; t < 27; ++t) {
        const int dz = t / 9 - 1, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
        const long long off = ((long long)dz * H + dy) * W + dx;
        const uint16_t* xa[kMB];
        short msk[kMB];
#pragma unroll
        for (int mb = 0; mb < kMB; ++mb) {
            const bool ok = (unsigned)(pz[mb] + dz) < (unsigned)D && (unsigned)(py[mb] + dy) < (unsigned)H &&
                            (unsigned)(px[mb] + dx) < (unsigned)W;
            msk[mb] = ok ? (short)-1 : (short)0;
            xa[mb] = xb + (ok ? pc[mb] + off : pc[mb]) * cxt;
        }
        for (int kb = 0; kb < KB; ++kb) {
            s4_t a[kMB], b[NB];
#pragma unroll
            for (int mb = 0; mb < kMB; ++mb) a[mb] = *reinterpret_cast<const s4_t*>(xa[mb] + kb * 16) & msk[mb];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) b[nb] = fr[((t * KB + kb) * NB + nb) * 64];
#pragma unroll
            for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[mb], b[nb], acc[mb][nb], 0, 0, 0);
        }
    }
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const long long p = p0 + 16 * mb + 4 * g + r;
            if (p >= npos) continue;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                float v = acc[mb][nb][r] + (bias ? bias[nb * 16 + li] : 0.0f);
                if (relu) v = fmaxf(v, 0.0f);
                y[p * cyt + cyo + nb * 16 + li] = f2bf(v);
            }
        }
}

// ------------------------------------------- conv forward from LDS planes
// The same convolution, bit for bit, with the input staged: a workgroup of 4
// waves takes R rows of a plane (R W <= 64 MB positions) and marches along z
// with three planes of R + 2 rows in LDS, zero-padded, so that a tap is an
// address offset without masks; plane z + 2 is fetched to registers while the
// matrix cores work on plane z.  Products are v_mfma_f32_16x16x32_bf16, which
// adds 32 terms in the order of two 16x16x16 ones (checked bit for bit), at
// twice their rate: the 27 KB 16-channel steps of the kernel above are taken in
// pairs, in its order; a lone last step is paired with zeros.  The weights are the
// row operand, so a lane ends with 4 consecutive channels of one position (one
// 8-byte store).  Weights stay in registers over the march when they fit.
// 32 x 56^3:
// 16 -> 16 from 781 to 214 us (its bytes take 80), 32 -> 16 432; the 14 convolutions
// of a prediction from 5.4 to 1.73 ms.  Bound by the step from plane to plane: fetch,
// store, barrier, 98 products of 18 cycles a wave.
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef short s8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));

// value e of the 8 bf16 of a 16-byte piece, and a piece from 8 values
__device__ __forceinline__ uint16_t piece_at(u4_t v, int e) { return (uint16_t)(v[e >> 1] >> (16 * (e & 1))); }
__device__ __forceinline__ u4_t piece_of(const uint16_t (&h)[8]) {
    u4_t v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (uint32_t)h[2 * e] | (uint32_t)h[2 * e + 1] << 16;
    return v;
}

constexpr int kCvPieces = 8;  // 16-byte pieces a thread fetches per plane at most

__host__ __device__ constexpr int cv_pixel(int KB) { return KB == 4 ? 72 : 16 * KB; }  // elements (64 channels: padded against bank conflicts)

template <int KB, int NB, int MB>
__global__ __launch_bounds__(256, 2) void k_conv3_planes(const uint16_t* __restrict__ x, int D, int H, int W, int cxt,
                                                         int cxo, const uint16_t* __restrict__ frag,
                                                         const float* __restrict__ bias, int relu,
                                                         uint16_t* __restrict__ y, int cyt, int cyo, int R, int ntile,
                                                         int zc) {
    constexpr int PS = cv_pixel(KB);
    extern __shared__ __align__(16) uint16_t xs[];  // [3][R + 2][W + 2][PS]
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, li = lane & 15, g = lane >> 4;
    const int tile = blockIdx.x % ntile, n = blockIdx.x / ntile;
    const int y0 = tile * R, z0 = blockIdx.y * zc, z1 = min(D, z0 + zc);
    const int rows = R + 2, pw = W + 2, plane = rows * pw * PS;
    for (int e = tid; e < 3 * plane / 8; e += 256) reinterpret_cast<u4_t*>(xs)[e] = u4_t{0, 0, 0, 0};

    // this lane's piece of the weights of 16-channel steps st, st + 1 (zeros past the last), block nb: k = 8g .. 8g + 7
    auto wfrag = [&](int st, int nb) -> bf8_t {
        const int s1 = st + (g >> 1);
        s4_t lo = {0, 0, 0, 0}, hi = {0, 0, 0, 0};
        if (s1 < 27 * KB) {
            const s4_t* f = reinterpret_cast<const s4_t*>(frag) + (s1 * NB + nb) * 64 + 32 * (g & 1) + li;
            lo = f[0];
            hi = f[16];
        }
        return __builtin_bit_cast(bf8_t, s8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w});
    };
    // positions of this wave's blocks wv, wv + 4, ...: LDS offset of the lane's 8
    // terms (8g of 32 channels, or 8 (g & 1) of one tap's 16) and index in the plane
    const int npos = min(R, H - y0) * W, nblk = (npos + 15) / 16;
    int base[MB], pos[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        const int q = (wv + 4 * j) * 16 + li, qc = min(q, npos - 1);
        const int yy = qc / W, xx = qc - yy * W;
        base[j] = (yy * pw + xx) * PS + (KB == 1 ? 8 * (g & 1) : 8 * g);
        pos[j] = q < npos ? (y0 + yy) * W + xx : -1;
    }
    // pieces this thread fetches: element offset in a plane of x (-1: none) and LDS offset in a staged plane
    int go[kCvPieces], lo[kCvPieces];
#pragma unroll
    for (int j = 0; j < kCvPieces; ++j) {
        const int e = tid + 256 * j, rowp = 2 * KB * W, r = e / rowp, q = e - r * rowp, yy = y0 + r - 1;
        go[j] = r < rows && (unsigned)yy < (unsigned)H ? (yy * W + q / (2 * KB)) * cxt + (q % (2 * KB)) * 8 : -1;
        lo[j] = (r * pw + q / (2 * KB) + 1) * PS + (q % (2 * KB)) * 8;
    }
    const long long hw = (long long)H * W;
    u4_t pre[kCvPieces];
    auto fetch = [&](int z) {
        const uint16_t* xz = x + ((long long)n * D + z) * hw * cxt + cxo;
        const bool zok = (unsigned)z < (unsigned)D;
#pragma unroll
        for (int j = 0; j < kCvPieces; ++j) {
            pre[j] = u4_t{0, 0, 0, 0};
            if (zok && go[j] >= 0) pre[j] = *reinterpret_cast<const u4_t*>(xz + go[j]);
        }
    };
    auto put = [&](int z) {
        uint16_t* d = xs + (z + 3) % 3 * plane;
#pragma unroll
        for (int j = 0; j < kCvPieces; ++j)
            if (go[j] >= 0) *reinterpret_cast<u4_t*>(d + lo[j]) = pre[j];
    };
    constexpr int NP = (27 * KB + 1) / 2;            // pairs of steps
    constexpr bool RES = KB <= 2 && NB == 1;  // all weights in 56 or 108 registers
    bf8_t wr[RES ? NP : 1][NB];
    if (RES) {
#pragma unroll
        for (int m = 0; m < NP; ++m) wr[m][0] = wfrag(2 * m, 0);
    }
    __syncthreads();
    fetch(z0 - 1);
    put(z0 - 1);
    fetch(z0);
    put(z0);
    fetch(z0 + 1);
    for (int z = z0; z < z1; ++z) {
        put(z + 1);
        __syncthreads();
        if (z + 1 < z1) fetch(z + 2);
        f4_t acc[MB][NB];
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[j][nb] = f4_t{0.f, 0.f, 0.f, 0.f};
        auto mac = [&](const bf8_t (&w)[NB], int off, bool half) {
#pragma unroll
            for (int j = 0; j < MB; ++j) {
                if (wv + 4 * j < nblk) {
                    u4_t v = *reinterpret_cast<const u4_t*>(xs + base[j] + off);
                    if (half) v = g < 2 ? v : u4_t{0, 0, 0, 0};
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[j][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[nb], __builtin_bit_cast(bf8_t, v), acc[j][nb], 0, 0, 0);
                }
            }
        };
        // LDS offset of tap t: plane z + t / 9 - 1, row and column shifts t / 3 % 3, t % 3
        auto tap = [&](int t) { return (z + t / 9 + 2) % 3 * plane + (t / 3 % 3 * pw + t % 3) * PS; };
        // pair m: steps 2m, 2m + 1, i.e. 32 channels of a tap or 16 channels of two taps (the last one alone)
        auto pair_off = [&](int m) {
            if (KB > 1) return tap(2 * m / KB) + 2 * m % KB * 16;
            const int oa = tap(2 * m), ob = tap(min(2 * m + 1, 26));
            return g < 2 ? oa : ob;
        };
        if constexpr (RES) {
#pragma unroll
            for (int m = 0; m < NP; ++m) mac(wr[m], pair_off(m), KB == 1 && m == NP - 1);
        } else {
            // weights are fetched three pairs ahead (from L2: 600 cycles; a pair's products take 36 to 290)
            bf8_t w[4][NB];
            auto get = [&](int m) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) w[m & 3][nb] = wfrag(2 * m, nb);
            };
#pragma unroll
            for (int u = 0; u < 3; ++u) get(u);
            constexpr int NL = (NP - 1) / 4 * 4;
#pragma unroll 1
            for (int m = 0; m < NL; m += 4) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) w[(u + 3) & 3][nb] = wfrag(2 * (m + u + 3), nb);
                    mac(w[u], pair_off(m + u), false);
                }
            }
#pragma unroll
            for (int m = NL; m < NP; ++m) {
                if (m + 3 < NP) get(m + 3);
                mac(w[m & 3], pair_off(m), KB == 1 && m == NP - 1);
            }
        }
        uint16_t* yb = y + ((long long)n * D + z) * hw * cyt + cyo + 4 * g;
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            if (pos[j] < 0) continue;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                s4_t o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float v = acc[j][nb][r] + (bias ? bias[nb * 16 + 4 * g + r] : 0.0f);
                    if (relu) v = fmaxf(v, 0.0f);
                    o[r] = (short)f2bf(v);
                }
                *reinterpret_cast<s4_t*>(yb + (long long)pos[j] * cyt + nb * 16) = o;
            }
        }
        __syncthreads();
    }
}

// --------------------------------------------------------- conv wgrad
// Partial sums of gW[t][i][o] = sum_p x[p + d_t][i] gz[p][o] over the rows
// (n, z, y) of one slice, on the matrix cores with K = positions: A[i][k] =
// x[p_k + d_t][i], B[k][o] = gz[p_k][o], 16 positions of one row per step.
// Block = 4 waves over interleaved rows, combined in wave order through LDS.
// part layout [slice][27][cin][cout].
__global__ __launch_bounds__(256) void k_conv3_wgrad(const uint16_t* __restrict__ x, int D, int H, int W,
                                                     long long nrows, int cxt, int cxo, int cin,
                                                     const uint16_t* __restrict__ gz, int cgt, int cgo,
                                                     int cout, long long rows_per_slice,
                                                     float* __restrict__ part) {
    __shared__ f4_t red[3][16][64];
    const int t = blockIdx.y;
    const long long slice = blockIdx.x;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
    const int dz = t / 9 - 1, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
    const int IB = (cin + 15) / 16, OB = cout / 16;
    f4_t acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = f4_t{0.f, 0.f, 0.f, 0.f};
    const long long r0 = slice * rows_per_slice;
    const long long r1 = r0 + rows_per_slice < nrows ? r0 + rows_per_slice : nrows;
    int chA[4];
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) {
        const int c = ib * 16 + li;
        chA[ib] = c < cin ? c : cin - 1;
    }
    for (long long r = r0 + wv; r < r1; r += 4) {
        const int yy = (int)(r % H);
        const int zz = (int)((r / H) % D);
        if ((unsigned)(zz + dz) >= (unsigned)D || (unsigned)(yy + dy) >= (unsigned)H) continue;
        const long long rowp = r * W;
        const long long nrowp = rowp + ((long long)dz * H + dy) * W;
        for (int x0 = 0; x0 < W; x0 += 16) {
            s4_t a[4], b[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int xk = x0 + 4 * g + v;
                const bool okb = xk < W;
                const bool oka = okb && (unsigned)(xk + dx) < (unsigned)W;
                const long long pa = oka ? nrowp + xk + dx : rowp;
                const long long pb = okb ? rowp + xk : rowp;
#pragma unroll
                for (int ib = 0; ib < 4; ++ib) {
                    if (ib < IB) {
                        const uint16_t va = x[pa * cxt + cxo + chA[ib]];
                        a[ib][v] = (oka && ib * 16 + li < cin) ? (short)va : (short)0;
                    }
                }
#pragma unroll
                for (int ob = 0; ob < 4; ++ob) {
                    if (ob < OB) {
                        const uint16_t vb = gz[pb * cgt + cgo + ob * 16 + li];
                        b[ob][v] = okb ? (short)vb : (short)0;
                    }
                }
            }
#pragma unroll
            for (int ib = 0; ib < 4; ++ib)
#pragma unroll
                for (int ob = 0; ob < 4; ++ob)
                    if (ib < IB && ob < OB)
                        acc[ib][ob] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[ib], b[ob], acc[ib][ob], 0, 0, 0);
        }
    }
    if (wv > 0) {
#pragma unroll
        for (int ib = 0; ib < 4; ++ib)
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) red[wv - 1][ib * 4 + ob][lane] = acc[ib][ob];
    }
    __syncthreads();
    if (wv != 0) return;
#pragma unroll
    for (int ib = 0; ib < 4; ++ib)
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            if (ib >= IB || ob >= OB) continue;
            f4_t s = acc[ib][ob];
            for (int w = 0; w < 3; ++w) s += red[w][ib * 4 + ob][lane];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = ib * 16 + 4 * g + r;
                if (i < cin)
                    part[((slice * 27 + t) * cin + i) * cout + ob * 16 + li] = s[r];
            }
        }
}

// ------------------------------------------- wgrad from LDS-staged rows
// The same sums with the rows staged once for all taps.  K = 32 positions of a
// row per v_mfma_f32_16x16x32_bf16; both operands need, per lane, one channel of
// 8 consecutive positions, i.e. columns of the channels-last rows:
// ds_read_tr16_b64 reads them transposed (16 lanes name the 8-byte pieces of a
// 4-position x 16-channel block, lane li gets its column li), so a tap's shift
// dx is a row offset.  The 9 input rows around a gradient row stay in LDS while
// y advances (3 new rows and the gradient row a step, fetched to registers while
// the matrix cores work on the step before); the taps are dealt to the 4 waves,
// the 28th "tap" (wave 3) has ones for its input and so sums the gradient: the
// bias gradient.
// Bound by LDS reads (a 1 KB operand per matrix instruction at one output
// block).  The per-tap kernel above re-reads x 27 times in 2-byte pieces: the 14
// weight gradients of an 8 x 56^3 pass took 13.1 ms there (and their bias sums
// 3.4 ms), 0.94 ms here; the 32 -> 16 one 167 us.
typedef __attribute__((address_space(3))) s4_t lds_s4_t;

// operand of 32 positions: rows 8g..8g+7 of the 16-channel block at p (32-byte
// rows `step` rows apart), column li; p already holds this lane's piece
__device__ __forceinline__ bf8_t tr_frag(const uint16_t* p, int step) {
    const s4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_t*)p);
    const s4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_t*)(p + 64 * step));
    return __builtin_bit_cast(bf8_t, s8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w});
}

constexpr int kWgX = 64;  // positions of a row chunk

// One tap of a slice's sums for one pair of 16-channel blocks, straight from memory,
// with inputs outside the volume left out instead of multiplied by 0 (xb, gb: the
// blocks' first channels; result as k_conv3_wgrad_rows has it).
__device__ f4_t wgrad_tap(const uint16_t* __restrict__ xb, int D, int H, int W, int cxt, const uint16_t* __restrict__ gb,
                          int cgt, long long r0, long long r1, int t, int lane) {
    const int li = lane & 15, g = lane >> 4;
    const int dz = t / 9 - 1, dy = t / 3 % 3 - 1, dx = t % 3 - 1;
    f4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (long long r = r0; r < r1; ++r) {
        const int yy = (int)(r % H), zz = (int)(r / H % D);
        if ((unsigned)(zz + dz) >= (unsigned)D || (unsigned)(yy + dy) >= (unsigned)H) continue;
        const long long nr = r + (long long)dz * H + dy;
        for (int x0 = 0; x0 < W; x0 += 32) {
            uint16_t a[8], b[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int xx = x0 + 8 * g + e;
                const bool ok = xx < W;
                a[e] = ok && (unsigned)(xx + dx) < (unsigned)W ? xb[(nr * W + xx + dx) * cxt + li] : (uint16_t)0;
                b[e] = ok ? gb[(r * W + xx) * cgt + li] : (uint16_t)0;
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8_t, piece_of(a)),
                                                          __builtin_bit_cast(bf8_t, piece_of(b)), acc, 0, 0, 0);
        }
    }
    return acc;
}

// IB x OB: the 16-channel blocks of this workgroup (blockIdx.y: which of them)
template <int IB, int OB>
__global__ __launch_bounds__(256) void k_conv3_wgrad_rows(const uint16_t* __restrict__ x, int D, int H, int W,
                                                          long long nrows, int cxt, int cxo, int cin,
                                                          const uint16_t* __restrict__ gz, int cgt, int cgo, int cout,
                                                          long long rows_per_slice, int nob, float* __restrict__ part,
                                                          float* __restrict__ bpart) {
    constexpr int XR = kWgX + 2;          // staged positions of an input row
    constexpr int NX = XR * IB * 2;       // 16-byte pieces of an input row
    constexpr int NG = kWgX * OB * 2;     // ... of a gradient row
    constexpr int NL = (3 * NX + NG + 255) / 256;
    __shared__ __align__(16) uint16_t xs[9][IB][XR][16];
    __shared__ __align__(16) uint16_t gs[OB][kWgX][16];
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, li = lane & 15, g = lane >> 4;
    const int ib0 = ((int)blockIdx.y / nob) * IB, ob0 = ((int)blockIdx.y % nob) * OB;
    const uint16_t* xb = x + cxo + ib0 * 16;
    const uint16_t* gb = gz + cgo + ob0 * 16;
    f4_t acc[7][IB][OB];
#pragma unroll
    for (int j = 0; j < 7; ++j)
#pragma unroll
        for (int a = 0; a < IB; ++a)
#pragma unroll
            for (int b = 0; b < OB; ++b) acc[j][a][b] = f4_t{0.f, 0.f, 0.f, 0.f};
    const long long r0 = (long long)blockIdx.x * rows_per_slice;
    const long long r1 = r0 + rows_per_slice < nrows ? r0 + rows_per_slice : nrows;
    const bf8_t ones = __builtin_bit_cast(bf8_t, s8_t{0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80});

    // piece q of input row (zz, yy) of sample row base, chunk x0: position q / (2 IB), then block and half
    auto ldx = [&](long long row, bool ok, int q, int x0) -> u4_t {
        const int pos = q / (2 * IB), xx = x0 + pos - 1;
        if (!ok || (unsigned)xx >= (unsigned)W) return u4_t{0, 0, 0, 0};
        return *reinterpret_cast<const u4_t*>(xb + (row * W + xx) * cxt + (q % (2 * IB)) * 8);
    };
    auto stx = [&](int slot, int q, u4_t v) {
        const int pos = q / (2 * IB), c = q % (2 * IB);
        *reinterpret_cast<u4_t*>(&xs[slot][c >> 1][pos][(c & 1) * 8]) = v;
    };
    for (int x0 = 0; x0 < W; x0 += kWgX) {
        const int nk = W - x0 > 32 ? 2 : 1;
        u4_t pre[NL];
        // what row r adds to the staged rows: input rows (z + dz, y + 1) and the gradient row
        auto fetch = [&](long long r) {
            const int yy = (int)(r % H), zz = (int)((r / H) % D);
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const int e = tid + 256 * j;
                if (e < 3 * NX) {
                    const int dz = e / NX - 1;
                    pre[j] = ldx(r + (long long)dz * H + 1, (unsigned)(zz + dz) < (unsigned)D && yy + 1 < H, e % NX, x0);
                } else if (e < 3 * NX + NG) {
                    const int q = e - 3 * NX, pos = q / (2 * OB);
                    pre[j] = x0 + pos < W ? *reinterpret_cast<const u4_t*>(gb + (r * W + x0 + pos) * cgt + (q % (2 * OB)) * 8)
                                          : u4_t{0, 0, 0, 0};
                }
            }
        };
        if (r0 < r1) fetch(r0);
        for (long long r = r0; r < r1; ++r) {
            const int yy = (int)(r % H), zz = (int)((r / H) % D);
            // ring slot of input row y + dy: 3 ((y + dy + 3) % 3) + (dz + 1)
            if (r == r0 || yy == 0) {  // rows y - 1 and y are not there yet
                for (int e = tid; e < 6 * NX; e += 256) {
                    const int w = e / NX, dz = w % 3 - 1, dy = w / 3 - 1;
                    const bool ok = (unsigned)(zz + dz) < (unsigned)D && yy + dy >= 0;
                    stx(3 * ((yy + dy + 3) % 3) + dz + 1, e % NX, ldx(r + (long long)dz * H + dy, ok, e % NX, x0));
                }
            }
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const int e = tid + 256 * j;
                if (e < 3 * NX) {
                    stx(3 * ((yy + 1) % 3) + e / NX, e % NX, pre[j]);
                } else if (e < 3 * NX + NG) {
                    const int q = e - 3 * NX, c = q % (2 * OB);
                    *reinterpret_cast<u4_t*>(&gs[c >> 1][q / (2 * OB)][(c & 1) * 8]) = pre[j];
                }
            }
            __syncthreads();
            if (r + 1 < r1) fetch(r + 1);
            for (int kb = 0; kb < nk; ++kb) {
                const int lrow = kb * 32 + 8 * g + (li >> 2), lch = 4 * (li & 3);
                bf8_t bfr[OB];
#pragma unroll
                for (int b = 0; b < OB; ++b) bfr[b] = tr_frag(&gs[b][lrow][lch], 1);
#pragma unroll
                for (int j = 0; j < 7; ++j) {
                    const int t = wv + 4 * j;
                    const int dz = t / 9, dy = (t / 3) % 3 - 1, dx = t % 3;
                    const int slot = t < 27 ? 3 * ((yy + dy + 3) % 3) + dz : 0;
#pragma unroll
                    for (int a = 0; a < IB; ++a) {
                        bf8_t af = tr_frag(&xs[slot][a][lrow + (t < 27 ? dx : 0)][lch], 1);
                        if (t == 27) af = ones;
#pragma unroll
                        for (int b = 0; b < OB; ++b)
                            acc[j][a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bfr[b], acc[j][a][b], 0, 0, 0);
                    }
                }
            }
            __syncthreads();
        }
    }
    unsigned over = 0;  // sums that overflowed
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const int t = wv + 4 * j;
#pragma unroll
        for (int a = 0; a < IB; ++a)
#pragma unroll
            for (int b = 0; b < OB; ++b) {
                const int o = (ob0 + b) * 16 + li;
                if (t == 27) {
                    if (bpart && ib0 == 0 && a == 0 && g == 0) bpart[(long long)blockIdx.x * cout + o] = acc[j][a][b][0];
                    continue;
                }
                const f4_t v = acc[j][a][b];
                if (__any(!(fabsf(v[0]) + fabsf(v[1]) + fabsf(v[2]) + fabsf(v[3]) < HUGE_VALF)))
                    over |= 1u << ((j * IB + a) * OB + b);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = (ib0 + a) * 16 + 4 * g + r;
                    if (i < cin) part[(((long long)blockIdx.x * 27 + t) * cin + i) * cout + o] = v[r];
                }
            }
    }
    // A row outside the volume, or a shift past a row's end, enters as products with 0,
    // which an infinite value turns into no number: sums that overflowed are done again.
    for (; over; over &= over - 1) {
        const int q = __ffs((int)over) - 1, b = q % OB, a = q / OB % IB, t = wv + 4 * (q / (OB * IB));
        const f4_t v = wgrad_tap(xb + a * 16, D, H, W, cxt, gb + b * 16, cgt, r0, r1, t, lane);
        for (int r = 0; r < 4; ++r) {
            const int i = (ib0 + a) * 16 + 4 * g + r;
            if (i < cin) part[(((long long)blockIdx.x * 27 + t) * cin + i) * cout + (ob0 + b) * 16 + li] = v[r];
        }
    }
}

// The same for the transposed up-sampling: per coarse row, the 4 child rows of
// the gradient; wave w = 2a + b holds the children (a, b, 0) and (a, b, 1),
// whose positions are every other row of the staged gradient.  bpart holds one
// partial bias sum per slice and wave.  (The three of an 8 x 56^3 pass: 3.0 ms
// as one thread per channel pair over its positions, 0.04 ms here.)
template <int IB, int OB>
__global__ __launch_bounds__(256) void k_up_wgrad_rows(const uint16_t* __restrict__ x, const uint16_t* __restrict__ gy,
                                                       int D, int H, int W, long long nrows, int cin, int cout, int cgt,
                                                       int cgo, long long rows_per_slice, int nob,
                                                       float* __restrict__ part, float* __restrict__ bpart) {
    constexpr int NX = kWgX * IB * 2, NG = 2 * kWgX * OB * 2;
    constexpr int NL = (NX + 4 * NG + 255) / 256;
    __shared__ __align__(16) uint16_t xs[IB][kWgX][16];
    __shared__ __align__(16) uint16_t gs[4][OB][2 * kWgX][16];
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, li = lane & 15, g = lane >> 4;
    const int ib0 = ((int)blockIdx.y / nob) * IB, ob0 = ((int)blockIdx.y % nob) * OB;
    const uint16_t* xb = x + ib0 * 16;
    const uint16_t* gb = gy + cgo + ob0 * 16;
    f4_t acc[2][IB][OB], accb[OB];
#pragma unroll
    for (int b = 0; b < OB; ++b) {
        accb[b] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int a = 0; a < IB; ++a) acc[c][a][b] = f4_t{0.f, 0.f, 0.f, 0.f};
    }
    const bf8_t ones = __builtin_bit_cast(bf8_t, s8_t{0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80});
    const long long r0 = (long long)blockIdx.x * rows_per_slice;
    const long long r1 = r0 + rows_per_slice < nrows ? r0 + rows_per_slice : nrows;
    for (int x0 = 0; x0 < W; x0 += kWgX) {
        const int nk = W - x0 > 32 ? 2 : 1;
        u4_t pre[NL];
        auto fetch = [&](long long r) {
            const long long nz = r / H;  // n D + z
            const int yy = (int)(r % H);
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const int e = tid + 256 * j;
                pre[j] = u4_t{0, 0, 0, 0};
                if (e < NX) {
                    const int pos = e / (2 * IB);
                    if (x0 + pos < W) pre[j] = *reinterpret_cast<const u4_t*>(xb + (r * W + x0 + pos) * cin + (e % (2 * IB)) * 8);
                } else if (e < NX + 4 * NG) {
                    const int w = (e - NX) / NG, q = (e - NX) % NG, pos = q / (2 * OB);
                    // fine row ((n 2D + 2z + a) 2H + 2y + b) = (2 nz + a) 2H + 2y + b
                    const long long fr = (2 * nz + (w >> 1)) * 2 * H + 2 * yy + (w & 1);
                    if (2 * x0 + pos < 2 * W)
                        pre[j] = *reinterpret_cast<const u4_t*>(gb + (fr * 2 * W + 2 * x0 + pos) * cgt + (q % (2 * OB)) * 8);
                }
            }
        };
        if (r0 < r1) fetch(r0);
        for (long long r = r0; r < r1; ++r) {
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const int e = tid + 256 * j;
                if (e < NX) {
                    const int c = e % (2 * IB);
                    *reinterpret_cast<u4_t*>(&xs[c >> 1][e / (2 * IB)][(c & 1) * 8]) = pre[j];
                } else if (e < NX + 4 * NG) {
                    const int w = (e - NX) / NG, q = (e - NX) % NG, c = q % (2 * OB);
                    *reinterpret_cast<u4_t*>(&gs[w][c >> 1][q / (2 * OB)][(c & 1) * 8]) = pre[j];
                }
            }
            __syncthreads();
            if (r + 1 < r1) fetch(r + 1);
            for (int kb = 0; kb < nk; ++kb) {
                const int lrow = kb * 32 + 8 * g + (li >> 2), lch = 4 * (li & 3);
                bf8_t af[IB];
#pragma unroll
                for (int a = 0; a < IB; ++a) af[a] = tr_frag(&xs[a][lrow][lch], 1);
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int b = 0; b < OB; ++b) {
                        const bf8_t bfr = tr_frag(&gs[wv][b][2 * lrow + c][lch], 2);
                        accb[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, bfr, accb[b], 0, 0, 0);
#pragma unroll
                        for (int a = 0; a < IB; ++a)
                            acc[c][a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bfr, acc[c][a][b], 0, 0, 0);
                    }
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int b = 0; b < OB; ++b) {
        const int o = (ob0 + b) * 16 + li;
        if (ib0 == 0 && g == 0) bpart[((long long)blockIdx.x * 4 + wv) * cout + o] = accb[b][0];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int a = 0; a < IB; ++a)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    part[(((long long)blockIdx.x * 8 + 2 * wv + c) * cin + (ib0 + a) * 16 + 4 * g + r) * cout + o] = acc[c][a][b][r];
    }
}

// out[j] = sum over slices of part[slice][j]: 16 groups of slices per output in
// a block (slice q in group q % 16, ascending), combined in order.  A chain of
// slices per output and thread, as a grid of one thread per output has it, took
// 26 us at 128 slices whatever the width.
constexpr int kSumCols = 64, kSumGroups = 16;
__global__ __launch_bounds__(kSumCols * kSumGroups) void k_sum_slices(const float* __restrict__ part, long long nslices,
                                                                      long long n, float* __restrict__ out) {
    __shared__ float red[kSumGroups][kSumCols];
    const int c = threadIdx.x % kSumCols, grp = threadIdx.x / kSumCols;
    const long long j = (long long)blockIdx.x * kSumCols + c;
    float s = 0.0f;
    if (j < n) {
#pragma unroll 4
        for (long long q = grp; q < nslices; q += kSumGroups) s += part[q * n + j];
    }
    red[grp][c] = s;
    __syncthreads();
    if (grp == 0 && j < n) {
        float t = red[0][c];
#pragma unroll
        for (int q = 1; q < kSumGroups; ++q) t += red[q][c];
        out[j] = t;
    }
}

// Column sums of a bf16 [npos][ct] block (channels [co, co + c), c <= 64):
// part[block][ch], 4 lane groups per block combined in order.
__global__ __launch_bounds__(256) void k_colsum_part(const uint16_t* __restrict__ g, long long npos, int ct, int co,
                                                     int c, long long chunk, float* __restrict__ part) {
    __shared__ float red[4][64];
    const int ch = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const long long p0 = blockIdx.x * chunk;
    const long long p1 = p0 + chunk < npos ? p0 + chunk : npos;
    float s = 0.0f;
    if (ch < c)
        for (long long p = p0 + grp; p < p1; p += 4) s += bf2f(g[p * ct + co + ch]);
    red[grp][ch] = s;
    __syncthreads();
    if (grp == 0 && ch < c) part[blockIdx.x * (long long)c + ch] = red[0][ch] + red[1][ch] + red[2][ch] + red[3][ch];
}

// ------------------------------------------------------------- relu mask
__global__ void k_relu_mask(const uint16_t* __restrict__ g, const uint16_t* __restrict__ y, long long npos, int ct,
                            int co, int c, uint16_t* __restrict__ go, int cot, int coo) {
    const long long n = npos * c;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long p = e / c;
        const int ch = (int)(e - p * c);
        const uint16_t yv = y[p * ct + co + ch];
        const bool pos = (yv & 0x8000u) == 0 && (yv & 0x7fffu) != 0;  // y > 0
        go[p * cot + coo + ch] = pos ? g[p * ct + co + ch] : (uint16_t)0;
    }
}

// ---------------------------------------------------------------- pooling
__device__ __forceinline__ long long child_pos(long long q, int Dh, int Hh, int Wh, int s) {
    // q indexes the pooled grid [n][Dh][Hh][Wh]; child s = a*4 + b*2 + c
    const int X = (int)(q % Wh);
    long long r = q / Wh;
    const int Y = (int)(r % Hh);
    r /= Hh;
    const int Z = (int)(r % Dh);
    const long long n = r / Dh;
    const int a = s >> 2, b = (s >> 1) & 1, c = s & 1;
    return ((n * (2 * Dh) + 2 * Z + a) * (2 * Hh) + 2 * Y + b) * (long long)(2 * Wh) + 2 * X + c;
}

__global__ void k_pool_fwd(const uint16_t* __restrict__ x, long long nq, int Dh, int Hh, int Wh, int ct, int co, int c,
                           uint16_t* __restrict__ y) {
    const long long n = nq * c;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long q = e / c;
        const int ch = (int)(e - q * c);
        uint16_t best = x[child_pos(q, Dh, Hh, Wh, 0) * ct + co + ch];
        float bv = bf2f(best);
        for (int s = 1; s < 8; ++s) {
            const uint16_t v = x[child_pos(q, Dh, Hh, Wh, s) * ct + co + ch];
            if (bf2f(v) > bv) {
                bv = bf2f(v);
                best = v;
            }
        }
        y[q * c + ch] = best;
    }
}

__global__ void k_pool_bwd(const uint16_t* __restrict__ x, const uint16_t* __restrict__ gy, long long nq, int Dh,
                           int Hh, int Wh, int ct, int co, int c, uint16_t* __restrict__ gx, int accumulate) {
    const long long n = nq * c;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long q = e / c;
        const int ch = (int)(e - q * c);
        int arg = 0;
        float bv = bf2f(x[child_pos(q, Dh, Hh, Wh, 0) * ct + co + ch]);
        for (int s = 1; s < 8; ++s) {
            const float v = bf2f(x[child_pos(q, Dh, Hh, Wh, s) * ct + co + ch]);
            if (v > bv) {
                bv = v;
                arg = s;
            }
        }
        const float gv = bf2f(gy[q * c + ch]);
        for (int s = 0; s < 8; ++s) {
            const long long idx = child_pos(q, Dh, Hh, Wh, s) * ct + co + ch;
            const float base = accumulate ? bf2f(gx[idx]) : 0.0f;
            gx[idx] = f2bf(s == arg ? base + gv : base);
        }
    }
}

// The mask and the pooling kernels on aligned 16-byte pieces of 8 channels (cp =
// c / 8 pieces a position): a lane moves 16 bytes where the kernels above move 2.
// Bound by memory.  On average over an 8 x 56^3 pass: mask 21.3 to 10.9 us, pooling
// 15.4 to 9.2 and 34.8 to 25.5 us.
__global__ void k_relu_mask8(const uint16_t* __restrict__ g, const uint16_t* __restrict__ y, long long npos, int ct,
                             int co, int cp, uint16_t* __restrict__ go, int cot, int coo) {
    const long long n = npos * cp;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long p = e / cp;
        const int q = 8 * (int)(e - p * cp);
        const u4_t gv = *reinterpret_cast<const u4_t*>(g + p * ct + co + q);
        const u4_t yv = *reinterpret_cast<const u4_t*>(y + p * ct + co + q);
        uint16_t o[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint16_t v = piece_at(yv, k);
            o[k] = (v & 0x8000u) == 0 && (v & 0x7fffu) != 0 ? piece_at(gv, k) : (uint16_t)0;  // y > 0
        }
        *reinterpret_cast<u4_t*>(go + p * cot + coo + q) = piece_of(o);
    }
}

__global__ void k_pool_fwd8(const uint16_t* __restrict__ x, long long nq, int Dh, int Hh, int Wh, int ct, int co, int cp,
                            uint16_t* __restrict__ y) {
    const long long n = nq * cp;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long q = e / cp;
        const int ch = 8 * (int)(e - q * cp);
        const long long p0 = child_pos(q, Dh, Hh, Wh, 0);  // child (a, b, c) lies a 4 Hh Wh + b 2 Wh + c further
        u4_t v[8];
#pragma unroll
        for (int s = 0; s < 8; ++s)
            v[s] = *reinterpret_cast<const u4_t*>(
                x + (p0 + (long long)(s >> 2) * 4 * Hh * Wh + (s >> 1 & 1) * 2 * Wh + (s & 1)) * ct + co + ch);
        uint16_t o[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            uint16_t best = piece_at(v[0], k);
#pragma unroll
            for (int s = 1; s < 8; ++s) {
                const uint16_t u = piece_at(v[s], k);
                best = bf2f(u) > bf2f(best) ? u : best;
            }
            o[k] = best;
        }
        *reinterpret_cast<u4_t*>(y + q * cp * 8 + ch) = piece_of(o);
    }
}

__global__ void k_pool_bwd8(const uint16_t* __restrict__ x, const uint16_t* __restrict__ gy, long long nq, int Dh, int Hh,
                            int Wh, int ct, int co, int cp, uint16_t* __restrict__ gx, int accumulate) {
    const long long n = nq * cp;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long q = e / cp;
        const int ch = 8 * (int)(e - q * cp);
        const long long p0 = child_pos(q, Dh, Hh, Wh, 0);
        u4_t v[8], gv[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const long long i = (p0 + (long long)(s >> 2) * 4 * Hh * Wh + (s >> 1 & 1) * 2 * Wh + (s & 1)) * ct + co + ch;
            v[s] = *reinterpret_cast<const u4_t*>(x + i);
            gv[s] = accumulate ? *reinterpret_cast<const u4_t*>(gx + i) : u4_t{0, 0, 0, 0};
        }
        const u4_t go = *reinterpret_cast<const u4_t*>(gy + q * cp * 8 + ch);
        int arg[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            arg[k] = 0;
            float bv = bf2f(piece_at(v[0], k));
#pragma unroll
            for (int s = 1; s < 8; ++s) {
                const float u = bf2f(piece_at(v[s], k));
                if (u > bv) {
                    bv = u;
                    arg[k] = s;
                }
            }
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            uint16_t o[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float bs = bf2f(piece_at(gv[s], k));
                o[k] = f2bf(s == arg[k] ? bs + bf2f(piece_at(go, k)) : bs);
            }
            const long long i = (p0 + (long long)(s >> 2) * 4 * Hh * Wh + (s >> 1 & 1) * 2 * Wh + (s & 1)) * ct + co + ch;
            *reinterpret_cast<u4_t*>(gx + i) = piece_of(o);
        }
    }
}

// ------------------------------------------------- transposed up-sampling
__global__ void k_up_fwd(const uint16_t* __restrict__ x, long long nout, int D, int H, int W, int cin,
                         const float* __restrict__ Wu, const float* __restrict__ b, int cout,
                         uint16_t* __restrict__ y, int cyt, int cyo) {
    const long long n = nout * cout;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long q = e / cout;
        const int o = (int)(e - q * cout);
        const int X = (int)(q % (2 * W));
        long long r = q / (2 * W);
        const int Y = (int)(r % (2 * H));
        r /= 2 * H;
        const int Z = (int)(r % (2 * D));
        const long long nb = r / (2 * D);
        const long long p = ((nb * D + (Z >> 1)) * H + (Y >> 1)) * W + (X >> 1);
        const int s = (Z & 1) * 4 + (Y & 1) * 2 + (X & 1);
        float acc = b[o];
        const uint16_t* xp = x + p * cin;
        const float* wp = Wu + (long long)s * cin * cout + o;
        for (int i = 0; i < cin; ++i) acc += bf2f(xp[i]) * wp[(long long)i * cout];
        y[q * cyt + cyo + o] = f2bf(acc);
    }
}

// Transposed up-sampling, one thread per coarse position and pair of children
// (c = 0, 1) for 16 output channels: the weights of a step (s, i) are the same
// for the whole wave and come as scalar operands, the input is read 8 channels
// at a time, and an output's sum runs over i as above.  (One thread per output
// fetched a weight and an input per multiply-add: the three of a 32-source
// prediction at 56^3 1.32 ms; here 0.25, of which the multiply-adds take 0.09.)
__global__ __launch_bounds__(256) void k_up_fwd_pos(const uint16_t* __restrict__ x, long long np, int D, int H, int W,
                                                    int cin, const float* __restrict__ Wu, const float* __restrict__ b,
                                                    int cout, uint16_t* __restrict__ y, int cyt, int cyo) {
    const long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (p >= np) return;
    const int s2 = 2 * (int)blockIdx.y, o0 = 16 * (int)blockIdx.z;
    float acc[2][16];
#pragma unroll
    for (int o = 0; o < 16; ++o) acc[0][o] = acc[1][o] = b[o0 + o];
    const u4_t* xp = reinterpret_cast<const u4_t*>(x + p * cin);
    const float* w = Wu + (long long)s2 * cin * cout + o0;
    for (int i0 = 0; i0 < cin; i0 += 8) {
        const u4_t v = xp[i0 >> 3];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float xv = bf2f(piece_at(v, e));
            const float* w0 = w + (long long)(i0 + e) * cout;
            const float* w1 = w0 + (long long)cin * cout;
#pragma unroll
            for (int o = 0; o < 16; ++o) {
                acc[0][o] = fmaf(xv, w0[o], acc[0][o]);
                acc[1][o] = fmaf(xv, w1[o], acc[1][o]);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        u4_t* q = reinterpret_cast<u4_t*>(y + child_pos(p, D, H, W, s2 + c) * cyt + cyo + o0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint16_t o[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = f2bf(acc[c][8 * h + e]);
            q[h] = piece_of(o);
        }
    }
}

// gx[p][i] = sum_s sum_o gy[child s of p][o] Wu[s][i][o]
__global__ void k_up_bwd_data(const uint16_t* __restrict__ gy, long long np, int D, int H, int W, int cin, int cout,
                              int cgt, int cgo, const float* __restrict__ Wu, uint16_t* __restrict__ gx) {
    const long long n = np * cin;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long p = e / cin;
        const int i = (int)(e - p * cin);
        float acc = 0.0f;
        for (int s = 0; s < 8; ++s) {
            const long long q = child_pos(p, D, H, W, s);
            const uint16_t* gp = gy + q * cgt + cgo;
            const float* wp = Wu + ((long long)s * cin + i) * cout;
            for (int o = 0; o < cout; ++o) acc += bf2f(gp[o]) * wp[o];
        }
        gx[p * cin + i] = f2bf(acc);
    }
}

// The data gradient likewise: one thread per coarse position for 16 input
// channels, weights as scalar operands, each sum over (s, o) in the order above.
// (The three of an 8 x 56^3 pass 1.70 ms as one thread per sum, 0.15 here.)
__global__ __launch_bounds__(256) void k_up_bwd_pos(const uint16_t* __restrict__ gy, long long np, int D, int H, int W,
                                                    int cin, int cout, int cgt, int cgo, const float* __restrict__ Wu,
                                                    uint16_t* __restrict__ gx) {
    const long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (p >= np) return;
    const int i0 = 16 * (int)blockIdx.y;
    float acc[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
    for (int s = 0; s < 8; ++s) {
        const u4_t* gp = reinterpret_cast<const u4_t*>(gy + child_pos(p, D, H, W, s) * cgt + cgo);
        for (int o0 = 0; o0 < cout; o0 += 16) {
            float g[16];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u4_t v = gp[(o0 >> 3) + h];
#pragma unroll
                for (int e = 0; e < 8; ++e) g[8 * h + e] = bf2f(piece_at(v, e));
            }
            const float* w = Wu + ((long long)s * cin + i0) * cout + o0;
#pragma unroll
            for (int i = 0; i < 16; ++i)
#pragma unroll
                for (int o = 0; o < 16; ++o) acc[i] = fmaf(g[o], w[(long long)i * cout + o], acc[i]);
        }
    }
    u4_t* q = reinterpret_cast<u4_t*>(gx + p * cin + i0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint16_t o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = f2bf(acc[8 * h + e]);
        q[h] = piece_of(o);
    }
}

// part[slice][s][i][o] = sum over the slice's coarse positions p of x[p][i] gy[child s of p][o]
__global__ __launch_bounds__(256) void k_up_wgrad_part(const uint16_t* __restrict__ x, const uint16_t* __restrict__ gy,
                                                       long long np, int D, int H, int W, int cin, int cout, int cgt,
                                                       int cgo, long long chunk, float* __restrict__ part) {
    const int s = blockIdx.y;
    const long long slice = blockIdx.x;
    const long long p0 = slice * chunk;
    const long long p1 = p0 + chunk < np ? p0 + chunk : np;
    const int npair = cin * cout;
    for (int pr = threadIdx.x; pr < npair; pr += blockDim.x) {
        const int i = pr / cout, o = pr - (pr / cout) * cout;
        float acc = 0.0f;
        for (long long p = p0; p < p1; ++p)
            acc += bf2f(x[p * cin + i]) * bf2f(gy[child_pos(p, D, H, W, s) * cgt + cgo + o]);
        part[((slice * 8 + s) * (long long)cin + i) * cout + o] = acc;
    }
}

// ------------------------------------------------------------------- head
__global__ void k_head_fwd(const uint16_t* __restrict__ x, long long npos, int cin, const float* __restrict__ w,
                           const float* __restrict__ b, float* __restrict__ y) {
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < npos; p += (long long)gridDim.x * blockDim.x) {
        float acc = b[0];
        for (int i = 0; i < cin; ++i) acc += bf2f(x[p * cin + i]) * w[i];
        y[p] = acc;
    }
}

__global__ void k_head_bwd_data(const float* __restrict__ gy, long long npos, int cin, const float* __restrict__ w,
                                uint16_t* __restrict__ gx) {
    const long long n = npos * cin;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long p = e / cin;
        gx[e] = f2bf(gy[p] * w[e - p * cin]);
    }
}

// The head on 16-byte pieces (cin a multiple of 8): one thread per position, the
// sum in the order above; its data gradient one piece per thread.
__global__ void k_head_fwd8(const uint16_t* __restrict__ x, long long npos, int cin, const float* __restrict__ w,
                            const float* __restrict__ b, float* __restrict__ y) {
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < npos; p += (long long)gridDim.x * blockDim.x) {
        float acc = b[0];
        const u4_t* xp = reinterpret_cast<const u4_t*>(x + p * cin);
        for (int i0 = 0; i0 < cin; i0 += 8) {
            const u4_t v = xp[i0 >> 3];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = fmaf(bf2f(piece_at(v, e)), w[i0 + e], acc);
        }
        y[p] = acc;
    }
}

__global__ void k_head_bwd_data8(const float* __restrict__ gy, long long npos, int cin, const float* __restrict__ w,
                                 uint16_t* __restrict__ gx) {
    const int cp = cin / 8;
    const long long n = npos * cp;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
        const long long p = e / cp;
        const int q = 8 * (int)(e - p * cp);
        const float g = gy[p];
        uint16_t o[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) o[k] = f2bf(g * w[q + k]);
        *reinterpret_cast<u4_t*>(gx + 8 * e) = piece_of(o);
    }
}

// part[block][col]: col < cin -> sum x[p][col] gy[p]; col == cin -> sum gy[p].
// The block's 256 threads are dealt to the cin / 8 pieces of a position (cp; one
// piece each if there are more threads than that), groups of positions summed in
// order through LDS: 8 x 56^3 x 16 from 569 us (2-byte loads, 2 positions at a
// time) to 16 us.
__global__ __launch_bounds__(256) void k_head_wgrad_part8(const uint16_t* __restrict__ x, const float* __restrict__ gy,
                                                          long long npos, int cin, long long chunk,
                                                          float* __restrict__ part) {
    __shared__ float red[256][9];
    const int cp = cin / 8, q = threadIdx.x % cp, grp = threadIdx.x / cp, ng = 256 / cp;
    const long long p0 = blockIdx.x * chunk;
    const long long p1 = p0 + chunk < npos ? p0 + chunk : npos;
    float s[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (grp < ng)
        for (long long p = p0 + grp; p < p1; p += ng) {
            const u4_t v = *reinterpret_cast<const u4_t*>(x + p * cin + 8 * q);
            const float g = gy[p];
#pragma unroll
            for (int e = 0; e < 8; ++e) s[e] += bf2f(piece_at(v, e)) * g;
            s[8] += g;
        }
#pragma unroll
    for (int e = 0; e < 9; ++e) red[threadIdx.x][e] = s[e];
    __syncthreads();
    for (int c = threadIdx.x; c <= cin; c += 256) {
        float t = 0.0f;
        for (int k = 0; k < ng; ++k) t += c < cin ? red[k * cp + c / 8][c % 8] : red[k * cp][8];
        part[blockIdx.x * (long long)(cin + 1) + c] = t;
    }
}

// part[block][col]: col < cin -> sum x[p][col] gy[p]; col == cin -> sum gy[p]
__global__ __launch_bounds__(256) void k_head_wgrad_part(const uint16_t* __restrict__ x, const float* __restrict__ gy,
                                                         long long npos, int cin, long long chunk,
                                                         float* __restrict__ part) {
    __shared__ float red[2][128];
    const int col = threadIdx.x & 127, grp = threadIdx.x >> 7;
    const long long p0 = blockIdx.x * chunk;
    const long long p1 = p0 + chunk < npos ? p0 + chunk : npos;
    float s = 0.0f;
    if (col <= cin)
        for (long long p = p0 + grp; p < p1; p += 2) s += (col < cin ? bf2f(x[p * cin + col]) : 1.0f) * gy[p];
    red[grp][col] = s;
    __syncthreads();
    if (grp == 0 && col <= cin) part[blockIdx.x * (long long)(cin + 1) + col] = red[0][col] + red[1][col];
}

// columns 0..cin-1 of the partials -> gw, column cin -> gb: one block per column,
// thread t takes blocks t, t + 256, ..., combined by a fixed tree (one thread per
// column walked all blocks: 52 us at 343; 4.9 us here)
__global__ __launch_bounds__(256) void k_head_finish(const float* __restrict__ part, long long nb, int cin,
                                                     float* __restrict__ gw, float* __restrict__ gb) {
    __shared__ float red[256];
    const int col = blockIdx.x;
    float s = 0.0f;
    for (long long q = threadIdx.x; q < nb; q += 256) s += part[q * (cin + 1) + col];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (col < cin)
            gw[col] = red[0];
        else
            gb[0] = red[0];
    }
}

// -------------------------------------------------------------------- loss
// part[block] = (sum m, sum m (y - t)^2) over the block's chunk
__global__ __launch_bounds__(256) void k_mse_part(const float* __restrict__ y, const float* __restrict__ t,
                                                  const float* __restrict__ m, long long n, long long chunk,
                                                  float* __restrict__ part) {
    __shared__ float rs[256], rm[256];
    const long long p0 = blockIdx.x * chunk;
    const long long p1 = p0 + chunk < n ? p0 + chunk : n;
    float ss = 0.0f, sm = 0.0f;
    for (long long i = p0 + threadIdx.x; i < p1; i += 256) {
        const float w = m ? m[i] : 1.0f;
        const float r = y[i] - t[i];
        ss += w * r * r;
        sm += w;
    }
    rs[threadIdx.x] = ss;
    rm[threadIdx.x] = sm;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) {
            rs[threadIdx.x] += rs[threadIdx.x + k];
            rm[threadIdx.x] += rm[threadIdx.x + k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = rm[0];
        part[2 * blockIdx.x + 1] = rs[0];
    }
}

// loss[0] = sum / max(count, 1); loss[1] = max(count, 1)
__global__ __launch_bounds__(256) void k_mse_final(const float* __restrict__ part, int nb, float* __restrict__ loss) {
    __shared__ float rs[256], rm[256];
    float ss = 0.0f, sm = 0.0f;
    for (int b = threadIdx.x; b < nb; b += 256) {
        sm += part[2 * b];
        ss += part[2 * b + 1];
    }
    rs[threadIdx.x] = ss;
    rm[threadIdx.x] = sm;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) {
            rs[threadIdx.x] += rs[threadIdx.x + k];
            rm[threadIdx.x] += rm[threadIdx.x + k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const float cnt = rm[0] > 1.0f ? rm[0] : 1.0f;
        loss[0] = rs[0] / cnt;
        loss[1] = cnt;
    }
}

__global__ void k_mse_grad(const float* __restrict__ y, const float* __restrict__ t, const float* __restrict__ m,
                           long long n, const float* __restrict__ loss, float* __restrict__ gy) {
    const float sc = 2.0f / loss[1];
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const float w = m ? m[i] : 1.0f;
        gy[i] = sc * w * (y[i] - t[i]);
    }
}

// ------------------------------------------------------------------- adam
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       long long n, float lr, float b1, float b2, float eps, float c1, float c2) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    }
}

// ------------------------------------------------------------- warm start
// Node position in the embedding: spherical (r, lat, lon) -> Cartesian km.
__device__ __forceinline__ void embed(int coord, double a0, double a1, double a2, double X[3]) {
    if (coord == 1) {
        const double ct = cos(a1);
        X[0] = a0 * ct * cos(a2);
        X[1] = a0 * ct * sin(a2);
        X[2] = a0 * sin(a1);
    } else {
        X[0] = a0;
        X[1] = a1;
        X[2] = a2;
    }
}

struct WarmGrid {
    int n[3], coord;
    double o[3], h[3];
};

// Four waves a block, a wave per row of the coarse grid (wave-uniform z, y), its
// lanes over x: what depends on a row or on x alone (the sines and cosines of
// the embedding) is formed once, not per position (32 x 56^3: 106 to 69 us).
__global__ __launch_bounds__(256) void k_warm_features(WarmGrid G, const double* __restrict__ s,
                                                       const double* __restrict__ xi, const double* __restrict__ eta,
                                                       const double* __restrict__ src_pos,
                                                       const double* __restrict__ src_par, int stride, int D, int H,
                                                       int W, uint16_t* __restrict__ feat) {
    const int q = blockIdx.y, lane = threadIdx.x & 63;
    const long long npos = (long long)D * H * W, nrow = (long long)D * H;
    double Xs[3];
    embed(G.coord, src_pos[3 * q], src_pos[3 * q + 1], src_pos[3 * q + 2], Xs);
    const double inv_s0 = 1.0 / src_par[3 * q];
    for (int x0 = 0; x0 < W; x0 += 64) {
        const int xx = x0 + lane, k = xx * stride;
        const double a2 = G.o[2] + k * G.h[2];
        const double c2 = G.coord == 1 ? cos(a2) : 0.0, s2 = G.coord == 1 ? sin(a2) : 0.0;
        for (long long r = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6))); r < nrow;
             r += 4LL * gridDim.x) {
            const int yy = (int)(r % H), zz = (int)(r / H);
            const int i = zz * stride, j = yy * stride;
            uint16_t f[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            if (xx < W && i < G.n[0] && j < G.n[1] && k < G.n[2]) {
                const long long node = ((long long)i * G.n[1] + j) * G.n[2] + k;
                const double a0 = G.o[0] + i * G.h[0], a1 = G.o[1] + j * G.h[1];
                double X[3] = {a0, a1, a2};
                if (G.coord == 1) {
                    const double ct = cos(a1);
                    X[0] = a0 * ct * c2;
                    X[1] = a0 * ct * s2;
                    X[2] = a0 * sin(a1);
                }
                const double d = sqrt((X[0] - Xs[0]) * (X[0] - Xs[0]) + (X[1] - Xs[1]) * (X[1] - Xs[1]) +
                                      (X[2] - Xs[2]) * (X[2] - Xs[2]));
                f[0] = f2bf((float)((s[node] * inv_s0 - 1.0) * NN_FEAT_S));
                f[1] = f2bf((float)(xi[node] * NN_FEAT_A));
                f[2] = f2bf((float)(eta[node] * NN_FEAT_A));
                f[3] = f2bf((float)(d * NN_FEAT_D));
            }
            if (xx < W) {
                uint16_t* o = feat + ((long long)q * npos + r * W + xx) * 16;
                // (8-byte stores: feat need not be 16-byte aligned)
                const u4_t v = piece_of(f);
                *reinterpret_cast<uint2*>(o) = make_uint2(v[0], v[1]);
                for (int e = 1; e < 4; ++e) *reinterpret_cast<uint2*>(o + 4 * e) = make_uint2(0u, 0u);
            }
        }
    }
}

__global__ void k_warm_target(WarmGrid G, const double* __restrict__ tau, int stride, int D, int H, int W,
                              float* __restrict__ target, float* __restrict__ mask) {
    const int q = blockIdx.y;
    const long long npos = (long long)D * H * W;
    const long long N = (long long)G.n[0] * G.n[1] * G.n[2];
    for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < npos; p += (long long)gridDim.x * blockDim.x) {
        const int xx = (int)(p % W);
        const int yy = (int)((p / W) % H);
        const int zz = (int)(p / ((long long)W * H));
        const int i = zz * stride, j = yy * stride, k = xx * stride;
        const bool ok = i < G.n[0] && j < G.n[1] && k < G.n[2];
        float tv = 0.0f;
        if (ok) tv = (float)((tau[q * N + ((long long)i * G.n[1] + j) * G.n[2] + k] - 1.0) * NN_TARGET_SCALE);
        target[q * npos + p] = tv;
        if (mask) mask[q * npos + p] = ok ? 1.0f : 0.0f;
    }
}

// tau_init = 1 + pred / NN_TARGET_SCALE, trilinear from the coarse nodes,
// clamped to [NN_TAU_INIT_MIN, NN_TAU_INIT_MAX] (NaN -> 1).  A wave per row of the
// grid, lanes over k, as k_warm_features: the row's four coarse rows and weights
// are wave-uniform (32 x 101^3: 263 us with per-node index arithmetic, 183 us here;
// the writes alone take 54).
__global__ __launch_bounds__(256) void k_warm_init(WarmGrid G, const float* __restrict__ pred, int stride, int D, int H,
                                                   int W, double* __restrict__ tau) {
    const int q = blockIdx.y, lane = threadIdx.x & 63;
    const long long N = (long long)G.n[0] * G.n[1] * G.n[2];
    const long long npos = (long long)D * H * W, nrow = (long long)G.n[0] * G.n[1];
    const float* pr = pred + q * npos;
    // coarse cell and upper weight of fine index x on an axis
    auto cell = [&](int a, int x, int& c0, int& c1, double& w1) {
        const int last = (G.n[a] - 1) / stride;
        c0 = min(x / stride, last);
        c1 = min(c0 + 1, last);
        w1 = c1 == c0 ? 0.0 : (double)(x - c0 * stride) / stride;
    };
    // this wave's rows: a contiguous run, so that (i, j) advances without divisions
    const long long wave = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long nw = 4LL * gridDim.x, r0 = nrow * wave / nw, r1 = nrow * (wave + 1) / nw;
    for (int k0 = 64 * (int)blockIdx.z; k0 < G.n[2]; k0 += 64 * (int)gridDim.z) {
        const int k = k0 + lane;
        int x0, x1;
        double wk;
        cell(2, min(k, G.n[2] - 1), x0, x1, wk);
        int i = (int)(r0 / G.n[1]), j = (int)(r0 % G.n[1]);
        for (long long r = r0; r < r1; ++r) {
            int z[2], y[2];
            double wi, wj;
            cell(0, i, z[0], z[1], wi);
            cell(1, j, y[0], y[1], wj);
            double v = 0.0;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int a = c >> 2, b = (c >> 1) & 1, d = c & 1;
                const double w = (a ? wi : 1.0 - wi) * (b ? wj : 1.0 - wj) * (d ? wk : 1.0 - wk);
                // (a corner of weight 0 takes no part, whatever it holds)
                const double t = fma(w, (double)pr[((long long)z[a] * H + y[b]) * W + (d ? x1 : x0)], v);
                v = w == 0.0 ? v : t;
            }
            double t = 1.0 + v / NN_TARGET_SCALE;
            if (t != t)
                t = 1.0;
            else
                t = fmin(fmax(t, NN_TAU_INIT_MIN), NN_TAU_INIT_MAX);
            if (k < G.n[2]) tau[q * N + r * G.n[2] + k] = t;
            if (++j == G.n[1]) {
                j = 0;
                ++i;
            }
        }
    }
}

// ===================================================== host: layer launches
int check_ptr(const void* p, const char* name, size_t align) {
    if (!p) return fail(TT_EINVAL, "%s is NULL", name);
    if (reinterpret_cast<uintptr_t>(p) % align) return fail(TT_EINVAL, "%s must be %zu-byte aligned", name, align);
    return TT_OK;
}

int check_dims(int nbatch, int D, int H, int W) {
    if (nbatch < 1 || D < 1 || H < 1 || W < 1) return fail(TT_EINVAL, "batch and spatial sizes must be >= 1");
    if ((long long)nbatch * D * H * W > (1LL << 40)) return fail(TT_EINVAL, "too many positions");
    return TT_OK;
}

int check_chan(int ct, int co, int c, const char* name) {
    if (c < 1 || co < 0 || co + c > ct) return fail(TT_EINVAL, "%s: channel range [%d, %d) outside %d", name, co, co + c, ct);
    return TT_OK;
}

// channel ranges that can be read in aligned 16-byte pieces
bool pieces16(const uint16_t* p, int ct, int co) {
    return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ct % 8 == 0 && co % 8 == 0;
}

// Rows of a k_conv3_planes tile (0: the staged form does not take these sizes):
// as many as its waves' blocks, the fetch registers and the LDS of two
// workgroups per CU hold (of one, if a single row needs that), evened out over H.
int conv3_plane_rows(int KB, int MB, int H, int W, size_t* lds) {
    auto bytes = [&](int r) { return (size_t)3 * (r + 2) * (W + 2) * cv_pixel(KB) * sizeof(uint16_t); };
    auto fits = [&](int r, size_t most) {
        return r * W <= 64 * MB && (r + 2) * 2 * KB * W <= 256 * kCvPieces && bytes(r) <= most;
    };
    int R = 0;
    while (R < H && fits(R + 1, 80 * 1024)) ++R;
    if (R == 0 && fits(1, 156 * 1024)) R = 1;
    if (R == 0) return 0;
    const int nt = (H + R - 1) / R;
    R = (H + nt - 1) / nt;
    *lds = bytes(R);
    return R;
}

template <int KB, int NB, int MB>
int conv3_planes(const uint16_t* x, int nbatch, int D, int H, int W, int cxt, int cxo, const uint16_t* frag,
                 const float* bias, int relu, uint16_t* y, int cyt, int cyo, int R, size_t lds, hipStream_t st) {
    const int ntile = (H + R - 1) / R;
    const long long nt = (long long)nbatch * ntile;
    // z chunks for one round of two workgroups a CU (a chunk fetches 2 planes more than it works on)
    long long nz = 512 / nt;
    nz = nz < 1 ? 1 : (nz > D ? D : nz);
    const int zc = (int)((D + nz - 1) / nz);
    NN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_conv3_planes<KB, NB, MB>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL((k_conv3_planes<KB, NB, MB>), dim3((unsigned)nt, (unsigned)((D + zc - 1) / zc)), dim3(256), lds, st,
                       x, D, H, W, cxt, cxo, frag, bias, relu, y, cyt, cyo, R, ntile, zc);
    NN_LAUNCHED();
    return TT_OK;
}

// 16-position blocks a wave of k_conv3_planes holds, as its accumulators leave
// registers for.  32 -> 16 channels, whose resident weights take 108 of them, has 6:
// with 8 the plane's tiles are larger and fewer (8 x 56^3 105.5 us instead of 99.4,
// 64^3 24.8 and 23.6, 24 x 100 x 100 31.1 and 29.4).
constexpr int cv_blocks(int KB, int NB) { return NB > 2 ? 4 : (KB == 2 && NB == 1 ? 6 : 8); }

template <int KB>
int conv3_planes_nb(int NB, const uint16_t* x, int nbatch, int D, int H, int W, int cxt, int cxo, const uint16_t* frag,
                    const float* bias, int relu, uint16_t* y, int cyt, int cyo, int R, size_t lds, hipStream_t st) {
    switch (NB) {
        case 1: return conv3_planes<KB, 1, cv_blocks(KB, 1)>(x, nbatch, D, H, W, cxt, cxo, frag, bias, relu, y, cyt, cyo, R, lds, st);
        case 2: return conv3_planes<KB, 2, cv_blocks(KB, 2)>(x, nbatch, D, H, W, cxt, cxo, frag, bias, relu, y, cyt, cyo, R, lds, st);
        case 3: return conv3_planes<KB, 3, cv_blocks(KB, 3)>(x, nbatch, D, H, W, cxt, cxo, frag, bias, relu, y, cyt, cyo, R, lds, st);
        default: return conv3_planes<KB, 4, cv_blocks(KB, 4)>(x, nbatch, D, H, W, cxt, cxo, frag, bias, relu, y, cyt, cyo, R, lds, st);
    }
}

int conv3_fwd(const uint16_t* x, int nbatch, int D, int H, int W, int cxt, int cxo, int cin, const uint16_t* frag,
              const float* bias, int cout, int relu, uint16_t* y, int cyt, int cyo, hipStream_t st) {
    const long long npos = (long long)nbatch * D * H * W;
    const unsigned blocks = blocks_of(npos, 4 * 16 * kMB);
    const int KB = cin / 16, NB = cout / 16;
    // staged planes take 16-byte pieces in and 8-byte ones out; 48 input channels
    // (an odd number of steps per tap) and rows wider than a tile go direct
    if (KB != 3 && pieces16(x, cxt, cxo) && reinterpret_cast<uintptr_t>(y) % 8 == 0 && cyt % 4 == 0 && cyo % 4 == 0 &&
        (long long)nbatch * H < (1 << 30) && (long long)H * W * cxt < (1LL << 31)) {
        size_t lds = 0;
        const int R = conv3_plane_rows(KB, cv_blocks(KB, NB), H, W, &lds);
        if (R > 0) {
            if (KB == 1) return conv3_planes_nb<1>(NB, x, nbatch, D, H, W, cxt, cxo, frag, bias, relu, y, cyt, cyo, R, lds, st);
            if (KB == 2) return conv3_planes_nb<2>(NB, x, nbatch, D, H, W, cxt, cxo, frag, bias, relu, y, cyt, cyo, R, lds, st);
            return conv3_planes_nb<4>(NB, x, nbatch, D, H, W, cxt, cxo, frag, bias, relu, y, cyt, cyo, R, lds, st);
        }
    }
    switch (NB) {
        case 1: hipLaunchKernelGGL(k_conv3_fwd<1>, dim3(blocks), dim3(256), 0, st, x, D, H, W, npos, cxt, cxo, KB, frag, bias, relu, y, cyt, cyo); break;
        case 2: hipLaunchKernelGGL(k_conv3_fwd<2>, dim3(blocks), dim3(256), 0, st, x, D, H, W, npos, cxt, cxo, KB, frag, bias, relu, y, cyt, cyo); break;
        case 3: hipLaunchKernelGGL(k_conv3_fwd<3>, dim3(blocks), dim3(256), 0, st, x, D, H, W, npos, cxt, cxo, KB, frag, bias, relu, y, cyt, cyo); break;
        default: hipLaunchKernelGGL(k_conv3_fwd<4>, dim3(blocks), dim3(256), 0, st, x, D, H, W, npos, cxt, cxo, KB, frag, bias, relu, y, cyt, cyo); break;
    }
    NN_LAUNCHED();
    return TT_OK;
}

// Slices of equal length that cover nrows rows, at most `most` of them.  The count
// is taken again after the length has been rounded up, so that no slice starts
// past the last row: the kernels read a slice's first rows unasked.
long long even_slices(long long nrows, long long most) {
    if (nrows < 1 || most < 1) return 1;
    const long long rows = (nrows + most - 1) / most;
    return (nrows + rows - 1) / rows;
}

// 512 slices give every CU two workgroups; a slice of fewer than 8 rows would
// stage more halo rows than it works on, which only pays while most of the chip is
// idle (rows in 8s and in up to 32 slices: 4^3 of 64 -> 64 channels 31.0 and 21.9 us,
// 8^3 31.5 and 27.4, 14^3 of 32 -> 32 30.6 and 28.0)
long long wgrad_slices(long long nrows) {
    return even_slices(nrows, std::min(std::max((nrows + 7) / 8, 32LL), std::min(nrows, 512LL)));
}

// partial weight gradients, then partial bias gradients, of every slice
size_t conv3_wgrad_floats(long long nrows, int cin, int cout) {
    return (size_t)wgrad_slices(nrows) * (27 * (size_t)cin * cout + cout);
}

int sum_slices(const float* part, long long ns, long long n, float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_sum_slices, dim3(blocks_of(n, kSumCols)), dim3(kSumCols * kSumGroups), 0, st, part, ns, n, out);
    NN_LAUNCHED();
    return TT_OK;
}

long long colsum_blocks(long long npos) {
    long long b = (npos + 4095) / 4096;
    return b < 1 ? 1 : (b > 1024 ? 1024 : b);
}

int colsum(const uint16_t* g, long long npos, int ct, int co, int c, float* out, float* work, hipStream_t st) {
    const long long nb = colsum_blocks(npos);
    const long long chunk = (npos + nb - 1) / nb;
    hipLaunchKernelGGL(k_colsum_part, dim3((unsigned)nb), dim3(256), 0, st, g, npos, ct, co, c, chunk, work);
    NN_LAUNCHED();
    return sum_slices(work, nb, c, out, st);
}

int conv3_wgrad(const uint16_t* x, int nbatch, int D, int H, int W, int cxt, int cxo, int cin, const uint16_t* gz,
                int cgt, int cgo, int cout, float* gW, float* gb, float* work, hipStream_t st) {
    const long long nrows = (long long)nbatch * D * H;
    const long long ns = wgrad_slices(nrows);
    const long long rps = (nrows + ns - 1) / ns;
    const long long n = 27LL * cin * cout;
    const int nib = (cin + 15) / 16, nob = cout / 16;
    // staged rows take whole 16-byte pieces of whole 16-channel blocks (the last
    // block's channels past cin are read and dropped); other layouts go per tap
    if (pieces16(x, cxt, cxo) && pieces16(gz, cgt, cgo) && cxo + nib * 16 <= cxt) {
        float* bpart = gb ? work + ns * n : nullptr;
        const int ib = nib % 2 == 0 ? 2 : 1, ob = nob % 2 == 0 ? 2 : 1;
        const dim3 grid((unsigned)ns, (unsigned)((nib / ib) * (nob / ob)));
#define NN_WG(A, B)                                                                                                   \
    hipLaunchKernelGGL((k_conv3_wgrad_rows<A, B>), grid, dim3(256), 0, st, x, D, H, W, nrows, cxt, cxo, cin, gz, cgt, cgo, \
                       cout, rps, nob / B, work, bpart)
        if (ib == 2 && ob == 2) NN_WG(2, 2);
        else if (ib == 2) NN_WG(2, 1);
        else if (ob == 2) NN_WG(1, 2);
        else NN_WG(1, 1);
#undef NN_WG
        NN_LAUNCHED();
        if (gb) {
            const int rc = sum_slices(bpart, ns, cout, gb, st);
            if (rc) return rc;
        }
        return sum_slices(work, ns, n, gW, st);
    }
    hipLaunchKernelGGL(k_conv3_wgrad, dim3((unsigned)ns, 27), dim3(256), 0, st, x, D, H, W, nrows, cxt, cxo, cin, gz,
                       cgt, cgo, cout, rps, work);
    NN_LAUNCHED();
    const int rc = sum_slices(work, ns, n, gW, st);
    if (rc) return rc;
    if (gb) return colsum(gz, nrows * W, cgt, cgo, cout, gb, work, st);
    return TT_OK;
}

size_t colsum_floats(long long npos, int c) { return (size_t)colsum_blocks(npos) * c; }

long long up_slices(long long np) {
    long long s = (np + 63) / 64;
    return s < 1 ? 1 : (s > 256 ? 256 : s);
}

long long up_row_slices(long long nrows) { return even_slices(nrows, std::min((nrows + 3) / 4, 512LL)); }

size_t up_work_floats(long long np, long long nrows, int cin, int cout) {
    const size_t a = (size_t)up_slices(np) * 8 * cin * cout;
    const size_t b = colsum_floats(np * 8, cout);
    const size_t c = (size_t)up_row_slices(nrows) * (8 * (size_t)cin * cout + 4 * (size_t)cout);
    return a > b ? (a > c ? a : c) : (b > c ? b : c);
}

int up_bwd(const uint16_t* x, const uint16_t* gy, int nbatch, int D, int H, int W, int cin, int cout, int cgt, int cgo,
           const float* Wu, uint16_t* gx, float* gW, float* gb, float* work, hipStream_t st) {
    const long long np = (long long)nbatch * D * H * W;
    if (gx && cin % 16 == 0 && cout % 16 == 0 && pieces16(gy, cgt, cgo) && pieces16(gx, cin, 0) && np < (1LL << 31)) {
        hipLaunchKernelGGL(k_up_bwd_pos, dim3(blocks_of(np, 256), cin / 16), dim3(256), 0, st, gy, np, D, H, W, cin, cout,
                           cgt, cgo, Wu, gx);
        NN_LAUNCHED();
    } else if (gx) {
        hipLaunchKernelGGL(k_up_bwd_data, dim3(grid_stride_blocks(np * cin)), dim3(256), 0, st, gy, np, D, H, W, cin,
                           cout, cgt, cgo, Wu, gx);
        NN_LAUNCHED();
    }
    if (cin % 16 == 0 && cout % 16 == 0 && pieces16(x, cin, 0) && pieces16(gy, cgt, cgo)) {
        const long long nrows = (long long)nbatch * D * H;
        const long long ns = up_row_slices(nrows), rps = (nrows + ns - 1) / ns, n = 8LL * cin * cout;
        float* bpart = work + ns * n;
        const int nib = cin / 16, nob = cout / 16, ib = nib % 2 == 0 ? 2 : 1, ob = nob % 2 == 0 ? 2 : 1;
        const dim3 grid((unsigned)ns, (unsigned)((nib / ib) * (nob / ob)));
#define NN_WG(A, B)                                                                                                \
    hipLaunchKernelGGL((k_up_wgrad_rows<A, B>), grid, dim3(256), 0, st, x, gy, D, H, W, nrows, cin, cout, cgt, cgo, rps, \
                       nob / B, work, bpart)
        if (ib == 2 && ob == 2) NN_WG(2, 2);
        else if (ib == 2) NN_WG(2, 1);
        else if (ob == 2) NN_WG(1, 2);
        else NN_WG(1, 1);
#undef NN_WG
        NN_LAUNCHED();
        const int rc = sum_slices(work, ns, n, gW, st);
        return rc ? rc : sum_slices(bpart, 4 * ns, cout, gb, st);
    }
    const long long ns = up_slices(np);
    const long long chunk = (np + ns - 1) / ns;
    hipLaunchKernelGGL(k_up_wgrad_part, dim3((unsigned)ns, 8), dim3(256), 0, st, x, gy, np, D, H, W, cin, cout, cgt,
                       cgo, chunk, work);
    NN_LAUNCHED();
    const long long n = 8LL * cin * cout;
    const int rc = sum_slices(work, ns, n, gW, st);
    if (rc) return rc;
    return colsum(gy, np * 8, cgt, cgo, cout, gb, work, st);
}

long long head_blocks(long long npos) {
    long long b = (npos + 4095) / 4096;
    return b < 1 ? 1 : (b > 1024 ? 1024 : b);
}

size_t head_work_floats(long long npos, int cin) { return (size_t)head_blocks(npos) * (cin + 1); }

int head_fwd(const uint16_t* x, long long npos, int cin, const float* w, const float* b, float* y, hipStream_t st) {
    if (pieces16(x, cin, 0))
        hipLaunchKernelGGL(k_head_fwd8, dim3(grid_stride_blocks(npos)), dim3(256), 0, st, x, npos, cin, w, b, y);
    else
        hipLaunchKernelGGL(k_head_fwd, dim3(grid_stride_blocks(npos)), dim3(256), 0, st, x, npos, cin, w, b, y);
    NN_LAUNCHED();
    return TT_OK;
}

int head_bwd(const uint16_t* x, const float* gy, long long npos, int cin, const float* w, uint16_t* gx, float* gw,
             float* gb, float* work, hipStream_t st) {
    if (gx && pieces16(gx, cin, 0)) {
        hipLaunchKernelGGL(k_head_bwd_data8, dim3(grid_stride_blocks(npos * (cin / 8))), dim3(256), 0, st, gy, npos, cin, w, gx);
        NN_LAUNCHED();
    } else if (gx) {
        hipLaunchKernelGGL(k_head_bwd_data, dim3(grid_stride_blocks(npos * cin)), dim3(256), 0, st, gy, npos, cin, w, gx);
        NN_LAUNCHED();
    }
    const long long nb = head_blocks(npos);
    const long long chunk = (npos + nb - 1) / nb;
    if (pieces16(x, cin, 0))
        hipLaunchKernelGGL(k_head_wgrad_part8, dim3((unsigned)nb), dim3(256), 0, st, x, gy, npos, cin, chunk, work);
    else
        hipLaunchKernelGGL(k_head_wgrad_part, dim3((unsigned)nb), dim3(256), 0, st, x, gy, npos, cin, chunk, work);
    NN_LAUNCHED();
    hipLaunchKernelGGL(k_head_finish, dim3(cin + 1), dim3(256), 0, st, work, nb, cin, gw, gb);
    NN_LAUNCHED();
    return TT_OK;
}

// ============================================================ U-Net plan
enum { E1A, E1B, E2A, E2B, E3A, E3B, BNA, BNB, D3A, D3B, D2A, D2B, D1A, D1B, NCONV };
enum { U3, U2, U1, NUP };

struct ConvDef {
    int ci, co, cip;     // input channels (real), output channels, padded input channels
    size_t w, b;         // parameter offsets (floats)
    size_t fw, fb;       // fragment offsets: forward, data-gradient (bf16 elements)
};
struct UpDef {
    int ci, co;
    size_t w, b;
};
struct Net {
    int c[4], in_ch;
    ConvDef conv[NCONV];
    UpDef up[NUP];
    size_t head_w, head_b, nparams, nfrag;
};

int make_net(const nn_unet_cfg* cfg, Net& N) {
    if (!cfg) return fail(TT_EINVAL, "cfg is NULL");
    for (int l = 0; l < 4; ++l)
        if (cfg->ch[l] < 16 || cfg->ch[l] % 16 || cfg->ch[l] > 64)
            return fail(TT_EINVAL, "cfg.ch[%d] = %d: channels must be multiples of 16 in [16, 64]", l, cfg->ch[l]);
    for (int l = 0; l < 3; ++l)
        if (2 * cfg->ch[l] > 64) return fail(TT_EINVAL, "decoder convolutions need 2 * ch[%d] <= 64", l);
    if (cfg->in_ch < 1 || cfg->in_ch > 16) return fail(TT_EINVAL, "cfg.in_ch must be in [1, 16]");
    std::memset(&N, 0, sizeof N);
    for (int l = 0; l < 4; ++l) N.c[l] = cfg->ch[l];
    N.in_ch = cfg->in_ch;
    const int c1 = N.c[0], c2 = N.c[1], c3 = N.c[2], c4 = N.c[3];
    const int io[NCONV][2] = {{N.in_ch, c1}, {c1, c1}, {c1, c2}, {c2, c2}, {c2, c3}, {c3, c3}, {c3, c4},
                              {c4, c4},      {2 * c3, c3}, {c3, c3}, {2 * c2, c2}, {c2, c2}, {2 * c1, c1}, {c1, c1}};
    size_t off = 0, fo = 0;
    for (int k = 0; k < NCONV; ++k) {
        ConvDef& C = N.conv[k];
        C.ci = io[k][0];
        C.co = io[k][1];
        C.cip = (C.ci + 15) / 16 * 16;
        C.w = off;
        off += 27 * (size_t)C.ci * C.co;
        C.b = off;
        off += C.co;
        C.fw = fo;
        fo += 27 * (size_t)C.cip * C.co;
        C.fb = fo;
        if (k != E1A) fo += 27 * (size_t)C.ci * C.co;
    }
    const int uio[NUP][2] = {{c4, c3}, {c3, c2}, {c2, c1}};
    for (int k = 0; k < NUP; ++k) {
        UpDef& U = N.up[k];
        U.ci = uio[k][0];
        U.co = uio[k][1];
        U.w = off;
        off += 8 * (size_t)U.ci * U.co;
        U.b = off;
        off += U.co;
    }
    N.head_w = off;
    off += c1;
    N.head_b = off;
    off += 1;
    N.nparams = off;
    N.nfrag = fo;
    return TT_OK;
}

// Activation and gradient buffers of one (batch, D, H, W) in the workspace.
struct Acts {
    long long P[4];
    uint16_t *a1, *cat1, *p1, *a2, *cat2, *p2, *a3, *cat3, *p3, *b1, *b2, *d3a, *d3b, *d2a, *d2b, *d1a, *d1b;
    uint16_t *gA[3], *gZ[3], *gcat[3], *gBa, *gBb, *gZ4, *gP[3];
    float* work;
    size_t bytes;
};

size_t aup(size_t v) { return (v + 255) & ~(size_t)255; }

int check_net_dims(int nbatch, int D, int H, int W) {
    if (check_dims(nbatch, D, H, W)) return TT_EINVAL;
    if (D % 8 || H % 8 || W % 8) return fail(TT_EINVAL, "U-Net spatial sizes must be multiples of 8 (got %d %d %d)", D, H, W);
    return TT_OK;
}

// Lays out the buffers from base (or only measures when base is NULL).
void layout(const Net& N, int nbatch, int D, int H, int W, int train, char* base, Acts& A) {
    std::memset(&A, 0, sizeof A);
    A.P[0] = (long long)nbatch * D * H * W;
    for (int l = 1; l < 4; ++l) A.P[l] = A.P[l - 1] / 8;
    const int c1 = N.c[0], c2 = N.c[1], c3 = N.c[2], c4 = N.c[3];
    size_t off = 0;
    auto take16 = [&](long long np, int c) -> uint16_t* {
        uint16_t* p = base ? reinterpret_cast<uint16_t*>(base + off) : nullptr;
        off += aup((size_t)np * c * sizeof(uint16_t));
        return p;
    };
    A.a1 = take16(A.P[0], c1);
    A.cat1 = take16(A.P[0], 2 * c1);
    A.p1 = take16(A.P[1], c1);
    A.a2 = take16(A.P[1], c2);
    A.cat2 = take16(A.P[1], 2 * c2);
    A.p2 = take16(A.P[2], c2);
    A.a3 = take16(A.P[2], c3);
    A.cat3 = take16(A.P[2], 2 * c3);
    A.p3 = take16(A.P[3], c3);
    A.b1 = take16(A.P[3], c4);
    A.b2 = take16(A.P[3], c4);
    A.d3a = take16(A.P[2], c3);
    A.d3b = take16(A.P[2], c3);
    A.d2a = take16(A.P[1], c2);
    A.d2b = take16(A.P[1], c2);
    A.d1a = take16(A.P[0], c1);
    A.d1b = take16(A.P[0], c1);
    if (train) {
        const int cl[3] = {c1, c2, c3};
        for (int l = 0; l < 3; ++l) {
            A.gA[l] = take16(A.P[l], cl[l]);
            A.gZ[l] = take16(A.P[l], cl[l]);
            A.gcat[l] = take16(A.P[l], 2 * cl[l]);
        }
        A.gBa = take16(A.P[3], c4);
        A.gBb = take16(A.P[3], c4);
        A.gZ4 = take16(A.P[3], c4);
        A.gP[0] = take16(A.P[1], c1);
        A.gP[1] = take16(A.P[2], c2);
        A.gP[2] = take16(A.P[3], c3);
        // reduction scratch: the largest of the layers' needs
        size_t wf = 0;
        const int lev[NCONV] = {0, 0, 1, 1, 2, 2, 3, 3, 2, 2, 1, 1, 0, 0};
        for (int k = 0; k < NCONV; ++k) {
            const long long np = A.P[lev[k]];
            const long long nrows = np / (W >> lev[k]);  // (n, z, y) rows of the level
            size_t f = conv3_wgrad_floats(nrows, N.conv[k].ci, N.conv[k].co);
            size_t g = colsum_floats(np, N.conv[k].co);
            if (f > wf) wf = f;
            if (g > wf) wf = g;
        }
        for (int k = 0; k < NUP; ++k) {
            const long long np = A.P[3 - k];
            const size_t f = up_work_floats(np, np / (W >> (3 - k)), N.up[k].ci, N.up[k].co);
            if (f > wf) wf = f;
        }
        const size_t hf = head_work_floats(A.P[0], c1);
        if (hf > wf) wf = hf;
        A.work = base ? reinterpret_cast<float*>(base + off) : nullptr;
        off += aup(wf * sizeof(float));
    }
    A.bytes = off;
}

int conv_layer_fwd(const Net& N, int k, const float* prm, const uint16_t* frag, const uint16_t* x, int cxt, int cxo,
                   int nbatch, int D, int H, int W, uint16_t* y, int cyt, int cyo, hipStream_t st) {
    const ConvDef& C = N.conv[k];
    return conv3_fwd(x, nbatch, D, H, W, cxt, cxo, C.cip, frag + C.fw, prm + C.b, C.co, 1, y, cyt, cyo, st);
}

int relu_mask(const uint16_t* g, const uint16_t* y, long long npos, int ct, int co, int c, uint16_t* go, int cot,
              int coo, hipStream_t st) {
    if (c % 8 == 0 && pieces16(g, ct, co) && pieces16(y, ct, co) && pieces16(go, cot, coo)) {
        hipLaunchKernelGGL(k_relu_mask8, dim3(grid_stride_blocks(npos * (c / 8))), dim3(256), 0, st, g, y, npos, ct, co,
                           c / 8, go, cot, coo);
        NN_LAUNCHED();
        return TT_OK;
    }
    hipLaunchKernelGGL(k_relu_mask, dim3(grid_stride_blocks(npos * c)), dim3(256), 0, st, g, y, npos, ct, co, c, go,
                       cot, coo);
    NN_LAUNCHED();
    return TT_OK;
}

int pool_fwd(const uint16_t* x, int nbatch, int D, int H, int W, int ct, int co, int c, uint16_t* y, hipStream_t st) {
    const long long nq = (long long)nbatch * (D / 2) * (H / 2) * (W / 2);
    if (c % 8 == 0 && pieces16(x, ct, co) && pieces16(y, c, 0)) {
        hipLaunchKernelGGL(k_pool_fwd8, dim3(grid_stride_blocks(nq * (c / 8))), dim3(256), 0, st, x, nq, D / 2, H / 2,
                           W / 2, ct, co, c / 8, y);
        NN_LAUNCHED();
        return TT_OK;
    }
    hipLaunchKernelGGL(k_pool_fwd, dim3(grid_stride_blocks(nq * c)), dim3(256), 0, st, x, nq, D / 2, H / 2, W / 2, ct,
                       co, c, y);
    NN_LAUNCHED();
    return TT_OK;
}

int pool_bwd(const uint16_t* x, const uint16_t* gy, int nbatch, int D, int H, int W, int ct, int co, int c,
             uint16_t* gx, int accumulate, hipStream_t st) {
    const long long nq = (long long)nbatch * (D / 2) * (H / 2) * (W / 2);
    if (c % 8 == 0 && pieces16(x, ct, co) && pieces16(gy, c, 0) && pieces16(gx, ct, co)) {
        hipLaunchKernelGGL(k_pool_bwd8, dim3(grid_stride_blocks(nq * (c / 8))), dim3(256), 0, st, x, gy, nq, D / 2, H / 2,
                           W / 2, ct, co, c / 8, gx, accumulate);
        NN_LAUNCHED();
        return TT_OK;
    }
    hipLaunchKernelGGL(k_pool_bwd, dim3(grid_stride_blocks(nq * c)), dim3(256), 0, st, x, gy, nq, D / 2, H / 2,
                       W / 2, ct, co, c, gx, accumulate);
    NN_LAUNCHED();
    return TT_OK;
}

int up_fwd(const uint16_t* x, int nbatch, int D, int H, int W, int cin, const float* Wu, const float* b, int cout,
           uint16_t* y, int cyt, int cyo, hipStream_t st) {
    const long long np = (long long)nbatch * D * H * W;
    // (a thread per position leaves the chip idle up to 512 of them: 7^3 of 64 -> 64
    // channels 10.7 us, 9.6 with a thread per output; 2 x 7^3 10.8 and 10.5, 14^3 of 64 -> 32
    // 11.3 and 17.3)
    if (np > 512 && cin % 8 == 0 && cout % 16 == 0 && pieces16(x, cin, 0) && pieces16(y, cyt, cyo) && np < (1LL << 31)) {
        hipLaunchKernelGGL(k_up_fwd_pos, dim3(blocks_of(np, 256), 4, cout / 16), dim3(256), 0, st, x, np, D, H, W, cin, Wu,
                           b, cout, y, cyt, cyo);
        NN_LAUNCHED();
        return TT_OK;
    }
    const long long nout = (long long)nbatch * D * H * W * 8;
    hipLaunchKernelGGL(k_up_fwd, dim3(grid_stride_blocks(nout * cout)), dim3(256), 0, st, x, nout, D, H, W, cin, Wu,
                       b, cout, y, cyt, cyo);
    NN_LAUNCHED();
    return TT_OK;
}

#define NN_TRY(expr)          \
    do {                      \
        int rc_ = (expr);     \
        if (rc_) return rc_;  \
    } while (0)

int unet_forward(const Net& N, const float* prm, const uint16_t* frag, const uint16_t* x, int nb, int D, int H, int W,
                 float* y, const Acts& A, hipStream_t st) {
    const int c1 = N.c[0], c2 = N.c[1], c3 = N.c[2], c4 = N.c[3];
    int d = D, h = H, w = W;
    // level 1
    NN_TRY(conv_layer_fwd(N, E1A, prm, frag, x, 16, 0, nb, d, h, w, A.a1, c1, 0, st));
    NN_TRY(conv_layer_fwd(N, E1B, prm, frag, A.a1, c1, 0, nb, d, h, w, A.cat1, 2 * c1, c1, st));
    NN_TRY(pool_fwd(A.cat1, nb, d, h, w, 2 * c1, c1, c1, A.p1, st));
    d /= 2, h /= 2, w /= 2;
    NN_TRY(conv_layer_fwd(N, E2A, prm, frag, A.p1, c1, 0, nb, d, h, w, A.a2, c2, 0, st));
    NN_TRY(conv_layer_fwd(N, E2B, prm, frag, A.a2, c2, 0, nb, d, h, w, A.cat2, 2 * c2, c2, st));
    NN_TRY(pool_fwd(A.cat2, nb, d, h, w, 2 * c2, c2, c2, A.p2, st));
    d /= 2, h /= 2, w /= 2;
    NN_TRY(conv_layer_fwd(N, E3A, prm, frag, A.p2, c2, 0, nb, d, h, w, A.a3, c3, 0, st));
    NN_TRY(conv_layer_fwd(N, E3B, prm, frag, A.a3, c3, 0, nb, d, h, w, A.cat3, 2 * c3, c3, st));
    NN_TRY(pool_fwd(A.cat3, nb, d, h, w, 2 * c3, c3, c3, A.p3, st));
    d /= 2, h /= 2, w /= 2;
    NN_TRY(conv_layer_fwd(N, BNA, prm, frag, A.p3, c3, 0, nb, d, h, w, A.b1, c4, 0, st));
    NN_TRY(conv_layer_fwd(N, BNB, prm, frag, A.b1, c4, 0, nb, d, h, w, A.b2, c4, 0, st));
    // decoder
    NN_TRY(up_fwd(A.b2, nb, d, h, w, c4, prm + N.up[U3].w, prm + N.up[U3].b, c3, A.cat3, 2 * c3, 0, st));
    d *= 2, h *= 2, w *= 2;
    NN_TRY(conv_layer_fwd(N, D3A, prm, frag, A.cat3, 2 * c3, 0, nb, d, h, w, A.d3a, c3, 0, st));
    NN_TRY(conv_layer_fwd(N, D3B, prm, frag, A.d3a, c3, 0, nb, d, h, w, A.d3b, c3, 0, st));
    NN_TRY(up_fwd(A.d3b, nb, d, h, w, c3, prm + N.up[U2].w, prm + N.up[U2].b, c2, A.cat2, 2 * c2, 0, st));
    d *= 2, h *= 2, w *= 2;
    NN_TRY(conv_layer_fwd(N, D2A, prm, frag, A.cat2, 2 * c2, 0, nb, d, h, w, A.d2a, c2, 0, st));
    NN_TRY(conv_layer_fwd(N, D2B, prm, frag, A.d2a, c2, 0, nb, d, h, w, A.d2b, c2, 0, st));
    NN_TRY(up_fwd(A.d2b, nb, d, h, w, c2, prm + N.up[U1].w, prm + N.up[U1].b, c1, A.cat1, 2 * c1, 0, st));
    d *= 2, h *= 2, w *= 2;
    NN_TRY(conv_layer_fwd(N, D1A, prm, frag, A.cat1, 2 * c1, 0, nb, d, h, w, A.d1a, c1, 0, st));
    NN_TRY(conv_layer_fwd(N, D1B, prm, frag, A.d1a, c1, 0, nb, d, h, w, A.d1b, c1, 0, st));
    NN_TRY(head_fwd(A.d1b, A.P[0], c1, prm + N.head_w, prm + N.head_b, y, st));
    return TT_OK;
}

// Backward of one conv + ReLU layer: g_out (gradient of the layer's ReLU
// output, in (gt, go)) -> gZ = g_out * (y > 0); weight and bias gradients from
// the layer input x; data gradient into gin (unless gin is NULL).
int conv_layer_bwd(const Net& N, int k, const uint16_t* frag, float* grad, const uint16_t* g_out, const uint16_t* y,
                   int yt, int yo, const uint16_t* x, int cxt, int cxo, int nb, int D, int H, int W, uint16_t* gZ,
                   uint16_t* gin, int cgt, float* work, hipStream_t st) {
    const ConvDef& C = N.conv[k];
    const long long np = (long long)nb * D * H * W;
    NN_TRY(relu_mask(g_out, y, np, yt, yo, C.co, gZ, C.co, 0, st));
    NN_TRY(conv3_wgrad(x, nb, D, H, W, cxt, cxo, C.ci, gZ, C.co, 0, C.co, grad + C.w, grad + C.b, work, st));
    if (gin) NN_TRY(conv3_fwd(gZ, nb, D, H, W, C.co, 0, C.co, frag + C.fb, nullptr, C.ci, 0, gin, cgt, 0, st));
    return TT_OK;
}

int unet_backward(const Net& N, const float* prm, const uint16_t* frag, const float* gy, const uint16_t* x, int nb,
                  int D, int H, int W, float* grad, const Acts& A, hipStream_t st) {
    const int c1 = N.c[0], c2 = N.c[1], c3 = N.c[2], c4 = N.c[3];
    float* wk = A.work;
    int d = D, h = H, w = W;
    // head
    NN_TRY(head_bwd(A.d1b, gy, A.P[0], c1, prm + N.head_w, A.gA[0], grad + N.head_w, grad + N.head_b, wk, st));
    // level-1 decoder
    NN_TRY(conv_layer_bwd(N, D1B, frag, grad, A.gA[0], A.d1b, c1, 0, A.d1a, c1, 0, nb, d, h, w, A.gZ[0], A.gA[0], c1, wk, st));
    NN_TRY(conv_layer_bwd(N, D1A, frag, grad, A.gA[0], A.d1a, c1, 0, A.cat1, 2 * c1, 0, nb, d, h, w, A.gZ[0], A.gcat[0], 2 * c1, wk, st));
    d /= 2, h /= 2, w /= 2;
    NN_TRY(up_bwd(A.d2b, A.gcat[0], nb, d, h, w, c2, c1, 2 * c1, 0, prm + N.up[U1].w, A.gA[1], grad + N.up[U1].w,
                  grad + N.up[U1].b, wk, st));
    NN_TRY(conv_layer_bwd(N, D2B, frag, grad, A.gA[1], A.d2b, c2, 0, A.d2a, c2, 0, nb, d, h, w, A.gZ[1], A.gA[1], c2, wk, st));
    NN_TRY(conv_layer_bwd(N, D2A, frag, grad, A.gA[1], A.d2a, c2, 0, A.cat2, 2 * c2, 0, nb, d, h, w, A.gZ[1], A.gcat[1], 2 * c2, wk, st));
    d /= 2, h /= 2, w /= 2;
    NN_TRY(up_bwd(A.d3b, A.gcat[1], nb, d, h, w, c3, c2, 2 * c2, 0, prm + N.up[U2].w, A.gA[2], grad + N.up[U2].w,
                  grad + N.up[U2].b, wk, st));
    NN_TRY(conv_layer_bwd(N, D3B, frag, grad, A.gA[2], A.d3b, c3, 0, A.d3a, c3, 0, nb, d, h, w, A.gZ[2], A.gA[2], c3, wk, st));
    NN_TRY(conv_layer_bwd(N, D3A, frag, grad, A.gA[2], A.d3a, c3, 0, A.cat3, 2 * c3, 0, nb, d, h, w, A.gZ[2], A.gcat[2], 2 * c3, wk, st));
    d /= 2, h /= 2, w /= 2;
    NN_TRY(up_bwd(A.b2, A.gcat[2], nb, d, h, w, c4, c3, 2 * c3, 0, prm + N.up[U3].w, A.gBa, grad + N.up[U3].w,
                  grad + N.up[U3].b, wk, st));
    // bottleneck
    NN_TRY(conv_layer_bwd(N, BNB, frag, grad, A.gBa, A.b2, c4, 0, A.b1, c4, 0, nb, d, h, w, A.gZ4, A.gBb, c4, wk, st));
    NN_TRY(conv_layer_bwd(N, BNA, frag, grad, A.gBb, A.b1, c4, 0, A.p3, c3, 0, nb, d, h, w, A.gZ4, A.gP[2], c3, wk, st));
    d *= 2, h *= 2, w *= 2;
    // level 3 encoder: skip gradient + pooled gradient
    NN_TRY(pool_bwd(A.cat3, A.gP[2], nb, d, h, w, 2 * c3, c3, c3, A.gcat[2], 1, st));
    NN_TRY(conv_layer_bwd(N, E3B, frag, grad, A.gcat[2], A.cat3, 2 * c3, c3, A.a3, c3, 0, nb, d, h, w, A.gZ[2], A.gA[2], c3, wk, st));
    NN_TRY(conv_layer_bwd(N, E3A, frag, grad, A.gA[2], A.a3, c3, 0, A.p2, c2, 0, nb, d, h, w, A.gZ[2], A.gP[1], c2, wk, st));
    d *= 2, h *= 2, w *= 2;
    NN_TRY(pool_bwd(A.cat2, A.gP[1], nb, d, h, w, 2 * c2, c2, c2, A.gcat[1], 1, st));
    NN_TRY(conv_layer_bwd(N, E2B, frag, grad, A.gcat[1], A.cat2, 2 * c2, c2, A.a2, c2, 0, nb, d, h, w, A.gZ[1], A.gA[1], c2, wk, st));
    NN_TRY(conv_layer_bwd(N, E2A, frag, grad, A.gA[1], A.a2, c2, 0, A.p1, c1, 0, nb, d, h, w, A.gZ[1], A.gP[0], c1, wk, st));
    d *= 2, h *= 2, w *= 2;
    NN_TRY(pool_bwd(A.cat1, A.gP[0], nb, d, h, w, 2 * c1, c1, c1, A.gcat[0], 1, st));
    NN_TRY(conv_layer_bwd(N, E1B, frag, grad, A.gcat[0], A.cat1, 2 * c1, c1, A.a1, c1, 0, nb, d, h, w, A.gZ[0], A.gA[0], c1, wk, st));
    NN_TRY(conv_layer_bwd(N, E1A, frag, grad, A.gA[0], A.a1, c1, 0, x, 16, 0, nb, d, h, w, A.gZ[0], nullptr, 0, wk, st));
    return TT_OK;
}

int warm_grid(const tt_grid* g, WarmGrid& W) {
    if (!g) return fail(TT_EINVAL, "grid is NULL");
    if (g->coord != 0 && g->coord != 1) return fail(TT_EINVAL, "grid.coord must be 0 or 1");
    for (int a = 0; a < 3; ++a) {
        if (g->n[a] < 1) return fail(TT_EINVAL, "grid.n[%d] must be >= 1", a);
        W.n[a] = g->n[a];
        W.o[a] = g->o[a];
        W.h[a] = g->h[a];
    }
    W.coord = g->coord;
    return TT_OK;
}

int check_coarse(const tt_grid* g, int stride, int D, int H, int W) {
    if (stride < 1) return fail(TT_EINVAL, "stride must be >= 1");
    if (D < 1 || H < 1 || W < 1) return fail(TT_EINVAL, "coarse sizes must be >= 1");
    const int c[3] = {D, H, W};
    for (int a = 0; a < 3; ++a)
        if ((g->n[a] - 1) / stride + 1 > c[a])
            return fail(TT_EINVAL, "coarse axis %d has %d nodes, needs >= %d", a, c[a], (g->n[a] - 1) / stride + 1);
    return TT_OK;
}

}  // namespace

// ================================================================= C ABI
extern "C" {

int nn_to_bf16(const float* x, int64_t n, uint16_t* y, void* stream) {
    if (n < 0) return fail(TT_EINVAL, "n < 0");
    if (n == 0) return TT_OK;
    NN_TRY(check_ptr(x, "x", 4));
    NN_TRY(check_ptr(y, "y", 2));
    hipLaunchKernelGGL(k_to_bf16, dim3(grid_stride_blocks(n)), dim3(256), 0, S(stream), x, (long long)n, y);
    NN_LAUNCHED();
    return TT_OK;
}

int nn_from_bf16(const uint16_t* x, int64_t n, float* y, void* stream) {
    if (n < 0) return fail(TT_EINVAL, "n < 0");
    if (n == 0) return TT_OK;
    NN_TRY(check_ptr(x, "x", 2));
    NN_TRY(check_ptr(y, "y", 4));
    hipLaunchKernelGGL(k_from_bf16, dim3(grid_stride_blocks(n)), dim3(256), 0, S(stream), x, (long long)n, y);
    NN_LAUNCHED();
    return TT_OK;
}

int nn_conv3_pack(const float* W, int cin, int cout, int flip, uint16_t* frag, void* stream) {
    NN_TRY(check_ptr(W, "W", 4));
    NN_TRY(check_ptr(frag, "frag", 8));
    if (cout < 16 || cout % 16 || cout > 64) return fail(TT_EINVAL, "cout must be a multiple of 16 in [16, 64]");
    if (cin < 1 || cin > 64) return fail(TT_EINVAL, "cin must be in [1, 64]");
    if (flip && cin % 16) return fail(TT_EINVAL, "flip = 1 needs cin a multiple of 16");
    const int KB = flip ? cout / 16 : (cin + 15) / 16;
    const int NB = flip ? cin / 16 : cout / 16;
    hipLaunchKernelGGL(k_conv3_pack, dim3(grid_stride_blocks(27LL * KB * NB * 256)), dim3(256), 0, S(stream), W, cin,
                       cout, KB, NB, flip, frag);
    NN_LAUNCHED();
    return TT_OK;
}

int nn_conv3_fwd(const uint16_t* x, int nbatch, int D, int H, int W, int cx_total, int cx_off, int cin,
                 const uint16_t* frag, const float* bias, int cout, int relu, uint16_t* y, int cy_total, int cy_off,
                 void* stream) {
    NN_TRY(check_dims(nbatch, D, H, W));
    NN_TRY(check_ptr(x, "x", 8));
    NN_TRY(check_ptr(frag, "frag", 8));
    NN_TRY(check_ptr(y, "y", 2));
    if (cin < 16 || cin % 16 || cin > 64) return fail(TT_EINVAL, "cin must be a multiple of 16 in [16, 64]");
    if (cout < 16 || cout % 16 || cout > 64) return fail(TT_EINVAL, "cout must be a multiple of 16 in [16, 64]");
    if (cx_total % 4 || cx_off % 4) return fail(TT_EINVAL, "cx_total and cx_off must be multiples of 4");
    NN_TRY(check_chan(cx_total, cx_off, cin, "x"));
    NN_TRY(check_chan(cy_total, cy_off, cout, "y"));
    return conv3_fwd(x, nbatch, D, H, W, cx_total, cx_off, cin, frag, bias, cout, relu, y, cy_total, cy_off, S(stream));
}

size_t nn_conv3_wgrad_work(int nbatch, int D, int H, int W, int cin, int cout) {
    if (nbatch < 1 || D < 1 || H < 1 || W < 1 || cin < 1 || cout < 1) return 0;
    const long long nrows = (long long)nbatch * D * H;
    const size_t a = conv3_wgrad_floats(nrows, cin, cout), b = colsum_floats(nrows * W, cout);
    return (a > b ? a : b) * sizeof(float);
}

int nn_conv3_wgrad(const uint16_t* x, int nbatch, int D, int H, int W, int cx_total, int cx_off, int cin,
                   const uint16_t* gz, int cg_total, int cg_off, int cout, float* gW, float* gb, float* work,
                   size_t work_bytes, void* stream) {
    NN_TRY(check_dims(nbatch, D, H, W));
    NN_TRY(check_ptr(x, "x", 2));
    NN_TRY(check_ptr(gz, "gz", 2));
    NN_TRY(check_ptr(gW, "gW", 4));
    NN_TRY(check_ptr(work, "work", 4));
    if (cin < 1 || cin > 64) return fail(TT_EINVAL, "cin must be in [1, 64]");
    if (cout < 16 || cout % 16 || cout > 64) return fail(TT_EINVAL, "cout must be a multiple of 16 in [16, 64]");
    NN_TRY(check_chan(cx_total, cx_off, cin, "x"));
    NN_TRY(check_chan(cg_total, cg_off, cout, "gz"));
    if (work_bytes < nn_conv3_wgrad_work(nbatch, D, H, W, cin, cout)) return fail(TT_EINVAL, "work too small");
    return conv3_wgrad(x, nbatch, D, H, W, cx_total, cx_off, cin, gz, cg_total, cg_off, cout, gW, gb, work, S(stream));
}

int nn_relu_mask(const uint16_t* g, const uint16_t* y, int64_t npos, int c_total, int c_off, int c, uint16_t* g_out,
                 int co_total, int co_off, void* stream) {
    if (npos < 0) return fail(TT_EINVAL, "npos < 0");
    if (npos == 0) return TT_OK;
    NN_TRY(check_ptr(g, "g", 2));
    NN_TRY(check_ptr(y, "y", 2));
    NN_TRY(check_ptr(g_out, "g_out", 2));
    NN_TRY(check_chan(c_total, c_off, c, "g"));
    NN_TRY(check_chan(co_total, co_off, c, "g_out"));
    return relu_mask(g, y, npos, c_total, c_off, c, g_out, co_total, co_off, S(stream));
}

int nn_pool_fwd(const uint16_t* x, int nbatch, int D, int H, int W, int c_total, int c_off, int c, uint16_t* y,
                void* stream) {
    NN_TRY(check_dims(nbatch, D, H, W));
    if (D % 2 || H % 2 || W % 2) return fail(TT_EINVAL, "pooling needs even sizes");
    NN_TRY(check_ptr(x, "x", 2));
    NN_TRY(check_ptr(y, "y", 2));
    NN_TRY(check_chan(c_total, c_off, c, "x"));
    return pool_fwd(x, nbatch, D, H, W, c_total, c_off, c, y, S(stream));
}

int nn_pool_bwd(const uint16_t* x, const uint16_t* gy, int nbatch, int D, int H, int W, int c_total, int c_off, int c,
                uint16_t* gx, int accumulate, void* stream) {
    NN_TRY(check_dims(nbatch, D, H, W));
    if (D % 2 || H % 2 || W % 2) return fail(TT_EINVAL, "pooling needs even sizes");
    NN_TRY(check_ptr(x, "x", 2));
    NN_TRY(check_ptr(gy, "gy", 2));
    NN_TRY(check_ptr(gx, "gx", 2));
    NN_TRY(check_chan(c_total, c_off, c, "x"));
    return pool_bwd(x, gy, nbatch, D, H, W, c_total, c_off, c, gx, accumulate, S(stream));
}

int nn_up_fwd(const uint16_t* x, int nbatch, int D, int H, int W, int cin, const float* Wup, const float* b, int cout,
              uint16_t* y, int cy_total, int cy_off, void* stream) {
    NN_TRY(check_dims(nbatch, D, H, W));
    NN_TRY(check_ptr(x, "x", 2));
    NN_TRY(check_ptr(Wup, "Wup", 4));
    NN_TRY(check_ptr(b, "b", 4));
    NN_TRY(check_ptr(y, "y", 2));
    if (cin < 1 || cout < 1) return fail(TT_EINVAL, "channel counts must be >= 1");
    NN_TRY(check_chan(cy_total, cy_off, cout, "y"));
    return up_fwd(x, nbatch, D, H, W, cin, Wup, b, cout, y, cy_total, cy_off, S(stream));
}

size_t nn_up_wgrad_work(int nbatch, int D, int H, int W, int cin, int cout) {
    if (nbatch < 1 || D < 1 || H < 1 || W < 1 || cin < 1 || cout < 1) return 0;
    return up_work_floats((long long)nbatch * D * H * W, (long long)nbatch * D * H, cin, cout) * sizeof(float);
}

int nn_up_bwd(const uint16_t* x, const uint16_t* gy, int nbatch, int D, int H, int W, int cin, int cout, int cg_total,
              int cg_off, const float* Wup, uint16_t* gx, float* gW, float* gb, float* work, size_t work_bytes,
              void* stream) {
    NN_TRY(check_dims(nbatch, D, H, W));
    NN_TRY(check_ptr(x, "x", 2));
    NN_TRY(check_ptr(gy, "gy", 2));
    NN_TRY(check_ptr(Wup, "Wup", 4));
    NN_TRY(check_ptr(gW, "gW", 4));
    NN_TRY(check_ptr(gb, "gb", 4));
    NN_TRY(check_ptr(work, "work", 4));
    if (cin < 1 || cout < 1 || cout > 64) return fail(TT_EINVAL, "channel counts must be in [1, 64]");
    NN_TRY(check_chan(cg_total, cg_off, cout, "gy"));
    if (work_bytes < nn_up_wgrad_work(nbatch, D, H, W, cin, cout)) return fail(TT_EINVAL, "work too small");
    return up_bwd(x, gy, nbatch, D, H, W, cin, cout, cg_total, cg_off, Wup, gx, gW, gb, work, S(stream));
}

int nn_head_fwd(const uint16_t* x, int64_t npos, int cin, const float* w, const float* b, float* y, void* stream) {
    if (npos < 1 || cin < 1 || cin > 127) return fail(TT_EINVAL, "need npos >= 1 and cin in [1, 127]");
    NN_TRY(check_ptr(x, "x", 2));
    NN_TRY(check_ptr(w, "w", 4));
    NN_TRY(check_ptr(b, "b", 4));
    NN_TRY(check_ptr(y, "y", 4));
    return head_fwd(x, (long long)npos, cin, w, b, y, S(stream));
}

size_t nn_head_work(int64_t npos, int cin) {
    if (npos < 1 || cin < 1) return 0;
    return head_work_floats(npos, cin) * sizeof(float);
}

int nn_head_bwd(const uint16_t* x, const float* gy, int64_t npos, int cin, const float* w, uint16_t* gx, float* gw,
                float* gb, float* work, size_t work_bytes, void* stream) {
    if (npos < 1 || cin < 1 || cin > 127) return fail(TT_EINVAL, "need npos >= 1 and cin in [1, 127]");
    NN_TRY(check_ptr(x, "x", 2));
    NN_TRY(check_ptr(gy, "gy", 4));
    NN_TRY(check_ptr(w, "w", 4));
    NN_TRY(check_ptr(gw, "gw", 4));
    NN_TRY(check_ptr(gb, "gb", 4));
    NN_TRY(check_ptr(work, "work", 4));
    if (work_bytes < nn_head_work(npos, cin)) return fail(TT_EINVAL, "work too small");
    return head_bwd(x, gy, npos, cin, w, gx, gw, gb, work, S(stream));
}

int nn_mse(const float* y, const float* t, const float* mask, int64_t n, float* loss, float* gy, void* stream) {
    if (n < 1) return fail(TT_EINVAL, "n must be >= 1");
    NN_TRY(check_ptr(y, "y", 4));
    NN_TRY(check_ptr(t, "t", 4));
    NN_TRY(check_ptr(loss, "loss", 4));
    NN_TRY(check_ptr(gy, "gy", 4));
    long long nb = (n + 4095) / 4096;  // (65536 a block: 22 blocks and 117 us at 8 x 56^3, 11 us here)
    if (nb > NN_MSE_MAX_BLOCKS) nb = NN_MSE_MAX_BLOCKS;
    const long long chunk = (n + nb - 1) / nb;
    hipStream_t st = S(stream);
    float* part = loss + 2;
    hipLaunchKernelGGL(k_mse_part, dim3((unsigned)nb), dim3(256), 0, st, y, t, mask, (long long)n, chunk, part);
    NN_LAUNCHED();
    hipLaunchKernelGGL(k_mse_final, dim3(1), dim3(256), 0, st, part, (int)nb, loss);
    NN_LAUNCHED();
    hipLaunchKernelGGL(k_mse_grad, dim3(grid_stride_blocks(n)), dim3(256), 0, st, y, t, mask, (long long)n, loss, gy);
    NN_LAUNCHED();
    return TT_OK;
}

int nn_adam(float* p, const float* g, float* m, float* v, int64_t n, int step, float lr, float beta1, float beta2,
            float eps, void* stream) {
    if (n < 1 || step < 1) return fail(TT_EINVAL, "need n >= 1 and step >= 1");
    NN_TRY(check_ptr(p, "p", 4));
    NN_TRY(check_ptr(g, "g", 4));
    NN_TRY(check_ptr(m, "m", 4));
    NN_TRY(check_ptr(v, "v", 4));
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, step)));
    hipLaunchKernelGGL(k_adam, dim3(grid_stride_blocks(n)), dim3(256), 0, S(stream), p, g, m, v, (long long)n, lr,
                       beta1, beta2, eps, c1, c2);
    NN_LAUNCHED();
    return TT_OK;
}

size_t nn_unet_nparams(const nn_unet_cfg* cfg) {
    Net N;
    return make_net(cfg, N) ? 0 : N.nparams;
}

size_t nn_unet_nfrag(const nn_unet_cfg* cfg) {
    Net N;
    return make_net(cfg, N) ? 0 : N.nfrag;
}

size_t nn_unet_workspace(const nn_unet_cfg* cfg, int nbatch, int D, int H, int W, int train) {
    Net N;
    if (make_net(cfg, N) || check_net_dims(nbatch, D, H, W)) return 0;
    Acts A;
    layout(N, nbatch, D, H, W, train, nullptr, A);
    return A.bytes;
}

int nn_unet_pack(const nn_unet_cfg* cfg, const float* params, uint16_t* frag, void* stream) {
    Net N;
    NN_TRY(make_net(cfg, N));
    NN_TRY(check_ptr(params, "params", 4));
    NN_TRY(check_ptr(frag, "frag", 8));
    for (int k = 0; k < NCONV; ++k) {
        const ConvDef& C = N.conv[k];
        NN_TRY(nn_conv3_pack(params + C.w, C.ci, C.co, 0, frag + C.fw, stream));
        if (k != E1A) NN_TRY(nn_conv3_pack(params + C.w, C.ci, C.co, 1, frag + C.fb, stream));
    }
    return TT_OK;
}

int nn_unet_forward(const nn_unet_cfg* cfg, const float* params, const uint16_t* frag, const uint16_t* x, int nbatch,
                    int D, int H, int W, float* y, void* ws, size_t ws_bytes, int train, void* stream) {
    Net N;
    NN_TRY(make_net(cfg, N));
    NN_TRY(check_net_dims(nbatch, D, H, W));
    NN_TRY(check_ptr(params, "params", 4));
    NN_TRY(check_ptr(frag, "frag", 8));
    NN_TRY(check_ptr(x, "x", 8));
    NN_TRY(check_ptr(y, "y", 4));
    NN_TRY(check_ptr(ws, "ws", 256));
    Acts A;
    layout(N, nbatch, D, H, W, train, static_cast<char*>(ws), A);
    if (ws_bytes < A.bytes) return fail(TT_EINVAL, "workspace too small: %zu < %zu", ws_bytes, A.bytes);
    return unet_forward(N, params, frag, x, nbatch, D, H, W, y, A, S(stream));
}

int nn_unet_backward(const nn_unet_cfg* cfg, const float* params, const uint16_t* frag, const uint16_t* x,
                     const float* gy, int nbatch, int D, int H, int W, float* grad, void* ws, size_t ws_bytes,
                     void* stream) {
    Net N;
    NN_TRY(make_net(cfg, N));
    NN_TRY(check_net_dims(nbatch, D, H, W));
    NN_TRY(check_ptr(params, "params", 4));
    NN_TRY(check_ptr(frag, "frag", 8));
    NN_TRY(check_ptr(x, "x", 8));
    NN_TRY(check_ptr(gy, "gy", 4));
    NN_TRY(check_ptr(grad, "grad", 4));
    NN_TRY(check_ptr(ws, "ws", 256));
    Acts A;
    layout(N, nbatch, D, H, W, 1, static_cast<char*>(ws), A);
    if (ws_bytes < A.bytes) return fail(TT_EINVAL, "workspace too small: %zu < %zu", ws_bytes, A.bytes);
    return unet_backward(N, params, frag, gy, x, nbatch, D, H, W, grad, A, S(stream));
}

int nn_warm_features(const tt_grid* grid, const double* s, const double* xi, const double* eta, int32_t nsrc,
                     const double* src_pos, const double* src_par, int32_t stride, int32_t D, int32_t H, int32_t W,
                     uint16_t* feat, void* stream) {
    WarmGrid G;
    NN_TRY(warm_grid(grid, G));
    if (nsrc < 1 || nsrc > 65535) return fail(TT_EINVAL, "nsrc must be in [1, 65535]");
    NN_TRY(check_coarse(grid, stride, D, H, W));
    NN_TRY(check_ptr(s, "s", 8));
    NN_TRY(check_ptr(xi, "xi", 8));
    NN_TRY(check_ptr(eta, "eta", 8));
    NN_TRY(check_ptr(src_pos, "src_pos", 8));
    NN_TRY(check_ptr(src_par, "src_par", 8));
    NN_TRY(check_ptr(feat, "feat", 8));
    unsigned bx = blocks_of((long long)D * H, 4);
    if (bx > 256) bx = 256;
    hipLaunchKernelGGL(k_warm_features, dim3(bx, nsrc), dim3(256), 0, S(stream), G, s, xi, eta, src_pos, src_par,
                       stride, D, H, W, feat);
    NN_LAUNCHED();
    return TT_OK;
}

int nn_warm_target(const tt_grid* grid, int32_t nsrc, const double* tau, int32_t stride, int32_t D, int32_t H,
                   int32_t W, float* target, float* mask, void* stream) {
    WarmGrid G;
    NN_TRY(warm_grid(grid, G));
    if (nsrc < 1 || nsrc > 65535) return fail(TT_EINVAL, "nsrc must be in [1, 65535]");
    NN_TRY(check_coarse(grid, stride, D, H, W));
    NN_TRY(check_ptr(tau, "tau", 8));
    NN_TRY(check_ptr(target, "target", 4));
    const long long npos = (long long)D * H * W;
    unsigned bx = blocks_of(npos, 256);
    if (bx > 4096) bx = 4096;
    hipLaunchKernelGGL(k_warm_target, dim3(bx, nsrc), dim3(256), 0, S(stream), G, tau, stride, D, H, W, target, mask);
    NN_LAUNCHED();
    return TT_OK;
}

int nn_warm_init(const tt_grid* grid, int32_t nsrc, const float* pred, int32_t stride, int32_t D, int32_t H, int32_t W,
                 double* tau_init, void* stream) {
    WarmGrid G;
    NN_TRY(warm_grid(grid, G));
    if (nsrc < 1 || nsrc > 65535) return fail(TT_EINVAL, "nsrc must be in [1, 65535]");
    NN_TRY(check_coarse(grid, stride, D, H, W));
    NN_TRY(check_ptr(pred, "pred", 4));
    NN_TRY(check_ptr(tau_init, "tau_init", 8));
    // waves take rows in runs, and the rows' 64-node pieces one after the other; a few
    // sources get more waves, of shorter runs and a piece each (101^3: 1 source 14.5 to
    // 10.8 us, 2 20.2 to 17.8, 4 31.3 to 28.6; 32 170 in runs of pieces, 176 a piece each)
    const unsigned pieces = nsrc < 8 ? (unsigned)((G.n[2] + 63) / 64) : 1u;
    const unsigned bx = std::min(blocks_of((long long)G.n[0] * G.n[1], 4), std::max(256u, 1024u / (nsrc * pieces)));
    hipLaunchKernelGGL(k_warm_init, dim3(bx, nsrc, pieces), dim3(256), 0, S(stream), G, pred, stride, D, H, W, tau_init);
    NN_LAUNCHED();
    return TT_OK;
}

}  // extern "C"
