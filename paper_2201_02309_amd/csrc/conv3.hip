// 3 x 3 x 3 convolutions of the dual-domain network (Sec. III-A: Conv3D with zero padding 1 and
// at most 16 channels on either side) on the float32 matrix cores of gfx950, with their
// gradients.  Volumes are [batch][depth][channel][height][width] or [batch][channel][depth]
// [height][width] (strides of batch, channel and depth given; rows contiguous).
//
//   k_conv3        y[co] = bias[co] + sum over ci, taps of w[co][ci][tap] x[ci] (forward; with the
//                  weights read transposed and flipped, the gradient with respect to x)
//   k_conv3_wgrad  dw[co][ci][tap] = sum over voxels of dy[co] x[ci] shifted by the tap, db[co] =
//                  sum of dy[co]: per-workgroup partials, then k_conv3_wsum adds them in float64
//                  in a fixed order (bit-reproducible)
//
//   k_prelu_grad   gradients of PReLU with one slope per channel, the layer after each convolution
//
// The convolutions' arithmetic is float32 (v_mfma_f32_16x16x4_f32: products exact to float32 fused into float32
// accumulators).  Bound by the matrix cores: a 16 -> 16 layer takes 13824 flop per voxel against
// 128 bytes; on 1 x 16 x 10 x 512 x 512 (36 Gflop) k_conv3 takes 0.34 ms and k_conv3_wgrad 0.35 ms,
// 105 Tflop/s, where a library float32 matrix product of 8192^3 reached 149 and torch's gradients
// (MIOpen on stacked copies of the input) took 0.6 ms and 1.1 ms with their layout conversions,
// besides the copies.
//
// A workgroup of 4 waves owns a kTH x kTW tile of the (height, width) plane and walks a range of
// depths: three planes of the tile with its one-voxel halo stay in LDS (every channel), the next
// plane's loads are in flight in registers while a plane is computed, so the input comes from
// memory about once.
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace kats {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kCT = 256;                 // threads
constexpr int kTH = 8, kTW = 32;         // tile
constexpr int kPH = kTH + 2, kPW = kTW + 2;
constexpr int kPE = kPH * kPW;           // samples of a channel's tile plane with its halo

// A tile plane's loads in flight: half-wave g takes channels g and g + 8, its lanes the tile's 32
// columns row by row (addresses: one offset per lane, the rest wave-uniform), then one load per
// channel for the halo columns (lane: side + 2 row).  Zero outside the volume.
template <int CH>
struct Plane {
    static constexpr int NC = (CH + 7) / 8;
    float v[NC][kPH], edge[NC];
    __device__ void load(const Conv3Args &a, const float *x, int z, int h0, int w0) {
        const int lane = threadIdx.x & 31, g = threadIdx.x >> 5;
        const bool zin = (unsigned)z < (unsigned)a.D;
        const float *xz = x + (long long)z * a.xd;
        const int side = lane & 1, er = lane >> 1;
        const bool win = w0 + lane < a.W;
        const int ew = side ? w0 + kTW : w0 - 1;
        const bool ein = er < kPH && (unsigned)(h0 - 1 + er) < (unsigned)a.H && (unsigned)ew < (unsigned)a.W;
        const unsigned at = (unsigned)g * (unsigned)a.xc + (unsigned)(w0 + lane);
        const unsigned eat = (unsigned)g * (unsigned)a.xc + (unsigned)(h0 - 1 + er) * (unsigned)a.W + (unsigned)ew;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const bool cin = zin && g + 8 * c < a.cin;
            const float *xc = xz + 8ll * c * a.xc;
#pragma unroll
            for (int r = 0; r < kPH; ++r) {
                const int h = h0 - 1 + r;
                v[c][r] = 0.0f;
                if ((unsigned)h < (unsigned)a.H && cin && win) v[c][r] = (xc + (long long)h * a.W)[at];
            }
            edge[c] = cin && ein ? xc[eat] : 0.0f;
        }
    }
    template <int CS>
    __device__ void store(float *lds) const {
        const int lane = threadIdx.x & 31, g = threadIdx.x >> 5;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (g + 8 * c < CH) {
                float *p = lds + (g + 8 * c) * CS;
#pragma unroll
                for (int r = 0; r < kPH; ++r) p[r * kPW + 1 + lane] = v[c][r];
                if ((lane >> 1) < kPH) p[(lane >> 1) * kPW + (lane & 1) * (kTW + 1)] = edge[c];
            }
    }
};

// Wave w computes rows 4 (w / 2) .. + 3 of columns 16 (w % 2) .. + 15: four 16 x 16 (output
// channel x column) accumulators.  Every weight sits in a register of its lane for the whole walk
// (27 taps x KK groups of 4 input channels); a row's samples serve the three taps that reach it
// (18 LDS reads for 36 matrix instructions).  CS = 48 (mod 64): the four channel groups of a wave's
// read lie in different banks.
template <int KK>
__global__ __launch_bounds__(kCT, 2) void k_conv3(Conv3Args a) {
    constexpr int CH = 4 * KK, CS = 368;
    static_assert(CS >= kPE, "channel stride");
    __shared__ float lds[3][CH * CS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n16 = lane & 15, k4 = lane >> 4;
    const int h0 = (blockIdx.x / a.tiles_w) * kTH, w0 = (blockIdx.x % a.tiles_w) * kTW;
    const int z0 = blockIdx.y * a.dseg, z1 = min(z0 + a.dseg, a.D);
    const float *x = a.x + blockIdx.z * a.xb;
    float *y = a.y + blockIdx.z * a.yb;

    float wr[27][KK];
#pragma unroll
    for (int t = 0; t < 27; ++t)
#pragma unroll
        for (int k = 0; k < KK; ++k) {
            const int ci = 4 * k + k4;
            wr[t][k] = ci < a.cin && n16 < a.cout ? a.w[n16 * a.wm + ci * a.wk + (a.flip ? 26 - t : t)] : 0.0f;
        }
    f32x4 bias = {0.0f, 0.0f, 0.0f, 0.0f};
    if (a.bias)
#pragma unroll
        for (int i = 0; i < 4; ++i) bias[i] = 4 * k4 + i < a.cout ? a.bias[4 * k4 + i] : 0.0f;

    Plane<CH> pl;
    for (int j = 0; j < 3; ++j) {
        pl.load(a, x, z0 - 1 + j, h0, w0);
        pl.template store<CS>(lds[j]);
    }
    __syncthreads();
    const int rows = 4 * (wave >> 1), col = 16 * (wave & 1) + n16;
    const int at = k4 * CS + rows * kPW + col;
    int s0 = 0, s1 = 1, s2 = 2;              // LDS planes of depths z - 1, z, z + 1
    for (int z = z0; z < z1; ++z) {
        const bool more = z + 1 < z1;
        if (more) pl.load(a, x, z + 2, h0, w0);
        f32x4 acc[4];
#pragma unroll
        for (int kd = 0; kd < 3; ++kd) {
            // each depth's taps are summed by themselves: shorter chains of roundings
            f32x4 part[4] = {};
            const float *L = &lds[kd == 0 ? s0 : (kd == 1 ? s1 : s2)][at];
#pragma unroll
            for (int k = 0; k < KK; ++k)
#pragma unroll
                for (int kw = 0; kw < 3; ++kw) {
                    float b[6];
#pragma unroll
                    for (int r = 0; r < 6; ++r) b[r] = L[4 * k * CS + r * kPW + kw];
#pragma unroll
                    for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            part[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr[9 * kd + 3 * kh + kw][k], b[r + kh],
                                                                           part[r], 0, 0, 0);
                }
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = kd ? acc[r] + part[r] : part[r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] += bias;
        // accumulator i of a lane: output channel 4 (lane / 16) + i, column lane % 16
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int h = h0 + rows + r, w = w0 + col;
            if (h < a.H && w < a.W)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int co = 4 * k4 + i;
                    if (co < a.cout) (y + z * a.yd + (long long)h * a.W)[(unsigned)co * (unsigned)a.yc + (unsigned)w] = acc[r][i];
                }
        }
        if (more) {
            __syncthreads();
            pl.template store<CS>(lds[s0]);
            const int s = s0;
            s0 = s1;
            s1 = s2;
            s2 = s;
            __syncthreads();
        }
    }
}

// Weight gradient.  Wave w takes the columns 4 w .. + 3 and 16 + 4 w .. + 3 of the tile, all its
// rows: the four columns are the K of a 16 x 16 x 4 product dy^T x per tap, 27 accumulators of
// (output channel x input channel).  dy comes straight from memory (one load per 27 products), x
// from the LDS planes (a row's samples serve three taps).  CS = 4 (mod 64): a wave reads 16
// channels x 4 columns from different banks.  Workgroups are persistent over (tile, depth range)
// tasks; a wave's sums are float32, the workgroup's four are added in LDS, the workgroups' in float64.
// The bias gradient may cancel to nothing: it is summed in float64 throughout, its partials stored
// whole, as the words of a double (a float and its remainder would turn an infinity into a NaN).
// Past the volume's edges dy is taken as 0, and so has to be the x it meets: the last row and column are
// neighbours of such samples, and 0 times a value that is not finite is no 0.  RW, RH: the width, the
// height is no multiple of the tile's.  A lane in the column past the edge then reads the zeros beside
// its own, a row past it takes a select.  16 -> 16 channels, without / with, us: 586 x 16 x 627 (RW)
// 839 / 848, 10 x 300 x 300 (both) 157.6 / 160.4; 10 x 512 x 512, which needs neither, 387.
template <bool RH, bool RW>
__global__ __launch_bounds__(kCT, 2) void k_conv3_wgrad(Conv3Args a, const float *__restrict__ dy,
                                                        float *__restrict__ part) {
    constexpr int CH = 16, CS = 388;
    static_assert(CS >= kPE && 3 * CH * CS >= kConv3Part, "LDS planes");
    __shared__ float lds[3 * CH * CS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n16 = lane & 15, k4 = lane >> 4;
    f32x4 acc[27];
#pragma unroll
    for (int t = 0; t < 27; ++t) acc[t] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
    double db = 0.0;
    const int plane_tiles = a.tiles_w * a.tiles_h, tasks = plane_tiles * a.nseg * a.B;
    for (int task = blockIdx.x; task < tasks; task += gridDim.x) {
        const int tile = task % plane_tiles, rest = task / plane_tiles;
        const int z0 = (rest % a.nseg) * a.dseg, z1 = min(z0 + a.dseg, a.D);
        const int h0 = (tile / a.tiles_w) * kTH, w0 = (tile % a.tiles_w) * kTW;
        const float *x = a.x + (rest / a.nseg) * a.xb;
        const float *g = dy + (rest / a.nseg) * a.yb;
        Plane<CH> pl;
        __syncthreads();                       // the previous task's planes are read
        for (int j = 0; j < 3; ++j) {
            pl.load(a, x, z0 - 1 + j, h0, w0);
            pl.template store<CS>(lds + j * CH * CS);
        }
        __syncthreads();
        int s0 = 0, s1 = 1, s2 = 2;
        for (int z = z0; z < z1; ++z) {
            const bool more = z + 1 < z1;
            if (more) pl.load(a, x, z + 2, h0, w0);
#pragma unroll 1
            for (int half = 0; half < 2; ++half) {
                const int col = 16 * half + 4 * wave + k4;
                const bool win = w0 + col < a.W;
                const int left = !RW || win ? 0 : 1;
                float gy[kTH];
#pragma unroll
                for (int r = 0; r < kTH; ++r) {
                    const int h = h0 + r, w = w0 + col;
                    gy[r] = 0.0f;
                    if (h < a.H && n16 < a.cout && win) gy[r] = (g + z * a.yd + (long long)h * a.W)[(unsigned)n16 * (unsigned)a.yc + (unsigned)w];
                    db += gy[r];
                }
#pragma unroll
                for (int kd = 0; kd < 3; ++kd) {
                    const float *L = lds + (kd == 0 ? s0 : (kd == 1 ? s1 : s2)) * CH * CS + n16 * CS + col;
#pragma unroll
                    for (int kw = 0; kw < 3; ++kw) {
                        float b[kPH];
#pragma unroll
                        for (int r = 0; r < kPH; ++r) b[r] = L[r * kPW + (kw ? kw : left)];
#pragma unroll
                        for (int r = 0; r < kTH; ++r)
#pragma unroll
                            for (int kh = 0; kh < 3; ++kh) {
                                const float xv = RH && kh == 0 && r > 0 ? (h0 + r < a.H ? b[r] : 0.0f) : b[r + kh];
                                acc[9 * kd + 3 * kh + kw] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    gy[r], xv, acc[9 * kd + 3 * kh + kw], 0, 0, 0);
                            }
                    }
                }
            }
            if (more) {
                __syncthreads();
                pl.template store<CS>(lds + s0 * CH * CS);
                const int s = s0;
                s0 = s1;
                s1 = s2;
                s2 = s;
                __syncthreads();
            }
        }
    }
    // the four waves' sums, in order, then this workgroup's partial: [tap][co][ci], db[co]
    __shared__ double dbs[16];
    for (int o = 16; o < 64; o <<= 1) db += __shfl_xor(db, o, 64);
    for (int w = 0; w < 4; ++w) {
        __syncthreads();
        if (wave != w) continue;
#pragma unroll
        for (int t = 0; t < 27; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float *s = lds + t * 256 + (4 * k4 + i) * 16 + n16;
                *s = w ? *s + acc[t][i] : acc[t][i];
            }
        if (lane < 16) {
            dbs[lane] = w ? dbs[lane] + db : db;
            lds[27 * 256 + lane] = __int_as_float(__double2hiint(dbs[lane]));
            lds[27 * 256 + 16 + lane] = __int_as_float(__double2loint(dbs[lane]));
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kConv3Part; e += kCT) part[(size_t)blockIdx.x * kConv3Part + e] = lds[e];
}

// dw[co][ci][tap] and db[co] = sums of the workgroups' partials: 16 elements per block (the bias's 16
// pairs in the last), 16 threads each taking every 16th partial in float64.
__global__ __launch_bounds__(kCT) void k_conv3_wsum(const float *__restrict__ part, int np, int cin, int cout,
                                                    float *__restrict__ dw, float *__restrict__ db) {
    __shared__ double sh[16][17];
    const int j = threadIdx.x & 15, g = threadIdx.x >> 4;
    const int e = blockIdx.x * 16 + j;
    double s = 0.0;
    if (e < 27 * 256) {
#pragma unroll 8
        for (int p = g; p < np; p += 16) s += (double)part[(size_t)p * kConv3Part + e];
    } else {
#pragma unroll 8
        for (int p = g; p < np; p += 16) {
            const float *h = part + (size_t)p * kConv3Part + e;
            s += __hiloint2double(__float_as_int(h[0]), __float_as_int(h[16]));
        }
    }
    sh[g][j] = s;
    __syncthreads();
    if (g != 0) return;
    for (int q = 1; q < 16; ++q) s += sh[q][j];
    if (e >= 27 * 256) {
        if (db && e - 27 * 256 < cout) db[e - 27 * 256] = (float)s;
        return;
    }
    const int t = e >> 8, co = (e >> 4) & 15, ci = e & 15;
    if (dw && co < cout && ci < cin) dw[(co * cin + ci) * 27 + t] = (float)s;
}

// PReLU gradient: dx = x > 0 ? dy : slope[c] dy, and the sum of x dy over a channel's x <= 0.  A
// block takes kPreluBlock samples of one (batch, depth, channel) plane; its sum
// (float64) is one partial, added per channel in a fixed order by
// k_prelu_sum.  Streams at the memory's rate: 91 us for the 1 x 16 x 10 x 512 x 512 layer (0.50 GB),
// where torch's kernel took 2.4 ms on the convolutions' [depth][channel] layout.
template <bool VEC>
__global__ __launch_bounds__(kCT) void k_prelu_grad(PreluArgs a, double *__restrict__ part) {
    __shared__ double sh[kCT / 64];
    const int plane = blockIdx.x / a.chunks, chunk = blockIdx.x - plane * a.chunks;
    const int c = plane % a.C, rest = plane / a.C;
    const int d = rest % a.D, b = rest / a.D;
    const float *x = a.x + b * a.xs[0] + c * a.xs[1] + d * a.xs[2];
    const float *g = a.dy + b * a.gs[0] + c * a.gs[1] + d * a.gs[2];
    float *o = a.dx + b * a.os[0] + c * a.os[1] + d * a.os[2];
    const float w = a.slope[c];
    double sum = 0.0;
    const long long e0 = (long long)chunk * kPreluBlock, e1 = min(e0 + kPreluBlock, a.n);
    auto one = [&](float xv, float gv) {
        // (no product where x > 0: an infinite cotangent times 0 would be a NaN)
        const bool on = xv > 0.0f;
        sum = on ? sum : fma((double)xv, (double)gv, sum);
        return on ? gv : w * gv;
    };
    if (VEC) {
#pragma unroll 4
        for (long long e = e0 + 4 * threadIdx.x; e < e1; e += 4 * kCT) {
            const float4 xv = *reinterpret_cast<const float4 *>(x + e), gv = *reinterpret_cast<const float4 *>(g + e);
            *reinterpret_cast<float4 *>(o + e) =
                make_float4(one(xv.x, gv.x), one(xv.y, gv.y), one(xv.z, gv.z), one(xv.w, gv.w));
        }
    } else {
#pragma unroll 8
        for (long long e = e0 + threadIdx.x; e < e1; e += kCT) o[e] = one(x[e], g[e]);
    }
    for (int q = 32; q > 0; q >>= 1) sum += __shfl_xor(sum, q, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

// one block per channel
__global__ __launch_bounds__(kCT) void k_prelu_sum(const double *__restrict__ part, int planes, int C, int chunks,
                                                   float *__restrict__ dslope) {
    __shared__ double sh[kCT / 64];
    double s = 0.0;
    const int n = planes / C * chunks;
    for (int i = threadIdx.x; i < n; i += kCT)
        s += part[((size_t)(i / chunks) * C + blockIdx.x) * chunks + i % chunks];
    for (int q = 32; q > 0; q >>= 1) s += __shfl_xor(s, q, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) dslope[blockIdx.x] = (float)(sh[0] + sh[1] + sh[2] + sh[3]);
}

// The three depth-shifted copies of x [B][C][D] side by side as channels, [B][D][3 C] dense planes of
// n samples: every plane is read once and written to the (at most) three depths that see it, and
// the two ends' missing depths are zeros.  The memory bounds it: 16 channels of 10 x 512 x 512 take
// 125 us (671 MB, 5.4 TB/s); padding, joining and reordering by torch's operators moved 2.3 GB for the
// same copies, 420 us a layer.
// V: samples per access.
template <int V>
__global__ __launch_bounds__(kCT) void k_stack3(Stack3Args a) {
    typedef float FV __attribute__((ext_vector_type(V)));
    const int plane = blockIdx.x;
    const int c = plane % a.C, rest = plane / a.C;
    const int d = rest % a.D, b = rest / a.D;
    const FV *x = reinterpret_cast<const FV *>(a.x + b * a.xs[0] + c * a.xs[1] + d * a.xs[2]);
    const long long depth = 3ll * a.C * a.n;                    // one output depth
    float *o = a.out + ((long long)b * a.D + d) * depth + (long long)c * a.n;
    // depth d sees this plane as its middle copy, d + 1 as its first, d - 1 as its last
    FV *mid = reinterpret_cast<FV *>(o + (long long)a.C * a.n);
    FV *first = reinterpret_cast<FV *>(d + 1 < a.D ? o + depth : o + 2ll * a.C * a.n);
    FV *last = reinterpret_cast<FV *>(d > 0 ? o - depth + 2ll * a.C * a.n : o);
    const bool in1 = d + 1 < a.D, in0 = d > 0;                  // otherwise: the end's zeros
    const FV zero = {};
    const long long m = a.n / V, step = (long long)gridDim.y * kCT;
#pragma unroll 4
    for (long long e = (long long)blockIdx.y * kCT + threadIdx.x; e < m; e += step) {
        const FV v = x[e];
        mid[e] = v;
        first[e] = in1 ? v : zero;
        last[e] = in0 ? v : zero;
    }
}

// Tiles and depth ranges: enough workgroups to fill the GPU twice over (two per CU), ranges not
// shorter than 4 depths (each re-reads two planes).
void split(Conv3Args &a) {
    a.tiles_w = (a.W + kTW - 1) / kTW;
    a.tiles_h = (a.H + kTH - 1) / kTH;
    const long long tiles = (long long)a.tiles_w * a.tiles_h * a.B;
    long long n = (1024 + tiles - 1) / tiles;
    const long long most = (a.D + 3) / 4;
    n = n < 1 ? 1 : (n > most ? most : n);
    a.dseg = (int)((a.D + n - 1) / n);
    a.nseg = (a.D + a.dseg - 1) / a.dseg;
}

}  // namespace

hipError_t launch_conv3(Conv3Args a, hipStream_t s) {
    split(a);
    const dim3 grid((unsigned)(a.tiles_w * a.tiles_h), (unsigned)a.nseg, (unsigned)a.B);
    switch ((a.cin + 3) / 4) {
        case 1: hipLaunchKernelGGL(k_conv3<1>, grid, dim3(kCT), 0, s, a); break;
        case 2: hipLaunchKernelGGL(k_conv3<2>, grid, dim3(kCT), 0, s, a); break;
        case 3: hipLaunchKernelGGL(k_conv3<3>, grid, dim3(kCT), 0, s, a); break;
        default: hipLaunchKernelGGL(k_conv3<4>, grid, dim3(kCT), 0, s, a); break;
    }
    return hipGetLastError();
}

hipError_t launch_conv3_wgrad(Conv3Args a, const float *dy, float *dw, float *db, float *part, hipStream_t s) {
    split(a);
    const long long tasks = (long long)a.tiles_w * a.tiles_h * a.nseg * a.B;
    const int blocks = (int)(tasks < kConv3Blocks ? tasks : kConv3Blocks);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kCT), 0, s, a, dy, part); };
    if (a.H % kTH) a.W % kTW ? go(k_conv3_wgrad<true, true>) : go(k_conv3_wgrad<true, false>);
    else a.W % kTW ? go(k_conv3_wgrad<false, true>) : go(k_conv3_wgrad<false, false>);
    hipLaunchKernelGGL(k_conv3_wsum, dim3(27 * 16 + 1), dim3(kCT), 0, s, (const float *)part, blocks, a.cin,
                       a.cout, dw, db);
    return hipGetLastError();
}

hipError_t launch_stack3(const Stack3Args &a, hipStream_t s) {
    // 16-byte accesses need every plane of both tensors on a 16-byte boundary
    const bool vec = ((a.n | a.xs[0] | a.xs[1] | a.xs[2]) & 3) == 0 && (((uintptr_t)a.x | (uintptr_t)a.out) & 15) == 0;
    const long long per = kCT * 4 * (vec ? 4 : 1);              // a block's samples in four accesses
    const long long chunks = (a.n + per - 1) / per;
    const dim3 grid((unsigned)(a.B * a.D * a.C), (unsigned)(chunks < 65535 ? chunks : 65535));
    if (vec)
        hipLaunchKernelGGL(k_stack3<4>, grid, dim3(kCT), 0, s, a);
    else
        hipLaunchKernelGGL(k_stack3<1>, grid, dim3(kCT), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_prelu_grad(PreluArgs a, float *dslope, double *part, hipStream_t s) {
    const int planes = a.B * a.D * a.C;
    a.chunks = (int)((a.n + kPreluBlock - 1) / kPreluBlock);
    // 16-byte loads need every plane of the three tensors on a 16-byte boundary
    long long any = a.n | (long long)(((uintptr_t)a.x | (uintptr_t)a.dy | (uintptr_t)a.dx) >> 2);
    for (int i = 0; i < 3; ++i) any |= a.xs[i] | a.gs[i] | a.os[i];
    if ((any & 3) == 0)
        hipLaunchKernelGGL(k_prelu_grad<true>, dim3(planes * a.chunks), dim3(kCT), 0, s, a, part);
    else
        hipLaunchKernelGGL(k_prelu_grad<false>, dim3(planes * a.chunks), dim3(kCT), 0, s, a, part);
    hipLaunchKernelGGL(k_prelu_sum, dim3(a.C), dim3(kCT), 0, s, (const double *)part, planes, a.C, a.chunks, dslope);
    return hipGetLastError();
}

}  // namespace kats
