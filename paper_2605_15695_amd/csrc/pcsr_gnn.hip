// Dense side of a GNN layer on fp32 matrix instructions (see pcsr_gnn.h).
//
// v_mfma_f32_16x16x4_f32: lane l holds A[i = l%16][k = l/16] and B[k = l/16][j = l%16]; the
// result register r of lane l is D[i = 4*(l/16) + r][j = l%16].  The order of k is free as long
// as A and B agree, which is what both kernels use to load 16 bytes per lane.
#include "pcsr_gnn.h"

#include <hip/hip_runtime.h>

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

constexpr int kWaves = 4;
constexpr int kLinearBlocks = 2048;
constexpr int kWgradBlocks = 512;
constexpr int kColsumBlocks = 512;

struct LinearArgs {
    long n;
    int a, b, w_transposed, relu;
    const float *X, *W, *bias, *mask, *aux;
    float *Y;
    float *ws_colsum; // one row of b per workgroup
    float *ws_dot;    // one value per workgroup
};

// A wavefront takes 32 rows of X at a time (16 where their registers would leave a SIMD with
// one wavefront).  D = op(W)-tile (16 outputs) x X^T (16 rows): a
// lane reads 16 bytes of one row per 16 inputs (component s of lane l is k = 4*(l/16) + s)
// and ends up with four consecutive outputs of one row, so loads and stores are 64-byte pieces of
// rows and X never goes through LDS; the weight fragments do (16 KB for 64 x 64), read as
// one ds_read_b128 per 4 matrix instructions.  Bound by memory: 2,000,000 x 64 -> 64 is 1.02 GB
// and 16.4 GFLOP (104 us at the fp32 matrix peak); measured 245 us without a mask, where the
// vendor GEMM took 290-320 us and left bias, ReLU and mask to passes of 150-230 us each.
// VEC: widths are multiples of 4 and the arrays 16-byte aligned.  RED: dot and/or column sums.
template <int KT, int NT, bool VEC, bool RED>
__global__ void __launch_bounds__(64 * kWaves, KT *NT <= 16 ? (RED ? 3 : 4) : 2) linear_kernel(LinearArgs p)
{
    constexpr int H = KT + NT >= 10 ? 1 : 2; // 16-row pieces per step
    __shared__ f4 wfrag[KT * NT * 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, q = lane >> 4;
    for (int f = tid; f < KT * NT * 64; f += 64 * kWaves) {
        const int l = f & 63, t = f >> 6, kt = t / NT, nt = t - kt * NT;
        const int out = nt * 16 + (l & 15), in0 = kt * 16 + 4 * (l >> 4);
        f4 w = {0.0f, 0.0f, 0.0f, 0.0f};
        if (out < p.b) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (in0 + s < p.a)
                    w[s] = p.w_transposed ? p.W[(long)(in0 + s) * p.b + out] : p.W[(long)out * p.a + in0 + s];
        }
        wfrag[f] = w;
    }
    f4 bias[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int o = nt * 16 + 4 * q + s;
            bias[nt][s] = (p.bias && o < p.b) ? p.bias[o] : 0.0f;
        }
    __syncthreads();

    f4 csum[RED ? NT : 1];
    float dot = 0.0f;
    if constexpr (RED) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) csum[nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    const long groups = (p.n + 16 * H - 1) / (16 * H);
    for (long g = (long)blockIdx.x * kWaves + wave; g < groups; g += (long)gridDim.x * kWaves) {
        // keeps the weight fragments in LDS: hoisted out of the loop they would fill the registers
        asm volatile("" ::: "memory");
        f4 x[H][KT];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            long row = (g * H + h) * 16 + r;
            row = row < p.n ? row : p.n - 1; // results of the rows past the end are dropped below
            const float *xr = p.X + row * p.a;
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) {
                const int c = kt * 16 + 4 * q;
                if constexpr (VEC) {
                    x[h][kt] = c < p.a ? *reinterpret_cast<const f4 *>(xr + c) : f4{0.0f, 0.0f, 0.0f, 0.0f};
                } else {
#pragma unroll
                    for (int s = 0; s < 4; ++s) x[h][kt][s] = c + s < p.a ? xr[c + s] : 0.0f;
                }
            }
        }
        f4 acc[H][NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int h = 0; h < H; ++h) acc[h][nt] = bias[nt];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const f4 w = wfrag[(kt * NT + nt) * 64 + lane];
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int h = 0; h < H; ++h) acc[h][nt] = mfma4(w[s], x[h][kt][s], acc[h][nt]);
            }
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const long row = (g * H + h) * 16 + r;
            if (row >= p.n) continue;
            const long at = row * p.b;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int c = nt * 16 + 4 * q;
                f4 v = acc[h][nt];
                if (p.relu) {
#pragma unroll
                    for (int s = 0; s < 4; ++s) v[s] = v[s] <= 0.0f ? 0.0f : v[s];
                }
                if constexpr (VEC) {
                    if (c < p.b) {
                        if constexpr (RED) {
                            if (p.aux) {
                                const f4 u = *reinterpret_cast<const f4 *>(p.aux + at + c);
                                dot += (v[0] * u[0] + v[1] * u[1]) + (v[2] * u[2] + v[3] * u[3]);
                            }
                        }
                        if (p.mask) {
                            const f4 m = *reinterpret_cast<const f4 *>(p.mask + at + c);
#pragma unroll
                            for (int s = 0; s < 4; ++s) v[s] = m[s] <= 0.0f ? 0.0f : v[s];
                        }
                        if constexpr (RED) csum[nt] += v;
                        if (p.Y) *reinterpret_cast<f4 *>(p.Y + at + c) = v;
                    }
                } else {
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        if (c + s < p.b) {
                            float e = v[s];
                            if constexpr (RED) {
                                if (p.aux) dot += e * p.aux[at + c + s];
                            }
                            if (p.mask && p.mask[at + c + s] <= 0.0f) e = 0.0f;
                            if constexpr (RED) csum[nt][s] += e;
                            if (p.Y) p.Y[at + c + s] = e;
                        }
                }
            }
        }
    }

    if constexpr (RED) {
        // the 16 row lanes, then the 4 wavefronts; fixed order, so the same bits on every run
        __syncthreads(); // the weight fragments are no longer read: their space is used again
        auto csh = reinterpret_cast<f4(*)[NT * 4]>(wfrag); // [kWaves], a quarter of it at most
        auto dsh = reinterpret_cast<float *>(wfrag + kWaves * NT * 4);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int m = 1; m < 16; m <<= 1) csum[nt][s] += __shfl_xor(csum[nt][s], m);
            if (r == 0) csh[wave][nt * 4 + q] = csum[nt];
        }
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) dot += __shfl_xor(dot, m);
        if (lane == 0) dsh[wave] = dot;
        __syncthreads();
        if (p.ws_colsum) {
            for (int c = tid; c < p.b; c += 64 * kWaves) {
                float t = 0.0f;
                for (int w = 0; w < kWaves; ++w) t += csh[w][c >> 2][c & 3];
                p.ws_colsum[(long)blockIdx.x * p.b + c] = t;
            }
        }
        if (p.ws_dot && tid == 0) p.ws_dot[blockIdx.x] = (dsh[0] + dsh[1]) + (dsh[2] + dsh[3]);
    }
}

struct WgradArgs {
    long n;
    int a, b;
    const float *G, *X;
    float *ws; // per workgroup of grid.x: b*a of dW, then b column sums
    int sums;
};

// dW = G^T X: the rows are the k of the matrix instruction, four per instruction.  With VG / VX
// a lane's 16-byte load of a row (columns T*(l%16) ...) feeds T tiles at once: tile t holds
// the columns T*i + t.  A workgroup keeps up to 64 x 64 of dW in its accumulators and walks
// 16 rows per wavefront and step, the next step's rows being loaded meanwhile; wider weights
// are cut into such squares by grid.y / grid.z.  Rows are dealt to about 2000 wavefronts,
// each leaves one partial dW, summed by sum_partials_kernel in a fixed order.
// 2,000,000 rows, 64 x 64: 197 us (5.2 TB/s of G and X) + 16 us for the sums; the vendor GEMM,
// which splits this shape over too few workgroups, took 2900 us.
template <int TG, bool VG, int TX, bool VX>
__global__ void __launch_bounds__(64 * kWaves) wgrad_kernel(WgradArgs p)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, q = lane >> 4;
    const int g0 = blockIdx.y * TG * 16, x0 = blockIdx.z * TX * 16;

    f4 acc[TG][TX];
    float gsum[TG];
#pragma unroll
    for (int i = 0; i < TG; ++i) {
        gsum[i] = 0.0f;
#pragma unroll
        for (int j = 0; j < TX; ++j) acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    auto load = [&](const float *base, int width, int off, long row, auto t_const, auto vec_const, float *d) {
        constexpr int T = decltype(t_const)::value;
        constexpr bool V = decltype(vec_const)::value;
        const bool ok = row < p.n;
        const float *src = base + row * width;
        if constexpr (V && T == 4) {
            const int col = off + 4 * c;
            f4 t = {0.0f, 0.0f, 0.0f, 0.0f};
            if (ok && col < width) t = *reinterpret_cast<const f4 *>(src + col);
#pragma unroll
            for (int s = 0; s < 4; ++s) d[s] = t[s];
        } else if constexpr (V && T == 2) {
            const int col = off + 2 * c;
            float2 t = make_float2(0.0f, 0.0f);
            if (ok && col < width) t = *reinterpret_cast<const float2 *>(src + col);
            d[0] = t.x;
            d[1] = t.y;
        } else {
#pragma unroll
            for (int s = 0; s < T; ++s) {
                const int col = off + 16 * s + c;
                d[s] = (ok && col < width) ? src[col] : 0.0f;
            }
        }
    };
    constexpr int U = 4; // 4 x 4 rows per step
    float gn[U][TG], xn[U][TX];
    auto fetch = [&](long row0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            load(p.G, p.b, g0, row0 + 4 * u + q, std::integral_constant<int, TG>{}, std::integral_constant<bool, VG>{},
                 gn[u]);
            load(p.X, p.a, x0, row0 + 4 * u + q, std::integral_constant<int, TX>{}, std::integral_constant<bool, VX>{},
                 xn[u]);
        }
    };
    const long step = (long)gridDim.x * kWaves * 4 * U;
    long row0 = ((long)blockIdx.x * kWaves + wave) * 4 * U;
    fetch(row0);
    for (; row0 < p.n; row0 += step) {
        float g[U][TG], x[U][TX];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int i = 0; i < TG; ++i) g[u][i] = gn[u][i];
#pragma unroll
            for (int j = 0; j < TX; ++j) x[u][j] = xn[u][j];
        }
        fetch(row0 + step);
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int i = 0; i < TG; ++i) {
                gsum[i] += g[u][i];
#pragma unroll
                for (int j = 0; j < TX; ++j) acc[i][j] = mfma4(g[u][i], x[u][j], acc[i][j]);
            }
        }
    }

    // the four wavefronts of the workgroup, in order
    __shared__ float red[TG * 16][TX * 16 + 1];
    __shared__ float gred[TG * 16];
    auto gcol = [](int i, int t) { return VG ? i * TG + t : t * 16 + i; };
    auto xcol = [](int j, int t) { return VX ? j * TX + t : t * 16 + j; };
#pragma unroll
    for (int i = 0; i < TG; ++i) {
        gsum[i] += __shfl_xor(gsum[i], 16);
        gsum[i] += __shfl_xor(gsum[i], 32);
    }
    for (int w = 0; w < kWaves; ++w) {
        if (wave == w) {
#pragma unroll
            for (int i = 0; i < TG; ++i) {
#pragma unroll
                for (int j = 0; j < TX; ++j)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        float &d = red[gcol(4 * q + s, i)][xcol(c, j)];
                        d = w ? d + acc[i][j][s] : acc[i][j][s];
                    }
                if (q == 0) {
                    float &d = gred[gcol(c, i)];
                    d = w ? d + gsum[i] : gsum[i];
                }
            }
        }
        __syncthreads();
    }
    float *out = p.ws + (long)blockIdx.x * ((long)p.b * p.a + p.b);
    for (int e = tid; e < TG * TX * 256; e += 64 * kWaves) {
        const int i = e / (TX * 16), j = e - i * (TX * 16);
        if (g0 + i < p.b && x0 + j < p.a) out[(long)(g0 + i) * p.a + x0 + j] = red[i][j];
    }
    if (p.sums && blockIdx.z == 0 && tid < TG * 16 && g0 + tid < p.b) out[(long)p.b * p.a + g0 + tid] = gred[tid];
}

// out[e] = sum over the parts of ws[part*len + e] for e < n0 (dst0), then dst1: 16 threads per
// element, each every 16th part in order, the 16 sums in order.
__global__ void __launch_bounds__(256) sum_partials_kernel(const float *ws, int parts, long stride, long n0, float *dst0,
                                                           long n1, float *dst1)
{
    __shared__ float sh[16][17];
    const int c = threadIdx.x & 15, j = threadIdx.x >> 4;
    const long e = (long)blockIdx.x * 16 + c;
    float t = 0.0f;
    if (e < n0 + n1)
        for (int s = j; s < parts; s += 16) t += ws[s * stride + e];
    sh[j][c] = t;
    __syncthreads();
    if (j == 0 && e < n0 + n1) {
        for (int k = 1; k < 16; ++k) t += sh[k][c];
        if (e < n0)
            dst0[e] = t;
        else
            dst1[e - n0] = t;
    }
}

// Column sums: 256 threads read consecutive elements of whole rows; a thread's column repeats
// every b / gcd(b, 256) steps, so widths up to 256 are taken with floor(256/b) rows per pass.
__global__ void __launch_bounds__(256) colsum_kernel(long n, int b, const float *G, float *ws)
{
    __shared__ float sh[256];
    const int rows = 256 / b;
    const int c = threadIdx.x % b, r = threadIdx.x / b;
    float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (r < rows) {
        const long step = (long)gridDim.x * rows;
        long row = (long)blockIdx.x * rows + r;
        for (; row + 3 * step < n; row += 4 * step)
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] += G[(row + u * step) * b + c];
        for (; row < n; row += step) t[0] += G[row * b + c];
    }
    sh[threadIdx.x] = (t[0] + t[1]) + (t[2] + t[3]);
    __syncthreads();
    if (threadIdx.x < b) {
        float s = 0.0f;
        for (int k = 0; k < rows; ++k) s += sh[k * b + threadIdx.x];
        ws[(long)blockIdx.x * b + threadIdx.x] = s;
    }
}

int to_code(hipError_t e) { return e == hipSuccess ? PCSR_OK : PCSR_E_HIP; }

int sum_partials(const float *ws, int parts, long stride, long n0, float *dst0, long n1, float *dst1, hipStream_t s)
{
    const long blocks = (n0 + n1 + 15) / 16;
    hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)blocks), dim3(256), 0, s, ws, parts, stride, n0, dst0, n1,
                       dst1);
    return to_code(hipGetLastError());
}

using LinearFn = void (*)(LinearArgs);
// tiles of 16 a width is rounded up to
int tiles(int w, bool vec)
{
    const int t = (w + 15) / 16;
    if (t <= 2) return t;
    if (t == 3) return vec ? 3 : 4;
    if (t == 4) return 4;
    if (t <= 6) return vec ? 6 : 8;
    return 8;
}
template <int KT, int NT> LinearFn pick_linear(bool vec, bool red)
{
    if (vec) return red ? &linear_kernel<KT, NT, true, true> : &linear_kernel<KT, NT, true, false>;
    if constexpr (KT != 3 && KT != 6 && NT != 3 && NT != 6)
        return red ? &linear_kernel<KT, NT, false, true> : &linear_kernel<KT, NT, false, false>;
    return nullptr;
}
template <int KT> LinearFn pick_linear_n(int nt, bool vec, bool red)
{
    switch (nt) {
    case 1: return pick_linear<KT, 1>(vec, red);
    case 2: return pick_linear<KT, 2>(vec, red);
    case 3: return pick_linear<KT, 3>(vec, red);
    case 4: return pick_linear<KT, 4>(vec, red);
    case 6: return pick_linear<KT, 6>(vec, red);
    case 8: return pick_linear<KT, 8>(vec, red);
    }
    return nullptr;
}
LinearFn pick_linear_kn(int kt, int nt, bool vec, bool red)
{
    switch (kt) {
    case 1: return pick_linear_n<1>(nt, vec, red);
    case 2: return pick_linear_n<2>(nt, vec, red);
    case 3: return pick_linear_n<3>(nt, vec, red);
    case 4: return pick_linear_n<4>(nt, vec, red);
    case 6: return pick_linear_n<6>(nt, vec, red);
    case 8: return pick_linear_n<8>(nt, vec, red);
    }
    return nullptr;
}

using WgradFn = void (*)(WgradArgs);
// how one operand of the weight gradient is read: tiles per workgroup and whether a lane's
// columns are consecutive (the row then has to be a multiple of that many floats)
struct Side {
    int t;
    bool v;
};
Side side(int w, const float *p)
{
    const uintptr_t at = reinterpret_cast<uintptr_t>(p);
    if (w <= 16) return {1, false};
    if (w <= 32) return {2, w % 2 == 0 && at % 8 == 0};
    return {4, w % 4 == 0 && at % 16 == 0};
}
template <int TG, bool VG> WgradFn pick_wgrad_x(Side x)
{
    if (x.t == 1) return &wgrad_kernel<TG, VG, 1, false>;
    if (x.t == 2) return x.v ? &wgrad_kernel<TG, VG, 2, true> : &wgrad_kernel<TG, VG, 2, false>;
    return x.v ? &wgrad_kernel<TG, VG, 4, true> : &wgrad_kernel<TG, VG, 4, false>;
}
WgradFn pick_wgrad(Side g, Side x)
{
    if (g.t == 1) return pick_wgrad_x<1, false>(x);
    if (g.t == 2) return g.v ? pick_wgrad_x<2, true>(x) : pick_wgrad_x<2, false>(x);
    return g.v ? pick_wgrad_x<4, true>(x) : pick_wgrad_x<4, false>(x);
}

bool width_ok(int w) { return w > 0 && w <= PCSR_GNN_MAX_WIDTH; }

} // namespace

extern "C" {

int64_t pcsr_gnn_workspace_floats(int32_t a, int32_t b)
{
    if (!width_ok(a) || !width_ok(b)) return 0;
    const int64_t wgrad = (int64_t)kWgradBlocks * ((int64_t)a * b + b), linear = (int64_t)kLinearBlocks * (b + 1);
    const int64_t col = (int64_t)kColsumBlocks * b;
    int64_t most = wgrad > linear ? wgrad : linear;
    return most > col ? most : col;
}

int pcsr_gnn_linear(int64_t n, int32_t a, int32_t b, const float *X, const float *W, int32_t w_transposed,
                    const float *bias, int32_t relu, const float *mask, const float *dot_aux, float *Y,
                    float *colsum_out, float *dot_out, float *ws, void *stream)
{
    const bool red = colsum_out || dot_out;
    if (n < 0 || !X || !W || (!Y && !red) || (red && !ws) || (dot_out && !dot_aux)) return PCSR_E_INVALID_ARG;
    if (!width_ok(a) || !width_ok(b)) return PCSR_E_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto aligned = [](const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
    const bool vec = a % 4 == 0 && b % 4 == 0 && aligned(X) && aligned(mask) && aligned(dot_aux) && aligned(Y);
    LinearFn fn = pick_linear_kn(tiles(a, vec), tiles(b, vec), vec, red);
    if (!fn) return PCSR_E_UNSUPPORTED;
    const long groups = (n + 31) / 32;
    long blocks = (groups + kWaves - 1) / kWaves;
    blocks = blocks < 1 ? 1 : (blocks > kLinearBlocks ? kLinearBlocks : blocks);
    LinearArgs p;
    p.n = n;
    p.a = a;
    p.b = b;
    p.w_transposed = w_transposed;
    p.relu = relu;
    p.X = X;
    p.W = W;
    p.bias = bias;
    p.mask = mask;
    p.aux = dot_out ? dot_aux : nullptr;
    p.Y = Y;
    p.ws_colsum = colsum_out ? ws : nullptr;
    p.ws_dot = dot_out ? ws + (long)kLinearBlocks * b : nullptr;
    hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, p);
    int rc = to_code(hipGetLastError());
    if (rc == PCSR_OK && colsum_out) rc = sum_partials(p.ws_colsum, (int)blocks, b, b, colsum_out, 0, nullptr, s);
    if (rc == PCSR_OK && dot_out) rc = sum_partials(p.ws_dot, (int)blocks, 1, 1, dot_out, 0, nullptr, s);
    return rc;
}

int pcsr_gnn_wgrad(int64_t n, int32_t a, int32_t b, const float *G, const float *X, float *dW, float *db,
                   float *ws, void *stream)
{
    if (n < 0 || !G || !X || !dW || !ws) return PCSR_E_INVALID_ARG;
    if (!width_ok(a) || !width_ok(b)) return PCSR_E_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Side sg = side(b, G), sx = side(a, X);
    const unsigned gy = (unsigned)((b + sg.t * 16 - 1) / (sg.t * 16)), gz = (unsigned)((a + sx.t * 16 - 1) / (sx.t * 16));
    long blocks = (n + 64 * kWaves - 1) / (64 * kWaves); // at least four steps of 16 rows per wavefront
    const long most = kWgradBlocks / (gy * gz);
    blocks = blocks < 1 ? 1 : (blocks > most ? most : blocks);
    WgradArgs p;
    p.n = n;
    p.a = a;
    p.b = b;
    p.G = G;
    p.X = X;
    p.ws = ws;
    p.sums = db != nullptr;
    hipLaunchKernelGGL(pick_wgrad(sg, sx), dim3((unsigned)blocks, gy, gz), dim3(64 * kWaves), 0, s, p);
    int rc = to_code(hipGetLastError());
    const long len = (long)a * b;
    if (rc == PCSR_OK) rc = sum_partials(ws, (int)blocks, len + b, len, dW, db ? b : 0, db, s);
    return rc;
}

int pcsr_gnn_colsum(int64_t n, int32_t b, const float *G, float *out, float *ws, void *stream)
{
    if (n < 0 || !G || !out || !ws) return PCSR_E_INVALID_ARG;
    if (!width_ok(b)) return PCSR_E_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int rows = 256 / b;
    long blocks = (n + rows * 4 - 1) / (rows * 4);
    blocks = blocks < 1 ? 1 : (blocks > kColsumBlocks ? kColsumBlocks : blocks);
    hipLaunchKernelGGL(colsum_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (long)n, b, G, ws);
    const int rc = to_code(hipGetLastError());
    return rc == PCSR_OK ? sum_partials(ws, (int)blocks, b, b, out, 0, nullptr, s) : rc;
}

} // extern "C"
