// Dense side of a GNN layer on fp32 matrix instructions (see pcsr_gnn.h).
//
// v_mfma_f32_16x16x4_f32: lane l holds A[i = l%16][k = l/16] and B[k = l/16][j = l%16]; the
// result register r of lane l is D[i = 4*(l/16) + r][j = l%16].  The order of k is free as long
// as A and B agree, which is what both kernels use to load 16 bytes per lane.
#include "pcsr_gnn.h"

#include <hip/hip_runtime.h>
#include <type_traits>
#include <utility>

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// fp32 products on the bf16 matrix instructions, which do 16 times the work (Henry, Tang, Heinecke: Leveraging the bfloat16
// Artificial Intelligence Datatype For Higher-Precision Computations, ARITH 2019, have the method).  A float is the sum of three
// bf16 numbers, to the last bit (8 of its 24 bits each), and a product of two floats that of the six products of their pieces that
// reach 2^-24 of it.  v_mfma_f32_16x16x32_bf16: lane l holds A[i = l%16][k = 8*(l/16) and on] and B likewise, eight numbers each;
// results as above.  The five smaller products are added up apart from the largest.  Against 64 bits, 2-norm of normal numbers: 0.50
// / 0.65e-7 over 64 / 128 of them, where the fp32 instructions are off by 1.44 / 2.03e-7.  One accumulator for all six is off by
// 0.93 / 1.53, but to one side: these instructions cut off what does not reach the last bit of a sum, and sums of 200,000 such
// results were off 5 to 10 times as much as before.  They do 2420 TFLOP/s here for 150: 2.7 times the rate with six of them.  Rows
// and weights are taken 2^16 times as large, and the sums 2^-32 times: bf16 reaches as low as 2^-133, floats to 2^-149, so that the
// last piece of the smallest number is whole, and no bit of a sum changes (rows of 2^-115 were off by 1.1e-6, of 2^-124 by 5.6e-4
// without).  It costs 0 to 2.7 % (2,000,000 rows: 128 -> 128 437 and 448 us, 96 -> 96 332 and 339, two layers of 64 293 and 301,
// backward the same).  Rows with numbers of 2^50 and more, infinities among them, and all rows where a weight or a bias reaches 2^16
// and 2^50, are left to the fp32 instructions, in a loop of their own that takes 6 times as long: an infinity has no pieces, and
// below that neither the products of two layers nor their pieces' overflow: 64 (64 * 2^50 * 2^16) * 2^16 * 2^32 = 2^126.
typedef unsigned u4 __attribute__((ext_vector_type(4)));
struct Pieces {
    u4 p[3]; // of eight floats
};
constexpr float kRowsBelow = 0x1p50f, kWeightsBelow = 0x1p16f, kLarger = 0x1p16f, kLargerSum = kLarger * kLarger;

__device__ __forceinline__ unsigned bf16_pair(float a, float b)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    const f2 t = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(t, b2)); // to nearest
}
__device__ __forceinline__ float bf16_low(unsigned p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float bf16_high(unsigned p) { return __builtin_bit_cast(float, p & 0xffff0000u); }
__device__ __forceinline__ Pieces split(float (&x)[8])
{
    Pieces s;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] *= kLarger;
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned t = bf16_pair(x[2 * i], x[2 * i + 1]);
            s.p[p][i] = t;
            if (p < 2) {
                x[2 * i] -= bf16_low(t);
                x[2 * i + 1] -= bf16_high(t);
            }
        }
    return s;
}
// two fragments of fp32 products, side by side: k = 32 to 32 as long as both operands are put together so
__device__ __forceinline__ Pieces split(const f4 &lo, const f4 &hi)
{
    float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return split(x);
}
__device__ __forceinline__ f4 mfma32(const u4 &a, const u4 &b, f4 c)
{
    typedef __bf16 b8 __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
}
// acc[i] + low[i] += A[i] B; side by side, since an instruction that adds to the sum of the last one waits for it.
template <int N> __device__ __forceinline__ void mfma_pieces(const Pieces (&a)[N], const Pieces &b, f4 *acc, f4 *low)
{
    constexpr int order[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
    for (int o = 0; o < 6; ++o)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            f4 &sum = o < 5 ? low[i] : acc[i];
            sum = mfma32(a[i].p[order[o][0]], b.p[order[o][1]], sum);
        }
}
// the largest magnitude so far; a NaN may be passed over: its pieces are NaN
__device__ __forceinline__ void largest(float a, float b, float &most)
{
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(most) : "v"(a), "v"(b));
}

constexpr int kWaves = 4;
constexpr int kLinearBlocks = 768; // three per compute unit
constexpr int kBackBlocks = 512;
constexpr int kWgradBlocks = 512; // of four wavefronts; 768 and 1024: 0.5 to 5 % slower at 2,000,000 rows, more below
constexpr int kWgradAhead = 2;
constexpr int kColsumBlocks = 512;

struct LinearArgs {
    long n;
    int a, b, w_transposed, relu;
    const float *X, *W, *bias, *mask, *aux;
    float *Y;
    float *ws_colsum; // one row of b per workgroup
    float *ws_dot;    // one value per workgroup
};

// A wavefront takes 16 rows of X at a time.  D = op(W)-tile (16 outputs) x X^T (16 rows): a
// lane reads 16 bytes of one row per 16 inputs (component s of lane l is k = 4*(l/16) + s)
// and ends up with four consecutive outputs of one row, so loads and stores are 64-byte pieces of
// rows, X never goes through LDS, and what comes out has the layout that goes in: two layers
// can be chained in registers (mlp_kernel).  The weight fragments are in LDS (16 KB for 64 x
// 64), read as one ds_read_b128 per 4 matrix instructions.
// Bound by memory: 2,000,000 x 64 -> 64 is 1.02 GB and 16.4 GFLOP (104 us at the fp32 matrix
// peak).  The next rows are requested before this step's products, and no more workgroups are
// started than run at once.  With bias and ReLU 186 us (piece_kernel, 5.5 TB/s), with a mask to read as
// well and column sums 268 (5.7 TB/s), where torch's product, bias and ReLU take 488.
// VEC: widths that are multiples of 4, arrays 16-byte aligned.  RED: dot and/or column sums.
constexpr int blocks_per_cu(int kt, int nt) { return kt + nt <= 8 ? 3 : 2; } // registers and LDS allow no more
// piece_kernel: eight wavefronts to one copy of the weights where two copies do not fit
constexpr int piece_waves(int kt, int nt) { return kt + nt > 12 ? 8 : 4; }
// Without conditions in its loop a wavefront keeps more loads and stores on their way, and fewer of them do: at 2,000,000 / 300,000
// / 65,536 rows one workgroup to a compute unit in place of two or three takes 0.88 / 0.80 / 0.73 of the time of 64 -> 64 before
// (two: 0.95, 0.86, 0.89), 48 -> 48 0.92 / 0.91 / 0.82, 128 -> 16 0.96 / 0.94 / 0.88, with a mask and column sums 0.99 / 0.97 /
// 0.95.  Narrower ones want two (16 -> 64 1.17 with one, 0.97 with two, 1.05 with three).  So do 64 columns of 96 and of 128 (one
// takes 1.04-1.20 of two at 300,000 rows, 0.96-1.07 at 2,000,000; with a mask and no sums 128 -> 64 had lost: 63 us for 56, now
// 53), 48 of 128 with a mask or sums (1.07-1.08; 0.91-0.96), and 16 -> 96 without, written by more than it is read (158 and 154 us
// in a training step of 2,000,000 rows; with a mask 305 and 323).
constexpr int piece_blocks_per_cu(int kt, int nt, bool red, bool mask)
{
    return kt + nt <= 5 || (kt >= 6 && nt == 4) || (kt == 8 && nt == 3 && (red || mask)) || (kt == 1 && nt == 6 && !red && !mask) ? 2 : 1;
}

// weight fragments of one layer: fragment (kt, nt), lane l, component s is
// W[out = 16 nt + l%16][in = 16 kt + 4 (l/16) + s] (transposed: W[in][out])
template <int KT, int NT>
__device__ __forceinline__ void stage_weights(f4 *wfrag, const float *W, int a, int b, int transposed)
{
    for (int f = threadIdx.x; f < KT * NT * 64; f += blockDim.x) {
        const int l = f & 63, t = f >> 6, kt = t / NT, nt = t - kt * NT;
        const int out = nt * 16 + (l & 15), in0 = kt * 16 + 4 * (l >> 4);
        f4 w = {0.0f, 0.0f, 0.0f, 0.0f};
        if (out < b) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (in0 + s < a) w[s] = transposed ? W[(long)(in0 + s) * b + out] : W[(long)out * a + in0 + s];
        }
        wfrag[f] = w;
    }
}

// acc += op(W) x for 16 rows, outputs 16 N0 to 16 (N0 + NS)
template <int KT, int NT, int N0 = 0, int NS = NT>
__device__ __forceinline__ void multiply(const f4 *wfrag, int lane, const f4 (&x)[KT], f4 (&acc)[NS])
{
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
        f4 w[NS];
#pragma unroll
        for (int nt = 0; nt < NS; ++nt) w[nt] = wfrag[(kt * NT + N0 + nt) * 64 + lane];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int nt = 0; nt < NS; ++nt) acc[nt] = mfma4(w[nt][s], x[kt][s], acc[nt]);
    }
}

// Where pieces are taken: where the matrix rate bounds a pass as much as memory does.  Elsewhere the work of splitting shows (us at
// 2,000,000 rows, fp32 products / pieces): 32 -> 32 92 / 113, 48 -> 64 157 / 174, 96 -> 16 162 / 178, 64 -> 64 alone 186 / 193; but
// 64 -> 128 333 / 315, 128 -> 64 315 / 302, 96 -> 96 359 / 336, 96 -> 128 451 / 361, 128 -> 128 558 / 434 (200,000 rows 77 / 53);
// two layers 16 -> 64 -> 64 237 / 225, 64 -> 64 -> 64 323 / 284 (200,000 rows 41 / 31) but 48 -> 48 -> 48 230 / 230; one layer
// backward 64 -> 64 327 / 300, 48 -> 48 226 / 226, 32 -> 32 151 / 156; two layers backward 64 from 32 450 / 410, 48 from 48 387 /
// 389.  64 from 48 and 64 backward have no registers for it (spilled, 587 -> 616).
constexpr bool split_piece(int kt, int nt) { return kt >= 4 && nt >= 4 && kt * nt > 16; }
constexpr bool split_mlp(int mt) { return mt == 4; }
constexpr bool split_back(int bt, int mt, int at, bool two) { return two ? mt == 4 && at <= 2 : bt * mt >= 12; }

// acc += op(W) x for 16 rows, with W in LDS as `words` of 16 bytes.  SPLIT: in pieces, but for sixteen inputs, where six products
// take as long.
constexpr std::true_type kInPieces{};
constexpr std::false_type kAsTheyAre{};
template <int KT, int NT, bool SPLIT> struct Product {
    static constexpr bool kSplit = SPLIT && KT > 1;
    static constexpr int kSteps = (KT + 1) / 2;
    static constexpr int words = kSplit ? kSteps * NT * 3 * 64 : KT * NT * 64;
    using Split = Pieces[kSteps];
    const f4 *frag;
    const float *W;
    int transposed;

    // Piece p of fragment (step, nt), lane l: W[out = 16 nt + l%16][in = 32 step + 16 (s/4) + 4 (l/16) + s%4], s < 8.  `most`: the
    // largest magnitude that this thread has seen.
    static __device__ __forceinline__ Product stage(f4 *frag, const float *W, int transposed, float &most)
    {
        constexpr int a = 16 * KT, b = 16 * NT;
        if constexpr (!kSplit) {
            stage_weights<KT, NT>(frag, W, a, b, transposed);
            if (SPLIT) // for what follows
                for (int i = threadIdx.x; i < a * b; i += blockDim.x) most = fmaxf(most, fabsf(W[i]));
        } else {
            for (int f = threadIdx.x; f < kSteps * NT * 64; f += blockDim.x) {
                const int l = f & 63, t = f >> 6, k = t / NT, out = (t - k * NT) * 16 + (l & 15);
                float w[8];
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const int in = 32 * k + 16 * (s >> 2) + 4 * (l >> 4) + (s & 3);
                    w[s] = in < a ? (transposed ? W[(long)in * b + out] : W[(long)out * a + in]) : 0.0f;
                }
#pragma unroll
                for (int s = 0; s < 8; s += 2) largest(w[s], w[s + 1], most);
                const Pieces x = split(w);
#pragma unroll
                for (int p = 0; p < 3; ++p) frag[(t * 3 + p) * 64 + l] = __builtin_bit_cast(f4, x.p[p]);
            }
        }
        return {frag, W, transposed};
    }

    static __device__ __forceinline__ void split_rows(const f4 (&x)[KT], Split &s)
    {
        if constexpr (kSplit) {
#pragma unroll
            for (int k = 0; k < kSteps; ++k) s[k] = split(x[2 * k], 2 * k + 1 < KT ? x[2 * k + 1] : f4{0.0f, 0.0f, 0.0f, 0.0f});
        }
    }
    // x[kt] without an index into registers
    template <int... I> static __device__ __forceinline__ f4 pick(const f4 (&x)[KT], int kt, std::integer_sequence<int, I...>)
    {
        f4 t = x[0];
        ((kt == I ? (void)(t = x[I]) : (void)0), ...);
        return t;
    }
    // Outputs 16 N0 to 16 (N0 + NS).  kAsTheyAre: seldom, so with no registers of its own and no room in LDS.
    template <int N0, int NS, class Form> __device__ __forceinline__ void add(Form, int lane, const f4 (&x)[KT], const Split &xs, f4 (&acc)[NS]) const
    {
        if constexpr (!kSplit) {
            multiply<KT, NT, N0, NS>(frag, lane, x, acc);
        } else if constexpr (Form::value) {
            constexpr int S = NS % 2 == 0 ? 2 : 1;
#pragma unroll
            for (int nt = 0; nt < NS; nt += S) {
                f4 low[S];
#pragma unroll
                for (int i = 0; i < S; ++i) {
                    low[i] = f4{0.0f, 0.0f, 0.0f, 0.0f};
                    acc[nt + i] *= kLargerSum;
                }
#pragma unroll
                for (int k = 0; k < kSteps; ++k) {
                    Pieces w[S];
#pragma unroll
                    for (int i = 0; i < S; ++i)
#pragma unroll
                        for (int p = 0; p < 3; ++p)
                            w[i].p[p] = __builtin_bit_cast(u4, frag[((k * NT + N0 + nt + i) * 3 + p) * 64 + lane]);
                    mfma_pieces<S>(w, xs[k], acc + nt, low);
                }
#pragma unroll
                for (int i = 0; i < S; ++i) acc[nt + i] = (acc[nt + i] + low[i]) * (1.0f / kLargerSum);
            }
        } else {
#pragma unroll 1
            for (int kt = 0; kt < KT; ++kt) {
                const f4 xk = pick(x, kt, std::make_integer_sequence<int, KT>{});
#pragma unroll
                for (int nt = 0; nt < NS; ++nt) {
                    const int out = (N0 + nt) * 16 + (lane & 15), in = kt * 16 + 4 * (lane >> 4);
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        acc[nt] = mfma4(transposed ? W[(in + s) * (16 * NT) + out] : W[out * (16 * KT) + in + s], xk[s], acc[nt]);
                    asm volatile("" ::: "memory");
                }
            }
        }
    }
    template <class Form> __device__ __forceinline__ void add(Form form, int lane, const f4 (&x)[KT], f4 (&acc)[NT]) const
    {
        Split xs;
        if constexpr (Form::value) split_rows(x, xs);
        add<0, NT>(form, lane, x, xs, acc);
    }
};

// whether all of this is small enough for pieces, in the whole wavefront
template <int T> __device__ __forceinline__ bool small_rows(const f4 (&x)[T])
{
    float most = 0.0f;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        largest(x[t][0], x[t][1], most);
        largest(x[t][2], x[t][3], most);
    }
    return __builtin_amdgcn_ballot_w64(!(most < kRowsBelow)) == 0;
}
// the same of the weights and of biases (null: none) as stage_bias has left them, for the workgroup; a barrier
template <int N, bool SPLIT> __device__ __forceinline__ bool small_weights(float most, const f4 *bias = nullptr, const f4 *other = nullptr)
{
    if (!SPLIT) {
        __syncthreads();
        return true;
    }
    float b = 0.0f;
    for (const f4 *one : {bias, other})
        for (int o = threadIdx.x; one && o < N; o += blockDim.x) b = fmaxf(b, fabsf(reinterpret_cast<const float *>(one)[o]));
    return !__syncthreads_or(!(most < kWeightsBelow) || !(b < kRowsBelow));
}

// the bias waits in LDS: in registers it would cost what the row pieces need
template <int NT> __device__ __forceinline__ void stage_bias(f4 *bias, const float *b, int width)
{
    for (int o = threadIdx.x; o < 16 * NT; o += blockDim.x)
        reinterpret_cast<float *>(bias)[o] = b && o < width ? b[o] : 0.0f;
}
template <int NT> __device__ __forceinline__ void start_from(const f4 *bias, int lane, f4 (&acc)[NT])
{
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = bias[nt * 4 + (lane >> 4)];
}

// Sixteen rows of exactly 16 T floats are one piece of memory.  It is read and written with the lanes
// side by side, T times 1 KB (lane l, step u: 16-byte word 64 u + l of the piece), and turned
// to and from the fragments through an LDS patch of the wavefront's own.  Straight from the fragments
// every access would touch 16 rows, 64 bytes of each: 16 -> 64 columns ran at 3.7 TB/s so, and run at
// 5.6 through the patch (2,000,000 rows, 115 us).
//
// Groups of 16 rows that are whole have a loop of their own: with no load or store in it that may be left out, but for the
// request of the next rows, the compiler counts what is in flight, and a wait for the next rows is not one for the stores before it.
constexpr std::integral_constant<long, 16> kWhole{};
constexpr int kSumRun = 8;
constexpr int patch_ld(int t) { return 16 * t + 4; } // floats per row
constexpr int patch_floats(int t) { return 16 * patch_ld(t); }

// LDS keeps the order of one wavefront's accesses: only the compiler has to keep it as well
__device__ __forceinline__ void patch_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// a scalar base and 32 bits of offset
__device__ __forceinline__ const f4 *at_byte(const float *base, unsigned off)
{
    return reinterpret_cast<const f4 *>(reinterpret_cast<const char *>(base) + off);
}
__device__ __forceinline__ f4 *at_byte(float *base, unsigned off)
{
    return reinterpret_cast<f4 *>(reinterpret_cast<char *>(base) + off);
}
// T: tiles of a row; S: of the part of it that is meant (from `piece` on), all of them or four
template <int T, int S> __device__ __forceinline__ unsigned piece_byte(int lane) // plus 1 KB times T/S times u
{
    return T == S ? 16u * (unsigned)lane : 64u * T * ((unsigned)lane / (4 * S)) + 16u * ((unsigned)lane % (4 * S));
}
template <int T, int S> __device__ __forceinline__ void load_piece(const float *piece, int lane, long rows, f4 (&x)[S])
{
    static_assert(T == S || S == 4);
    if (rows >= 16) {
#pragma unroll
        for (int u = 0; u < S; ++u) x[u] = *at_byte(piece + u * 256 * (T / S), piece_byte<T, S>(lane));
    } else { // zeros past the end
#pragma unroll
        for (int u = 0; u < S; ++u) {
            x[u] = f4{0.0f, 0.0f, 0.0f, 0.0f};
            if ((u * 64 + lane) / (4 * S) < rows) x[u] = *at_byte(piece + u * 256 * (T / S), piece_byte<T, S>(lane));
        }
    }
}
template <int T, int S> __device__ __forceinline__ void store_piece(float *piece, int lane, long rows, const f4 (&x)[S])
{
#pragma unroll
    for (int u = 0; u < S; ++u)
        if (rows >= 16 || (u * 64 + lane) / (4 * S) < rows) *at_byte(piece + u * 256 * (T / S), piece_byte<T, S>(lane)) = x[u];
}
// straight to the fragments
template <int T> __device__ __forceinline__ void load_frags(const float *piece, int lane, long rows, f4 (&x)[T])
{
    const unsigned at = 4u * ((lane & 15) * (16 * T) + 4 * (lane >> 4));
    if (rows >= 16 || (lane & 15) < rows) {
#pragma unroll
        for (int t = 0; t < T; ++t) x[t] = *at_byte(piece + t * 16, at);
    } else {
#pragma unroll
        for (int t = 0; t < T; ++t) x[t] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }
}
template <int T> __device__ __forceinline__ void store_frags(float *piece, int lane, long rows, const f4 (&x)[T])
{
    const unsigned at = 4u * ((lane & 15) * (16 * T) + 4 * (lane >> 4));
    if (rows >= 16 || (lane & 15) < rows) {
#pragma unroll
        for (int t = 0; t < T; ++t) *at_byte(piece + t * 16, at) = x[t];
    }
}
template <int T, int LD> __device__ __forceinline__ void piece_to_patch(float *patch, int lane, const f4 (&x)[T])
{
#pragma unroll
    for (int u = 0; u < T; ++u) {
        const int i = u * 64 + lane;
        *reinterpret_cast<f4 *>(patch + i / (4 * T) * LD + i % (4 * T) * 4) = x[u];
    }
}
template <int T, int LD> __device__ __forceinline__ void patch_to_piece(const float *patch, int lane, f4 (&x)[T])
{
#pragma unroll
    for (int u = 0; u < T; ++u) {
        const int i = u * 64 + lane;
        x[u] = *reinterpret_cast<const f4 *>(patch + i / (4 * T) * LD + i % (4 * T) * 4);
    }
}
template <int T, int LD> __device__ __forceinline__ void frags_to_patch(float *patch, int lane, const f4 (&x)[T])
{
#pragma unroll
    for (int t = 0; t < T; ++t) *reinterpret_cast<f4 *>(patch + (lane & 15) * LD + t * 16 + 4 * (lane >> 4)) = x[t];
}
template <int T> __device__ __forceinline__ void frags_to_piece(float *patch, int lane, f4 (&x)[T])
{
    patch_fence();
    frags_to_patch<T, patch_ld(T)>(patch, lane, x);
    patch_fence();
    patch_to_piece<T, patch_ld(T)>(patch, lane, x);
}
template <int T> __device__ __forceinline__ void relu_rows(f4 (&x)[T]) // NaN stays NaN
{
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int s = 0; s < 4; ++s) x[t][s] = x[t][s] <= 0.0f ? 0.0f : x[t][s];
}
template <int T> __device__ __forceinline__ void mask_rows(f4 (&x)[T], const f4 (&m)[T])
{
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int s = 0; s < 4; ++s) x[t][s] = m[t][s] <= 0.0f ? 0.0f : x[t][s];
}

// fragments of rows past the end: what a sum over rows must not count (a product of zeros plus the bias)
template <int T> __device__ __forceinline__ void clear_past_end(int lane, long rows, f4 (&x)[T])
{
    if (rows >= 16) return; // all but the last of a wavefront's groups
    if ((lane & 15) >= rows) {
#pragma unroll
        for (int t = 0; t < T; ++t) x[t] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }
}

template <int KT, int NT, bool VEC, bool RED>
__global__ void __launch_bounds__(64 * kWaves, blocks_per_cu(KT, NT)) linear_kernel(LinearArgs p)
{
    __shared__ f4 wfrag[KT * NT * 64], bias[NT * 4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, q = lane >> 4;
    stage_weights<KT, NT>(wfrag, p.W, p.a, p.b, p.w_transposed);
    stage_bias<NT>(bias, p.bias, p.b);
    __syncthreads();

    f4 csum[RED ? NT : 1];
    float dot = 0.0f;
    if constexpr (RED) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) csum[nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    const long groups = (p.n + 15) >> 4, stride = (long)gridDim.x * kWaves;
    auto fetch = [&](long g, f4 (&x)[KT]) {
        long row = g * 16 + r;
        row = row < p.n ? row : p.n - 1; // results of the rows past the end are dropped below
        const float *xr = p.X + row * p.a;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            const int c = kt * 16 + 4 * q;
            if constexpr (VEC) {
                x[kt] = c < p.a ? *reinterpret_cast<const f4 *>(xr + c) : f4{0.0f, 0.0f, 0.0f, 0.0f};
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) x[kt][s] = c + s < p.a ? xr[c + s] : 0.0f;
            }
        }
    };
    long g = (long)blockIdx.x * kWaves + wave;
    f4 xn[KT]; // the next rows are requested before this step's products
    if (g < groups) fetch(g, xn);
    for (; g < groups; g += stride) {
        // keeps the weight fragments in LDS: hoisted out of the loop they would fill the registers
        asm volatile("" ::: "memory");
        f4 x[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) x[kt] = xn[kt];
        if (g + stride < groups) fetch(g + stride, xn);
        f4 acc[NT];
        start_from<NT>(bias, lane, acc);
        multiply<KT, NT>(wfrag, lane, x, acc);
        const long row = g * 16 + r;
        if (row >= p.n) continue;
        const long at = row * p.b;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int c = nt * 16 + 4 * q;
            f4 v = acc[nt];
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

// Sums over a workgroup in a fixed order.  `lds` may be the patches.
template <int T, bool FRAGS>
__device__ __forceinline__ void collect_colsum(float *lds, const f4 (&csum)[T], float *out)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __syncthreads();
    f4 *s = reinterpret_cast<f4 *>(lds) + wave * T * 64; // word i: columns 4 (i mod 4T) and on
#pragma unroll
    for (int u = 0; u < T; ++u) s[FRAGS ? (lane & 15) * (4 * T) + 4 * u + (lane >> 4) : u * 64 + lane] = csum[u];
    __syncthreads();
    for (int c = tid; c < 16 * T; c += blockDim.x) {
        float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int i = 0; i < (int)blockDim.x / 4; i += 4) // 64 or 128 of them
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] += lds[(i + u) * (16 * T) + c];
        out[c] = (t[0] + t[1]) + (t[2] + t[3]);
    }
}
__device__ __forceinline__ void collect_dot(float *lds, float dot, float *out)
{
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) dot += __shfl_xor(dot, m);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = dot;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = (lds[0] + lds[1]) + (lds[2] + lds[3]);
        if (blockDim.x == 512) t += (lds[4] + lds[5]) + (lds[6] + lds[7]);
        *out = t;
    }
}

// Exact widths, a = 16 KT and b = 16 NT: as linear_kernel, in pieces.
template <int KT, int NT, bool RED>
__global__ void __launch_bounds__(64 * piece_waves(KT, NT), RED || piece_waves(KT, NT) == 8 ? 2 : blocks_per_cu(KT, NT)) piece_kernel(LinearArgs p)
{
    // Eight tiles of outputs in two halves: the patch of one leaves room for the weights' pieces.
    constexpr int kW = piece_waves(KT, NT), kHalves = NT == 8 ? 2 : 1, NS = NT / kHalves, kPatch = patch_floats(NS);
    using Weights = Product<KT, NT, split_piece(KT, NT)>;
    __shared__ f4 wfrag[Weights::words], bias[NT * 4];
    __shared__ __align__(16) float patches[kW * kPatch];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *patch = patches + wave * kPatch;
    stage_bias<NT>(bias, p.bias, 16 * NT);
    float most = 0.0f;
    const auto W = Weights::stage(wfrag, p.W, p.w_transposed, most);
    bool in_pieces = small_weights<16 * NT, Weights::kSplit>(most, bias);

    f4 csum[RED ? NT : 1], csums[RED ? NT : 1]; // sums of kSumRun groups are put apart
    float dot = 0.0f, dots = 0.0f;
    [[maybe_unused]] int run = 0;
    auto put_apart = [&] {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            csums[nt] += csum[nt];
            csum[nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        dots += dot;
        dot = 0.0f;
        run = 0;
    };
    if constexpr (RED) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) csum[nt] = csums[nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    const long full = p.n >> 4, stride = (long)gridDim.x * kW;
    long g = (long)blockIdx.x * kW + wave;
    f4 xn[KT]; // the next rows are requested before this step's products
    auto load = [&](long g, auto rows) { load_frags<KT>(p.X + g * (256 * KT), lane, rows, xn); };
    // aux, mask, store: which of these arrays there are, as constants in the loops of the layers' own calls
    auto step = [&](auto form, long g, auto rows, auto aux, auto mask, auto store, auto next) {
        asm volatile("" ::: "memory"); // as in linear_kernel
        f4 x[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) x[kt] = xn[kt];
        next();
        if (decltype(form)::value && Weights::kSplit && !small_rows(x)) { // asked for once the next rows have been
            in_pieces = false;
            return;
        }
        typename Weights::Split xs;
        if constexpr (decltype(form)::value) Weights::split_rows(x, xs);
        auto half = [&](auto h) {
            constexpr int N0 = decltype(h)::value * NS;
            f4 y[NS], m[NS]; // aux, or the mask; callers have one of them
            if (aux || mask) load_piece<NT, NS>((aux ? p.aux : p.mask) + g * (256 * NT) + 16 * N0, lane, rows, m);
            start_from<NS>(bias + 4 * N0, lane, y);
            W.template add<N0, NS>(form, lane, x, xs, y);
            if (p.relu) relu_rows<NS>(y);
            if constexpr (RED) clear_past_end<NS>(lane, rows, y);
            frags_to_piece<NS>(patch, lane, y);
            if (aux) {
#pragma unroll
                for (int t = 0; t < NS; ++t)
                    dot += (y[t][0] * m[t][0] + y[t][1] * m[t][1]) + (y[t][2] * m[t][2] + y[t][3] * m[t][3]);
                if (mask) load_piece<NT, NS>(p.mask + g * (256 * NT) + 16 * N0, lane, rows, m);
            }
            if (mask) mask_rows<NS>(y, m);
            if constexpr (RED) {
#pragma unroll
                for (int t = 0; t < NS; ++t) csum[N0 + t] += y[t];
            }
            if (store) store_piece<NT, NS>(p.Y + g * (256 * NT) + 16 * N0, lane, rows, y);
        };
        half(std::integral_constant<int, 0>{});
        if constexpr (kHalves == 2) half(std::integral_constant<int, 1>{});
        if constexpr (RED)
            if (++run == kSumRun) put_apart();
    };
    auto walk = [&](auto aux, auto mask, auto store) {
        if (g < full) load(g, kWhole);
        for (; g < full; g += stride) {
            step(kInPieces, g, kWhole, aux, mask, store, [&] {
                if (g + stride < full) load(g + stride, kWhole);
            });
            if (Weights::kSplit && !in_pieces) break;
        }
    };
    const std::true_type yes;
    const std::false_type no;
    const bool aux = RED && p.aux, mask = p.mask, store = p.Y;
    if (!in_pieces) {
    } else if constexpr (RED) {
        if (aux && !mask && store)
            walk(yes, no, yes);
        else if (!aux && mask && store)
            walk(no, yes, yes);
        else
            walk(aux, mask, store);
    } else if (mask) {
        walk(no, yes, yes);
    } else {
        walk(no, no, yes);
    }
    if (const long rows = p.n - g * 16; rows > 0 && in_pieces) { // the rows that are left over
        load(g, rows);
        step(kInPieces, g, rows, aux, mask, store, [] {});
    }
    if constexpr (Weights::kSplit) {
        for (; !in_pieces && g * 16 < p.n; g += stride) {
            load(g, p.n - g * 16);
            step(kAsTheyAre, g, p.n - g * 16, aux, mask, store, [] {});
        }
    }
    if constexpr (RED) {
        put_apart();
        if (p.ws_colsum) {
            float *out = p.ws_colsum + (long)blockIdx.x * (16 * NT);
            static_assert(kPatch >= NS * 256, "collect_colsum's words in the patches");
#pragma unroll
            for (int h = 0; h < kHalves; ++h) {
                f4 sums[NS];
#pragma unroll
                for (int t = 0; t < NS; ++t) sums[t] = csums[h * NS + t];
                collect_colsum<NS, false>(patches, sums, out + h * (16 * NS));
            }
        }
        if (p.ws_dot) collect_dot(patches, dots, p.ws_dot + blockIdx.x);
    }
}

// Two layers in one pass: Z = relu(X W1^T + b1), Y = Z W2^T + b2 (relu).  Exact widths: a = 16 KT,
// both layers 16 MT outputs.  Z is stored for the backward pass and not read back: 2,000,000 x 64
// -> 64 -> 64 takes 310-335 us where two piece_kernel passes take 370.
struct MlpArgs {
    long n;
    int relu;
    const float *X, *W1, *b1, *W2, *b2;
    float *Z, *Y;
};
constexpr int mlp_blocks_per_cu(int kt, int mt) { return kt + mt > 5 && split_mlp(mt) ? 2 : 3; }
template <int KT, int MT> __global__ void __launch_bounds__(64 * kWaves, mlp_blocks_per_cu(KT, MT)) mlp_kernel(MlpArgs p)
{
    constexpr int kPatch = patch_floats(MT);
    __shared__ f4 w1[Product<KT, MT, split_mlp(MT)>::words], w2[Product<MT, MT, split_mlp(MT)>::words], bias1[MT * 4], bias2[MT * 4];
    __shared__ __align__(16) float patches[kWaves * kPatch];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *patch = patches + wave * kPatch;
    stage_bias<MT>(bias1, p.b1, 16 * MT);
    stage_bias<MT>(bias2, p.b2, 16 * MT);
    float most = 0.0f;
    const auto W1 = Product<KT, MT, split_mlp(MT)>::stage(w1, p.W1, 0, most);
    const auto W2 = Product<MT, MT, split_mlp(MT)>::stage(w2, p.W2, 0, most);
    constexpr bool kSplit = split_mlp(MT);
    bool in_pieces = small_weights<16 * MT, kSplit>(most, bias1, bias2);
    const long full = p.n >> 4, stride = (long)gridDim.x * kWaves;
    long g = (long)blockIdx.x * kWaves + wave;
    f4 xn[KT];
    auto load = [&](long g, auto rows) { load_frags<KT>(p.X + g * (256 * KT), lane, rows, xn); };
    auto step = [&](auto form, long g, auto rows, auto next) {
        asm volatile("" ::: "memory"); // as in linear_kernel
        f4 x[KT], z[MT], y[MT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) x[kt] = xn[kt];
        next();
        if (decltype(form)::value && kSplit && !small_rows(x)) { // as in piece_kernel
            in_pieces = false;
            return;
        }
        start_from<MT>(bias1, lane, z);
        W1.add(form, lane, x, z);
        relu_rows<MT>(z);
        start_from<MT>(bias2, lane, y);
        W2.add(form, lane, z, y);
        if (p.relu) relu_rows<MT>(y);
        frags_to_piece<MT>(patch, lane, z);
        store_piece<MT, MT>(p.Z + g * (256 * MT), lane, rows, z);
        frags_to_piece<MT>(patch, lane, y);
        store_piece<MT, MT>(p.Y + g * (256 * MT), lane, rows, y);
    };
    if (g < full && in_pieces) load(g, kWhole);
    for (; g < full && in_pieces; g += stride) {
        step(kInPieces, g, kWhole, [&] {
            if (g + stride < full) load(g + stride, kWhole);
        });
        if (kSplit && !in_pieces) break;
    }
    if (const long rows = p.n - g * 16; rows > 0 && in_pieces) { // the rows that are left over
        load(g, rows);
        step(kInPieces, g, rows, [] {});
    }
    if constexpr (kSplit) {
        for (; !in_pieces && g * 16 < p.n; g += stride) {
            load(g, p.n - g * 16);
            step(kAsTheyAre, g, p.n - g * 16, [] {});
        }
    }
}

// Backward of one layer, or of the two of a GIN layer, in one pass over its arrays:
//   dW2 = G^T Z, db2 = sums of G, G1 = (G W2) masked by Z > 0,
// and with TWO   dW1 = G1^T A, db1 = sums of G1, dA = G1 W1, dot = sum(dA * H);
// without it G1 is stored and its column sums are taken.  Exact widths: G 16 BT, Z 16 MT, A and H
// 16 AT.  The products with the weights run on registers as in mlp_kernel.  For those with
// G^T and G1^T the rows are the k of the matrix instruction, so 16 rows of both operands are
// turned in an LDS patch of the wavefront's own: written as they are held, read T consecutive
// columns of one row per lane, which feeds T tiles (tile t holds the columns T*i + t, as in
// wgrad_kernel).  G, Z, A and H are read once and G1 never leaves the registers: 2.6 GB for
// 2,000,000 x 64 (TWO) where the separate kernels move 5.6 GB, 550-595 us where they take 920 (650-700 with conditions
// on loads and stores in the loop); what bounds it is the matrix rate (65.5 GFLOP,
// 428 us; matrix cores 84 % busy) with two wavefronts to a SIMD, all that the accumulators leave room for.  Without TWO,
// masked and with column sums, 317 us for 468.
struct BackArgs {
    long n;
    int masked;
    const float *G, *Z, *W2, *A, *H, *W1;
    float *out;    // dA, or G1 (may be null)
    float *ws;     // per workgroup: dW2, db2, then dW1, db1, dot (TWO) or the sums of G1
    long ws_stride;
};
// floats per row: 16 lanes that write 16 bytes of a row each meet all 64 banks (16 t + 16 had four of them on
// the same ones: conflicts 19 % of the LDS cycles for 52, 2,000,000 x 64 656-662 us for 672); rows of 16 are dense as they are
constexpr int back_ld(int t) { return t == 1 ? 16 : 16 * t + 4; }

// acc += P^T Q over the 16 rows in the patch; psum: column sums of P
template <int PT, int QT>
__device__ __forceinline__ void turned_product(const float *patch, int lane, f4 (&acc)[PT][QT], float (&psum)[PT])
{
    constexpr int LP = back_ld(PT), LQ = back_ld(QT);
    const int c = lane & 15, q = lane >> 4;
    const float *qpatch = patch + 16 * LP;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        float a[PT], b[QT];
#pragma unroll
        for (int t = 0; t < PT; ++t) a[t] = patch[(4 * u + q) * LP + PT * c + t];
#pragma unroll
        for (int t = 0; t < QT; ++t) b[t] = qpatch[(4 * u + q) * LQ + QT * c + t];
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            psum[i] += a[i];
#pragma unroll
            for (int j = 0; j < QT; ++j) acc[i][j] = mfma4(a[i], b[j], acc[i][j]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}
// the four wavefronts' accumulators, in order, to out[16 PT x 16 QT] and sums[16 PT]; `red`: LDS
template <int PT, int QT>
__device__ __forceinline__ void collect(float *red, const f4 (&acc)[PT][QT], float (&psum)[PT], float *out, float *sums)
{
    constexpr int LD = QT * 16 + 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, q = lane >> 4;
    float *sred = red + PT * 16 * LD;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
        psum[i] += __shfl_xor(psum[i], 16);
        psum[i] += __shfl_xor(psum[i], 32);
    }
    __syncthreads();
    for (int w = 0; w < kWaves; ++w) {
        if (wave == w) {
#pragma unroll
            for (int i = 0; i < PT; ++i) {
#pragma unroll
                for (int j = 0; j < QT; ++j)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        float &d = red[((4 * q + s) * PT + i) * LD + c * QT + j];
                        d = w ? d + acc[i][j][s] : acc[i][j][s];
                    }
                if (q == 0) {
                    float &d = sred[c * PT + i];
                    d = w ? d + psum[i] : psum[i];
                }
            }
        }
        __syncthreads();
    }
    for (int e = tid; e < PT * QT * 256; e += 64 * kWaves) out[e] = red[(e / (QT * 16)) * LD + e % (QT * 16)];
    if (tid < PT * 16) sums[tid] = sred[tid];
    __syncthreads();
}

template <int BT, int MT, int AT, bool TWO>
__global__ void __launch_bounds__(64 * kWaves, 2) back_kernel(BackArgs p)
{
    constexpr int kPatch1 = 16 * (back_ld(BT) + back_ld(MT)), kPatch2 = TWO ? 16 * (back_ld(MT) + back_ld(AT)) : 0;
    constexpr int kPatch = kPatch1 > kPatch2 ? kPatch1 : kPatch2;
    constexpr int kRed1 = BT * 16 * (MT * 16 + 1) + BT * 16, kRed2 = TWO ? MT * 16 * (AT * 16 + 1) + MT * 16 : 0;
    constexpr int kRed = kRed1 > kRed2 ? kRed1 : kRed2;
    constexpr bool kSplit = split_back(BT, MT, AT, TWO);
    __shared__ f4 w2[Product<BT, MT, kSplit>::words];
    __shared__ f4 w1[TWO ? Product<MT, AT, kSplit>::words : 1];
    __shared__ __align__(16) float lds[kWaves * kPatch > kRed ? kWaves * kPatch : kRed];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *patch = lds + wave * kPatch;
    float most = 0.0f;
    const auto W2 = Product<BT, MT, kSplit>::stage(w2, p.W2, 1, most);
    const auto W1 = [&] {
        if constexpr (TWO) return Product<MT, AT, kSplit>::stage(w1, p.W1, 1, most);
        else return 0;
    }();
    bool in_pieces = small_weights<0, kSplit>(most);

    const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f4 acc2[BT][MT], acc1[TWO ? MT : 1][TWO ? AT : 1], csum[MT];
    float sum2[BT], sum1[TWO ? MT : 1], dot = 0.0f;
#pragma unroll
    for (int i = 0; i < BT; ++i) {
        sum2[i] = 0.0f;
#pragma unroll
        for (int j = 0; j < MT; ++j) acc2[i][j] = zero;
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) csum[i] = zero;
    if constexpr (TWO) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            sum1[i] = 0.0f;
#pragma unroll
            for (int j = 0; j < AT; ++j) acc1[i][j] = zero;
        }
    }

    constexpr int LG = back_ld(BT), LZ = back_ld(MT), LA = back_ld(AT);
    const long full = p.n >> 4, stride = (long)gridDim.x * kWaves;
    long g = (long)blockIdx.x * kWaves + wave;
    f4 gg[BT], zz[MT], aa[TWO ? AT : 1];
    constexpr bool kLateZ = TWO && MT + AT > 7; // no registers to hold the next rows of Z as well from early on
    auto load_g = [&](long g, auto rows) { load_frags<BT>(p.G + g * (256 * BT), lane, rows, gg); };
    auto load_z = [&](long g, auto rows) { load_frags<MT>(p.Z + g * (256 * MT), lane, rows, zz); };
    auto load_a = [&](long g, auto rows) {
        if constexpr (TWO) load_piece<AT, AT>(p.A + g * (256 * AT), lane, rows, aa);
    };
    // the next rows of G, Z and A go into the same registers once these are in the patch and used;
    // the products that follow cover the wait
    auto step = [&](auto form, long g, auto rows, auto next_g, auto next_z, auto next_a) {
        f4 g1[MT];
        patch_fence();
        frags_to_patch<BT, LG>(patch, lane, gg);
        frags_to_patch<MT, LZ>(patch + 16 * LG, lane, zz);
#pragma unroll
        for (int t = 0; t < MT; ++t) g1[t] = zero;
        W2.add(form, lane, gg, g1);
        if (TWO || p.masked) mask_rows<MT>(g1, zz);
        patch_fence(); // keeps weight fragments and patches in LDS, and what follows below
        if constexpr (!TWO) {
            next_g();
            next_z();
            if (p.out) store_frags<MT>(p.out + g * (256 * MT), lane, rows, g1);
            clear_past_end<MT>(lane, rows, g1); // zeros times an infinite weight are no zeros
#pragma unroll
            for (int t = 0; t < MT; ++t) csum[t] += g1[t];
            turned_product<BT, MT>(patch, lane, acc2, sum2);
        } else {
            next_g();
            if constexpr (!kLateZ) next_z();
            turned_product<BT, MT>(patch, lane, acc2, sum2);
            patch_fence();
            frags_to_patch<MT, LZ>(patch, lane, g1);
            piece_to_patch<AT, LA>(patch + 16 * LZ, lane, aa);
            patch_fence();
            if (p.H) load_frags<AT>(p.H + g * (256 * AT), lane, rows, aa);
            f4 da[AT];
#pragma unroll
            for (int t = 0; t < AT; ++t) da[t] = zero;
            W1.add(form, lane, g1, da);
            if (p.H && (rows >= 16 || (lane & 15) < rows)) {
#pragma unroll
                for (int t = 0; t < AT; ++t)
                    dot += (da[t][0] * aa[t][0] + da[t][1] * aa[t][1]) + (da[t][2] * aa[t][2] + da[t][3] * aa[t][3]);
            }
            if constexpr (kLateZ) next_z();
            next_a();
            if (p.out) store_frags<AT>(p.out + g * (256 * AT), lane, rows, da);
            patch_fence();
            turned_product<MT, AT>(patch, lane, acc1, sum1);
        }
    };
    if (g < full && in_pieces) {
        load_g(g, kWhole);
        load_z(g, kWhole);
        load_a(g, kWhole);
    }
    for (; g < full && in_pieces; g += stride) {
        if (kSplit && !small_rows(gg)) {
            in_pieces = false;
            break;
        }
        const long after = g + stride < full ? g + stride : g;
        step(kInPieces, g, kWhole, [&] { load_g(after, kWhole); }, [&] { load_z(after, kWhole); }, [&] { load_a(after, kWhole); });
    }
    auto load_all = [&](long g, auto rows) {
        load_g(g, rows);
        load_z(g, rows);
        load_a(g, rows);
    };
    if (const long rows = p.n - g * 16; rows > 0 && in_pieces) { // the rows that are left over
        load_all(g, rows);
        in_pieces = !kSplit || small_rows(gg);
        if (in_pieces) step(kInPieces, g, rows, [] {}, [] {}, [] {});
    }
    if constexpr (kSplit) {
        for (; !in_pieces && g * 16 < p.n; g += stride) {
            load_all(g, p.n - g * 16);
            step(kAsTheyAre, g, p.n - g * 16, [] {}, [] {}, [] {});
        }
    }

    float *ws = p.ws + (long)blockIdx.x * p.ws_stride;
    collect<BT, MT>(lds, acc2, sum2, ws, ws + BT * MT * 256);
    ws += BT * MT * 256 + BT * 16;
    if constexpr (TWO) {
        collect<MT, AT>(lds, acc1, sum1, ws, ws + MT * AT * 256);
        collect_dot(lds, dot, ws + MT * AT * 256 + MT * 16);
    } else {
        collect_colsum<MT, true>(lds, csum, ws);
    }
}

// Bound by memory whatever the layout.  Arrays larger than the memory-side cache leave it as they are read (2,000,000 rows, 16 x 64
// 114 -> 104 us, 128 x 16 194 -> 170, 32 x 32 91 -> 82; 300,000 rows, which fit, are 3-4 % slower so at 128 x 16, and left there
// for the next kernel).  Only a side that one square reads: the others' reads come from L2 (128 x 32 215 -> 190 us, with both sides
// 222), and so does the rest of a line of 128 bytes that two squares of 48 columns share (in a training step of 2,000,000 rows 96 x
// 16 192 us so, 172 kept).  Wider shapes lose (96 x 96 398 -> 483).
constexpr bool wgrad_light(int tg, int tx) { return tg * tx <= 8; }
constexpr long kMemorySideCache = 256l << 20;

struct WgradArgs {
    long n;
    int a, b;
    const float *G, *X;
    float *ws; // per workgroup: b*a of dW, then b column sums
    int sums;
    int squares_x;      // of dW, side by side along X: 1 or 2
    int squares;        // of a workgroup: 1, 2 or 4; grid.y has the others
    int once_g, once_x; // nothing will be read again that is read of G / of X
    long unchecked;     // rows before which a lane may read past the end of its row
};

// dW = G^T X: the rows are the k of the matrix instruction, four per instruction.  A lane reads T consecutive columns of a row
// (T*(l%16) and on), which feed T tiles: tile t holds the columns T*i + t.  A wavefront keeps up to 64 x 64 of dW in its
// accumulators and walks 16 rows a step; the rows of the next two steps are on their way (requested right after the products that
// free their registers: no copies between two sets).  Weights wider than 64 are cut into two or four squares.  Long inputs:
// workgroups of eight wavefronts take all squares over the same rows.  Short ones are in the caches, and what a workgroup leaves
// costs more than the second read of them: four wavefronts to a square, fewer partial dW of fewer rows each.  Rows are dealt to 512
// to 2048 wavefronts.  Those of a workgroup and square are added through LDS, and each workgroup leaves one partial of its squares,
// summed by sum_partials_kernel in a fixed order.  Whole steps read without conditions.  Where a width is rounded up, lanes past the
// end of a row read the next one's columns, whose sums nobody stores; the last rows, where that would pass the end of the array,
// and steps of fewer rows take loads that check both.  Four-byte addresses do for loads of any width.  2,000,000 rows, with the sums,
// beside conditions on every load and squares of 64 as workgroups of their own: 128 x 128 676 -> 581 us (matrix cores 78 % busy at
// 2.0 GHz), 96 x 96 692 -> 389, 64 x 64 203 -> 182, 48 x 48 187 -> 139, 128 x 16 187 -> 170, 16 x 64 108 -> 104; 32,768 rows: 128 x
// 128 23.9 -> 23.1, 64 x 128 18.0 -> 15.9, 96 x 96 22.7 -> 16.4.  torch's product of the transposed G takes 2900 at 64 x 64.
template <int TG, int TX>
__global__ void __launch_bounds__(2 * 64 * kWaves, 2) wgrad_kernel(WgradArgs p)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;
    const int squares = p.squares, row_waves = (int)(blockDim.x >> 6) / squares;
    const int square = wave & (squares - 1), row_wave = wave / squares, of_dw = (int)blockIdx.y * squares + square;
    const int g0 = of_dw / p.squares_x * TG * 16, x0 = of_dw % p.squares_x * TX * 16;

    f4 acc[TG][TX];
    float gsum[TG];
#pragma unroll
    for (int i = 0; i < TG; ++i) {
        gsum[i] = 0.0f;
#pragma unroll
        for (int j = 0; j < TX; ++j) acc[i][j] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    constexpr int U = 4; // 4 x 4 rows per step
    const unsigned gat = 4u * (unsigned)(q * p.b + g0 + TG * c), xat = 4u * (unsigned)(q * p.a + x0 + TX * c);
    struct Rows {
        float g[U][TG], x[U][TX];
    };
    auto fetch = [&](long row0, Rows &r, auto once_g, auto once_x) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float *g = reinterpret_cast<const float *>(reinterpret_cast<const char *>(p.G + (row0 + 4 * u) * p.b) + gat);
            const float *x = reinterpret_cast<const float *>(reinterpret_cast<const char *>(p.X + (row0 + 4 * u) * p.a) + xat);
#pragma unroll
            for (int i = 0; i < TG; ++i) r.g[u][i] = once_g ? __builtin_nontemporal_load(g + i) : g[i];
#pragma unroll
            for (int j = 0; j < TX; ++j) r.x[u][j] = once_x ? __builtin_nontemporal_load(x + j) : x[j];
        }
    };
    auto fetch_checked = [&](long row0, Rows &r) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long row = row0 + 4 * u + q;
#pragma unroll
            for (int i = 0; i < TG; ++i) {
                const int col = g0 + TG * c + i;
                const bool in = row < p.n && col < p.b;
                const float v = p.G[in ? row * p.b + col : 0];
                r.g[u][i] = in ? v : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < TX; ++j) {
                const int col = x0 + TX * c + j;
                const bool in = row < p.n && col < p.a;
                const float v = p.X[in ? row * p.a + col : 0];
                r.x[u][j] = in ? v : 0.0f;
            }
        }
    };
    auto products = [&](const Rows &r) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int i = 0; i < TG; ++i) {
                gsum[i] += r.g[u][i];
#pragma unroll
                for (int j = 0; j < TX; ++j) acc[i][j] = mfma4(r.g[u][i], r.x[u][j], acc[i][j]);
            }
        }
    };
    const long step = (long)gridDim.x * row_waves * 4 * U;
    const long whole = p.unchecked - 4 * U; // the last row a step may begin at
    long row0 = ((long)blockIdx.x * row_waves + row_wave) * 4 * U;
    Rows r[kWgradAhead];
    auto walk = [&](auto once_g, auto once_x) {
#pragma unroll
        for (int d = 0; d < kWgradAhead; ++d)
            if (row0 + d * step <= whole) fetch(row0 + d * step, r[d], once_g, once_x);
        for (; row0 + (kWgradAhead - 1) * step <= whole; row0 += kWgradAhead * step) {
#pragma unroll
            for (int d = 0; d < kWgradAhead; ++d) {
                products(r[d]);
                const long next = row0 + (d + kWgradAhead) * step;
                asm volatile("" ::: "memory"); // requested here, not where they are used
                fetch(next <= whole ? next : row0, r[d], once_g, once_x);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int d = 0; d < kWgradAhead; ++d)
            if (row0 <= whole) {
                products(r[d]);
                row0 += step;
            }
    };
    const std::true_type yes;
    const std::false_type no;
    if constexpr (wgrad_light(TG, TX)) {
        if (p.once_g && p.once_x)
            walk(yes, yes);
        else if (p.once_g)
            walk(yes, no);
        else if (p.once_x)
            walk(no, yes);
        else
            walk(no, no);
    } else {
        walk(no, no);
    }
    for (; row0 < p.n; row0 += step) {
        fetch_checked(row0, r[0]);
        products(r[0]);
    }

#pragma unroll
    for (int i = 0; i < TG; ++i) {
        gsum[i] += __shfl_xor(gsum[i], 16);
        gsum[i] += __shfl_xor(gsum[i], 32);
    }
    float *out = p.ws + (long)blockIdx.x * ((long)p.b * p.a + p.b);
    float *sums = p.sums && x0 == 0 ? out + (long)p.b * p.a : nullptr;
    // The wavefronts of a square, in order, lane by lane as they hold it; the last one ends with the sum.
    __shared__ f4 red[4][TG * TX * 64];
    __shared__ float gred[2 * kWaves][TG * 16];
    if (q == 0) {
#pragma unroll
        for (int i = 0; i < TG; ++i) gred[wave][TG * c + i] = gsum[i];
    }
    f4 *held = red[square] + lane;
    for (int w = 0; w < row_waves; ++w) {
        if (row_wave == w) {
            if (w) {
                f4 t[TG][TX]; // requested together
#pragma unroll
                for (int i = 0; i < TG; ++i)
#pragma unroll
                    for (int j = 0; j < TX; ++j) t[i][j] = held[(i * TX + j) * 64];
#pragma unroll
                for (int i = 0; i < TG; ++i)
#pragma unroll
                    for (int j = 0; j < TX; ++j) acc[i][j] = t[i][j] + acc[i][j];
            }
            if (w + 1 < row_waves) {
#pragma unroll
                for (int i = 0; i < TG; ++i)
#pragma unroll
                    for (int j = 0; j < TX; ++j) held[(i * TX + j) * 64] = acc[i][j];
            }
        }
        __syncthreads();
    }
    if (row_wave == row_waves - 1) {
#pragma unroll
        for (int i = 0; i < TG; ++i) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int row = g0 + (4 * q + s) * TG + i, col = x0 + TX * c;
                if (row < p.b) {
#pragma unroll
                    for (int j = 0; j < TX; ++j)
                        if (col + j < p.a) out[(long)row * p.a + col + j] = acc[i][j][s];
                }
            }
        }
    }
    if (sums && row_wave == 0 && lane < TG * 16 && g0 + lane < p.b) {
        float t = gred[wave][lane];
        for (int w = 1; w < row_waves; ++w) t += gred[wave + w * squares][lane];
        sums[g0 + lane] = t;
    }
}

// out[e] = sum over the parts of ws[part*len + e] for e < n0 (dst0), then dst1: 16 threads per
// element, each every 16th part in order, the 16 sums in order.  Eight loads in flight: 512 parts of 64 x 64 in 5 us
// where one after the other took 10.
__global__ void __launch_bounds__(256) sum_partials_kernel(const float *ws, int parts, long stride, long n0, float *dst0,
                                                           long n1, float *dst1)
{
    __shared__ float sh[16][17];
    const int c = threadIdx.x & 15, j = threadIdx.x >> 4;
    const long e = (long)blockIdx.x * 16 + c;
    float t = 0.0f;
    if (e < n0 + n1) {
        int s = j;
        for (; s + 7 * 16 < parts; s += 8 * 16) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = ws[(s + k * 16) * stride + e];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] += v[k + 4];
            t += (v[0] + v[2]) + (v[1] + v[3]);
        }
        for (; s < parts; s += 16) t += ws[s * stride + e];
    }
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
template <int KT, int NT> LinearFn pick_linear(int mode, bool red)
{
    if (mode == 2) return red ? &piece_kernel<KT, NT, true> : &piece_kernel<KT, NT, false>;
    if (mode == 1) return red ? &linear_kernel<KT, NT, true, true> : &linear_kernel<KT, NT, true, false>;
    if constexpr (KT != 3 && KT != 6 && NT != 3 && NT != 6)
        return red ? &linear_kernel<KT, NT, false, true> : &linear_kernel<KT, NT, false, false>;
    return nullptr;
}
template <int KT> LinearFn pick_linear_n(int nt, int mode, bool red)
{
    switch (nt) {
    case 1: return pick_linear<KT, 1>(mode, red);
    case 2: return pick_linear<KT, 2>(mode, red);
    case 3: return pick_linear<KT, 3>(mode, red);
    case 4: return pick_linear<KT, 4>(mode, red);
    case 6: return pick_linear<KT, 6>(mode, red);
    case 8: return pick_linear<KT, 8>(mode, red);
    }
    return nullptr;
}
LinearFn pick_linear_kn(int kt, int nt, int mode, bool red)
{
    switch (kt) {
    case 1: return pick_linear_n<1>(nt, mode, red);
    case 2: return pick_linear_n<2>(nt, mode, red);
    case 3: return pick_linear_n<3>(nt, mode, red);
    case 4: return pick_linear_n<4>(nt, mode, red);
    case 6: return pick_linear_n<6>(nt, mode, red);
    case 8: return pick_linear_n<8>(nt, mode, red);
    }
    return nullptr;
}

using WgradFn = void (*)(WgradArgs);
// Squares of one side of the weight gradient, and their tiles: as few columns of padding as two squares allow.
// 2,000,000 rows, 96 x 96: 48 + 48 columns a side 473 us, 64 + 64 (the work of 128 x 128) 700.
int wgrad_squares(int w) { return w > 64 ? 2 : 1; }
int wgrad_tiles(int w)
{
    const int squares = wgrad_squares(w);
    return (w + 16 * squares - 1) / (16 * squares);
}
template <int TG> WgradFn pick_wgrad_x(int tx)
{
    switch (tx) {
    case 1: return &wgrad_kernel<TG, 1>;
    case 2: return &wgrad_kernel<TG, 2>;
    case 3: return &wgrad_kernel<TG, 3>;
    }
    return &wgrad_kernel<TG, 4>;
}
WgradFn pick_wgrad(int tg, int tx)
{
    switch (tg) {
    case 1: return pick_wgrad_x<1>(tx);
    case 2: return pick_wgrad_x<2>(tx);
    case 3: return pick_wgrad_x<3>(tx);
    }
    return pick_wgrad_x<4>(tx);
}

// workgroups for groups of 16 rows, one wavefront each
long row_blocks(long n, long most, int waves = kWaves)
{
    const long blocks = ((n + 15) / 16 + waves - 1) / waves;
    return blocks < 1 ? 1 : (blocks > most ? most : blocks);
}

// 16, 32, 48 or 64: tiles of the fused kernels, else 0
int exact_tiles(int w) { return w > 0 && w <= 64 && w % 16 == 0 ? w / 16 : 0; }
bool aligned16(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

using MlpFn = void (*)(MlpArgs);
template <int KT> MlpFn pick_mlp_m(int mt)
{
    switch (mt) {
    case 1: return &mlp_kernel<KT, 1>;
    case 2: return &mlp_kernel<KT, 2>;
    case 3: return &mlp_kernel<KT, 3>;
    case 4: return &mlp_kernel<KT, 4>;
    }
    return nullptr;
}
using BackFn = void (*)(BackArgs);
template <int MT> BackFn pick_back_two(int at)
{
    switch (at) {
    case 1: return &back_kernel<MT, MT, 1, true>;
    case 2: return &back_kernel<MT, MT, 2, true>;
    case 3: return &back_kernel<MT, MT, 3, true>;
    case 4: return &back_kernel<MT, MT, 4, true>;
    }
    return nullptr;
}
template <int BT> BackFn pick_back_one(int mt)
{
    switch (mt) {
    case 1: return &back_kernel<BT, 1, 1, false>;
    case 2: return &back_kernel<BT, 2, 1, false>;
    case 3: return &back_kernel<BT, 3, 1, false>;
    case 4: return &back_kernel<BT, 4, 1, false>;
    }
    return nullptr;
}

bool width_ok(int w) { return w > 0 && w <= PCSR_GNN_MAX_WIDTH; }

} // namespace

extern "C" {

int64_t pcsr_gnn_workspace_floats(int32_t a, int32_t b)
{
    if (!width_ok(a) || !width_ok(b)) return 0;
    const int64_t wgrad = (int64_t)kWgradBlocks * ((int64_t)a * b + b), linear = (int64_t)kLinearBlocks * (b + 1);
    const int64_t col = (int64_t)kColsumBlocks * (a > b ? a : b);
    const int64_t side = a > b ? a : b, back = (int64_t)kBackBlocks * (side * b + side * a + 2 * side + 64);
    int64_t most = wgrad > linear ? wgrad : linear;
    most = most > back ? most : back;
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
    const int kt = tiles(a, vec), nt = tiles(b, vec);
    const bool exact = vec && a == 16 * kt && b == 16 * nt;
    LinearFn fn = pick_linear_kn(kt, nt, exact ? 2 : vec, red);
    if (!fn) return PCSR_E_UNSUPPORTED;
    const int waves = exact ? piece_waves(kt, nt) : kWaves;
    const long blocks = row_blocks(n, 256 * (exact ? piece_blocks_per_cu(kt, nt, red, mask != nullptr) : blocks_per_cu(kt, nt)), waves);
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
    hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(64 * waves), 0, s, p);
    int rc = to_code(hipGetLastError());
    if (rc == PCSR_OK && colsum_out) rc = sum_partials(p.ws_colsum, (int)blocks, b, b, colsum_out, 0, nullptr, s);
    if (rc == PCSR_OK && dot_out) rc = sum_partials(p.ws_dot, (int)blocks, 1, 1, dot_out, 0, nullptr, s);
    return rc;
}

int pcsr_gnn_mlp(int64_t n, int32_t a, int32_t m, const float *X, const float *W1, const float *b1, const float *W2,
                 const float *b2, int32_t relu, float *Z, float *Y, void *stream)
{
    if (n < 0 || !X || !W1 || !W2 || !Z || !Y) return PCSR_E_INVALID_ARG;
    const int kt = exact_tiles(a), mt = exact_tiles(m);
    if (!kt || !mt || !aligned16(X) || !aligned16(Z) || !aligned16(Y)) return PCSR_E_UNSUPPORTED;
    MlpFn fn = kt == 1 ? pick_mlp_m<1>(mt) : kt == 2 ? pick_mlp_m<2>(mt) : kt == 3 ? pick_mlp_m<3>(mt) : pick_mlp_m<4>(mt);
    const MlpArgs p = {(long)n, relu, X, W1, b1, W2, b2, Z, Y};
    hipLaunchKernelGGL(fn, dim3((unsigned)row_blocks(n, 256 * mlp_blocks_per_cu(kt, mt))), dim3(64 * kWaves), 0, static_cast<hipStream_t>(stream), p);
    return to_code(hipGetLastError());
}

int pcsr_gnn_mlp_backward(int64_t n, int32_t a, int32_t m, const float *G, const float *Z, const float *A,
                          const float *H, const float *W1, const float *W2, float *dA, float *dW1, float *db1,
                          float *dW2, float *db2, float *dot, float *ws, void *stream)
{
    if (n < 0 || !G || !Z || !A || !W1 || !W2 || !dW1 || !db1 || !dW2 || !db2 || (dot && !H) || !ws)
        return PCSR_E_INVALID_ARG;
    const int at = exact_tiles(a), mt = exact_tiles(m);
    if (!at || !mt || !aligned16(G) || !aligned16(Z) || !aligned16(A) || !aligned16(H) || !aligned16(dA))
        return PCSR_E_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    BackFn fn = mt == 1   ? pick_back_two<1>(at)
                : mt == 2 ? pick_back_two<2>(at)
                : mt == 3 ? pick_back_two<3>(at)
                          : pick_back_two<4>(at);
    const long n2 = (long)m * m, n1 = (long)m * a, len = n2 + m + n1 + m + 1;
    BackArgs p = {};
    p.n = n;
    p.G = G;
    p.Z = Z;
    p.W2 = W2;
    p.A = A;
    p.H = dot ? H : nullptr;
    p.W1 = W1;
    p.out = dA;
    p.ws = ws;
    p.ws_stride = len;
    const long blocks = row_blocks(n, kBackBlocks);
    hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, p);
    int rc = to_code(hipGetLastError());
    if (rc == PCSR_OK) rc = sum_partials(ws, (int)blocks, len, n2, dW2, m, db2, s);
    if (rc == PCSR_OK) rc = sum_partials(ws + n2 + m, (int)blocks, len, n1, dW1, m, db1, s);
    if (rc == PCSR_OK && dot) rc = sum_partials(ws + len - 1, (int)blocks, len, 1, dot, 0, nullptr, s);
    return rc;
}

int pcsr_gnn_linear_backward(int64_t n, int32_t a, int32_t b, const float *G, const float *X, const float *W,
                             int32_t masked, float *dX, float *dW, float *db, float *colsum, float *ws, void *stream)
{
    if (n < 0 || !G || !X || !W || !dW || !ws) return PCSR_E_INVALID_ARG;
    const int bt = exact_tiles(b), at = exact_tiles(a);
    if (!bt || !at || !aligned16(G) || !aligned16(X) || !aligned16(dX)) return PCSR_E_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    BackFn fn = bt == 1   ? pick_back_one<1>(at)
                : bt == 2 ? pick_back_one<2>(at)
                : bt == 3 ? pick_back_one<3>(at)
                          : pick_back_one<4>(at);
    const long n2 = (long)a * b, len = n2 + b + a;
    BackArgs p = {};
    p.n = n;
    p.masked = masked;
    p.G = G;
    p.Z = X;
    p.W2 = W;
    p.out = dX;
    p.ws = ws;
    p.ws_stride = len;
    const long blocks = row_blocks(n, kBackBlocks);
    hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(64 * kWaves), 0, s, p);
    int rc = to_code(hipGetLastError());
    if (rc == PCSR_OK) rc = sum_partials(ws, (int)blocks, len, n2, dW, db ? b : 0, db, s);
    if (rc == PCSR_OK && colsum) rc = sum_partials(ws + n2 + b, (int)blocks, len, a, colsum, 0, nullptr, s);
    return rc;
}

int pcsr_gnn_wgrad(int64_t n, int32_t a, int32_t b, const float *G, const float *X, float *dW, float *db,
                   float *ws, void *stream)
{
    if (n < 0 || !G || !X || !dW || !ws) return PCSR_E_INVALID_ARG;
    if (!width_ok(a) || !width_ok(b)) return PCSR_E_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int tg = wgrad_tiles(b), tx = wgrad_tiles(a);
    WgradArgs p;
    const int squares_g = wgrad_squares(b), squares_x = wgrad_squares(a), all = squares_g * squares_x;
    // Squares as workgroups of their own, where dW is cut, up to 131,072 rows (us beside all squares in one: 128 x 128 32,768 rows
    // 23.1 / 27.3, 65,536 31.8 / 35.4, 131,072 49.1 / 52.3; 64 x 128 15.9 / 20.1, 23.8 / 23.5 and 32.5 / 32.2; 300,000 rows, the
    // old form, 112 / 101 and 62 / 55).
    const bool apart = all == 1 || n <= (1 << 17);
    const int waves = apart ? kWaves : 2 * kWaves;
    const long most = kWgradBlocks / (apart ? all : 2);
    long blocks = (n + 64 * kWaves - 1) / (64 * kWaves); // at least four steps of 16 rows per wavefront of a square of its own
    blocks = blocks < 1 ? 1 : (blocks > most ? most : blocks);
    const bool large = (double)n * 4.0 * (a + b) > (double)kMemorySideCache;
    p.squares_x = squares_x;
    p.squares = apart ? 1 : all;
    p.once_g = large && squares_x == 1 && (squares_g == 1 || tg % 2 == 0);
    p.once_x = large && squares_g == 1 && (squares_x == 1 || tx % 2 == 0);
    // rows that the columns past a row's end reach into
    const long past_g = (16 * tg * squares_g - 1) / b, past_x = (16 * tx * squares_x - 1) / a;
    p.unchecked = n - (past_g > past_x ? past_g : past_x);
    p.n = n;
    p.a = a;
    p.b = b;
    p.G = G;
    p.X = X;
    p.ws = ws;
    p.sums = db != nullptr;
    hipLaunchKernelGGL(pick_wgrad(tg, tx), dim3((unsigned)blocks, (unsigned)(all / p.squares)), dim3(64 * waves), 0, s, p);
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
