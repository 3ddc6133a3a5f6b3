// Learned per-column correction: coarsening, column features, a three-layer
// perceptron trained and evaluated with BF16 matrix-core (MFMA) products and
// FP32 accumulation, Adam in FP32, and the application of the predicted
// tendencies to a coarse state.
//
// Matrix products use gfx950's v_mfma_f32_16x16x32_bf16: one instruction
// adds a 16 x 32 by 32 x 16 BF16 product to a 16 x 16 FP32 tile.  Every
// operand is kept with its contraction index contiguous and padded to 32
// (activations and errors also transposed, for the weight gradients; weights
// in both orders), so that a lane reads its eight values of an MFMA operand as
// one 16-byte word straight from memory: the network is small (395 -> 256 ->
// 256 -> 237), its operands stay in L2, and what bounds a product is the
// latency of its loads, which are issued several chunks ahead.
#include <cmath>
#include <cstdint>
#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "fv3_internal.hpp"

namespace fv3 {

#define DEVI __device__ __forceinline__

typedef uint16_t bf16_t;
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// round to nearest even, the bit-exact rounding the oracle applies
DEVI bf16_t to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return (bf16_t)((u >> 16) | 0x40);
    uint32_t lsb = (u >> 16) & 1u;
    u += 0x7fffu + lsb;
    return (bf16_t)(u >> 16);
}

// ------------------------------------------------------------- products
constexpr int PADK = 32;   // widths and the transposed row count are padded to this
constexpr int pad32(int x) { return (x + PADK - 1) / PADK * PADK; }

// acc[x][y] += A rows m0 + 16 x .. by B rows n0 + 16 y .. over K (a multiple
// of 32), both with k contiguous.  Chunks of 32 in ascending order, one MFMA
// per chunk and tile; the loads of PF chunks are in flight ahead of them.
template <int TM, int TN, int PF>
DEVI void product(const bf16_t *A, long lda, const bf16_t *B, long ldb, int m0, int n0, int K, v4f (&acc)[TM][TN])
{
    const int lane = (int)threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const bf16_t *pa[TM], *pb[TN];
#pragma unroll
    for (int x = 0; x < TM; x++) pa[x] = A + (long)(m0 + 16 * x + r) * lda + 8 * g;
#pragma unroll
    for (int y = 0; y < TN; y++) pb[y] = B + (long)(n0 + 16 * y + r) * ldb + 8 * g;
    const int nc = K / 32;
    v8s ca[PF][TM], cb[PF][TN], na[PF][TM], nb_[PF][TN];
    auto load = [&](int c0, v8s (&a)[PF][TM], v8s (&b)[PF][TN]) {
#pragma unroll
        for (int q = 0; q < PF; q++) {
            const long o = 32L * min(c0 + q, nc - 1);   // chunks past the end repeat the last and are not used
#pragma unroll
            for (int x = 0; x < TM; x++) a[q][x] = *(const v8s *)(pa[x] + o);
#pragma unroll
            for (int y = 0; y < TN; y++) b[q][y] = *(const v8s *)(pb[y] + o);
        }
    };
    load(0, ca, cb);
    for (int c0 = 0; c0 < nc; c0 += PF) {
        if (c0 + PF < nc) load(c0 + PF, na, nb_);
#pragma unroll
        for (int q = 0; q < PF; q++) {
            if (c0 + q < nc) {
#pragma unroll
                for (int x = 0; x < TM; x++)
#pragma unroll
                    for (int y = 0; y < TN; y++)
                        acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(v8bf, ca[q][x]), __builtin_bit_cast(v8bf, cb[q][y]), acc[x][y], 0, 0, 0);
            }
        }
#pragma unroll
        for (int q = 0; q < PF; q++) {
#pragma unroll
            for (int x = 0; x < TM; x++) ca[q][x] = na[q][x];
#pragma unroll
            for (int y = 0; y < TN; y++) cb[q][y] = nb_[q][y];
        }
    }
}

// Epilogue outputs of a layer product; null pointers are skipped.  Rows from
// `rows` up to the next multiple of 32 are zero in the transposed copies (they
// are contracted over).
struct LayerOut {
    float *f;          // FP32 [row][ld]
    bf16_t *b, *bt;    // BF16 [row][ld] and [column][ldt]
    int ld;
    long ldt;
};
enum { LY_TANH = 0, LY_OUT = 1, LY_LOSS = 2, LY_BACK = 3 };

// One layer over all rows: 64 x 64 per block, 32 x 32 per wavefront (1024
// wavefronts at 4096 x 256).
//   LY_TANH  tanh(x W + b)
//   LY_OUT   x W + b into Y (rows x out)
//   LY_LOSS  error of the mean squared loss, scale (x W + b - T), and the
//            squared residuals summed per row and 16 columns
//   LY_BACK  (error W^T) (1 - h^2), h the layer's FP32 activation
// One wavefront tile takes four chunks ahead: 13 chunks are 4 load latencies
// instead of 13 with two barriers each (55 -> 24 us at 13824 x 256 x 400).
template <int KIND>
__global__ void __launch_bounds__(256) k_layer(int rows, int N, int K, const bf16_t *A, long lda, const bf16_t *B,
                                               long ldb, const float *bias, const float *h, LayerOut O, float *Y,
                                               const float *T, int out, float scale, float *sq)
{
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int m0 = (int)blockIdx.y * 64 + (w >> 1) * 32, n0 = (int)blockIdx.x * 64 + (w & 1) * 32;
    if (m0 >= pad32(rows) || n0 >= N) return;
    v4f acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; x++)
#pragma unroll
        for (int y = 0; y < 2; y++) acc[x][y] = v4f{0.f, 0.f, 0.f, 0.f};
    product<2, 2, 4>(A, lda, B, ldb, m0, n0, K, acc);
    // a lane holds rows 4g .. 4g + 3 of column r of each 16 x 16 tile
#pragma unroll
    for (int x = 0; x < 2; x++)
#pragma unroll
        for (int y = 0; y < 2; y++) {
            const int n = n0 + 16 * y + r;
            const float bn = KIND == LY_BACK ? 0.f : bias[n];
            bf16_t tb[4];
            float s4[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int m = m0 + 16 * x + 4 * g + q;
                const bool in = m < rows;
                float v = acc[x][y][q];
                s4[q] = 0.f;
                if constexpr (KIND == LY_TANH) v = tanhf(v + bn);
                if constexpr (KIND == LY_OUT) {
                    if (in && n < out) Y[(long)m * out + n] = v + bn;
                }
                if constexpr (KIND == LY_LOSS) {
                    const bool real = in && n < out;
                    const float res = real ? v + bn - T[(long)m * out + n] : 0.f;
                    v = scale * res;
                    s4[q] = res * res;
                }
                if constexpr (KIND == LY_BACK) {
                    const float a = in ? h[(long)m * O.ld + n] : 0.f;
                    v = v * (1.f - a * a);
                }
                if constexpr (KIND != LY_OUT) {
                    const bf16_t hb = to_bf16(v);
                    if (in) {
                        if (O.f) O.f[(long)m * O.ld + n] = v;
                        if (O.b) O.b[(long)m * O.ld + n] = hb;
                    }
                    tb[q] = in ? hb : (bf16_t)0;
                }
            }
            if constexpr (KIND != LY_OUT) {
                typedef bf16_t b4 __attribute__((ext_vector_type(4)));
                if (O.bt) *(b4 *)(O.bt + (long)n * O.ldt + m0 + 16 * x + 4 * g) = b4{tb[0], tb[1], tb[2], tb[3]};
            }
            if constexpr (KIND == LY_LOSS) {
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    float s = s4[q];
                    for (int d = 8; d > 0; d >>= 1) s += __shfl_xor(s, d, 16);
                    const int m = m0 + 16 * x + 4 * g + q;
                    if (r == 0 && m < rows) sq[(long)m * (N / 16) + (n0 + 16 * y) / 16] = s;
                }
            }
        }
}

// Weight gradients of the three layers in one launch: gW = (inputs)^T
// (errors), contracted over the rows, one 16 x 16 tile per wavefront (about
// 930 wavefronts; whole 64 x 64 tiles would be 16 blocks a layer, each with
// the serial walk of all rows), eight chunks of loads ahead.
struct GradW {
    const bf16_t *a[3], *b[3];
    float *g[3];
    int mt[3], nt[3];   // 16 x 16 tiles
};
__global__ void __launch_bounds__(256) k_wgrad(int K, long ldt, GradW G)
{
    const int lane = (int)threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    int u = (int)blockIdx.x * 4 + ((int)threadIdx.x >> 6), l = 0;
    while (l < 3 && u >= G.mt[l] * G.nt[l]) {
        u -= G.mt[l] * G.nt[l];
        l++;
    }
    if (l == 3) return;
    const bf16_t *a = l == 0 ? G.a[0] : l == 1 ? G.a[1] : G.a[2], *b = l == 0 ? G.b[0] : l == 1 ? G.b[1] : G.b[2];
    float *c = l == 0 ? G.g[0] : l == 1 ? G.g[1] : G.g[2];
    const int nt = l == 0 ? G.nt[0] : l == 1 ? G.nt[1] : G.nt[2];
    const int m0 = 16 * (u / nt), n0 = 16 * (u % nt);
    v4f acc[1][1] = {{v4f{0.f, 0.f, 0.f, 0.f}}};
    product<1, 1, 8>(a, ldt, b, ldt, m0, n0, K, acc);
#pragma unroll
    for (int q = 0; q < 4; q++) c[(long)(m0 + 4 * g + q) * (16 * nt) + n0 + r] = acc[0][0][q];
}

// ------------------------------------------------------------ elementwise
// rows x cols FP32 to BF16 [row][ldy], columns padded with zeros, and (yt)
// transposed [column][ldt] with zeros in rows .. pad32(rows)
__global__ void __launch_bounds__(256) k_to_bf16(const float *x, int rows, int cols, bf16_t *y, int ldy, bf16_t *yt,
                                                 long ldt)
{
    __shared__ bf16_t t[64][66];
    const int r0 = (int)blockIdx.y * 64, c0 = (int)blockIdx.x * 64, tx = (int)threadIdx.x & 63, ty = (int)threadIdx.x >> 6;
#pragma unroll 4
    for (int q = 0; q < 16; q++) {
        const int r = r0 + ty + 4 * q, c = c0 + tx;
        const bf16_t v = r < rows && c < cols ? to_bf16(x[(long)r * cols + c]) : (bf16_t)0;
        if (r < rows && c < ldy) y[(long)r * ldy + c] = v;
        t[ty + 4 * q][tx] = v;
    }
    if (!yt) return;
    __syncthreads();
#pragma unroll 4
    for (int q = 0; q < 16; q++) {
        const int c = c0 + ty + 4 * q, r = r0 + tx;
        if (c < ldy && r < pad32(rows)) yt[(long)c * ldt + r] = t[tx][ty + 4 * q];
    }
}

// Bias gradients: column sums of the errors of the three layers in two
// deterministic passes: partial sums of 256-row chunks in row order (threads
// along columns, 16 rows of loads ahead of the sum), then the chunks in order.
struct ColSum {
    const float *x[3];
    int ld[3], cb[3];   // width, blocks of 64 columns
    float *part;        // [layer][chunk][column], layers `stride` apart
    long stride;
};
__global__ void __launch_bounds__(64) k_colsum_partial(ColSum S, int rows)
{
    int b = (int)blockIdx.x, l = 0;
    while (b >= (l == 0 ? S.cb[0] : l == 1 ? S.cb[1] : S.cb[2])) {
        b -= l == 0 ? S.cb[0] : S.cb[1];
        l++;
    }
    const float *x = l == 0 ? S.x[0] : l == 1 ? S.x[1] : S.x[2];
    const int ld = l == 0 ? S.ld[0] : l == 1 ? S.ld[1] : S.ld[2];
    const int c = b * 64 + (int)threadIdx.x;
    if (c >= ld) return;
    const int r0 = (int)blockIdx.y * 256, r1 = min(rows, r0 + 256);
    float s = 0.f;
    for (int r = r0; r < r1; r += 16) {
        float v[16];
#pragma unroll
        for (int q = 0; q < 16; q++) v[q] = x[(long)min(r + q, r1 - 1) * ld + c];
#pragma unroll
        for (int q = 0; q < 16; q++)
            if (r + q < r1) s += v[q];
    }
    S.part[l * S.stride + (long)blockIdx.y * ld + c] = s;
}
DEVI float colsum_final(const float *part, int chunks, int ld, int c)
{
    float s = 0.f;
    for (int q = 0; q < chunks; q++) s += part[(long)q * ld + c];
    return s;
}

// The parameters of the three layers as one list of elements: per layer the
// padded weight matrix, then the bias.
struct Params {
    float *W[3], *b[3], *mW[3], *vW[3], *mb[3], *vb[3], *gW[3], *gb[3];
    bf16_t *Wb[3], *WbT[3];
    int kp[3], np[3];      // padded input and output widths
    int in[3], on[3];      // true widths
    const float *part;     // bias gradient partials (or null: gb is given)
    long stride;
    int chunks;
};
// bias gradients from their partials
__global__ void k_bias_final(Params P)
{
    const int l = (int)blockIdx.y, c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (c < P.np[l]) P.gb[l][c] = colsum_final(P.part + l * P.stride, P.chunks, P.np[l], c);
}
// Adam on the FP32 master parameters (all layers, one launch); refreshes both
// BF16 copies of the weights; bias gradients are summed from their partials
__global__ void __launch_bounds__(256) k_adam(Params P, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int l = (int)blockIdx.y;
    const long wc = (long)P.kp[l] * P.np[l], e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= wc + P.np[l]) return;
    const bool isw = e < wc;
    const long q = isw ? e : e - wc;
    float gg;
    if (isw) {
        gg = P.gW[l][q];
    } else {
        gg = colsum_final(P.part + l * P.stride, P.chunks, P.np[l], (int)q);
        P.gb[l][q] = gg;
    }
    float *p = isw ? P.W[l] : P.b[l], *m = isw ? P.mW[l] : P.mb[l], *v = isw ? P.vW[l] : P.vb[l];
    float mm = b1 * m[q] + (1.f - b1) * gg;
    float vv = b2 * v[q] + (1.f - b2) * gg * gg;
    m[q] = mm;
    v[q] = vv;
    float mh = mm / c1, vh = vv / c2;
    float pn = p[q] - lr * mh / (sqrtf(vh) + eps);
    p[q] = pn;
    if (isw) {
        const bf16_t h = to_bf16(pn);
        const int r = (int)(q / P.np[l]), c = (int)(q - (long)r * P.np[l]);
        P.Wb[l][q] = h;
        P.WbT[l][(long)c * P.kp[l] + r] = h;
    }
}

// true-size parameters (or gradients) to one packed array and back: W1 (in x
// h1), b1, W2, b2, W3, b3, row-major
__global__ void k_pack(Params P, int grads, float *flat)
{
    const int l = (int)blockIdx.y;
    long off = 0;
    for (int k = 0; k < l; k++) off += (long)P.in[k] * P.on[k] + P.on[k];
    const long wc = (long)P.in[l] * P.on[l], e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= wc + P.on[l]) return;
    const float *W = grads ? P.gW[l] : P.W[l], *b = grads ? P.gb[l] : P.b[l];
    flat[off + e] = e < wc ? W[e / P.on[l] * P.np[l] + e % P.on[l]] : b[e - wc];
}
// packed parameters into the padded arrays, Adam state reset
__global__ void k_unpack(Params P, const float *flat)
{
    const int l = (int)blockIdx.y;
    long off = 0;
    for (int k = 0; k < l; k++) off += (long)P.in[k] * P.on[k] + P.on[k];
    const long wc = (long)P.kp[l] * P.np[l], e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= wc + P.np[l]) return;
    if (e < wc) {
        const int r = (int)(e / P.np[l]), c = (int)(e - (long)r * P.np[l]);
        const float v = r < P.in[l] && c < P.on[l] ? flat[off + (long)r * P.on[l] + c] : 0.f;
        P.W[l][e] = v;
        P.mW[l][e] = P.vW[l][e] = 0.f;
        P.Wb[l][e] = to_bf16(v);
        P.WbT[l][(long)c * P.kp[l] + r] = to_bf16(v);
    } else {
        const int c = (int)(e - wc);
        P.b[l][c] = c < P.on[l] ? flat[off + (long)P.in[l] * P.on[l] + c] : 0.f;
        P.mb[l][c] = P.vb[l][c] = 0.f;
    }
}

// sum of the squared residuals in FP64, one block, fixed order (16 loads
// ahead of the sums: 62 -> 9 us for 65536 values)
__global__ void __launch_bounds__(1024) k_loss(const float *sq, long count, double *loss)
{
    __shared__ double s[1024];
    double a = 0.0;
    for (long e0 = threadIdx.x; e0 < count; e0 += 16 * 1024) {
        float v[16];
#pragma unroll
        for (int q = 0; q < 16; q++) v[q] = e0 + q * 1024 < count ? sq[e0 + q * 1024] : 0.f;
#pragma unroll
        for (int q = 0; q < 16; q++) a += (double)v[q];
    }
    s[threadIdx.x] = a;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = s[0];
}

}  // namespace fv3

// ====================================================================
// network object
// ====================================================================
struct fv3_mlp {
    int in, h1, h2, out;        // true sizes
    int limit, maxrows;         // most rows of a call; rows the arrays hold
    long step, ldt;             // Adam steps taken; row stride of the transposed arrays
    fv3::Params P;              // parameters, Adam moments, gradients, BF16 copies
    // activations and errors for up to maxrows rows: FP32, BF16, BF16 transposed
    fv3::bf16_t *Xb, *XbT, *H1b, *H1bT, *H2b, *H2bT, *dYb, *dYbT, *dZ2b, *dZ2bT, *dZ1bT;
    float *H1, *H2, *dY, *dZ2, *dZ1, *sq, *part, *flat;
    double *loss;
    int device;
    mutable std::mutex mu;      // `flat` holds one download at a time
};

namespace fv3 {
namespace {

template <class T>
bool dalloc(T **p, long count)
{
    if (hipMalloc((void **)p, count * sizeof(T)) != hipSuccess) return false;
    return hipMemset(*p, 0, count * sizeof(T)) == hipSuccess;
}

template <int KIND>
void layer(int rows, int N, int K, const bf16_t *A, const bf16_t *B, const float *bias, const float *h,
           const LayerOut &O, float *Y, const float *T, int out, float scale, float *sq, hipStream_t st)
{
    dim3 grd((unsigned)((N + 63) / 64), (unsigned)((rows + 63) / 64));
    hipLaunchKernelGGL(k_layer<KIND>, grd, dim3(256), 0, st, rows, N, K, A, (long)K, B, (long)K, bias, h, O, Y, T, out,
                       scale, sq);
}

// forward pass on `rows` rows of X (FP32, in columns): with Y the outputs,
// else the activations the backward pass needs and the output errors
void forward(fv3_mlp *n, const float *X, int rows, float *Y, const float *T, hipStream_t st)
{
    const bool train = Y == nullptr;
    const Params &P = n->P;
    hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)((P.kp[0] + 63) / 64), (unsigned)((rows + 63) / 64)), dim3(256), 0, st,
                       X, rows, n->in, n->Xb, P.kp[0], train ? n->XbT : nullptr, n->ldt);
    layer<LY_TANH>(rows, P.np[0], P.kp[0], n->Xb, P.WbT[0], P.b[0], nullptr,
                   LayerOut{train ? n->H1 : nullptr, n->H1b, train ? n->H1bT : nullptr, P.np[0], n->ldt}, nullptr, nullptr,
                   0, 0.f, nullptr, st);
    layer<LY_TANH>(rows, P.np[1], P.kp[1], n->H1b, P.WbT[1], P.b[1], nullptr,
                   LayerOut{train ? n->H2 : nullptr, n->H2b, train ? n->H2bT : nullptr, P.np[1], n->ldt}, nullptr, nullptr,
                   0, 0.f, nullptr, st);
    if (!train)
        layer<LY_OUT>(rows, P.np[2], P.kp[2], n->H2b, P.WbT[2], P.b[2], nullptr, LayerOut{}, Y, nullptr, n->out, 0.f,
                      nullptr, st);
    else
        layer<LY_LOSS>(rows, P.np[2], P.kp[2], n->H2b, P.WbT[2], P.b[2], nullptr,
                       LayerOut{n->dY, n->dYb, n->dYbT, P.np[2], n->ldt}, nullptr, T, n->out,
                       2.0f / (float)((long)rows * n->out), n->sq, st);
}

// gradients of the mean squared error over rows x out: gW, and the partials
// of the bias gradients
void backward(fv3_mlp *n, int rows, hipStream_t st)
{
    Params &P = n->P;
    layer<LY_BACK>(rows, P.np[1], P.np[2], n->dYb, P.Wb[2], nullptr, n->H2,
                   LayerOut{n->dZ2, n->dZ2b, n->dZ2bT, P.np[1], n->ldt}, nullptr, nullptr, 0, 0.f, nullptr, st);
    layer<LY_BACK>(rows, P.np[0], P.np[1], n->dZ2b, P.Wb[1], nullptr, n->H1,
                   LayerOut{n->dZ1, nullptr, n->dZ1bT, P.np[0], n->ldt}, nullptr, nullptr, 0, 0.f, nullptr, st);
    GradW G{{n->XbT, n->H1bT, n->H2bT}, {n->dZ1bT, n->dZ2bT, n->dYbT}, {P.gW[0], P.gW[1], P.gW[2]}, {}, {}};
    ColSum S{{n->dZ1, n->dZ2, n->dY}, {}, {}, n->part, P.stride};
    int tiles = 0, cbs = 0;
    for (int l = 0; l < 3; l++) {
        G.mt[l] = P.kp[l] / 16;
        G.nt[l] = P.np[l] / 16;
        tiles += G.mt[l] * G.nt[l];
        S.ld[l] = P.np[l];
        S.cb[l] = (P.np[l] + 63) / 64;
        cbs += S.cb[l];
    }
    P.chunks = (rows + 255) / 256;
    hipLaunchKernelGGL(k_wgrad, dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, st, pad32(rows), n->ldt, G);
    hipLaunchKernelGGL(k_colsum_partial, dim3((unsigned)cbs, (unsigned)P.chunks), dim3(64), 0, st, S, rows);
}

// launch over the elements of every layer's weights and bias
dim3 param_grid(const Params &P, bool padded)
{
    long most = 0;
    for (int l = 0; l < 3; l++) {
        const long c = padded ? (long)P.kp[l] * P.np[l] + P.np[l] : (long)P.in[l] * P.on[l] + P.on[l];
        most = c > most ? c : most;
    }
    return dim3((unsigned)((most + 255) / 256), 3);
}

}  // namespace
}  // namespace fv3

using namespace fv3;

namespace {
fv3_status mfail(fv3_status s, const char *m) { return set_error(s, m); }

bool on_device(const fv3_mlp *n)
{
    int cur = -1;
    return hipGetDevice(&cur) == hipSuccess && cur == n->device;
}

// The parameter transfers may be called with any device current: the
// network's for the duration of one, then the caller's again.
struct OnDevice {
    int prev = -1;
    bool ok, moved = false;
    explicit OnDevice(const fv3_mlp *n)
    {
        ok = hipGetDevice(&prev) == hipSuccess;
        if (ok && prev != n->device) ok = moved = hipSetDevice(n->device) == hipSuccess;
    }
    ~OnDevice()
    {
        if (moved) (void)hipSetDevice(prev);
    }
};

// parameters (or gradients) of the padded arrays into `flat`
bool pack(const fv3_mlp *n, int grads, hipStream_t st)
{
    Params P = n->P;
    float *flat = n->flat;
    void *a[] = {&P, &grads, &flat};
    return hipLaunchKernel((const void *)k_pack, param_grid(P, false), dim3(256), a, 0, st) == hipSuccess;
}
// `flat` into the padded arrays
bool unpack(fv3_mlp *n, hipStream_t st)
{
    Params P = n->P;
    const float *flat = n->flat;
    void *a[] = {&P, &flat};
    return hipLaunchKernel((const void *)k_unpack, param_grid(P, true), dim3(256), a, 0, st) == hipSuccess;
}
}  // namespace

extern "C" {

fv3_status fv3_mlp_create(int in, int h1, int h2, int out, int maxrows, const float *params, fv3_mlp **outp)
{
    if (!outp || !params || in < 1 || h1 < 16 || h2 < 16 || out < 1 || maxrows < 1 || (h1 % 16) || (h2 % 16))
        return mfail(FV3_EINVAL, "bad network sizes (hidden widths must be multiples of 16)");
    fv3_mlp *n = new fv3_mlp();
    n->in = in; n->h1 = h1; n->h2 = h2; n->out = out;
    n->limit = (maxrows + 15) / 16 * 16;
    n->maxrows = (maxrows + 63) / 64 * 64;   // whole product tiles
    n->ldt = n->maxrows;
    n->step = 0;
    if (hipGetDevice(&n->device) != hipSuccess) {
        delete n;
        return mfail(FV3_EDEVICE, "no current HIP device");
    }
    Params &P = n->P;
    const int wi[3] = {in, h1, h2}, wo[3] = {h1, h2, out};
    bool ok = true;
    int wmax = 0;
    long flat = 0;
    for (int l = 0; l < 3; l++) {
        P.in[l] = wi[l];
        P.on[l] = wo[l];
        P.kp[l] = pad32(wi[l]);
        P.np[l] = pad32(wo[l]);
        wmax = std::max(wmax, std::max(P.kp[l], P.np[l]));
        flat += (long)wi[l] * wo[l] + wo[l];
        // operand rows are read in whole tiles of up to 64
        const long kr = (P.kp[l] + 63) / 64 * 64, nr = (P.np[l] + 63) / 64 * 64, wc = (long)P.kp[l] * P.np[l];
        ok = ok && dalloc(&P.W[l], wc) && dalloc(&P.mW[l], wc) && dalloc(&P.vW[l], wc) && dalloc(&P.gW[l], wc) &&
             dalloc(&P.b[l], P.np[l]) && dalloc(&P.mb[l], P.np[l]) && dalloc(&P.vb[l], P.np[l]) &&
             dalloc(&P.gb[l], P.np[l]) && dalloc(&P.Wb[l], kr * P.np[l]) && dalloc(&P.WbT[l], nr * P.kp[l]);
    }
    const long R = n->maxrows, X = P.kp[0], A = P.np[0], B = P.np[1], O = P.np[2];
    P.stride = (R / 256 + 1) * (long)wmax;
    ok = ok && dalloc(&n->Xb, R * X) && dalloc(&n->XbT, R * X) && dalloc(&n->H1b, R * A) && dalloc(&n->H1bT, R * A) &&
         dalloc(&n->H2b, R * B) && dalloc(&n->H2bT, R * B) && dalloc(&n->dYb, R * O) && dalloc(&n->dYbT, R * O) &&
         dalloc(&n->dZ2b, R * B) && dalloc(&n->dZ2bT, R * B) && dalloc(&n->dZ1bT, R * A) && dalloc(&n->H1, R * A) &&
         dalloc(&n->H2, R * B) && dalloc(&n->dY, R * O) && dalloc(&n->dZ2, R * B) && dalloc(&n->dZ1, R * A) &&
         dalloc(&n->sq, R * (O / 16)) && dalloc(&n->part, 3 * P.stride) && dalloc(&n->flat, flat) &&
         dalloc(&n->loss, 1);
    P.part = n->part;
    if (!ok) {
        fv3_mlp_free(n);
        return mfail(FV3_ENOMEM, "device allocation failed");
    }
    *outp = n;
    fv3_status s = fv3_mlp_set_params(n, params);
    if (s != FV3_OK) {
        fv3_mlp_free(n);
        *outp = nullptr;
    }
    return s;
}

fv3_status fv3_mlp_free(fv3_mlp *n)
{
    if (!n) return FV3_OK;
    (void)hipDeviceSynchronize();
    const Params &P = n->P;
    for (int l = 0; l < 3; l++) {
        void *ps[] = {P.W[l], P.b[l], P.mW[l], P.vW[l], P.mb[l], P.vb[l], P.gW[l], P.gb[l], P.Wb[l], P.WbT[l]};
        for (void *p : ps)
            if (p) (void)hipFree(p);
    }
    void *ps[] = {n->Xb, n->XbT, n->H1b, n->H1bT, n->H2b, n->H2bT, n->dYb, n->dYbT, n->dZ2b, n->dZ2bT, n->dZ1bT,
                  n->H1, n->H2, n->dY, n->dZ2, n->dZ1, n->sq, n->part, n->flat, n->loss};
    for (void *p : ps)
        if (p) (void)hipFree(p);
    delete n;
    return FV3_OK;
}

// packed parameter order: W1 (in x h1), b1, W2 (h1 x h2), b2, W3 (h2 x out), b3, row-major, unpadded
static long packed_count(const fv3_mlp *n)
{
    return (long)n->in * n->h1 + n->h1 + (long)n->h1 * n->h2 + n->h2 + (long)n->h2 * n->out + n->out;
}

fv3_status fv3_mlp_set_params(fv3_mlp *n, const float *params)
{
    if (!n || !params) return mfail(FV3_EINVAL, "NULL argument");
    std::lock_guard<std::mutex> lock(n->mu);
    OnDevice dev(n);
    if (!dev.ok || hipDeviceSynchronize() != hipSuccess ||
        hipMemcpy(n->flat, params, (size_t)packed_count(n) * 4, hipMemcpyHostToDevice) != hipSuccess ||
        !unpack(n, nullptr))
        return mfail(FV3_EDEVICE, "parameter upload failed");
    n->step = 0;
    return hipDeviceSynchronize() == hipSuccess ? FV3_OK : mfail(FV3_EDEVICE, "sync failed");
}

fv3_status fv3_mlp_get_params(const fv3_mlp *n, float *params)
{
    if (!n || !params) return mfail(FV3_EINVAL, "NULL argument");
    std::lock_guard<std::mutex> lock(n->mu);
    OnDevice dev(n);
    if (!dev.ok || hipDeviceSynchronize() != hipSuccess) return mfail(FV3_EDEVICE, "sync failed");
    if (!pack(n, 0, nullptr) || hipMemcpy(params, n->flat, (size_t)packed_count(n) * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return mfail(FV3_EDEVICE, "parameter download failed");
    return FV3_OK;
}

long fv3_mlp_param_count(const fv3_mlp *n) { return n ? packed_count(n) : 0; }

fv3_status fv3_mlp_forward(fv3_mlp *n, const float *X, int rows, float *Y, void *stream)
{
    if (!n || !X || !Y || rows < 1 || rows > n->limit) return mfail(FV3_EINVAL, "bad arguments");
    if (!on_device(n)) return mfail(FV3_EDEVICE, "current HIP device differs from the network's device");
    hipStream_t st = (hipStream_t)stream;
    forward(n, X, rows, Y, nullptr, st);
    return hipGetLastError() == hipSuccess ? FV3_OK : mfail(FV3_EDEVICE, "launch failed");
}

fv3_status fv3_mlp_gradients(fv3_mlp *n, const float *X, const float *T, int rows, float *grads, void *stream)
{
    if (!n || !X || !T || !grads || rows < 1 || rows > n->limit) return mfail(FV3_EINVAL, "bad arguments");
    if (!on_device(n)) return mfail(FV3_EDEVICE, "current HIP device differs from the network's device");
    hipStream_t st = (hipStream_t)stream;
    forward(n, X, rows, nullptr, T, st);
    backward(n, rows, st);
    int wmax = std::max(n->P.np[0], std::max(n->P.np[1], n->P.np[2]));
    hipLaunchKernelGGL(k_bias_final, dim3((unsigned)((wmax + 63) / 64), 3), dim3(64), 0, st, n->P);
    std::lock_guard<std::mutex> lock(n->mu);
    if (!pack(n, 1, st) || hipMemcpyAsync(grads, n->flat, (size_t)packed_count(n) * 4, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return mfail(FV3_EDEVICE, "gradient download failed");
    return FV3_OK;
}

fv3_status fv3_mlp_train_step(fv3_mlp *n, const float *X, const float *T, int rows, float lr, double *loss,
                              void *stream)
{
    if (!n || !X || !T || rows < 1 || rows > n->limit) return mfail(FV3_EINVAL, "bad arguments");
    if (!on_device(n)) return mfail(FV3_EDEVICE, "current HIP device differs from the network's device");
    hipStream_t st = (hipStream_t)stream;
    forward(n, X, rows, nullptr, T, st);
    backward(n, rows, st);
    n->step++;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    float c1 = 1.f - powf(b1, (float)n->step), c2 = 1.f - powf(b2, (float)n->step);
    hipLaunchKernelGGL(k_adam, param_grid(n->P, true), dim3(256), 0, st, n->P, lr, b1, b2, eps, c1, c2);
    if (loss) {
        hipLaunchKernelGGL(k_loss, dim3(1), dim3(1024), 0, st, (const float *)n->sq, (long)rows * (n->P.np[2] / 16), n->loss);
        double s = 0.0;
        if (hipMemcpyAsync(&s, n->loss, sizeof(s), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return mfail(FV3_EDEVICE, "loss read failed");
        *loss = s / ((double)rows * n->out);
    }
    return hipGetLastError() == hipSuccess ? FV3_OK : mfail(FV3_EDEVICE, "launch failed");
}

}  // extern "C"
