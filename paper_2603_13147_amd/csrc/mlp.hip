// mlp.hip - the learned scheduler's network on gfx950: forward, loss,
// backward and Adam kernels for training, and the per-round trace features.
//
// Network: 12 round features -> 64 -> 64 -> 5 outputs, ReLU hidden layers.
// Weights are kept in FP32 (master copy) and used as BF16 (round to nearest
// even) in every product; inputs and hidden activations are rounded to BF16;
// accumulation is FP32.  The outputs are a push logit, a dense logit and
// three delta-class logits.
//
// Both training passes run on the matrix cores, one wave per tile of 16
// rows.  The forward pass is three BF16 products with FP32 accumulation
// (v_mfma_f32_16x16x16_bf16): the BF16 inputs and weights are exactly the
// values the network defines, and the products of two BF16 values are exact
// in FP32.  Each hidden layer goes through the wave's LDS tile between the
// accumulator layout of one product and the operand layout of the next.
// The backward pass keeps the gradient signals in FP32 (the straight-through
// rule passes them unrounded), so its products are FP32 ones
// (v_mfma_f32_16x16x4_f32): dH2 = dL W3, dH1 = dZ2 W2, and the weight
// gradients dZ^T H summed over the wave's tiles in accumulators; the waves
// of a workgroup are reduced in LDS and each workgroup adds one value per
// parameter to the global gradient.
//
// The features of a traced round are computed by the same device function the
// sweep uses when it decides that round, so a network trained on trace
// features sees exactly the inputs it is given at decision time.
#include <math.h>
#include <string.h>

#include "llp_host.h"
#include "llp_sched.h"

namespace llp {

constexpr int NI = LLP_MLP_IN, NH = LLP_MLP_HID, NO = LLP_MLP_OUT;
constexpr int OFF_W1 = 0, OFF_B1 = NH * NI, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH, OFF_W3 = OFF_B2 + NH,
              OFF_B3 = OFF_W3 + NO * NH, NPAR = OFF_B3 + NO;
static_assert(NPAR == LLP_MLP_PARAMS, "parameter layout");

// Rounding to bf16 (nearest even) by the conversion instruction: the same
// values as f32_to_bf16, a sixth of the code.
__device__ __forceinline__ unsigned short bf16_bits(float f) { return __builtin_bit_cast(unsigned short, (__bf16)f); }
__device__ __forceinline__ float bf16_round(float f) { return (float)(__bf16)f; }
__device__ __forceinline__ float bfw(const float* p, int i) { return bf16_round(p[i]); }

constexpr int MB = 256;            // threads per workgroup
constexpr int MW = MB / LLP_WAVE;  // waves per workgroup
constexpr int MT = 16;             // rows per tile (the matrix products' M)

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Operand layouts of the two products, for lane l (wave64):
//   16x16x16 bf16: A[i][k] at i = l % 16, k = 4 (l / 16) + q (q = 0..3);
//                  B[k][j] at k = 4 (l / 16) + q, j = l % 16
//   16x16x4 f32:   A[i][k] at i = l % 16, k = l / 16; B[k][j] at k = l / 16, j = l % 16
//   both:          D[i][j] at i = 4 (l / 16) + q, j = l % 16
__device__ __forceinline__ f32x4 mma_bf16(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ short bfbits(float f) { return (short)bf16_bits(f); }

// 16 bytes at any address (the caller's arrays are only aligned to their type).
template <class V>
__device__ __forceinline__ V ld16(const void* p) {
    V v;
    __builtin_memcpy(&v, p, 16);
    return v;
}
__device__ __forceinline__ bf16x4 bf4(f32x4 f) {
    bf16x4 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = bfbits(f[q]);
    return r;
}
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave per workgroup: the waves share nothing, and a small batch then
// spreads over as many CUs as it has tiles.  A lane's operands are four
// consecutive values of a weight row, read 16 bytes at a time with no branch
// between the loads, and the activations leave by whole 32-byte pieces of
// their rows: 859 rows 4.1 us (14.9 with a load, and a
// branch, per value), 2^18 rows 30 (65).  A small batch's time is that of
// fetching the code once, so the conversions use the packed instruction.
// act[row][0..63] = h1, act[row][64..127] = h2 (bf16 bits)
__global__ void __launch_bounds__(LLP_WAVE) k_mlp_forward(int B, const float* P, const float* X, float* logits,
                                                          unsigned short* act) {
    __shared__ __align__(16) unsigned short h[MT * NH];   // the hidden tile, row-major
    const int l = lane();
    const int lr = l & 15, lg = l >> 4;          // operand row / column, and k group
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    // B operands (the transposed weights), as bf16; rows of W1 have 12 values
    bf16x4 bw1[4], bw2[4][4], bw3[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const f32x4 f = ld16<f32x4>(P + OFF_W1 + (nt * 16 + lr) * NI + 4 * min(lg, 2));
        bw1[nt] = bf4(lg < 3 ? f : z);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) bw2[ks][nt] = bf4(ld16<f32x4>(P + OFF_W2 + (nt * 16 + lr) * NH + ks * 16 + 4 * lg));
        const f32x4 f = ld16<f32x4>(P + OFF_W3 + min(lr, NO - 1) * NH + ks * 16 + 4 * lg);
        bw3[ks] = bf4(lr < NO ? f : z);
    }
    float b1[4], b2[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        b1[nt] = bfw(P, OFF_B1 + nt * 16 + lr);
        b2[nt] = bfw(P, OFF_B2 + nt * 16 + lr);
    }
    const float b3 = bfw(P, OFF_B3 + min(lr, NO - 1));
    const int ntiles = (B + MT - 1) / MT;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const long long r0 = (long long)tile * MT;
        // layer 1: X (16 x 12, padded to 16) times W1^T; rows past the batch repeat its last
        const long long xr = r0 + lr < B ? r0 + lr : B - 1;
        const f32x4 xf = ld16<f32x4>(X + xr * NI + 4 * min(lg, 2));
        const bf16x4 ax = bf4(lg < 3 ? xf : z);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const f32x4 d = mma_bf16(ax, bw1[nt], z);
#pragma unroll
            for (int q = 0; q < 4; ++q) h[(4 * lg + q) * NH + nt * 16 + lr] = bf16_bits(fmaxf(d[q] + b1[nt], 0.f));
        }
        // the hidden layers: the tile in LDS turns the accumulator layout into
        // the operand layout of the next product
#pragma unroll
        for (int layer = 0; layer < 2; ++layer) {
            wave_lds_sync();
            bf16x4 ah[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) ah[ks] = *(const bf16x4*)(h + lr * NH + ks * 16 + 4 * lg);
            // this layer's activations to act (rows of the tile inside the batch):
            // lane l has 16 values of row l / 4
            const uint4 a0 = *(const uint4*)(h + l * 16), a1 = *(const uint4*)(h + l * 16 + 8);
            const long long row = r0 + (l >> 2);
            if (row < B) {
                unsigned short* dst = act + row * 2 * NH + layer * NH + (l & 3) * 16;
                __builtin_memcpy(dst, &a0, 16);
                __builtin_memcpy(dst + 8, &a1, 16);
            }
            wave_lds_sync();
            if (layer == 0) {
                // layer 2: H1 W2^T
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) {
                    f32x4 d = z;
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) d = mma_bf16(ah[ks], bw2[ks][nt], d);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        h[(4 * lg + q) * NH + nt * 16 + lr] = bf16_bits(fmaxf(d[q] + b2[nt], 0.f));
                }
            } else {
                // layer 3: H2 W3^T (5 of 16 columns used)
                f32x4 d = z;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) d = mma_bf16(ah[ks], bw3[ks], d);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const long long row = r0 + 4 * lg + q;
                    if (row < B && lr < NO) logits[row * NO + lr] = d[q] + b3;
                }
            }
        }
    }
}

// Loss over the batch: mean of BCE(o0, push) + BCE(o1, dense) +
// softmax-CE(o2..o4, delta class).  labels are round codes: mode in bits 0-1
// (2 = push, 1 = dense), delta class in bits 8-9.  d = d loss / d logits of a
// row (scaled by inv); returns the row's term.
__device__ __forceinline__ float loss_row(const float* o, int code, float inv, float (&d)[NO]) {
    const int mode = code & 3, dc = min((code >> 8) & 3, 2);
    const float y0 = mode == 2 ? 1.f : 0.f, y1 = mode == 1 ? 1.f : 0.f;
    // numerically stable BCE with logits: max(o,0) - o*y + log(1 + exp(-|o|))
    float l = 0.f;
    for (int k = 0; k < 2; ++k) {
        const float z = o[k], y = k == 0 ? y0 : y1;
        l += fmaxf(z, 0.f) - z * y + log1pf(expf(-fabsf(z)));
        const float s = 1.f / (1.f + expf(-z));
        d[k] = (s - y) * inv;
    }
    const float mx = fmaxf(o[2], fmaxf(o[3], o[4]));
    const float e2 = expf(o[2] - mx), e3 = expf(o[3] - mx), e4 = expf(o[4] - mx);
    const float se = e2 + e3 + e4;
    const float lse = mx + logf(se);
    l += lse - o[2 + dc];
    d[2] = (e2 / se - (dc == 0 ? 1.f : 0.f)) * inv;
    d[3] = (e3 / se - (dc == 1 ? 1.f : 0.f)) * inv;
    d[4] = (e4 / se - (dc == 2 ? 1.f : 0.f)) * inv;
    return l;
}

// The workgroup's rows [r0, r1): writes dL where store is set; their terms'
// sum, valid in thread 0.  Deterministic.
__device__ float loss_rows(long long r0, long long r1, float inv, const float* L, const int* labels, float* dL,
                           bool store, float* part) {
    float acc = 0.f;
    for (long long row = r0 + threadIdx.x; row < r1; row += blockDim.x) {
        float d[NO];
        acc += loss_row(L + row * NO, labels[row], inv, d);
        if (store)
#pragma unroll
            for (int k = 0; k < NO; ++k) dL[row * NO + k] = d[k];
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, LLP_WAVE);
    if (lane() == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    float t = 0.f;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) t += part[k];
    return t;
}

// One workgroup for up to LOSS_ONE rows.  A larger batch takes three launches,
// with a workgroup per LOSS_CHUNK rows: each leaves its rows' sum in the first
// gradient of its rows (k_mlp_loss_part), one workgroup adds the sums
// (k_mlp_loss_sum), and the gradients are written (k_mlp_loss_grad).  Gradients
// written over the logits themselves take one workgroup at any size, as the
// sums would replace logits still to be read.  859 rows:
// 5.1 us in one launch; 2^18 rows: 11 us against 664 in one workgroup.
constexpr int LOSS_ONE = 4096;
constexpr int LOSS_CHUNK = 1024;

__global__ void __launch_bounds__(1024) k_mlp_loss(int B, const float* L, const int* labels, float* dL, float* loss) {
    __shared__ float part[1024 / LLP_WAVE];
    const float inv = 1.f / (float)(B > 0 ? B : 1);
    const float t = loss_rows(0, B, inv, L, labels, dL, true, part);
    if (threadIdx.x == 0) *loss = t * inv;
}

__global__ void __launch_bounds__(256) k_mlp_loss_part(int B, const float* L, const int* labels, float* dL) {
    __shared__ float part[256 / LLP_WAVE];
    const long long r0 = (long long)blockIdx.x * LOSS_CHUNK, r1 = min(r0 + LOSS_CHUNK, (long long)B);
    const float t = loss_rows(r0, r1, 1.f / (float)B, L, labels, dL, false, part);
    if (threadIdx.x == 0) dL[r0 * NO] = t;
}

__global__ void __launch_bounds__(1024) k_mlp_loss_sum(int B, const float* dL, float* loss) {
    __shared__ float part[1024 / LLP_WAVE];
    const int chunks = (int)(((long long)B + LOSS_CHUNK - 1) / LOSS_CHUNK);
    float acc = 0.f;
    for (int c = threadIdx.x; c < chunks; c += 1024) acc += dL[(long long)c * LOSS_CHUNK * NO];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, LLP_WAVE);
    if (lane() == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int k = 0; k < 1024 / LLP_WAVE; ++k) t += part[k];
        *loss = t * (1.f / (float)B);
    }
}

__global__ void __launch_bounds__(256) k_mlp_loss_grad(int B, const float* L, const int* labels, float* dL) {
    const long long row = (long long)blockIdx.x * 256 + threadIdx.x;
    if (row >= B) return;
    float d[NO];
    loss_row(L + row * NO, labels[row], 1.f / (float)B, d);
#pragma unroll
    for (int k = 0; k < NO; ++k) dL[row * NO + k] = d[k];
}

// Backward: grad += d loss / d params (straight through the bf16 rounding).
// Per tile of 16 rows, with each wave's tiles in LDS as FP32 (rows past the
// batch are zero and contribute nothing):
//   dH2 = dL W3 (K = 5, padded to 8), dZ2 = dH2 where H2 > 0;
//   gW3 += dL^T H2, gW2 += dZ2^T H1;
//   dH1 = dZ2 W2 (W2 from LDS), dZ1 = dH1 where H1 > 0; gW1 += dZ1^T X;
//   the biases' gradients are the column sums of dL, dZ2 and dZ1.
// A small batch is one tile per wave, a chain of LDS reads and FP32 matrix
// products behind one fetch of the code: loads go 16 bytes at a time, all in
// flight, and the loops over K stay rolled.  A large one is bound by those
// products at two waves a SIMD (the registers allow no more) and by the
// workgroups' atomic adds to the same 5317 words: 859 rows 12.0 us (42.3 with
// a load per value and LDS atomics for the waves' sums), 2^18 rows 104 (239).
struct __align__(16) BwdWave {
    float x[MT][16];              // bf16 inputs, columns 12..15 zero
    float d[MT][8];               // dL, columns 5..7 zero
    unsigned short h1[MT][NH];    // bf16 bits as stored by the forward pass
    unsigned short h2[MT][NH];
    float z[MT][NH];              // dZ2, then dZ1
};
struct BwdSums {   // one wave's: 16 tiles of dW2, 4 each of dW1 and dW3, and the biases
    f32x4 tile[24][LLP_WAVE];
    f32x4 bias[LLP_WAVE];
};
struct BwdShared {
    union {
        struct {
            float w2[NH * NH];  // bf16 W2, row-major [out][in]
            BwdWave wv[MW];
        };
        BwdSums sums[MW / 2];
    };
};

static_assert(sizeof(BwdShared) <= 64 * 1024, "backward LDS within the default per-workgroup limit");

__global__ void __launch_bounds__(MB, 2) k_mlp_backward(int B, const float* P, const float* X,
                                                     const unsigned short* act, const float* dL, float* grad) {
    extern __shared__ __align__(16) unsigned char smem[];
    BwdShared& sh = *reinterpret_cast<BwdShared*>(smem);
    const int l = lane(), w = threadIdx.x >> 6;
    const int lr = l & 15, lg = l >> 4;
    // W2, 16 bytes per thread and load, all in flight
    f32x4 w2[NH * NH / 4 / MB];
#pragma unroll
    for (int i = 0; i < NH * NH / 4 / MB; ++i) w2[i] = ld16<f32x4>(P + OFF_W2 + 4 * (threadIdx.x + i * MB));
    // W3 as the B operand of dH2 = dL W3: B[k][j] = W3[k][j], k = ks * 4 + lg (< 5)
    float bw3[2][4];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int k = ks * 4 + lg;
            const float f = bfw(P, OFF_W3 + min(k, NO - 1) * NH + nt * 16 + lr);
            bw3[ks][nt] = k < NO ? f : 0.f;
        }
#pragma unroll
    for (int i = 0; i < NH * NH / 4 / MB; ++i) {
        f32x4 f;
#pragma unroll
        for (int q = 0; q < 4; ++q) f[q] = bf16_round(w2[i][q]);
        *(f32x4*)(sh.w2 + 4 * (threadIdx.x + i * MB)) = f;
    }
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    f32x4 g2[4][4], g1[4], g3[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        g1[a] = z;
        g3[a] = z;
#pragma unroll
        for (int b = 0; b < 4; ++b) g2[a][b] = z;
    }
    float gb1 = 0.f, gb2 = 0.f, gb3 = 0.f;   // lane l: column l (gb3: l < 5)
    __syncthreads();
    BwdWave& t = sh.wv[w];
    const int ntiles = (B + MT - 1) / MT;
    for (int tile = blockIdx.x * MW + w; tile < ntiles; tile += gridDim.x * MW) {
        const long long r0 = (long long)tile * MT;
        // the tile's rows into LDS, the lane's pieces loaded together: 64 bytes
        // of the 256 of activation row l / 4, 16 of the 48 of input row l / 3,
        // and two of the tile's 80 logit gradients; rows past the batch are zero
        {
            const int ar = l >> 2, ap = l & 3, xr = min(l / 3, MT - 1), xp = l % 3;
            const bool ain = r0 + ar < B, xin = l < 48 && r0 + xr < B;
            const unsigned short* asrc = act + (ain ? r0 + ar : 0) * 2 * NH + ap * 32;
            uint4 av[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i] = ld16<uint4>(asrc + 8 * i);
            const f32x4 xv = ld16<f32x4>(X + (xin ? r0 + xr : 0) * NI + 4 * xp);
            const int last = (int)min((long long)MT, B - r0) * NO;   // the tile's gradients
            const float d0 = dL[r0 * NO + min(l, last - 1)], d1 = dL[r0 * NO + min(l + 64, last - 1)];
            unsigned short* ah = ap < 2 ? &t.h1[ar][ap * 32] : &t.h2[ar][(ap - 2) * 32];
#pragma unroll
            for (int i = 0; i < 4; ++i) *(uint4*)(ah + 8 * i) = ain ? av[i] : make_uint4(0u, 0u, 0u, 0u);
            f32x4 xw;
#pragma unroll
            for (int q = 0; q < 4; ++q) xw[q] = xin ? bf16_round(xv[q]) : 0.f;
            *(f32x4*)(l < 48 ? &t.x[xr][4 * xp] : &t.x[l - 48][12]) = xw;
            t.d[l / NO][l % NO] = l < last ? d0 : 0.f;
            if (l < MT * NO - 64) t.d[(l + 64) / NO][(l + 64) % NO] = l + 64 < last ? d1 : 0.f;
            if (l < MT) t.d[l][5] = t.d[l][6] = t.d[l][7] = 0.f;
        }
        wave_lds_sync();
        // dZ2 = (dL W3) where H2 > 0
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            f32x4 d = z;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) d = mma_f32(t.d[lr][ks * 4 + lg], bw3[ks][nt], d);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = 4 * lg + q, c = nt * 16 + lr;
                t.z[row][c] = bf16_to_f32(t.h2[row][c]) > 0.f ? d[q] : 0.f;
            }
        }
        wave_lds_sync();
        // gW3 += dL^T H2 (rows of the output: 5 of 16) and gW2 += dZ2^T H1, K = the tile's rows
#pragma unroll 1
        for (int ks = 0; ks < 4; ++ks) {
            const int k = ks * 4 + lg;
            const float a3 = lr < 8 ? t.d[k][lr] : 0.f;
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                g3[nt] = mma_f32(a3, bf16_to_f32(t.h2[k][nt * 16 + lr]), g3[nt]);
                const float b = bf16_to_f32(t.h1[k][nt * 16 + lr]);
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) g2[mt][nt] = mma_f32(t.z[k][mt * 16 + lr], b, g2[mt][nt]);
            }
        }
        // bias gradients: column sums
        {
            float s2 = 0.f;
            for (int row = 0; row < MT; ++row) s2 += t.z[row][l];
            gb2 += s2;
        }
        if (l < NO) {
            float s3 = 0.f;
            for (int row = 0; row < MT; ++row) s3 += t.d[row][l];
            gb3 += s3;
        }
        // dZ1 = (dZ2 W2) where H1 > 0, into the dZ2 tile once every lane has read it
        f32x4 dh[4] = {z, z, z, z};
#pragma unroll 2
        for (int ks = 0; ks < 16; ++ks) {
            const float a = t.z[lr][ks * 4 + lg];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) dh[nt] = mma_f32(a, sh.w2[(ks * 4 + lg) * NH + nt * 16 + lr], dh[nt]);
        }
        wave_lds_sync();
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = 4 * lg + q, c = nt * 16 + lr;
                t.z[row][c] = bf16_to_f32(t.h1[row][c]) > 0.f ? dh[nt][q] : 0.f;
            }
        wave_lds_sync();
        // gW1 += dZ1^T X
#pragma unroll 1
        for (int ks = 0; ks < 4; ++ks) {
            const int k = ks * 4 + lg;
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) g1[mt] = mma_f32(t.z[k][mt * 16 + lr], t.x[k][lr], g1[mt]);
        }
        {
            float s1 = 0.f;
            for (int row = 0; row < MT; ++row) s1 += t.z[row][l];
            gb1 += s1;
        }
        wave_lds_sync();
    }
    // The waves' sums meet in LDS: the upper half's are added to the lower's,
    // the last two waves' to one another tile by tile, and each wave adds a
    // quarter of the tiles to the gradient. LDS float atomics in place of this,
    // four waves on the same 5317 words, took 24 of a launch's 37 us.
    auto put = [&](BwdSums& to) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) to.tile[6 * nt + mt][l] = g2[mt][nt];
            to.tile[6 * nt + 4][l] = g1[nt];
            to.tile[6 * nt + 5][l] = g3[nt];
        }
        to.bias[l] = f32x4{gb1, gb2, gb3, 0.f};
    };
    static_assert(MW == 4, "two waves send, two receive");
    __syncthreads();   // every wave has left its tiles
    if (w >= 2) put(sh.sums[w - 2]);
    __syncthreads();
    if (w < 2) {
        BwdSums& from = sh.sums[w];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) g2[mt][nt] += from.tile[6 * nt + mt][l];
            g1[nt] += from.tile[6 * nt + 4][l];
            g3[nt] += from.tile[6 * nt + 5][l];
        }
        const f32x4 b = from.bias[l];
        gb1 += b[0];
        gb2 += b[1];
        gb3 += b[2];
        put(from);
    }
    __syncthreads();
    auto add = [&](int i, float v) {
        if (v != 0.f) atomicAdd(&grad[i], v);
    };
#pragma unroll 1
    for (int k = w; k < 24; k += MW) {
        const f32x4 v = sh.sums[0].tile[k][l] + sh.sums[1].tile[k][l];
        const int nt = k / 6, mt = k % 6;
        int at, step;   // the tile's element (row 4 lg, column lr) and its stride by rows
        bool in = true;
        if (mt < 4) {
            step = NH;
            at = OFF_W2 + (mt * 16 + 4 * lg) * NH + nt * 16 + lr;
        } else if (mt == 4) {
            step = NI;
            at = OFF_W1 + (nt * 16 + 4 * lg) * NI + lr;
            in = lr < NI;
        } else {
            step = NH;
            at = OFF_W3 + 4 * lg * NH + nt * 16 + lr;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (in && (mt < 5 || 4 * lg + q < NO)) add(at + q * step, v[q]);
    }
    if (w == 0) {
        const f32x4 v = sh.sums[0].bias[l] + sh.sums[1].bias[l];
        add(OFF_B1 + l, v[0]);
        add(OFF_B2 + l, v[1]);
        if (l < NO) add(OFF_B3 + l, v[2]);
    }
}

__global__ void k_mlp_adam(const float* g, float* p, float* m1, float* m2, int step, float lr) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NPAR) return;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.f - b1) * gi;
    const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    p[i] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

// features[r][12] of traced rounds r = 1..rounds, as the sweep computes them
// when it decides round r (history from the record of round r-1; the
// hybrid's code for the round from the same parameters the sweep uses).
__global__ void k_trace_features(long long rounds, const llp_trace_rec* tr, int n, int m, SchedParams sp, float* F) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    SchedHist h;
    memset(&h, 0, sizeof(h));
    for (long long r = 1; r <= rounds; ++r) {
        const llp_trace_rec t = tr[r - 1];
        float f[12];
        round_features(f, (int)r, t.in_count, (int)t.in_edges, n, m, h, hybrid_code(sp, (int)t.in_edges, m));
        for (int k = 0; k < 12; ++k) F[(r - 1) * 12 + k] = f[k];
        const long long prev_adv = h.adv_total;
        h.r = (int)r;
        h.mode = t.mode & 3;
        h.cl_count = t.in_count;
        h.cl_edges = (int)t.in_edges;
        h.wl_count = t.out_count;
        h.wl_edges = (int)t.out_edges;
        h.adv_total = prev_adv + t.in_count;
    }
}

// one wave per tile of MT rows, waves of them per workgroup, at most per_cu waves for each CU
static int mlp_grid(int B, int waves, int per_cu) {
    int g = (B + MT * waves - 1) / (MT * waves);
    int cap = device_info().cus * per_cu / waves;
    if (g > cap) g = cap;
    return g < 1 ? 1 : g;
}

}  // namespace llp

extern "C" {

int llp_mlp_forward(int32_t B, const float* params, const float* x, float* logits, uint16_t* act, void* stream) {
    if (B < 0 || !params || (B > 0 && (!x || !logits || !act))) return llp::fail(LLP_E_ARG, "bad forward arguments");
    if (B == 0) return LLP_OK;
    hipLaunchKernelGGL(llp::k_mlp_forward, dim3(llp::mlp_grid(B, 1, 16)), dim3(LLP_WAVE), 0, (hipStream_t)stream, B, params,
                       x, logits, act);
    return llp::hip_check(hipGetLastError(), "k_mlp_forward");
}

int llp_mlp_loss(int32_t B, const float* logits, const int32_t* labels, float* dlogits, float* loss, void* stream) {
    if (B < 0 || !loss || (B > 0 && (!logits || !labels || !dlogits))) return llp::fail(LLP_E_ARG, "bad loss arguments");
    hipStream_t st = (hipStream_t)stream;
    if (B <= llp::LOSS_ONE || dlogits == logits) {
        hipLaunchKernelGGL(llp::k_mlp_loss, dim3(1), dim3(1024), 0, st, B, logits, labels, dlogits, loss);
    } else {
        const int chunks = (int)(((long long)B + llp::LOSS_CHUNK - 1) / llp::LOSS_CHUNK);
        const int blocks = (int)(((long long)B + 255) / 256);
        hipLaunchKernelGGL(llp::k_mlp_loss_part, dim3(chunks), dim3(256), 0, st, B, logits, labels, dlogits);
        hipLaunchKernelGGL(llp::k_mlp_loss_sum, dim3(1), dim3(1024), 0, st, B, (const float*)dlogits, loss);
        hipLaunchKernelGGL(llp::k_mlp_loss_grad, dim3(blocks), dim3(256), 0, st, B, logits, labels, dlogits);
    }
    return llp::hip_check(hipGetLastError(), "k_mlp_loss");
}

int llp_mlp_backward(int32_t B, const float* params, const float* x, const uint16_t* act, const float* dlogits,
                     float* grad, void* stream) {
    if (B < 0 || !params || !grad || (B > 0 && (!x || !act || !dlogits)))
        return llp::fail(LLP_E_ARG, "bad backward arguments");
    if (B == 0) return LLP_OK;
    hipLaunchKernelGGL(llp::k_mlp_backward, dim3(llp::mlp_grid(B, llp::MW, 2 * llp::MW)), dim3(llp::MB), sizeof(llp::BwdShared),
                       (hipStream_t)stream, B, params, x, act, dlogits, grad);
    return llp::hip_check(hipGetLastError(), "k_mlp_backward");
}

int llp_mlp_adam(const float* grad, float* params, float* m1, float* m2, int32_t step, float lr, void* stream) {
    if (!grad || !params || !m1 || !m2 || step < 1) return llp::fail(LLP_E_ARG, "bad Adam arguments");
    hipLaunchKernelGGL(llp::k_mlp_adam, dim3((LLP_MLP_PARAMS + 255) / 256), dim3(256), 0, (hipStream_t)stream, grad,
                       params, m1, m2, step, lr);
    return llp::hip_check(hipGetLastError(), "k_mlp_adam");
}

int llp_trace_features(int64_t rounds, const llp_trace_rec* trace, int32_t n, int64_t m, int32_t kind,
                       float* features, void* stream) {
    if (rounds < 0 || n <= 0 || m < 0 || m > 0x7fffffffll || (rounds > 0 && (!trace || !features)))
        return llp::fail(LLP_E_ARG, "bad trace-feature arguments");
    if (kind != LLP_KIND_SSSP && kind != LLP_KIND_BFS && kind != LLP_KIND_JOBS)
        return llp::fail(LLP_E_ARG, "kind must be LLP_KIND_SSSP, LLP_KIND_BFS or LLP_KIND_JOBS");
    if (rounds == 0) return LLP_OK;
    llp::SchedParams sp;
    memset(&sp, 0, sizeof(sp));
    llp::hybrid_params(kind, n, m, true, &sp);
    hipLaunchKernelGGL(llp::k_trace_features, dim3(1), dim3(64), 0, (hipStream_t)stream, (long long)rounds, trace, n,
                       (int)m, sp, features);
    return llp::hip_check(hipGetLastError(), "k_trace_features");
}

}  // extern "C"
