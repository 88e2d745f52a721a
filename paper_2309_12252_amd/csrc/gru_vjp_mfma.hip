// Vector-Jacobian product of the GRU cell on the matrix cores (fp32, n = 16, 32 or 64, d <= 16): the same
// quantities as gru_vjp_kernel (Sec. 3.1.1 eq. 7, outer bracket) -- dL/dx per position, dL/dy0, and partial
// rows of dL/dtheta for the fixed-order reduction -- with every contraction as 16 x 16 x 4 MFMAs.
//
// A wavefront takes 16 consecutive positions as the column tile (lane = 16 g + c: column c, lane group g).
//   1. gate pre-activations  a_r, a_z = U h + W x + b,  q = U_c h + b_hc,  a_c' = W_c x + b_c : rows of the
//      weights are the A operands (U resident in registers, W read from LDS), h and x of the 16 positions
//      the B operands (lane (g, c) supplies entry 4m + g of position c in k-step m);
//   2. cotangents in accumulator layout (lane (g, c): rows 4g .. 4g+3 of a 16-row block, position c), where
//      lam and h arrive as 16-byte loads:  dac = lam (1 - z)(1 - c^2), daz = lam (h - c) z (1 - z),
//      dq = dac r, dar = dac q r (1 - r);
//   3. dL/dx = sum over gates of W_g^T d_g straight from those registers: k-step v takes the rows
//      {16 I + 4g + v}, and the A operand's columns are picked to match;
//   4. dU_g += d_g H^T and dW_g += d_g X^T have the positions on the k index: the cotangent blocks cross a
//      wavefront-private LDS tile to become A operands, h and x are read a second time as B operands
//      (lane (g, j): entry j of position 4m + g);
//   5. the bias sums stay per lane and are added over the 16 columns once, at the end.
// Accumulators live in registers over all passes; every wavefront writes one partial row.
#include "deer_common.h"

namespace deer {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kDP = 16;   // inputs are padded to 16 columns (zeros)
constexpr int kLD = 17;   // LDS row stride of the 16-column blocks

typedef float acc4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ acc4 mfma(float a, float b, acc4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int N>
__global__ __launch_bounds__(kThreads, N == 32 ? 2 : 1) void gru_vjp_mfma_kernel(GruVjpParams p) {
    constexpr int NB = N / 16;   // 16-row blocks
    constexpr int KH = N / 4;    // k-steps over the state
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float* sW = reinterpret_cast<float*>(smem_raw);   // [3N][kLD] input weights, columns >= d zero
    float* sB = sW + 3 * N * kLD;                      // [4N] biases r | z | c | hc
    float* sD = sB + 4 * N;                            // [kWaves][5][N][kLD] cotangent blocks (dar, daz, dac, dq, z lam)
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, c = lane & 15;
    const int d = p.d;
    const float* __restrict__ theta = reinterpret_cast<const float*>(p.theta);
    const float* __restrict__ U = theta + 3 * N * d;
    const float* __restrict__ bias = U + 3 * N * N;
    const float* __restrict__ x = reinterpret_cast<const float*>(p.x);
    const float* __restrict__ y0 = reinterpret_cast<const float*>(p.y0);
    const float* __restrict__ y = reinterpret_cast<const float*>(p.y);
    const float* __restrict__ lam = reinterpret_cast<const float*>(p.lam);
    float* __restrict__ dx = reinterpret_cast<float*>(p.dx);
    float* __restrict__ dy0 = reinterpret_cast<float*>(p.dy0);

    for (int q = tid; q < 3 * N * kLD; q += kThreads) {
        const int row = q / kLD, col = q - row * kLD;
        sW[q] = (col < d) ? theta[row * d + col] : 0.0f;
    }
    for (int q = tid; q < 4 * N; q += kThreads) sB[q] = bias[q];
    // hidden-to-hidden weights as A operands: uA[gate][I][m] = U_gate[16 I + c][4 m + g]
    float uA[3][NB][KH];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
            for (int m = 0; m < KH; ++m) uA[a][I][m] = U[(a * N + 16 * I + c) * N + 4 * m + g];
    __syncthreads();

    float* myD = sD + (size_t)wave * 5 * N * kLD;
    acc4 accU[3][NB][NB], accW[3][NB], accB[4][NB];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            accW[a][I] = acc4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int J = 0; J < NB; ++J) accU[a][I][J] = acc4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int I = 0; I < NB; ++I) accB[a][I] = acc4{0.f, 0.f, 0.f, 0.f};

    const long long total = (long long)p.B * p.T;
    const long long tiles = (total + 15) / 16;
    // state in front of position s (y0 at the first position of a sequence); positions past the end read position 0
    const bool narrow = total < (1LL << 31);   // 32-bit division is several times cheaper than the 64-bit one
    auto hrow = [&](long long s) -> const float* {
        const long long sc = s < total ? s : 0;
        const long long bi = narrow ? (long long)((unsigned)sc / (unsigned)p.T) : sc / p.T;
        return (sc - bi * p.T == 0) ? (y0 + bi * N) : (y + (sc - 1) * N);
    };

    // operands of one tile, in the layouts described above
    struct Operands {
        float hB[KH], xB[4];
        acc4 lamA[NB], hA[NB];
        float hK[4][NB], xK[4];
    };
    auto request = [&](long long tile, Operands& o) {
        const long long s0 = tile * 16;
        const long long sc = s0 + c;            // this lane's column position
        const bool live = sc < total;
        const long long scl = live ? sc : 0;
        const float* hc = hrow(sc);
#pragma unroll
        for (int m = 0; m < KH; ++m) o.hB[m] = hc[4 * m + g];
#pragma unroll
        for (int m = 0; m < 4; ++m) o.xB[m] = (4 * m + g < d) ? x[scl * d + 4 * m + g] : 0.0f;
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            const float4 lv = *reinterpret_cast<const float4*>(lam + scl * N + 16 * I + 4 * g);
            const float4 hv = *reinterpret_cast<const float4*>(hc + 16 * I + 4 * g);
            o.lamA[I] = live ? acc4{lv.x, lv.y, lv.z, lv.w} : acc4{0.f, 0.f, 0.f, 0.f};
            o.hA[I] = acc4{hv.x, hv.y, hv.z, hv.w};
        }
        // second view for the products over positions: lane (g, j) reads entry j of position 4 m + g
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const long long sp = s0 + 4 * m + g;
            const float* hp = hrow(sp);
#pragma unroll
            for (int J = 0; J < NB; ++J) o.hK[m][J] = hp[16 * J + c];
            o.xK[m] = (c < d && sp < total) ? x[sp * d + c] : 0.0f;
        }
    };
    const long long tstride = (long long)gridDim.x * kWaves;
    for (long long tile = (long long)blockIdx.x * kWaves + wave; tile < tiles; tile += tstride) {
        const long long s0 = tile * 16;
        const long long sc = s0 + c;
        const bool live = sc < total;
        // (requesting the next tile's operands one pass ahead costs a wavefront of occupancy and measured slower)
        Operands o;
        request(tile, o);
        const float (&hB)[KH] = o.hB;
        const float (&xB)[4] = o.xB;
        const acc4 (&lamA)[NB] = o.lamA;
        const acc4 (&hA)[NB] = o.hA;
        const float (&hK)[4][NB] = o.hK;
        const float (&xK)[4] = o.xK;

        // ---- 1. gates ----
        acc4 dar[NB], daz[NB], dac[NB], dq[NB];
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            acc4 ar, az, aq, ac;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                ar[v] = sB[16 * I + 4 * g + v];
                az[v] = sB[N + 16 * I + 4 * g + v];
                ac[v] = sB[2 * N + 16 * I + 4 * g + v];
                aq[v] = sB[3 * N + 16 * I + 4 * g + v];
            }
#pragma unroll
            for (int m = 0; m < KH; ++m) {
                ar = mfma(uA[0][I][m], hB[m], ar);
                az = mfma(uA[1][I][m], hB[m], az);
                aq = mfma(uA[2][I][m], hB[m], aq);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                ar = mfma(sW[(16 * I + c) * kLD + 4 * m + g], xB[m], ar);
                az = mfma(sW[(N + 16 * I + c) * kLD + 4 * m + g], xB[m], az);
                ac = mfma(sW[(2 * N + 16 * I + c) * kLD + 4 * m + g], xB[m], ac);
            }
            // ---- 2. cotangents ----
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float r = feed_sigmoid(ar[v]), z = feed_sigmoid(az[v]);
                const float cc = feed_tanh(ac[v] + r * aq[v]);
                const float lm = lamA[I][v], hi = hA[I][v];
                const float dcand = lm * (1.0f - z);
                const float vac = dcand * (1.0f - cc * cc);
                dac[I][v] = vac;
                daz[I][v] = lm * (hi - cc) * z * (1.0f - z);
                dq[I][v] = vac * r;
                dar[I][v] = vac * aq[v] * r * (1.0f - r);
                const int row = 16 * I + 4 * g + v;
                myD[(0 * N + row) * kLD + c] = dar[I][v];
                myD[(1 * N + row) * kLD + c] = daz[I][v];
                myD[(2 * N + row) * kLD + c] = dac[I][v];
                myD[(3 * N + row) * kLD + c] = dq[I][v];
                myD[(4 * N + row) * kLD + c] = z * lm;
            }
            accB[0][I] += dar[I];
            accB[1][I] += daz[I];
            accB[2][I] += dac[I];
            accB[3][I] += dq[I];
        }

        // ---- 3. dL/dx: rows (input index) 4g + v of position c ----
        if (dx) {
            acc4 ax = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int I = 0; I < NB; ++I)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    // k-step v: lane group g supplies row 16 I + 4g + v of the cotangent; A[i = c][k = g] = W[that row][c]
                    const int row = 16 * I + 4 * g + v;
                    ax = mfma(sW[row * kLD + c], dar[I][v], ax);
                    ax = mfma(sW[(N + row) * kLD + c], daz[I][v], ax);
                    ax = mfma(sW[(2 * N + row) * kLD + c], dac[I][v], ax);
                }
            if (live) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (4 * g + v < d) dx[sc * d + 4 * g + v] = ax[v];
            }
        }

        // ---- 4. dU += d H^T, dW += d X^T (k = positions) ----
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                // A[i = c -> row 16 I + c][k = g -> position 4 m + g]
                const int at = (16 * I + c) * kLD + 4 * m + g;
                const float tr = myD[0 * N * kLD + at], tz = myD[1 * N * kLD + at];
                const float tc = myD[2 * N * kLD + at], tq = myD[3 * N * kLD + at];
#pragma unroll
                for (int J = 0; J < NB; ++J) {
                    accU[0][I][J] = mfma(tr, hK[m][J], accU[0][I][J]);
                    accU[1][I][J] = mfma(tz, hK[m][J], accU[1][I][J]);
                    accU[2][I][J] = mfma(tq, hK[m][J], accU[2][I][J]);
                }
                accW[0][I] = mfma(tr, xK[m], accW[0][I]);
                accW[1][I] = mfma(tz, xK[m], accW[1][I]);
                accW[2][I] = mfma(tc, xK[m], accW[2][I]);
            }

        // ---- dL/dy0 = J_1^T lam_1 at the first position of a sequence (rare: one column of a few tiles) ----
        if (dy0) {
            for (int c0 = 0; c0 < 16; ++c0) {
                const long long sp = s0 + c0;
                if (sp >= total) break;
                const long long bi = sp / p.T;
                if (sp - bi * p.T != 0) continue;
                if (lane < N) {
                    float s = myD[(4 * N + lane) * kLD + c0];   // z_j lam_j
                    for (int i = 0; i < N; ++i) {
                        s += U[(0 * N + i) * N + lane] * myD[(0 * N + i) * kLD + c0];
                        s += U[(1 * N + i) * N + lane] * myD[(1 * N + i) * kLD + c0];
                        s += U[(2 * N + i) * N + lane] * myD[(3 * N + i) * kLD + c0];
                    }
                    dy0[bi * N + lane] = s;
                }
            }
        }
    }

    // ---- partial row of this wavefront ----
    const long long P = 3LL * N * d + 3LL * N * N + 4LL * N;
    float* __restrict__ prow = reinterpret_cast<float*>(p.partial) + ((long long)blockIdx.x * kWaves + wave) * P;
    float* pU = prow + 3LL * N * d;
    float* pb = pU + 3LL * N * N;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = a * N + 16 * I + 4 * g + v;
                if (c < d) prow[(long long)row * d + c] = accW[a][I][v];
#pragma unroll
                for (int J = 0; J < NB; ++J) pU[(long long)row * N + 16 * J + c] = accU[a][I][J][v];
            }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float s = accB[a][I][v];
                s += __shfl_xor(s, 1);
                s += __shfl_xor(s, 2);
                s += __shfl_xor(s, 4);
                s += __shfl_xor(s, 8);
                if (c == 0) pb[a * N + 16 * I + 4 * g + v] = s;
            }
}

// n = 64: the sums of one wavefront would not fit its registers (48 blocks), so the four wavefronts of a workgroup take the same 16
// positions and 16 rows of every gate each: gates, cotangents and sums of these rows need nothing from the other wavefronts but
// the input gradient, whose four parts meet in LDS (one barrier a tile, double-buffered).  One partial row per workgroup.
// Bound: fp32 matrix instructions, 132 of 32 cycles a wavefront and tile (25 us at 49,865 positions).  The vector-ALU kernel took 742 us
// there (d = 7), this one 66 us (58 with one chain of sums over all tiles and the biases and W columns in registers).
__global__ __launch_bounds__(kThreads, 2) void gru_vjp_mfma64_kernel(GruVjpParams p) {
    constexpr int N = 64, NB = 4;
    __shared__ __align__(16) float sD[kWaves][5][16][kLD];    // dar, daz, dac, dq, z lam of the wavefront's rows
    __shared__ float sX[2][kWaves][16][kLD];                  // input gradient: parts of the wavefronts
    __shared__ float sY[kWaves][N];                           // dL/dy0: the same
    __shared__ __align__(16) float sH[2][16][N + 4];          // state in front of the sixteen positions
    __shared__ __align__(16) acc4 sWT[3][kThreads];           // W columns for dL/dx (row 4 g + v of the wavefront's, column c)
    __shared__ __align__(16) float sBias[4][N];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15, d = p.d, row0 = 16 * wave;
    const float* __restrict__ theta = reinterpret_cast<const float*>(p.theta);
    const float* __restrict__ U = theta + 3 * N * d;
    const float* __restrict__ bias = U + 3 * N * N;
    const float* __restrict__ x = reinterpret_cast<const float*>(p.x);
    const float* __restrict__ y0 = reinterpret_cast<const float*>(p.y0);
    const float* __restrict__ y = reinterpret_cast<const float*>(p.y);
    const float* __restrict__ lam = reinterpret_cast<const float*>(p.lam);
    float* __restrict__ dx = reinterpret_cast<float*>(p.dx);
    float* __restrict__ dy0 = reinterpret_cast<float*>(p.dy0);

    // operands A of this wavefront's rows; the state and the input supply entry 16 K + 4 g + v and 4 m + g
    // (what is used once a tile waits in LDS: registers)
    acc4 uA[3][NB];
    float wA[3][4];   // W rows
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int K = 0; K < NB; ++K)
#pragma unroll
            for (int v = 0; v < 4; ++v) uA[a][K][v] = U[(a * N + row0 + c) * N + 16 * K + 4 * g + v];
        acc4 wT;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const float w = theta[(a * N + row0 + c) * d + min(4 * m + g, d - 1)], t = theta[(a * N + row0 + 4 * g + m) * d + min(c, d - 1)];
            wA[a][m] = 4 * m + g < d ? w : 0.0f;
            wT[m] = c < d ? t : 0.0f;
        }
        sWT[a][tid] = wT;   // (read by the same lane)
    }
    sBias[tid / N][tid % N] = bias[tid];
    __syncthreads();

    const acc4 zero = {0.f, 0.f, 0.f, 0.f};
    acc4 accU[3][NB], accW[3], accB[4];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        accW[a] = zero;
#pragma unroll
        for (int J = 0; J < NB; ++J) accU[a][J] = zero;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) accB[a] = zero;

    const long long total = (long long)p.B * p.T, tiles = (total + 15) / 16;
    auto hrow = [&](long long s) -> const float* {   // state in front of position s (positions past the end read position 0)
        const long long sc = s < total ? s : 0, bi = sc / p.T;
        return (sc - bi * p.T == 0) ? (y0 + bi * N) : (y + (sc - 1) * N);
    };
    int buf = 0;
    static_assert(kThreads == 4 * N, "one bias entry per thread");
    for (long long tile = blockIdx.x; tile < tiles; tile += gridDim.x, buf ^= 1) {
        const long long s0 = tile * 16, sc = s0 + c;
        const bool live = sc < total;
        const long long scl = live ? sc : 0;
        const float* hc = hrow(sc);
        acc4 h[NB];
        float xB[4], xK[4];
#pragma unroll
        for (int K = 0; K < NB; ++K) {
            const float4 t = *reinterpret_cast<const float4*>(hc + 16 * K + 4 * g);
            h[K] = acc4{t.x, t.y, t.z, t.w};
        }
        const float4 lv = *reinterpret_cast<const float4*>(lam + scl * N + row0 + 4 * g), hv = *reinterpret_cast<const float4*>(hc + row0 + 4 * g);
        const acc4 lm = live ? acc4{lv.x, lv.y, lv.z, lv.w} : zero, hw = {hv.x, hv.y, hv.z, hv.w};
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const long long sp = s0 + 4 * m + g;
            const float a = x[scl * d + min(4 * m + g, d - 1)], b = x[(sp < total ? sp : 0) * d + min(c, d - 1)];
            xB[m] = 4 * m + g < d ? a : 0.0f;
            xK[m] = (c < d && sp < total) ? b : 0.0f;
        }
        const float* bs = &sBias[0][row0 + 4 * g];
        acc4 ar = *reinterpret_cast<const acc4*>(bs), az = *reinterpret_cast<const acc4*>(bs + N), ac = *reinterpret_cast<const acc4*>(bs + 2 * N), aq = *reinterpret_cast<const acc4*>(bs + 3 * N);
#pragma unroll
        for (int K = 0; K < NB; ++K)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                ar = mfma(uA[0][K][v], h[K][v], ar);
                az = mfma(uA[1][K][v], h[K][v], az);
                aq = mfma(uA[2][K][v], h[K][v], aq);
            }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            ar = mfma(wA[0][m], xB[m], ar);
            az = mfma(wA[1][m], xB[m], az);
            ac = mfma(wA[2][m], xB[m], ac);
        }
        acc4 dar, daz, dac, dq;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float r = feed_sigmoid(ar[v]), z = feed_sigmoid(az[v]);
            const float cc = feed_tanh(ac[v] + r * aq[v]);
            dac[v] = lm[v] * (1.0f - z) * (1.0f - cc * cc);
            daz[v] = lm[v] * (hw[v] - cc) * z * (1.0f - z);
            dq[v] = dac[v] * r;
            dar[v] = dac[v] * aq[v] * r * (1.0f - r);
            const int row = 4 * g + v;
            sD[wave][0][row][c] = dar[v];
            sD[wave][1][row][c] = daz[v];
            sD[wave][2][row][c] = dac[v];
            sD[wave][3][row][c] = dq[v];
            sD[wave][4][row][c] = z * lm[v];
        }
        accB[0] += dar; accB[1] += daz; accB[2] += dac; accB[3] += dq;
        *reinterpret_cast<acc4*>(&sH[buf][c][row0 + 4 * g]) = hw;
        if (dx) {   // rows (input index) 4 g + v of position c, this wavefront's share of the sum over rows
            acc4 ax = zero, bx = zero, cx = zero;
            const acc4 wr = sWT[0][tid], wz = sWT[1][tid], wc = sWT[2][tid];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                ax = mfma(wr[v], dar[v], ax);
                bx = mfma(wz[v], daz[v], bx);
                cx = mfma(wc[v], dac[v], cx);
            }
            ax += bx + cx;
#pragma unroll
            for (int v = 0; v < 4; ++v) sX[buf][wave][c][4 * g + v] = ax[v];
        }
        __syncthreads();
        if (dx) {
            const int q = tid >> 4, k = tid & 15;
            if (s0 + q < total && k < d) dx[(s0 + q) * d + k] = (sX[buf][0][q][k] + sX[buf][1][q][k]) + (sX[buf][2][q][k] + sX[buf][3][q][k]);
        }
        // the tile's sixteen positions by themselves, then added to the sums (one chain over all tiles of a workgroup rounds at the size of the sums)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float tu[4], tw[4];   // cotangents in front of U and W (block c: dq and dac)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                tw[m] = sD[wave][a][c][4 * m + g];
                tu[m] = a == 2 ? sD[wave][3][c][4 * m + g] : tw[m];
            }
#pragma unroll
            for (int J = 0; J < NB; ++J) {
                acc4 s = zero;
#pragma unroll
                for (int m = 0; m < 4; ++m) s = mfma(tu[m], sH[buf][4 * m + g][16 * J + c], s);
                accU[a][J] += s;
            }
            acc4 s = zero;
#pragma unroll
            for (int m = 0; m < 4; ++m) s = mfma(tw[m], xK[m], s);
            accW[a] += s;
        }
        // dL/dy0 = J_1^T lam_1 where a sequence starts among the sixteen positions (rare; the same for the whole workgroup)
        if (dy0) {
            const long long b0 = (s0 + p.T - 1) / p.T;   // first sequence that starts at s0 or later
            if (b0 < p.B && b0 * p.T < s0 + 16) {
                for (long long bi = b0; bi < p.B && bi * p.T < s0 + 16; ++bi) {
                    const int q = (int)(bi * p.T - s0);
                    // short partial sums, z lambda last (one chain of 192 products on top of it was twice as far off)
                    float part[3] = {0.0f, 0.0f, 0.0f};
                    for (int i = 0; i < 16; ++i) {
                        part[0] += U[(0 * N + row0 + i) * N + lane] * sD[wave][0][i][q];
                        part[1] += U[(1 * N + row0 + i) * N + lane] * sD[wave][1][i][q];
                        part[2] += U[(2 * N + row0 + i) * N + lane] * sD[wave][3][i][q];
                    }
                    sY[wave][lane] = part[0] + (part[1] + part[2]);
                    __syncthreads();
                    if (tid < N) dy0[bi * N + tid] = ((sY[0][tid] + sY[1][tid]) + (sY[2][tid] + sY[3][tid])) + sD[tid / 16][4][tid % 16][q];
                    __syncthreads();
                }
            }
        }
    }

    const long long P = 3LL * N * d + 3LL * N * N + 4LL * N;
    float* __restrict__ prow = reinterpret_cast<float*>(p.partial) + (long long)blockIdx.x * P;
    float* pU = prow + 3LL * N * d;
    float* pb = pU + 3LL * N * N;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = a * N + row0 + 4 * g + v;
            if (c < d) prow[(long long)row * d + c] = accW[a][v];
#pragma unroll
            for (int J = 0; J < NB; ++J) pU[(long long)row * N + 16 * J + c] = accU[a][J][v];
        }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float s = accB[a][v];
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o);
            if (c == 0) pb[a * N + row0 + 4 * g + v] = s;
        }
}

template <int N>
hipError_t launch_n(const GruVjpParams& p, hipStream_t s) {
    const size_t shmem = ((size_t)3 * N * kLD + 4 * N + (size_t)kWaves * 5 * N * kLD) * sizeof(float);
    hipLaunchKernelGGL((gru_vjp_mfma_kernel<N>), dim3((unsigned)p.blocks), dim3(kThreads), shmem, s, p);
    return hipGetLastError();
}

}  // namespace

bool gru_vjp_mfma_supported(int dtype, int n, int d) { return dtype == 0 && (n == 16 || n == 32 || n == 64) && d >= 1 && d <= kDP; }

// one partial row per wavefront, at n = 64 per workgroup; added in a fixed order
hipError_t launch_gru_vjp_mfma(const GruVjpParams& p, hipStream_t s) {
    if (!gru_vjp_mfma_supported(0, p.n, p.d) || p.blocks < 1) return hipErrorInvalidValue;
    int rows = p.blocks * kWaves;
    hipError_t e;
    if (p.n == 64) {
        const long long tiles = ((long long)p.B * p.T + 15) / 16;
        rows = tiles < p.blocks ? (int)tiles : p.blocks;
        hipLaunchKernelGGL(gru_vjp_mfma64_kernel, dim3((unsigned)rows), dim3(kThreads), 0, s, p);
        e = hipGetLastError();
    } else {
        e = p.n == 16 ? launch_n<16>(p, s) : launch_n<32>(p, s);
    }
    if (e != hipSuccess) return e;
    return launch_partial_reduce(0, p.partial, p.dtheta, 3LL * p.n * p.d + 3LL * p.n * p.n + 4LL * p.n, rows, s);
}

}  // namespace deer
