// Newton step and dual scan of the GRU at n = 16 and 32 in fp32 (n = 64: chunk_gru64.hip): chunks of the sequence are reduced to one affine map
// each, the maps are folded, and sixteen chunks per wavefront are then walked side by side (Sec. 3.1 eq. 3 and 5, Sec. 3.1.1
// eq. 7, Sec. 3.3 eq. 10).
//
// A sequence is cut into chunks of Lc positions, sixteen consecutive chunks form a group.
//   1. chunk_totals_kernel: every chunk's map x -> M x + v (the composition of its pairs).  The only part that multiplies
//      matrices by matrices; a wavefront streams through its positions with one running product in registers.  The maps
//      of a workgroup's 4, 8 or 16 chunks (a unit) are then composed into the unit's map.
//   2. chunk_walk_kernel: a wavefront owns one group.  It folds the maps of the units in front of it into the group's
//      carry and the maps of its own chunks into sixteen carries, which are the columns of a 16 x 16 matrix-core tile; the
//      sixteen chunks are then walked position by position, every step being a product of a constant weight matrix with
//      the sixteen column vectors (J is never formed: J e = z e + p_z (U_z e) + s_r (U_c e) + s_t (U_r e)).
// Nothing in a launch waits for another workgroup, the number of wavefronts does not depend on the length (the chunk does),
// and the state that travels between the two launches is one map per chunk.
//
// Bound: issue.  The matrix instructions and the vector ALU of a SIMD do not overlap.  The reduction of a Newton step has both factors of a
// product split in two fp16 numbers (split_f16.h): a position costs 12 matrix instructions of 18 cycles and 120 vector instructions of 2.4 at n = 32 (3 and 40 at n =
// 16) beside its share of the gates (60 fp32 matrix instructions for sixteen positions), in the place of 32 fp32 matrix instructions of 32 cycles and 72 (4 and 20).
// Two wavefronts a SIMD (registers, LDS) issue in 71 % of the time.  Newton step, reduction alone, fp32 products before / now: n = 32, d = 8, 16 x 100,000
// positions 1,150 / 757 us; n = 16, d = 6, 32 x 17,984 positions 101 / 91 us (the walk 212 and 43; the single-pass scan 2,650 and 240 for the whole step).  Assembling
// the factor of the next position behind the products of this one: 6 and 3 % slower (20 more vector instructions a position).
//
// The split reduction (Newton steps): every column of the product has a power of two of its own, looked at before each sixteen positions (ColumnScale).  The
// entries of J are split as they are: an absolute error of 2^-25 each, and nothing of one below that; a column that falls by 2^-k between two looks
// is known to 2^(k-28) of its largest entry at worst.  A step's maps multiply a correction, so what they lose is lost against the correction and the next step
// takes it up: 2-norm errors of the trajectory against 64 bits, fp32 / split products (mean of 8 solves) 1.344e-7 / 1.344e-7 (n = 32), 1.153e-7 / 1.153e-7
// (n = 16).  Steps from far iterates keep fp32 products.  A product that leaves the range of fp16 leaves infinities or NaN; the wavefront sees them at the next
// look and goes on with fp32 products from the chunk that it had in work at the look before.
// The dual scan keeps fp32 products: its maps multiply the cotangent itself, which may have faded by many powers of ten when it reaches the first
// positions.  With split products dL/dy0 of a loss on the last state had lost 3e-5 to 0.3 of itself behind chunks of 16 positions that keep 0.1 to 0.3 of
// the state a step, and 1e-6 with fp32 ones.
//
// Everything is in correction form: with e = y_new - y the recurrence of a Newton step is e_i = J_i e_{i-1} + (f_i - y_i),
// e_0 = 0, so neither J h nor a right-hand side is needed and rounding is relative to the correction.
//
// Matrix-core layout (16x16x4, lane (g = lane / 16, r = lane % 16)): operand A supplies A[r][4g + v] and operand B
// B[4g + v][r] in the v-th of four instructions of a 16-wide contraction, the accumulator holds D[4g + v][r] in register v.  So an
// accumulator is a valid B operand, four consecutive scalars of a row-major matrix are an A operand, and an accumulator of
// X is the A operand of its transpose.
#include "chunk_common.h"
#include "split_f16.h"

namespace deer {

namespace {

// weights in LDS: rows of [U_gate | W_gate], W in the order the input operand takes its columns (step s of lane group g:
// column DS g + s), zero beyond d; then the four bias vectors
template <int N, int DS>
struct Weights {
    static constexpr int LD = N + 4 * DS + 4;
    float row[3][N][LD];
    float bias[4][N];
};

template <int N, int DS, int THREADS>
__device__ __forceinline__ void fill_weights(Weights<N, DS>& w, const float* __restrict__ th, int d, int tid) {
    const float* __restrict__ U = th + 3 * N * d;
    const float* __restrict__ bias = U + 3 * N * N;
    constexpr int NU = 3 * N * (N / 4), NW = 3 * N * 4 * DS, KU = (NU + THREADS - 1) / THREADS, KW = (NW + THREADS - 1) / THREADS;
    Acc u[KU];
    float v[KW];
    // all requests first
#pragma unroll
    for (int k = 0; k < KU; ++k) u[k] = load4(U + 4 * min(tid + k * THREADS, NU - 1));
#pragma unroll
    for (int k = 0; k < KW; ++k) {
        const int i = min(tid + k * THREADS, NW - 1), c = i % (4 * DS);
        v[k] = th[(i / (4 * DS)) * d + min(c, d - 1)];
        v[k] = c < d ? v[k] : 0.f;
    }
    const float bv = bias[min(tid, 4 * N - 1)];
#pragma unroll
    for (int k = 0; k < KU; ++k) {
        const int i = tid + k * THREADS, row = i / (N / 4);
        if (i < NU) store4(&w.row[row / N][row % N][4 * (i % (N / 4))], u[k]);
    }
#pragma unroll
    for (int k = 0; k < KW; ++k) {
        const int i = tid + k * THREADS, row = i / (4 * DS);
        if (i < NW) w.row[row / N][row % N][N + i % (4 * DS)] = v[k];
    }
    static_assert(THREADS >= 4 * N, "one bias entry per thread");
    if (tid < 4 * N) w.bias[tid / N][tid % N] = bv;
}

// Four scalars of row `row` of [U | W]: operand A of a product with that row block (lane (g, r): row r), and equally operand
// B of the transposed product.
template <int N, int DS>
__device__ __forceinline__ Acc u_row(const Weights<N, DS>& w, int gate, int row, int K, int g) {
    return load4(&w.row[gate][row][16 * K + 4 * g]);
}
template <int N, int DS>
__device__ __forceinline__ void w_row(float* o, const Weights<N, DS>& w, int gate, int row, int g) {
    vload<float, DS>(o, &w.row[gate][row][N + DS * g]);
}


// ------------------------------------------------------------------------------------------------------------------
// Maps of the chunks.  Forward: the total of a chunk is P = J_L .. J_1, and Q = P^T is built from the last position to the
// first, Q <- J_i^T Q, because the vector then needs no chain of its own: v = sum over i of (J_L .. J_{i+1}) r_i, four
// multiply-adds per 16 rows with the running Q.  Dual: the map of the times [a, b) is N = J_{a+1}^T .. J_b^T, and S = N^T =
// J_b .. J_{a+1} is built from the first to the last, S <- J_i S, with v = sum over j of (J_j .. J_{a+1})^T g_j.  In both
// the accumulator of the running product is the map in the order of an A operand, so it leaves with 16-byte stores as M
// row-major.
// The gates of sixteen positions at a time are matrix products with the positions as columns (dual: as rows, which gives
// the row factors to the lanes that assemble J instead of its transpose); the row factors reach the assembly through an
// LDS slice of the wavefront.
// ------------------------------------------------------------------------------------------------------------------
template <int N, int DS, bool REV, bool FAR>
__global__ __launch_bounds__(256, N == 16 ? 3 : 2) void chunk_totals_kernel(ChunkParams p) {
    constexpr int NB = N / 16, MS = map_size<N>();
    constexpr bool SPLIT = !FAR && !REV;
    __shared__ __align__(16) Weights<N, DS> sW;
    // forward: [kind: p_z, s_r, s_t, z, residual][position][row]; dual: [position][row][p_z, s_r, s_t, z], then [position][row] of g
    constexpr int PS = REV ? N : N + 4, KS = 16 * PS;   // (forward: sixteen positions' rows of 16 bytes fall on different banks)
    __shared__ __align__(16) float sF[4][5 * KS];

    if (step_closed(p.gate, FAR)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int b = (int)(blockIdx.x % (unsigned)p.B), unit = (int)(blockIdx.x / (unsigned)p.B);

    const int T = p.T, d = p.d, Lc = p.Lc;
    const int chunks = (T + Lc - 1) / Lc;
    const float* __restrict__ yb = p.y + (long long)b * T * N;
    const float* __restrict__ xb = p.x + (long long)b * T * d;
    const float* __restrict__ y0b = p.y0 ? p.y0 + (long long)b * N : nullptr;
    const float* __restrict__ gb = REV ? p.g + (long long)b * T * N : nullptr;
    const int first = unit * p.per_unit, cpw = p.per_unit / 4;   // first chunk, chunks of a wavefront
    float* __restrict__ tot = p.tot + ((long long)b * chunks + first) * MS;
    float* __restrict__ sFw = sF[wave];

    const int q_lo = cpw * wave, q_hi = min(q_lo + cpw, chunks - first);   // chunks of this wavefront (inside the unit)
    const int lo = (first + q_lo) * Lc;
    const int hi = min(T, (first + q_hi) * Lc);
    int top = hi;   // forward: one past the first position that is still to be reduced

    // operands of one block: state in front of each position (16-byte pieces: operand of the products and the rows of
    // this lane's accumulators), the vector the residual is taken against (forward: the iterate at the position; dual: g), x
    Acc hB[NB], oB[NB];
    float xB[DS];
    auto request = [&](int blk) {
        int pos = (REV ? lo + 16 * blk : top - 16 * (blk + 1)) + r;
        pos = min(max(pos, lo), hi - 1);
        const float* hp = REV ? yb + (long long)pos * N : (pos > 0 ? yb + (long long)(pos - 1) * N : y0b);
        const float* op = (REV ? gb : yb) + (long long)pos * N;
#pragma unroll
        for (int K = 0; K < NB; ++K) {
            hB[K] = hp ? load4(hp + 16 * K + 4 * g) : zero4();
            oB[K] = load4(op + 16 * K + 4 * g);
        }
        load_x<DS>(xB, xb + (long long)(REV ? min(pos + 1, T - 1) : pos) * d, d, g);
    };
    if (q_lo < q_hi) request(0);
    fill_weights<N, DS, 256>(sW, p.theta, p.d, tid);
    __syncthreads();

    // weights of the assembly: ua[gate][X][Y][v] multiplies the factor of J's row
    //   forward: J[16Y + 4g + v][16X + r] (operand A of J^T);  dual: J[16X + r][16Y + 4g + v] (operand A of J)
    float ua[3][NB][NB][4];
#pragma unroll
    for (int gate = 0; gate < 3; ++gate)
#pragma unroll
        for (int X = 0; X < NB; ++X)
#pragma unroll
            for (int Y = 0; Y < NB; ++Y)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    ua[gate][X][Y][v] = REV ? sW.row[gate][16 * X + r][16 * Y + 4 * g + v] : sW.row[gate][16 * Y + 4 * g + v][16 * X + r];
    float dsel[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) dsel[v] = (4 * g + v == r) ? 1.f : 0.f;

    bool wide = !SPLIT, again = false;   // products of fp32 factors; a product of the other kind was not finite
    int q = REV ? q_lo : q_hi - 1, kept = q;   // chunk being reduced; the same when all was last seen to be finite
    while (q_lo < q_hi) {
        const float unit_q = wide ? 1.f : (float)(1 << ColumnScale::kStart);
        Acc Q[NB][NB];
        float vec[NB];
        ColumnScale scale[NB];
        auto reset = [&]() {
#pragma unroll
            for (int X = 0; X < NB; ++X) {
                vec[X] = 0.f;
                scale[X].reset(!wide);
#pragma unroll
                for (int C = 0; C < NB; ++C)
#pragma unroll
                    for (int v = 0; v < 4; ++v) Q[X][C][v] = (X == C) ? dsel[v] * unit_q : 0.f;
            }
        };
        reset();

        int edge = REV ? min(T, (first + q + 1) * Lc) - 1 : (first + q) * Lc;   // the chunk's last position in traversal order
        const int blocks = (top - lo + 15) / 16;

        for (int blk = 0; blk < blocks; ++blk) {
            const int base = REV ? lo + 16 * blk : top - 16 * (blk + 1);
            if (SPLIT && !wide) {
                // (in front of the gates: nothing waits for it there)
                float sum = 0.f;   // (not a finite number if one of its terms is none)
#pragma unroll
                for (int C = 0; C < NB; ++C) {
                    float m = 0.f;
#pragma unroll
                    for (int X = 0; X < NB; ++X)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            m = fmaxf(m, fabsf(Q[X][C][v]));
                            sum += 0.f * Q[X][C][v];
                        }
                    const float f = scale[C].next(max_groups(m));
#pragma unroll
                    for (int X = 0; X < NB; ++X) Q[X][C] *= f;
                }
                if (__ballot(again || sum != 0.f)) {
                    again = true;
                    break;
                }
                kept = q;
            }
            // ---- gates of the sixteen positions ----
            if constexpr (!REV) {
#pragma unroll
                for (int I = 0; I < NB; ++I) {
                    Acc ar = load4(&sW.bias[0][16 * I + 4 * g]), az = load4(&sW.bias[1][16 * I + 4 * g]);
                    Acc ac = load4(&sW.bias[2][16 * I + 4 * g]), aq = load4(&sW.bias[3][16 * I + 4 * g]);
#pragma unroll
                    for (int K = 0; K < NB; ++K) {
                        const Acc ur = u_row(sW, 0, 16 * I + r, K, g), uz = u_row(sW, 1, 16 * I + r, K, g), uc = u_row(sW, 2, 16 * I + r, K, g);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            ar = mfma(ur[v], hB[K][v], ar);
                            az = mfma(uz[v], hB[K][v], az);
                            aq = mfma(uc[v], hB[K][v], aq);
                        }
                    }
                    float wr[DS], wz[DS], wc[DS];
                    w_row(wr, sW, 0, 16 * I + r, g); w_row(wz, sW, 1, 16 * I + r, g); w_row(wc, sW, 2, 16 * I + r, g);
#pragma unroll
                    for (int s = 0; s < DS; ++s) {
                        ar = mfma(wr[s], xB[s], ar);
                        az = mfma(wz[s], xB[s], az);
                        ac = mfma(wc[s], xB[s], ac);
                    }
                    Acc fpz, fsr, fst, fz, fr;
                    GruGates o[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        o[v] = gru_gates(ar[v], az[v], ac[v], aq[v], hB[I][v]);
                        fpz[v] = o[v].pz; fsr[v] = o[v].sr; fst[v] = o[v].st; fz[v] = o[v].z;
                    }
                    if constexpr (FAR) {
                        Acc hr = zero4(), hz = zero4(), hc = zero4();
#pragma unroll
                        for (int K = 0; K < NB; ++K) {
                            const Acc ur = u_row(sW, 0, 16 * I + r, K, g), uz = u_row(sW, 1, 16 * I + r, K, g), uc = u_row(sW, 2, 16 * I + r, K, g);
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                hr = mfma(ur[v], hB[K][v], hr);
                                hz = mfma(uz[v], hB[K][v], hz);
                                hc = mfma(uc[v], hB[K][v], hc);
                            }
                        }
#pragma unroll
                        for (int v = 0; v < 4; ++v) fr[v] = gru_rhs(o[v], hr[v], hz[v], hc[v]);
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v) fr[v] = o[v].f - oB[I][v];
                    }
                    float* q = sFw + r * PS + 16 * I + 4 * g;
                    store4(q, fpz); store4(q + KS, fsr); store4(q + 2 * KS, fst); store4(q + 3 * KS, fz); store4(q + 4 * KS, fr);
                }
            } else {
                // the state entries of the rows this lane evaluates (positions 4g + v, row 16 I + r) come through the slice too
#pragma unroll
                for (int K = 0; K < NB; ++K) {
                    store4(sFw + 64 * N + r * N + 16 * K + 4 * g, oB[K]);
                    store4(sFw + r * N + 16 * K + 4 * g, hB[K]);
                }
                wave_lds_fence();
                float hr[NB][4];
#pragma unroll
                for (int I = 0; I < NB; ++I)
#pragma unroll
                    for (int v = 0; v < 4; ++v) hr[I][v] = sFw[(4 * g + v) * N + 16 * I + r];
                wave_lds_fence();
#pragma unroll
                for (int I = 0; I < NB; ++I) {
                    const float br = sW.bias[0][16 * I + r], bz = sW.bias[1][16 * I + r], bc = sW.bias[2][16 * I + r], bq = sW.bias[3][16 * I + r];
                    Acc ar = {br, br, br, br}, az = {bz, bz, bz, bz}, ac = {bc, bc, bc, bc}, aq = {bq, bq, bq, bq};
#pragma unroll
                    for (int K = 0; K < NB; ++K) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            ar = mfma(hB[K][v], ua[0][I][K][v], ar);
                            az = mfma(hB[K][v], ua[1][I][K][v], az);
                            aq = mfma(hB[K][v], ua[2][I][K][v], aq);
                        }
                    }
                    float wr[DS], wz[DS], wc[DS];
                    w_row(wr, sW, 0, 16 * I + r, g); w_row(wz, sW, 1, 16 * I + r, g); w_row(wc, sW, 2, 16 * I + r, g);
#pragma unroll
                    for (int s = 0; s < DS; ++s) {
                        ar = mfma(xB[s], wr[s], ar);
                        az = mfma(xB[s], wz[s], az);
                        ac = mfma(xB[s], wc[s], ac);
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const GruGates o = gru_gates(ar[v], az[v], ac[v], aq[v], hr[I][v]);
                        store4(sFw + ((4 * g + v) * N + 16 * I + r) * 4, Acc{o.pz, o.sr, o.st, o.z});
                    }
                }
            }
            wave_lds_fence();
            if (blk + 1 < blocks) request(blk + 1);

            // ---- the running product takes the positions of the block in one after the other ----
            const int c_lo = REV ? 0 : max(lo - base, 0), c_hi = REV ? min(hi - base, 16) : 16, cnt = c_hi - c_lo;
            auto at = [&](int k) { return REV ? c_lo + k : c_hi - 1 - k; };
            // factor and right-hand side of the position in column c
            auto assemble = [&](int c, float (&a)[NB][NB][4], Acc (&rv)[NB]) {
                if constexpr (!REV) {
#pragma unroll
                    for (int Y = 0; Y < NB; ++Y) {
                        const float* o = sFw + c * PS + 16 * Y + 4 * g;
                        const Acc pz = load4(o), sr = load4(o + KS), st = load4(o + 2 * KS), z = load4(o + 3 * KS);
                        rv[Y] = load4(o + 4 * KS);
#pragma unroll
                        for (int X = 0; X < NB; ++X)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                float j = pz[v] * ua[1][X][Y][v] + (sr[v] * ua[2][X][Y][v] + st[v] * ua[0][X][Y][v]);
                                if (X == Y) j += dsel[v] * z[v];
                                a[X][Y][v] = j;
                            }
                    }
                } else {
#pragma unroll
                    for (int X = 0; X < NB; ++X) {
                        rv[X] = load4(sFw + 64 * N + c * N + 16 * X + 4 * g);
                        const Acc ff = load4(sFw + (c * N + 16 * X + r) * 4);
#pragma unroll
                        for (int Y = 0; Y < NB; ++Y)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                float j = ff[0] * ua[1][X][Y][v] + (ff[1] * ua[2][X][Y][v] + ff[2] * ua[0][X][Y][v]);
                                if (X == Y) j += dsel[v] * ff[3];
                                a[X][Y][v] = j;
                            }
                    }
                }
            };
            auto add_vector = [&](const Acc (&rv)[NB]) {
#pragma unroll
                for (int C = 0; C < NB; ++C) {
                    float s = SPLIT ? 0.f : vec[C];
#pragma unroll
                    for (int K = 0; K < NB; ++K)
#pragma unroll
                        for (int v = 0; v < 4; ++v) s += Q[K][C][v] * rv[K][v];
                    vec[C] = SPLIT ? vec[C] + s * scale[C].down : s;
                }
            };
            // at the end of a chunk its map leaves: M[16 C + r][16 X + 4g + v] = Q[X][C][v]
            auto finish = [&](int c) {
                if (base + c != edge) return;
                float* o = tot + (long long)q * MS;
                float sum = 0.f;   // (not a finite number if one of its terms is none)
#pragma unroll
                for (int C = 0; C < NB; ++C) {
#pragma unroll
                    for (int X = 0; X < NB; ++X) {
                        if (SPLIT)
#pragma unroll
                            for (int v = 0; v < 4; ++v) sum += 0.f * Q[X][C][v];
                        Acc m = Q[X][C];
                        if (SPLIT)
#pragma unroll
                            for (int v = 0; v < 4; ++v) m[v] = __builtin_amdgcn_ldexpf(m[v], -scale[C].e);
                        store4(o + (16 * C + r) * N + 16 * X + 4 * g, m);
                    }
                    const float s = sum_groups(vec[C]);
                    if (g == 0) o[N * N + 16 * C + r] = s;
                }
                again |= sum != 0.f;
                reset();
                q += REV ? 1 : -1;
                edge = REV ? min(T, (first + q + 1) * Lc) - 1 : (first + q) * Lc;
            };
#pragma unroll 2
            for (int k = 0; k < cnt; ++k) {
                float a[NB][NB][4];
                Acc rv[NB], Qn[NB][NB];
                assemble(at(k), a, rv);
                add_vector(rv);
                if (SPLIT && !wide) {
                    auto row = [&](int X, int Y) { return Acc{a[X][Y][0], a[X][Y][1], a[X][Y][2], a[X][Y][3]}; };
                    if constexpr (N == 16) {
                        Qn[0][0] = split_product(split4(row(0, 0)), split4(Q[0][0]), zero4());
                    } else {
                        Split8 A[NB], B[NB];
#pragma unroll
                        for (int X = 0; X < NB; ++X) {
                            A[X] = split8(row(X, 0), row(X, NB - 1));
                            B[X] = split8(Q[0][X], Q[NB - 1][X]);
                        }
#pragma unroll
                        for (int part = 0; part < 3; ++part)
#pragma unroll
                            for (int X = 0; X < NB; ++X)
#pragma unroll
                                for (int C = 0; C < NB; ++C)
                                    Qn[X][C] = mfma16(part == 0 ? A[X].lo : A[X].hi, part == 1 ? B[C].lo : B[C].hi, part == 0 ? zero4() : Qn[X][C]);
                    }
                } else {
#pragma unroll
                    for (int X = 0; X < NB; ++X)
#pragma unroll
                        for (int C = 0; C < NB; ++C) Qn[X][C] = zero4();
#pragma unroll
                    for (int K = 0; K < NB; ++K)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
#pragma unroll
                            for (int X = 0; X < NB; ++X)
#pragma unroll
                                for (int C = 0; C < NB; ++C) Qn[X][C] = mfma(a[X][K][v], Q[K][C][v], Qn[X][C]);
                }
#pragma unroll
                for (int X = 0; X < NB; ++X)
#pragma unroll
                    for (int C = 0; C < NB; ++C) Q[X][C] = Qn[X][C];
                finish(at(k));
            }
            wave_lds_fence();
        }
        if (wide || !__ballot(again)) break;
        wide = true;
        q = kept;
        top = min(T, (first + q + 1) * Lc);
        request(0);
    }
    __syncthreads();

    // the units of the group that nothing follows need no map
    const int pu = 16 / p.per_unit;
    const bool needed = REV ? unit >= pu : unit < (p.groups - 1) * pu;
    if (needed && wave <= NB)
        compose_unit<N, REV>(tot, p.sup + ((long long)b * p.units + unit) * MS, min(p.per_unit, chunks - first), wave, g, r);
}

// ------------------------------------------------------------------------------------------------------------------
// The walk: one wavefront per group, its sixteen chunks are the columns of every product.
// ------------------------------------------------------------------------------------------------------------------
// SPLIT (n = 32, not from far iterates): the products with the state and with the correction have their factors split in two fp16 numbers, a scale
// to every column from its largest entry; U keeps all its digits for the state (a third part), which the trajectory sees, and its small entries theirs next to large ones (Split8Weights).
// Bound: issue, one or two wavefronts a SIMD: a step takes 12 fp32 matrix instructions (the input's) and 42 of 18 cycles in the place of 108 fp32 ones.  16 x
// 100,000 positions, d = 8: 314 us with fp32 products, now 212; 2-norm error of the trajectory against 64 bits 1.347e-7, now 1.309e-7.
template <int N, int DS, bool REV, bool SPLIT>
__global__ __launch_bounds__(256, N == 16 ? 3 : 2) void chunk_walk_kernel(ChunkParams p) {
    constexpr int NB = N / 16;
    static_assert(!SPLIT || (N == 32 && !REV), "");
    __shared__ unsigned s_max[4];
    __shared__ __align__(16) float sB[4 * N];
    if (step_closed(p.gate, p.far != 0)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int T = p.T, d = p.d, Lc = p.Lc;
    const float* __restrict__ th = p.theta;
    const float* __restrict__ U = th + 3 * N * d;
    if (tid < 4 * N) sB[tid] = U[3 * N * N + tid];
    // sixteen inputs: W waits in LDS, its registers go to the parts of U (with both in registers five spilled: a solve at 16 x 50,000, d = 16, 2,632 us, now 2,534)
    constexpr bool WLDS = SPLIT && DS == 4;
    __shared__ __align__(16) Acc sW[WLDS ? 3 * NB : 1][64];
    auto w_entry = [&](int gate, int I, int l, int s) {
        const int c = DS * (l >> 4) + s;
        return c < d ? th[(gate * N + 16 * I + (l & 15)) * d + c] : 0.f;
    };
    if constexpr (WLDS)
        for (int q = tid; q < 3 * NB * 64; q += 256)
#pragma unroll
            for (int s = 0; s < DS; ++s) sW[q / 64][q % 64][s] = w_entry(q / 64 / NB, q / 64 % NB, q % 64, s);
    __syncthreads();

    const unsigned id = blockIdx.x * 4u + (unsigned)wave;
    const int b = (int)(id % (unsigned)p.B), grp = (int)(id / (unsigned)p.B);
    unsigned emax = 0u;   // largest |y_new - y| as raw bits (a NaN compares above everything)
    if (grp < p.groups) {
        const int chunks = (T + Lc - 1) / Lc, nq = min(16, chunks - 16 * grp);
        // addresses relative to the group's first position
        const long long first = (long long)b * T + (long long)16 * grp * Lc;
        const float* __restrict__ yb = p.y + first * N;
        const float* __restrict__ xb = p.x + first * d;
        const float* __restrict__ gb = REV ? p.g + first * N : nullptr;
        float* __restrict__ ob = p.out + first * N;
        const int a = r * Lc, end = T - 16 * grp * Lc;   // this column's first position, one past the last that exists
        auto row = [&](int rel) { return (unsigned)min(max(rel, 0), end - 1); };

        // What step t reads: forward y at the position (the state in front of the next one), dual y and g at the position;
        // both the input of the cell the step evaluates.  Requested R - 1 steps ahead: a step is shorter than a trip to the last-level
        // cache.  Slots are named by t mod R, so nothing moves between registers.
        constexpr int R = (REV && N == 32) ? 2 : 4;
        Acc yr[R][NB], gr[REV ? R : 1][NB];
        float xr[R][DS];
        auto ask_y = [&](int j, int t) {
            const unsigned o = row(REV ? a + Lc - 1 - t : a + t) * N + 4 * g;
#pragma unroll
            for (int K = 0; K < NB; ++K) {
                yr[j][K] = load4(yb + o + 16 * K);
                if constexpr (REV) gr[j][K] = load4(gb + o + 16 * K);
            }
        };
        auto ask_x = [&](int j, int t) {
            const unsigned o = row(REV ? a + Lc - t : a + t) * (unsigned)d;
#pragma unroll
            for (int s = 0; s < DS; ++s) xr[j][s] = xb[o + min(DS * g + s, d - 1)];
        };
        if constexpr (!REV) {
            const bool start = a == 0 && grp == 0;
            const float* __restrict__ y0b = p.y0 ? p.y0 + (long long)b * N : nullptr;
            const float* hp = start ? y0b : yb + (long long)(min(a, end) - 1) * N;
#pragma unroll
            for (int K = 0; K < NB; ++K) yr[R - 1][K] = hp ? load4(hp + 16 * K + 4 * g) : zero4();
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (REV || j < R - 1) ask_y(j, j);
            ask_x(j, j);
        }

        Acc u[3][NB][NB];      // U_gate as operand A
        Split8Weights us[3][SPLIT ? NB : 1];   // its parts, U 2^eu with entries below 2^8
        int eu = 0;
        Acc ut[REV ? 3 : 1][REV ? NB : 1][REV ? NB : 1];   // dual: U_gate^T as operand A
        float w[3][NB][DS];
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int I = 0; I < NB; ++I) {
#pragma unroll
                for (int K = 0; K < NB; ++K) {
                    u[gate][I][K] = load4(U + (gate * N + 16 * I + r) * N + 16 * K + 4 * g);
                    if constexpr (REV)
#pragma unroll
                        for (int v = 0; v < 4; ++v) ut[gate][I][K][v] = U[(gate * N + 16 * K + 4 * g + v) * N + 16 * I + r];
                }
                if constexpr (!WLDS)
#pragma unroll
                    for (int s = 0; s < DS; ++s) w[gate][I][s] = w_entry(gate, I, lane, s);
            }

        if constexpr (SPLIT) {
            float m = 0.f;
#pragma unroll
            for (int gate = 0; gate < 3; ++gate)
#pragma unroll
                for (int I = 0; I < NB; ++I)
#pragma unroll
                    for (int K = 0; K < NB; ++K)
#pragma unroll
                        for (int v = 0; v < 4; ++v) m = fmaxf(m, fabsf(u[gate][I][K][v]));
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
            eu = min(8 - exponent(max_groups(m)), 100);
            const float up = __builtin_amdgcn_ldexpf(1.f, eu);
#pragma unroll
            for (int gate = 0; gate < 3; ++gate)
#pragma unroll
                for (int I = 0; I < NB; ++I) us[gate][I] = split8_weights(u[gate][I][0] * up, u[gate][I][NB - 1] * up);
        }

        Acc e[NB];   // forward: correction of the state in front of the position; dual: lambda at the time after it
        Acc x[REV ? 1 : NB];   // forward: the new state in front of the position
        const bool far = !REV && p.far;
        fold_carries<N, REV>(p, b, grp, nq, g, r, e, far, [&](int row) { return p.y0 ? p.y0[(long long)b * N + row] : 0.f; });
        if constexpr (!REV)
#pragma unroll
            for (int K = 0; K < NB; ++K) {
                x[K] = far ? e[K] : yr[R - 1][K] + e[K];
                if (far) e[K] = x[K] - yr[R - 1][K];
            }

        for (int t0 = 0; t0 < Lc; t0 += R) {   // Lc is a multiple of four
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int t = t0 + j, rel = REV ? a + Lc - 1 - t : a + t;
                const bool live = rel < end;
                Acc (&h)[NB] = yr[REV ? j : (j + R - 1) % R];
                // gates (forward: of the position, dual: of the one after it)
                Acc y[NB];
                Acc lr[NB], lz[NB], lc[NB];
                Split8 hs, es;
                Half8 small_h, small_e;
                float down_h = 1.f, down_e = 1.f;
                if constexpr (SPLIT) {
                    auto split_column = [&](const Acc (&x)[NB], Split8& s) {
                        float m = 0.f;
#pragma unroll
                        for (int K = 0; K < NB; ++K)
#pragma unroll
                            for (int v = 0; v < 4; ++v) m = fmaxf(m, fabsf(x[K][v]));
                        const int k = min(13 - exponent(max_groups(m)), 100);
                        const float f = __builtin_amdgcn_ldexpf(1.f, k);
                        s = split8(x[0] * f, x[NB - 1] * f);
                        return __builtin_amdgcn_ldexpf(1.f, -k - eu);
                    };
                    down_h = split_column(h, hs);
                    down_e = split_column(e, es);
                    small_h = split_small(hs.hi);
                    small_e = split_small(es.hi);
                }
#pragma unroll
                for (int I = 0; I < NB; ++I) {
                    const float* bs = sB + 16 * I + 4 * g;
                    Acc ar = load4(bs), az = load4(bs + N), ac = load4(bs + 2 * N), aq = load4(bs + 3 * N);
                    Acc er = zero4(), ez = zero4(), ec = zero4();
                    if constexpr (SPLIT) {
                        auto state = [&](int gate) {
                            Acc t = mfma16(us[gate][I].rest, small_h, zero4());
                            t = mfma16(us[gate][I].lo, small_h, t);
                            t = mfma16(us[gate][I].hi, hs.lo, t);
                            return mfma16(us[gate][I].hi, hs.hi, t);
                        };
                        auto correction = [&](int gate) {
                            Acc t = mfma16(us[gate][I].lo, small_e, zero4());
                            t = mfma16(us[gate][I].hi, es.lo, t);
                            return mfma16(us[gate][I].hi, es.hi, t);
                        };
                        const Acc tr = state(0), tz = state(1), tc = state(2);
                        er = correction(0);
                        ez = correction(1);
                        ec = correction(2);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            ar[v] += tr[v] * down_h;
                            az[v] += tz[v] * down_h;
                            aq[v] += tc[v] * down_h;
                        }
                    } else
#pragma unroll
                    for (int K = 0; K < NB; ++K)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            ar = mfma(u[0][I][K][v], h[K][v], ar);
                            az = mfma(u[1][I][K][v], h[K][v], az);
                            aq = mfma(u[2][I][K][v], h[K][v], aq);
                            if constexpr (!REV) {
                                er = mfma(u[0][I][K][v], e[K][v], er);
                                ez = mfma(u[1][I][K][v], e[K][v], ez);
                                ec = mfma(u[2][I][K][v], e[K][v], ec);
                            }
                        }
                    if constexpr (WLDS) {
                        int at = lane;
                        asm volatile("" : "+v"(at));   // (or the reads leave the loop)
#pragma unroll
                        for (int gate = 0; gate < 3; ++gate) {
                            const Acc o = sW[gate * NB + I][at];
#pragma unroll
                            for (int s = 0; s < DS; ++s) w[gate][I][s] = o[s];
                        }
                    }
#pragma unroll
                    for (int s = 0; s < DS; ++s) {
                        ar = mfma(w[0][I][s], xr[j][s], ar);
                        az = mfma(w[1][I][s], xr[j][s], az);
                        ac = mfma(w[2][I][s], xr[j][s], ac);
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const GruGates k = gru_gates(ar[v], az[v], ac[v], aq[v], h[I][v]);
                        if constexpr (!REV) {
                            y[I][v] = k.c + (k.z * (x[REV ? 0 : I][v] - k.c) + down_e * (k.pz * ez[v] + (k.sr * ec[v] + k.st * er[v])));
                        } else {
                            const float l = e[I][v];
                            lz[I][v] = k.pz * l;
                            lc[I][v] = k.sr * l;
                            lr[I][v] = k.st * l;
                            y[I][v] = k.z * l;
                        }
                    }
                }
                if constexpr (REV) {
                    // lambda_pos = g_pos + J_{pos+1}^T lambda_{pos+1}.  The products are added up by themselves: with g or z lambda in the accumulator
                    // every instruction rounds at the size of lambda (dL/dx at n = 27 was 2.65e-7 off, now 2.12e-7, the single-pass scan 2.14e-7)
#pragma unroll
                    for (int I = 0; I < NB; ++I) {
                        Acc s0 = zero4(), s1 = zero4();
#pragma unroll
                        for (int K = 0; K < NB; ++K)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                s0 = mfma(ut[1][I][K][v], lz[K][v], s0);
                                s1 = mfma(ut[2][I][K][v], lc[K][v], s1);
                                s0 = mfma(ut[0][I][K][v], lr[K][v], s0);
                            }
#pragma unroll
                        for (int v = 0; v < 4; ++v) y[I][v] = gr[REV ? j : 0][I][v] + (y[I][v] + (s0[v] + s1[v]));
                    }
                }
                const unsigned o = (unsigned)(rel * N + 4 * g);
                if (live) {
#pragma unroll
                    for (int I = 0; I < NB; ++I) store4(ob + o + 16 * I, y[I]);
                }
                const unsigned mask = live ? 0x7fffffffu : 0u;
#pragma unroll
                for (int I = 0; I < NB; ++I)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if constexpr (!REV) {
                            x[REV ? 0 : I][v] = y[I][v];
                            e[I][v] = y[I][v] - yr[j][I][v];
                            emax = max(emax, __float_as_uint(e[I][v]) & mask);
                        } else {
                            e[I][v] = live ? y[I][v] : 0.f;   // nothing follows the last time
                        }
                    }
                if constexpr (!REV) ask_y((j + R - 1) % R, t - 1 + R);
                else ask_y(j, t + R);
                ask_x(j, t + R);
            }
        }
    }
    if (!REV && p.err) {
        // one read-modify-write per workgroup: all wavefronts end at about the same time and queue on one address
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) emax = max(emax, (unsigned)__shfl_xor((int)emax, o));
        if (lane == 0) s_max[wave] = emax;
        __syncthreads();
        if (tid == 0) {
            emax = max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3]));
            err_atomic_max(p.err, __uint_as_float(min(emax, 0x7f800000u)));
        }
    }
}

// ------------------------------------------------------------------------------------------------------------------
// n = 16: the dual walk with the vector-Jacobian product inside (as in chunk_cells.hip).  lambda_i = g_i + J_{i+1}^T lambda_{i+1} needs the
// cotangents of the pre-activations at position i + 1, which are all that dL/dx, dL/dtheta and (at the first position) dL/dy0 are made of;
// one more step takes the first position of a sequence.  The sums over positions have the columns on the contraction index:
// cotangents, state and input cross a slice of LDS.  J^T lambda is added up without g (see the walk above), and a
// position's sixteen columns by themselves before they join the sums (see chunk_cells.hip; chunks of 32 positions: 3.9e-7 -> 2.4e-7).  At n = 32 the sums (72 registers more) would leave one wavefront per SIMD.
// Measured, d = 6, 32 x 17,984 positions: walk 43 us and a kernel of its own for the product 126 us; now 79 us in all.
// ------------------------------------------------------------------------------------------------------------------
template <int DS>
__global__ __launch_bounds__(256, 2) void chunk_dual16_kernel(ChunkParams p) {
    constexpr int N = 16, SLICE = 1600;   // six tiles of [column][16]; at the end the wavefront's row of dL/dtheta (at most 1,600 scalars)
    __shared__ __align__(16) float sT[4][SLICE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int T = p.T, d = p.d, Lc = p.Lc;
    const float* __restrict__ th = p.theta;
    const float* __restrict__ U = th + 3 * N * d;
    const float* __restrict__ bias = U + 3 * N * N;
    float* __restrict__ S = sT[wave];
    const unsigned id = blockIdx.x * 4u + (unsigned)wave;
    const int b = (int)(id % (unsigned)p.B), grp = (int)(id / (unsigned)p.B);
    Acc aU[3], aW[3], aB[4];   // blocks r, z, c; bias sums of this column's rows: r, z, c, hidden part of c
#pragma unroll
    for (int q = 0; q < 3; ++q) aU[q] = aW[q] = zero4();
#pragma unroll
    for (int q = 0; q < 4; ++q) aB[q] = zero4();
    store4(S + 1280 + 4 * lane, zero4());   // (input columns past 4 DS are never written)
    wave_lds_fence();
    if (grp < p.groups) {
        const int chunks = (T + Lc - 1) / Lc, nq = min(16, chunks - 16 * grp);
        const long long first = (long long)b * T + (long long)16 * grp * Lc;
        const float* __restrict__ yb = p.y + first * N;
        const float* __restrict__ xb = p.x + first * d;
        const float* __restrict__ gb = p.g + first * N;
        float* __restrict__ dxb = p.dx ? p.dx + first * d : nullptr;
        const int a = r * Lc, end = T - 16 * grp * Lc;
        auto row = [&](int rel) { return (unsigned)min(max(rel, 0), end - 1); };
        constexpr int R = 2;
        Acc yr[R], gr[R];
        float xr[R][DS];
        auto ask = [&](int j, int t) {
            const unsigned o = row(a + Lc - 1 - t) * N + 4 * g, ox = row(a + Lc - t) * (unsigned)d;
            yr[j] = load4(yb + o);
            gr[j] = load4(gb + o);
#pragma unroll
            for (int s = 0; s < DS; ++s) xr[j][s] = xb[ox + min(DS * g + s, d - 1)];
        };
#pragma unroll
        for (int j = 0; j < R; ++j) ask(j, j);
        Acc u[3], ut[3], wt[3], bs[4];   // U_gate, U_gate^T and W_gate^T as operand A
        float w[3][DS];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            u[q] = load4(U + (q * N + r) * N + 4 * g);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = q * N + 4 * g + v;
                const float x = th[k * d + min(r, d - 1)];
                ut[q][v] = U[k * N + r];
                wt[q][v] = r < d ? x : 0.f;
            }
#pragma unroll
            for (int s = 0; s < DS; ++s) {
                const float x = th[(q * N + r) * d + min(DS * g + s, d - 1)];
                w[q][s] = DS * g + s < d ? x : 0.f;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) bs[q] = load4(bias + q * N + 4 * g);
        Acc ev[1];   // lambda at the position the step evaluates
        fold_carries<N, true>(p, b, grp, nq, g, r, ev, false, [](int) { return 0.f; });
        Acc e = ev[0];

        // one step at position `at` (relative) with state h in front of it: y = J^T lambda
        auto step = [&](const Acc& h, const float (&x)[DS], int at, Acc& y) {
            Acc ar = bs[0], az = bs[1], ac = bs[2], aq = bs[3];
#pragma unroll
            for (int s = 0; s < DS; ++s) {
                ar = mfma(w[0][s], x[s], ar);
                az = mfma(w[1][s], x[s], az);
                ac = mfma(w[2][s], x[s], ac);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                ar = mfma(u[0][v], h[v], ar);
                az = mfma(u[1][v], h[v], az);
                aq = mfma(u[2][v], h[v], aq);
            }
            Acc dr, dz, dc, dq;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const GruGates k = gru_gates(ar[v], az[v], ac[v], aq[v], h[v]);
                dr[v] = k.st * e[v];
                dz[v] = k.pz * e[v];
                dc[v] = k.sc * e[v];
                dq[v] = k.sr * e[v];
                y[v] = k.z * e[v];
            }
            float* o = S + r * 16 + 4 * g;
            store4(o, dr); store4(o + 256, dz); store4(o + 512, dq); store4(o + 768, dc); store4(o + 1024, h);
#pragma unroll
            for (int s = 0; s < DS; ++s) S[1280 + r * 16 + DS * g + s] = x[s];
            aB[0] += dr; aB[1] += dz; aB[2] += dc; aB[3] += dq;
            Acc s1 = zero4(), dx = zero4();
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s1 = mfma(ut[1][v], dz[v], s1);
                s1 = mfma(ut[0][v], dr[v], s1);
                dx = mfma(wt[0][v], dr[v], dx);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s1 = mfma(ut[2][v], dq[v], s1);
                dx = mfma(wt[1][v], dz[v], dx);
                dx = mfma(wt[2][v], dc[v], dx);
            }
            y += s1;
            if (dxb && at < end) {
                float* t = dxb + (long long)at * d + 4 * g;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (4 * g + v < d) t[v] = dx[v];
            }
            wave_lds_fence();
            const float* q = S + g * 16 + r;   // row m of four: + 64 m
            float hk[4], xk[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                hk[m] = q[64 * m + 1024];
                xk[m] = q[64 * m + 1280];
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) {   // r, z, c (hidden part 512, input part 768)
                Acc pU = zero4(), pW = zero4();
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const float t = q[64 * m + 256 * i];
                    pU = mfma(t, hk[m], pU);
                    pW = mfma(i == 2 ? q[64 * m + 768] : t, xk[m], pW);
                }
                aU[i] += pU;
                aW[i] += pW;
            }
            wave_lds_fence();
        };
        for (int t0 = 0; t0 < Lc; t0 += R) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int t = t0 + j, rel = a + Lc - 1 - t;
                const bool live = rel < end;
                Acc y;
                step(yr[j], xr[j], rel + 1, y);
#pragma unroll
                for (int v = 0; v < 4; ++v) e[v] = live ? gr[j][v] + y[v] : 0.f;   // nothing follows the last position
                ask(j, t + R);
            }
        }
        if (grp == 0) {   // the first position of the sequence
            const Acc h = p.y0 ? load4(p.y0 + (long long)b * N + 4 * g) : zero4();
            Acc y;
#pragma unroll
            for (int v = 0; v < 4; ++v) e[v] = r == 0 ? e[v] : 0.f;
            step(h, xr[0], r == 0 ? 0 : end, y);
            if (p.dy0 && r == 0)
#pragma unroll
                for (int v = 0; v < 4; ++v) p.dy0[(long long)b * N + 4 * g + v] = y[v];
        }
    }
    // ---- the workgroup's row of dL/dtheta ----
    const int U0 = 3 * N * d, b0 = U0 + 3 * N * N, P = b0 + 4 * N;
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = q * N + 4 * g + v;
            S[U0 + k * N + r] = aU[q][v];
            if (r < d) S[k * d + r] = aW[q][v];
        }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const Acc s = row_sums4(aB[q], r);
        if (r == 0) store4(S + b0 + q * N + 4 * g, s);
    }
    __syncthreads();
    for (int q = tid; q < P; q += 256) p.partial[(long long)blockIdx.x * P + q] = (sT[0][q] + sT[1][q]) + (sT[2][q] + sT[3][q]);
}

template <int N, int DS, bool REV>
hipError_t launch_nd(const ChunkParams& p, hipStream_t s) {
    const dim3 units((unsigned)((long long)p.B * p.units));
    if (!REV && p.far) hipLaunchKernelGGL((chunk_totals_kernel<N, DS, REV, !REV>), units, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((chunk_totals_kernel<N, DS, REV, false>), units, dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int rows = (int)chunk_rows(p);
    if constexpr (N == 16 && REV) {
        hipLaunchKernelGGL((chunk_dual16_kernel<DS>), dim3((unsigned)rows), dim3(256), 0, s, p);
        e = hipGetLastError();
        return e != hipSuccess ? e : launch_partial_reduce(0, p.partial, p.dtheta, 3LL * N * p.d + 3LL * N * N + 4 * N, rows, s);
    } else {
        constexpr bool SPLIT = N == 32 && !REV;
        if (SPLIT && !p.far) hipLaunchKernelGGL((chunk_walk_kernel<N, DS, REV, SPLIT>), dim3((unsigned)rows), dim3(256), 0, s, p);
        else hipLaunchKernelGGL((chunk_walk_kernel<N, DS, REV, false>), dim3((unsigned)rows), dim3(256), 0, s, p);
        return hipGetLastError();
    }
}

template <int N, bool REV>
hipError_t launch_n(const ChunkParams& p, hipStream_t s) {
    if (p.d <= 4) return launch_nd<N, 1, REV>(p, s);
    if (p.d <= 8) return launch_nd<N, 2, REV>(p, s);
    return launch_nd<N, 4, REV>(p, s);
}

}  // namespace

bool chunk_gru_supported(int dtype, int n, int d) { return dtype == 0 && (n == 16 || n == 32 || n == 64) && d >= 1 && d <= 16; }

size_t chunk_map_bytes(int n) { return ((size_t)n * n + n) * sizeof(float); }

long long chunk_rows(const ChunkParams& p) { return ((long long)p.B * p.groups + 3) / 4; }

bool chunk_params_valid(const ChunkParams& p) {
    return p.Lc >= 4 && p.Lc % 4 == 0 && (p.per_unit == 4 || p.per_unit == 8 || p.per_unit == 16) &&
           p.groups == (int)((p.T + 16LL * p.Lc - 1) / (16LL * p.Lc)) &&
           p.units == (int)((p.T + (long long)p.per_unit * p.Lc - 1) / ((long long)p.per_unit * p.Lc));
}

hipError_t launch_chunk_gru(int n, const ChunkParams& p, hipStream_t s) {
    if (!chunk_gru_supported(0, n, p.d) || !chunk_params_valid(p)) return hipErrorInvalidValue;
    if (n == 64) return launch_chunk_gru64(p, s);
    const bool rev = p.g != nullptr;
    if (rev && n == 16 ? !p.partial || !p.dtheta : !p.out) return hipErrorInvalidValue;
    if (n == 16) return rev ? launch_n<16, true>(p, s) : launch_n<16, false>(p, s);
    return rev ? launch_n<32, true>(p, s) : launch_n<32, false>(p, s);
}

}  // namespace deer
