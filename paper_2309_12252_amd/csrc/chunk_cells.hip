// Newton step and dual scan of the LSTM and the LEM by chunks in fp32 (the scheme of chunk_gru.hip: maps of chunks, then a walk of
// sixteen chunks per wavefront), equations and factors of the cells in cell_lstm.hip.
//
// The state is two parts of u <= 16 units, (h | c) or (y | z); kernels hold UP = 8 or 16 units a part, the rest zero (zero
// weights and zero state stay zero), and read and write the caller's rows of 2u scalars directly.  The Jacobian never exists
// in memory, and the reduction uses its structure: a step of either cell is two triangular steps,
//     LSTM   c' = f c + M h,             h' = D U_o h + a c'            M = sum of diag(factor) U over i, f, g
//     LEM    z' = (1 - s1) z + M y,      y' = (1 - s2) y + F U_2 y + E U_y z'       M = C1 U_1 + C2 U_z
// (in the differentials), so at UP = 16 the running product is multiplied by two or three u x u factors instead of one of
// 2u x 2u.  At UP = 8 both parts share one 16 x 16 block: one dense factor (LSTM) or one per triangular step (LEM).
//
// Lane (g, r) of a wavefront evaluates units 4g .. 4g + 3 of position (column) r; at UP = 8 lanes g and g + 2 evaluate the same units
// (the products with U then contract over 8 entries in two instructions: lane groups 0, 1 supply two of their four
// units, groups 2, 3 the other two), groups 0, 1 answer for the rows of the first part, 2, 3 for those of the second.
//
// Bound: issue (matrix and vector instructions of a SIMD do not overlap).  Above 8 units the reduction of a Newton step has the factors of its
// products split in two fp16 numbers, as in chunk_gru.hip (the dual scan has fp32 products, for the reason given there).  Measured, a Newton step (Jacobian kernel and
// scan before / both launches now): LSTM u = 8, d = 4, 16 x 50,000 positions 710 / 211 us; LEM u = 16, d = 6, 32 x 17,984 positions 2,280 / 359 us (reduction 348 with
// fp32 products, now 289).
#include "chunk_common.h"
#include "split_f16.h"

#include <type_traits>

namespace deer {

namespace {

enum { LSTM = 0, LEM = 1 };

// Row factors of one unit.  LSTM: a = factor of U_i, b = of U_f, c = of U_g in dc', d = of U_o in dh', e = of dc' in dh', f = f.
// LEM: a = factor of U_1, b = of U_z in dz', c = of U_2, d = of U_y in dy', e = 1 - s2, f = 1 - s1.
struct Factors {
    float n0, n1;   // new state, first and second part
    float a, b, c, d, e, f;
    float g0, g1;   // what the linear terms leave of it: LSTM c' - f c; LEM y' - (1 - s2) y, z' - (1 - s1) z
};

template <int CELL, int UP, int DS>
struct Cell {
    static constexpr int KS = UP / 4;   // matrix instructions of a contraction over the units
    float u[4][KS];    // operand A: row r (mod UP) of U_gate
    float w[4][DS];
    Acc b[4];

    // entry of the contraction that lane group g supplies in instruction s
    static __device__ __forceinline__ int kappa(int g, int s) { return UP == 16 ? 4 * g + s : 4 * (g & 1) + (g < 2 ? s : 2 + s); }
    // operand B from the four units of a lane
    static __device__ __forceinline__ float operand(const Acc& v, int g, int s) {
        if constexpr (UP == 16) return v[s];
        else {
            const float lo = v[s], hi = v[s + 2];   // (both by constant index)
            return g < 2 ? lo : hi;
        }
    }
    __device__ __forceinline__ void load(const float* __restrict__ th, int n, int d, int g, int r) {
        const float* __restrict__ U = th + 4 * n * d;
        const float* __restrict__ bias = U + 4 * n * n;
        const int row = min(r % UP, n - 1);
        const bool in = r % UP < n;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int k = kappa(g, s);
                const float v = U[(q * n + row) * n + min(k, n - 1)];
                u[q][s] = in && k < n ? v : 0.f;
            }
#pragma unroll
            for (int s = 0; s < DS; ++s) {
                const int k = DS * g + s;
                const float v = th[(q * n + row) * d + min(k, d - 1)];
                w[q][s] = in && k < d ? v : 0.f;
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int j = (4 * g + v) % UP;
                const float t = bias[q * n + min(j, n - 1)];
                b[q][v] = j < n ? t : 0.f;
            }
        }
    }
    // U_gate times a vector whose units the lanes hold, added to acc
    __device__ __forceinline__ Acc times(int q, const Acc& x, Acc acc, int g) const {
#pragma unroll
        for (int s = 0; s < KS; ++s) acc = mfma(u[q][s], operand(x, g, s), acc);
        return acc;
    }
    // the cell at the lane's four units of sixteen positions
    __device__ __forceinline__ void eval(Factors (&o)[4], const Acc& s0, const Acc& s1, const float (&x)[DS], float dt, int g) const {
        Acc a[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] = b[q];
#pragma unroll
            for (int s = 0; s < DS; ++s) a[q] = mfma(w[q][s], x[s], a[q]);
            if (CELL == LSTM || q < 3) a[q] = times(q, s0, a[q], g);
        }
        if constexpr (CELL == LSTM) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float i = feed_sigmoid(a[0][v]), f = feed_sigmoid(a[1][v]), gg = feed_tanh(a[2][v]), oo = feed_sigmoid(a[3][v]);
                const float cn = f * s1[v] + i * gg, tc = feed_tanh(cn);
                o[v].g0 = 0.f;
                o[v].g1 = i * gg;
                o[v].n0 = oo * tc;
                o[v].n1 = cn;
                o[v].a = gg * i * (1.f - i);
                o[v].b = s1[v] * f * (1.f - f);
                o[v].c = i * (1.f - gg * gg);
                o[v].d = tc * oo * (1.f - oo);
                o[v].e = oo * (1.f - tc * tc);
                o[v].f = f;
            }
        } else {
            Acc zn;
            const float inv = 1.f / dt;
            float s2[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float t1 = dt * feed_sigmoid(a[0][v]), gz = feed_tanh(a[2][v]);
                s2[v] = dt * feed_sigmoid(a[1][v]);
                zn[v] = (1.f - t1) * s1[v] + t1 * gz;
                o[v].n1 = zn[v];
                o[v].g1 = t1 * gz;
                o[v].a = t1 * (1.f - t1 * inv) * (gz - s1[v]);
                o[v].b = t1 * (1.f - gz * gz);
                o[v].f = 1.f - t1;
            }
            a[3] = times(3, zn, a[3], g);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float gy = feed_tanh(a[3][v]);
                o[v].g0 = s2[v] * gy;
                o[v].n0 = (1.f - s2[v]) * s0[v] + o[v].g0;
                o[v].c = s2[v] * (1.f - s2[v] * inv) * (gy - s0[v]);
                o[v].d = s2[v] * (1.f - gy * gy);
                o[v].e = 1.f - s2[v];
            }
        }
    }
};

// four consecutive units of one part of a row of 2 n scalars (units past n: zero)
template <bool VEC>
__device__ __forceinline__ Acc load_units(const float* __restrict__ part, int j0, int n) {
    Acc o = zero4();
    if constexpr (VEC) {
        const Acc t = load4(part + min(j0, n - 4));
        if (j0 < n) o = t;
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float t = part[min(j0 + v, n - 1)];
            o[v] = j0 + v < n ? t : 0.f;
        }
    }
    return o;
}
template <bool VEC>
__device__ __forceinline__ void store_units(float* __restrict__ part, int j0, int n, Acc x) {
    if constexpr (VEC) {
        if (j0 < n) store4(part + j0, x);
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (j0 + v < n) part[j0 + v] = x[v];
    }
}

// ------------------------------------------------------------------------------------------------------------------
// Maps of the chunks.  Forward: Q <- J_i^T Q from the last position to the first (Q = P^T); dual: S <- J_i S from the first to the last; see
// chunk_gru.hip.  The factors of sixteen positions sit in the wavefront's LDS slice, [kind][position][row].
// ------------------------------------------------------------------------------------------------------------------
template <int CELL, int UP> struct Slice;
template <int CELL> struct Slice<CELL, 16> { static constexpr int kinds = 8; };   // a .. f, then the vector's two parts; row = unit
template <> struct Slice<LSTM, 8> { static constexpr int kinds = 6; };            // factors of U_i, U_f, U_g, U_o, diagonal, vector; row of the state
template <> struct Slice<LEM, 8> { static constexpr int kinds = 4; };             // two factors and the diagonal of the row's step, vector

// Product with a 16 x 16 factor: of fp32 scalars, or of both factors split in two fp16 numbers
template <bool SPLIT>
struct Product16 {
    static __device__ __forceinline__ auto left(const Acc& a) {
        if constexpr (SPLIT) return split4(a);
        else return a;
    }
    static __device__ __forceinline__ auto right(const Acc& b) {
        if constexpr (SPLIT) return split4(b);
        else return b;
    }
    template <typename A, typename B>
    static __device__ __forceinline__ Acc add(const A& a, const B& b, Acc c) {
        if constexpr (SPLIT) {
            return split_product(a, b, c);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) c = mfma(a[v], b[v], c);
            return c;
        }
    }
};

template <int CELL, int UP, int DS, bool VEC, bool REV, bool FAR>
__global__ __launch_bounds__(256, 2) void cell_totals_kernel(ChunkParams p) {
    constexpr int N = 2 * UP, NB = N / 16, MS = map_size<N>(), KINDS = Slice<CELL, UP>::kinds;
    constexpr bool SPLIT = UP == 16 && !FAR && !REV;   // (a factor of 16 x 16 a position: the split costs what it saves, LSTM u = 8, 16 x 50,000, 120 us with fp32 products, 133)
    __shared__ __align__(16) float sF[4][KINDS * 256];
    if (step_closed(p.gate, FAR)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int b = (int)(blockIdx.x % (unsigned)p.B), unit = (int)(blockIdx.x / (unsigned)p.B);
    const int T = p.T, d = p.d, Lc = p.Lc, n = p.cell_units, ld = 2 * n;
    const float dt = p.dt;
    const int chunks = (T + Lc - 1) / Lc, first = unit * p.per_unit, cpw = p.per_unit / 4;
    const float* __restrict__ yb = p.y + (long long)b * T * ld;
    const float* __restrict__ xb = p.x + (long long)b * T * d;
    const float* __restrict__ y0b = p.y0 ? p.y0 + (long long)b * ld : nullptr;
    const float* __restrict__ gb = REV ? p.g + (long long)b * T * ld : nullptr;
    float* __restrict__ tot = p.tot + ((long long)b * chunks + first) * MS;
    float* __restrict__ sFw = sF[wave];
    const int q_lo = cpw * wave, q_hi = min(q_lo + cpw, chunks - first);   // chunks of this wavefront (inside the unit)
    const int lo = (first + q_lo) * Lc, hi = min(T, (first + q_hi) * Lc);
    int top = hi;   // forward: one past the first position that is still to be reduced
    const int j0 = (4 * g) % UP;   // this lane's units

    Acc s0, s1, v0, v1;
    float x[DS];
    auto request = [&](int blk) {
        int pos = (REV ? lo + 16 * blk : top - 16 * (blk + 1)) + r;
        pos = min(max(pos, lo), hi - 1);
        const float* sp = REV ? yb + (long long)pos * ld : (pos > 0 ? yb + (long long)(pos - 1) * ld : y0b);
        const float* vp = (REV ? gb : yb) + (long long)pos * ld;
        s0 = sp ? load_units<VEC>(sp, j0, n) : zero4();
        s1 = sp ? load_units<VEC>(sp + n, j0, n) : zero4();
        v0 = load_units<VEC>(vp, j0, n);
        v1 = load_units<VEC>(vp + n, j0, n);
        load_x<DS>(x, xb + (long long)(REV ? min(pos + 1, T - 1) : pos) * d, d, g);
    };
    if (q_lo < q_hi) {
        request(0);
        Cell<CELL, UP, DS> cell;
        cell.load(p.theta, n, d, g, r);
        // weights of the assembly
        //   UP = 16: forward U_gate[4g + v][r], dual U_gate[r][4g + v] (the gate operands)
        //   UP = 8: the block of J (LSTM) or of its two steps (LEM) that entry (4g + v, r) of operand A^T (forward) or (r, 4g + v)
        //   (dual) lies in
        float wa[4][4], dm[4], im[4];
        {
            const float* __restrict__ U = p.theta + 4 * n * d;
            auto at = [&](int q, int row, int col) {
                const float t = U[(q * n + min(row, n - 1)) * n + min(col, n - 1)];
                return row < n && col < n ? t : 0.f;
            };
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = REV ? r : 4 * g + v, col = REV ? 4 * g + v : r;   // entry of J (UP = 8: rows 0..7 first part)
                if constexpr (UP == 16) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) wa[q][v] = at(q, row, col);
                    dm[v] = im[v] = 0.f;
                } else if constexpr (CELL == LSTM) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) wa[q][v] = col < 8 ? at(q, row & 7, col) : 0.f;
                    dm[v] = (col == 8 + (row & 7)) ? 1.f : 0.f;
                    im[v] = 0.f;
                } else {
                    // second step (rows of y): U_2 in front of y, U_y in front of z; first step (rows of z): U_1, U_z in front of y
                    wa[0][v] = row < 8 ? (col < 8 ? at(1, row, col) : at(3, row, col - 8)) : 0.f;
                    wa[1][v] = row >= 8 && col < 8 ? at(0, row - 8, col) : 0.f;
                    wa[2][v] = row >= 8 && col < 8 ? at(2, row - 8, col) : 0.f;
                    wa[3][v] = 0.f;
                    dm[v] = (row == col && row < 8) ? 1.f : 0.f;    // diagonal 1 - s2 in the second step, 1 in the first
                    im[v] = (row == col && row >= 8) ? 1.f : 0.f;   // 1 in the second step, 1 - s1 in the first
                }
            }
        }
        float dsel[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) dsel[v] = (4 * g + v == r) ? 1.f : 0.f;

        Acc Q[NB][NB];
        float vec[NB], unit_q = SPLIT ? (float)(1 << ColumnScale::kStart) : 1.f;
        ColumnScale scale[NB];
        auto reset = [&]() {
#pragma unroll
            for (int X = 0; X < NB; ++X) {
                vec[X] = 0.f;
                scale[X].reset(unit_q != 1.f);
#pragma unroll
                for (int C = 0; C < NB; ++C)
#pragma unroll
                    for (int v = 0; v < 4; ++v) Q[X][C][v] = (X == C) ? dsel[v] * unit_q : 0.f;
            }
        };
        bool wide = !SPLIT, again = false;   // products of fp32 factors; a product of the other kind was not finite
        int q = REV ? q_lo : q_hi - 1, kept = q;   // chunk being reduced; the same when all was last seen to be finite
        for (;;) {
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
                {
                    Factors k[4];
                    cell.eval(k, s0, s1, x, dt, g);
                    Acc r0 = v0, r1 = v1;
                    if constexpr (!REV) {
                        if constexpr (FAR) {   // the cell minus J times its state
                            // (one product after the other: registers)
                            Acc q, j1;   // j1: second part of J times the state
#pragma unroll
                            for (int i = 0; i < 3; ++i) {
                                if (CELL == LEM && i == 1) continue;
                                const Acc t = cell.times(i, s0, zero4(), g);
#pragma unroll
                                for (int v = 0; v < 4; ++v) q[v] = i == 0 ? k[v].a * t[v] : q[v] + (CELL == LSTM && i == 2 ? k[v].c : k[v].b) * t[v];
                                __builtin_amdgcn_sched_barrier(0);
                            }
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                j1[v] = k[v].f * s1[v] + q[v];
                                r1[v] = k[v].g1 - q[v];
                            }
                            __builtin_amdgcn_sched_barrier(0);
                            const Acc t3 = cell.times(3, CELL == LSTM ? s0 : j1, zero4(), g);
#pragma unroll
                            for (int v = 0; v < 4; ++v) r0[v] = CELL == LSTM ? k[v].n0 - (k[v].d * t3[v] + k[v].e * j1[v]) : k[v].g0 - k[v].d * t3[v];
                            if constexpr (CELL == LEM) {
                                __builtin_amdgcn_sched_barrier(0);
                                const Acc t1 = cell.times(1, s0, zero4(), g);
#pragma unroll
                                for (int v = 0; v < 4; ++v) r0[v] -= k[v].c * t1[v];
                            }
                        } else {
#pragma unroll
                            for (int v = 0; v < 4; ++v) { r0[v] = k[v].n0 - v0[v]; r1[v] = k[v].n1 - v1[v]; }
                        }
                    }
                    Acc o[KINDS];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if constexpr (UP == 16) {
                            o[0][v] = k[v].a; o[1][v] = k[v].b; o[2][v] = k[v].c; o[3][v] = k[v].d; o[4][v] = k[v].e; o[5][v] = k[v].f;
                            o[6][v] = r0[v]; o[KINDS - 1][v] = r1[v];
                        } else if constexpr (CELL == LSTM) {
                            const float s = g < 2 ? k[v].e : 1.f;   // rows of h: dh' = d U_o h + e dc'
                            o[0][v] = s * k[v].a; o[1][v] = s * k[v].b; o[2][v] = s * k[v].c;
                            o[3][v] = g < 2 ? k[v].d : 0.f;
                            o[4][v] = s * k[v].f;
                            o[KINDS - 1][v] = g < 2 ? r0[v] : r1[v];
                        } else {
                            o[0][v] = g < 2 ? k[v].c : k[v].a;
                            o[1][v] = g < 2 ? k[v].d : k[v].b;
                            o[2][v] = g < 2 ? k[v].e : k[v].f;
                            o[KINDS - 1][v] = g < 2 ? r0[v] : r1[v];
                        }
                    }
#pragma unroll
                    for (int i = 0; i < KINDS; ++i) store4(sFw + i * 256 + r * 16 + 4 * g, o[i]);
                }
                wave_lds_fence();
                if (blk + 1 < blocks) request(blk + 1);

                const int c_lo = REV ? 0 : max(lo - base, 0), c_hi = REV ? min(hi - base, 16) : 16;
                // the running product takes in the position in column c
                auto advance = [&](auto split, int c) {
                    using P = Product16<decltype(split)::value>;
                    const float* fp = sFw + c * 16;   // factors of the position: of rows 4g + v, or of row r
                    auto rows = [&](int i) { return load4(fp + i * 256 + 4 * g); };
                    auto row_r = [&](int i) { return fp[i * 256 + r]; };
                    // a factor of operand A: forward it goes with the contraction index 4g + v, dual with the row r
                    auto fac = [&](int i) {
                        if constexpr (!REV) return rows(i);
                        else { const float t = row_r(i); return Acc{t, t, t, t}; }
                    };
                    if constexpr (UP == 16) {
                        const Acc r0 = rows(6), r1 = rows(KINDS - 1);
#pragma unroll
                        for (int C = 0; C < NB; ++C) {
                            float s = SPLIT ? 0.f : vec[C];
#pragma unroll
                            for (int v = 0; v < 4; ++v) s += Q[0][C][v] * r0[v] + Q[NB - 1][C][v] * r1[v];
                            vec[C] = SPLIT ? vec[C] + s * scale[C].down : s;
                        }
                        const Acc fa = fac(0), fb = fac(1), fc = fac(2), fd = fac(3), fe = rows(4), ff = rows(5);
                        Acc m, n2, n3;   // M; LSTM: D U_o; LEM: E U_y and F U_2
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            if constexpr (CELL == LSTM) {
                                m[v] = fa[v] * wa[0][v] + (fb[v] * wa[1][v] + fc[v] * wa[2][v]);
                                n2[v] = fd[v] * wa[3][v];
                            } else {
                                m[v] = fa[v] * wa[0][v] + fb[v] * wa[2][v];
                                n2[v] = fd[v] * wa[3][v];
                                n3[v] = fc[v] * wa[1][v];
                            }
                        }
                        const auto lm = P::left(m), ln2 = P::left(n2);
                        decltype(P::left(n3)) ln3;
                        if constexpr (CELL == LEM) ln3 = P::left(n3);
#pragma unroll
                        for (int C = 0; C < NB; ++C) {
                            Acc &Q0 = Q[0][C], &Q1 = Q[NB - 1][C];
                            if constexpr (CELL == LSTM && !REV) {
                                // Z = Q1 + e Q0;  Q0 <- (D U_o)^T Q0 + M^T Z,  Q1 <- f Z
                                Acc z;
#pragma unroll
                                for (int v = 0; v < 4; ++v) z[v] = Q1[v] + fe[v] * Q0[v];
                                Q0 = P::add(lm, P::right(z), P::add(ln2, P::right(Q0), zero4()));
#pragma unroll
                                for (int v = 0; v < 4; ++v) Q1[v] = ff[v] * z[v];
                            } else if constexpr (CELL == LSTM) {
                                // S1 <- f S1 + M S0,  S0 <- D U_o S0 + e S1
                                Acc t, w;
#pragma unroll
                                for (int v = 0; v < 4; ++v) t[v] = ff[v] * Q1[v];
                                t = P::add(lm, P::right(Q0), t);
                                w = P::add(ln2, P::right(Q0), zero4());
#pragma unroll
                                for (int v = 0; v < 4; ++v) Q0[v] = w[v] + fe[v] * t[v];
                                Q1 = t;
                            } else if constexpr (!REV) {
                                // Z = Q1 + (E U_y)^T Q0;  Q0 <- (1 - s2) Q0 + (F U_2)^T Q0 + M^T Z,  Q1 <- (1 - s1) Z
                                Acc t;
#pragma unroll
                                for (int v = 0; v < 4; ++v) t[v] = fe[v] * Q0[v];
                                const auto q0 = P::right(Q0);
                                const Acc z = P::add(ln2, q0, Q1);
                                Q0 = P::add(lm, P::right(z), P::add(ln3, q0, t));
#pragma unroll
                                for (int v = 0; v < 4; ++v) Q1[v] = ff[v] * z[v];
                            } else {
                                // S1 <- (1 - s1) S1 + M S0,  S0 <- (1 - s2) S0 + F U_2 S0 + E U_y S1
                                Acc t, w;
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    t[v] = ff[v] * Q1[v];
                                    w[v] = fe[v] * Q0[v];
                                }
                                t = P::add(lm, P::right(Q0), t);
                                w = P::add(ln2, P::right(t), P::add(ln3, P::right(Q0), w));
                                Q0 = w;
                                Q1 = t;
                            }
                        }
                    } else {
                        const Acc rv = rows(KINDS - 1);
                        float s = SPLIT ? 0.f : vec[0];
#pragma unroll
                        for (int v = 0; v < 4; ++v) s += Q[0][0][v] * rv[v];
                        vec[0] = SPLIT ? vec[0] + s * scale[0].down : s;
                        if constexpr (CELL == LSTM) {
                            const Acc fi = fac(0), ff = fac(1), fg = fac(2), fo = fac(3), fd = fac(4);
                            Acc a;
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                a[v] = fi[v] * wa[0][v] + (ff[v] * wa[1][v] + (fg[v] * wa[2][v] + (fo[v] * wa[3][v] + fd[v] * dm[v])));
                            Q[0][0] = P::add(P::left(a), P::right(Q[0][0]), zero4());
                        } else {
                            const Acc f0 = fac(0), f1 = fac(1), fd = fac(2);
                            // factor of the second step: F in front of y, E in front of z
                            Acc a1, a2;
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int col = REV ? 4 * g + v : r;
                                a2[v] = (col < 8 ? f0[v] : f1[v]) * wa[0][v] + (fd[v] * dm[v] + im[v]);
                                a1[v] = f0[v] * wa[1][v] + (f1[v] * wa[2][v] + (fd[v] * im[v] + dm[v]));
                            }
                            const Acc t = P::add(P::left(REV ? a1 : a2), P::right(Q[0][0]), zero4());
                            Q[0][0] = P::add(P::left(REV ? a2 : a1), P::right(t), zero4());
                        }
                    }
                    if (base + c == edge) {
                        // the chunk's map: M[16 C + r][16 X + 4g + v] = Q[X][C][v]
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
                    }
                };
#pragma unroll 2
                for (int k = 0; k < c_hi - c_lo; ++k) {
                    const int c = REV ? c_lo + k : c_hi - 1 - k;
                    if (SPLIT && !wide) advance(std::bool_constant<SPLIT>{}, c);
                    else advance(std::false_type{}, c);
                }
                wave_lds_fence();
            }
            if (wide || !__ballot(again)) break;
            wide = true;
            unit_q = 1.f;
            q = kept;
            top = min(T, (first + q + 1) * Lc);
            request(0);
        }
    }
    __syncthreads();
    // the units of the group that nothing follows need no map
    const int pu = 16 / p.per_unit;
    const bool needed = REV ? unit >= pu : unit < (p.groups - 1) * pu;
    if (needed && wave <= NB) compose_unit<N, REV>(tot, p.sup + ((long long)b * p.units + unit) * MS, min(p.per_unit, chunks - first), wave, g, r);
}

// ------------------------------------------------------------------------------------------------------------------
// The walk: one wavefront per group, its sixteen chunks are the columns of every product.
// ------------------------------------------------------------------------------------------------------------------
template <int CELL, int UP, int DS, bool VEC>
__global__ __launch_bounds__(256, 2) void cell_walk_kernel(ChunkParams p) {
    constexpr int N = 2 * UP;
    __shared__ unsigned s_max[4];
    if (step_closed(p.gate, p.far != 0)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int T = p.T, d = p.d, Lc = p.Lc, n = p.cell_units, ld = 2 * n;
    const float dt = p.dt;
    const unsigned id = blockIdx.x * 4u + (unsigned)wave;
    const int b = (int)(id % (unsigned)p.B), grp = (int)(id / (unsigned)p.B);
    unsigned emax = 0u;   // largest |y_new - y| as raw bits (a NaN compares above everything)
    if (grp < p.groups) {
        const int chunks = (T + Lc - 1) / Lc, nq = min(16, chunks - 16 * grp);
        const long long first = (long long)b * T + (long long)16 * grp * Lc;
        const int j0 = (4 * g) % UP;
        const bool part0 = UP == 16 || g < 2, part1 = UP == 16 || g >= 2;   // parts this lane writes
        const float* __restrict__ yb = p.y + first * ld;
        const float* __restrict__ xb = p.x + first * d;
        float* __restrict__ ob = p.out + first * ld;
        const int a = r * Lc, end = T - 16 * grp * Lc;
        auto row = [&](int rel) { return (unsigned)min(max(rel, 0), end - 1); };

        // requested R - 1 steps ahead; slots named by t mod R
        constexpr int R = 4;
        Acc y0r[R], y1r[R];
        float xr[R][DS];
        auto ask_y = [&](int j, int t) {
            const unsigned o = row(a + t) * (unsigned)ld;
            y0r[j] = load_units<VEC>(yb + o, j0, n);
            y1r[j] = load_units<VEC>(yb + o + n, j0, n);
        };
        auto ask_x = [&](int j, int t) {
            const unsigned o = row(a + t) * (unsigned)d;
#pragma unroll
            for (int s = 0; s < DS; ++s) xr[j][s] = xb[o + min(DS * g + s, d - 1)];
        };
        {
            const bool start = a == 0 && grp == 0;
            const float* __restrict__ y0b = p.y0 ? p.y0 + (long long)b * ld : nullptr;
            const float* hp = start ? y0b : yb + (long long)(min(a, end) - 1) * ld;
            y0r[R - 1] = hp ? load_units<VEC>(hp, j0, n) : zero4();
            y1r[R - 1] = hp ? load_units<VEC>(hp + n, j0, n) : zero4();
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (j < R - 1) ask_y(j, j);
            ask_x(j, j);
        }
        Cell<CELL, UP, DS> cell;
        cell.load(p.theta, n, d, g, r);
        // correction of the state in front of the position, and the new state there
        Acc e0, e1, x0, x1;
        const bool far = p.far;
        {
            Acc e[N / 16];
            fold_carries<N, false>(p, b, grp, nq, g, r, e, far, [&](int row) {
                const int unit = row % UP;
                return p.y0 && unit < n ? p.y0[(long long)b * ld + (row / UP) * n + unit] : 0.f;
            });
            if constexpr (UP == 16) {
                e0 = e[0];
                e1 = e[N / 16 - 1];
            } else {
                Acc o;
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] = __shfl_xor(e[0][v], 32);
                e0 = g < 2 ? e[0] : o;
                e1 = g < 2 ? o : e[0];
            }
        }

        x0 = far ? e0 : y0r[R - 1] + e0;
        x1 = far ? e1 : y1r[R - 1] + e1;
        if (far) {
            e0 = x0 - y0r[R - 1];
            e1 = x1 - y1r[R - 1];
        }

        for (int t0 = 0; t0 < Lc; t0 += R) {   // Lc is a multiple of four
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int t = t0 + j, rel = a + t;
                const bool live = rel < end;
                const int jh = (j + R - 1) % R;
                Factors k[4];
                cell.eval(k, y0r[jh], y1r[jh], xr[j], dt, g);
                Acc n0, n1;
                if constexpr (CELL == LSTM) {
                    const Acc ti = cell.times(0, e0, zero4(), g), tf = cell.times(1, e0, zero4(), g);
                    const Acc tg = cell.times(2, e0, zero4(), g), to = cell.times(3, e0, zero4(), g);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float q = k[v].a * ti[v] + (k[v].b * tf[v] + k[v].c * tg[v]);
                        n1[v] = k[v].g1 + (k[v].f * x1[v] + q);
                        n0[v] = k[v].n0 + (k[v].d * to[v] + k[v].e * (k[v].f * e1[v] + q));
                    }
                } else {
                    const Acc t1 = cell.times(0, e0, zero4(), g), t2 = cell.times(1, e0, zero4(), g), tz = cell.times(2, e0, zero4(), g);
                    Acc dz;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float q = k[v].a * t1[v] + k[v].b * tz[v];
                        dz[v] = k[v].f * e1[v] + q;
                        n1[v] = k[v].g1 + (k[v].f * x1[v] + q);
                    }
                    const Acc ty = cell.times(3, dz, zero4(), g);
#pragma unroll
                    for (int v = 0; v < 4; ++v) n0[v] = k[v].g0 + (k[v].e * x0[v] + (k[v].c * t2[v] + k[v].d * ty[v]));
                }
                if (live) {
                    float* o = ob + (long long)rel * ld;
                    if (part0) store_units<VEC>(o, j0, n, n0);
                    if (part1) store_units<VEC>(o + n, j0, n, n1);
                }
                const unsigned mask = live ? 0x7fffffffu : 0u;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    x0[v] = n0[v];
                    x1[v] = n1[v];
                    e0[v] = n0[v] - y0r[j][v];
                    e1[v] = n1[v] - y1r[j][v];
                    emax = max(emax, max(__float_as_uint(e0[v]) & mask, __float_as_uint(e1[v]) & mask));
                }
                ask_y((j + R - 1) % R, t - 1 + R);
                ask_x(j, t + R);
            }
        }
    }
    if (p.err) {
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
// The dual walk with the vector-Jacobian product inside: lambda_i = g_i + J_{i+1}^T lambda_{i+1} needs the cotangents of the pre-activations
// at position i + 1, which are all that dL/dx, dL/dtheta and (at the first position) dL/dy0 are made of, so neither lambda nor the
// gates go through memory.  A step evaluates the cell behind the position it solves for; one more step takes the first position of
// the sequence.  The sums over positions have the columns on the contraction index: cotangents, state and input cross a slice of LDS.
// UP = 16: dU per block, and dW^T with the bias sums as a ninth row (the input rows are followed by a row of ones).  UP = 8: two
// blocks share a tile whose columns are (state | input).  A position's sixteen columns are added up by themselves and then to the sums: one
// accumulator over all 16 Lc positions had a relative error in dL/dtheta of 3.5e-7 (LSTM and LEM), against 2.7e-7 and 2.9e-7 of
// a kernel that sums 16 positions at a time; now 2.3e-7.  J^T lambda is added up without the cotangent, as in chunk_gru.hip.  dL/dx leaves before
// the sums, so that the pre-activations' cotangents end there (17 to 32 registers spilled otherwise).
// Measured, gradient with a kernel of its own for the vector-Jacobian product / now, us: LSTM u = 8, d = 4, 16 x 50,000 positions 455 / 245; LEM u = 16, d = 6, 32 x 17,984 positions 1,020 / 490.
// ------------------------------------------------------------------------------------------------------------------
template <int CELL, int UP, int DS, bool VEC>
__global__ __launch_bounds__(256, 2) void cell_dual_kernel(ChunkParams p) {
    constexpr int N = 2 * UP, KS = UP / 4, TILES = UP == 16 ? 4 : 2;
    constexpr int ST = 256 * TILES, XT = ST + (CELL == LEM ? 512 : 256);   // state tile (LEM: then the new z), UP = 16: input tile
    constexpr int USED = UP == 16 ? XT + 256 : XT, ROW = 4 * UP * 8 + 4 * UP * UP + 4 * UP;
    constexpr int SLICE = USED > ROW ? USED : ROW;   // (at the end the wavefront's row of dL/dtheta takes the place of its slice)
    __shared__ __align__(16) float sT[4][SLICE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int T = p.T, d = p.d, Lc = p.Lc, n = p.cell_units, ld = 2 * n;
    const float dt = p.dt;
    const unsigned id = blockIdx.x * 4u + (unsigned)wave;
    const int b = (int)(id % (unsigned)p.B), grp = (int)(id / (unsigned)p.B);
    float* __restrict__ S = sT[wave];
    // UP = 16: aU[q] = dU_q, aW[q] = (dW_q | db_q)^T.  UP = 8: aU[t] = blocks 2t, 2t + 1 by (state | input), aU[2] = block y by (z' | input);
    // aW[t] = this lane's bias sums of the blocks.
    Acc aU[4], aW[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) aU[q] = aW[q] = zero4();
    for (int q = lane; q < SLICE; q += 64) S[q] = 0.f;
    if (UP == 16 && lane < 16) S[XT + lane * 16 + 8] = 1.f;
    wave_lds_fence();
    if (grp < p.groups) {
        const int chunks = (T + Lc - 1) / Lc, nq = min(16, chunks - 16 * grp);
        const long long first = (long long)b * T + (long long)16 * grp * Lc;
        const int j0 = (4 * g) % UP;
        const float* __restrict__ yb = p.y + first * ld;
        const float* __restrict__ xb = p.x + first * d;
        const float* __restrict__ gb = p.g + first * ld;
        float* __restrict__ dxb = p.dx ? p.dx + first * d : nullptr;
        const int a = r * Lc, end = T - 16 * grp * Lc;
        auto row = [&](int rel) { return (unsigned)min(max(rel, 0), end - 1); };
        constexpr int R = 2;
        Acc y0r[R], y1r[R], g0r[R], g1r[R];
        float xr[R][DS];
        auto ask = [&](int j, int t) {
            const unsigned o = row(a + Lc - 1 - t) * (unsigned)ld, ox = row(a + Lc - t) * (unsigned)d;
            y0r[j] = load_units<VEC>(yb + o, j0, n);
            y1r[j] = load_units<VEC>(yb + o + n, j0, n);
            g0r[j] = load_units<VEC>(gb + o, j0, n);
            g1r[j] = load_units<VEC>(gb + o + n, j0, n);
#pragma unroll
            for (int s = 0; s < DS; ++s) xr[j][s] = xb[ox + min(DS * g + s, d - 1)];
        };
#pragma unroll
        for (int j = 0; j < R; ++j) ask(j, j);
        Cell<CELL, UP, DS> cell;
        cell.load(p.theta, n, d, g, r);
        float ut[4][KS], wt[4][KS];   // U_gate^T and W_gate^T as operand A
        {
            const float* __restrict__ U = p.theta + 4 * n * d;
            const int col = min(r % UP, n - 1), xc = min(r, d - 1);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const int k = Cell<CELL, UP, DS>::kappa(g, s), kc = min(k, n - 1);
                    const float v = U[(q * n + kc) * n + col], x = p.theta[(q * n + kc) * d + xc];
                    ut[q][s] = k < n && r % UP < n ? v : 0.f;
                    wt[q][s] = k < n && r < d ? x : 0.f;
                }
        }
        auto times_t = [&](const float (&m)[KS], const Acc& x, Acc acc) {
#pragma unroll
            for (int s = 0; s < KS; ++s) acc = mfma(m[s], Cell<CELL, UP, DS>::operand(x, g, s), acc);
            return acc;
        };
        Acc e0, e1;   // lambda at the position the step evaluates
        {
            Acc e[N / 16];
            fold_carries<N, true>(p, b, grp, nq, g, r, e, false, [](int) { return 0.f; });
            if constexpr (UP == 16) {
                e0 = e[0];
                e1 = e[N / 16 - 1];
            } else {
                Acc o;
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] = __shfl_xor(e[0][v], 32);
                e0 = g < 2 ? e[0] : o;
                e1 = g < 2 ? o : e[0];
            }
        }
        // one step at position `at` (relative) with state (s0 | s1) in front of it: (n0 | n1) = J^T lambda
        auto step = [&](const Acc& s0, const Acc& s1, const float (&x)[DS], int at, Acc& n0, Acc& n1) {
            Factors k[4];
            cell.eval(k, s0, s1, x, dt, g);
            Acc da[4], zn;
            if constexpr (CELL == LSTM) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float dc = e1[v] + k[v].e * e0[v];
                    da[0][v] = k[v].a * dc;
                    da[1][v] = k[v].b * dc;
                    da[2][v] = k[v].c * dc;
                    da[3][v] = k[v].d * e0[v];
                    n1[v] = k[v].f * dc;
                }
                n0 = times_t(ut[0], da[0], zero4());
                n0 = times_t(ut[1], da[1], n0);
                const Acc s2 = times_t(ut[2], da[2], zero4());
                n0 += times_t(ut[3], da[3], s2);
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    da[3][v] = k[v].d * e0[v];
                    da[1][v] = k[v].c * e0[v];
                    zn[v] = k[v].n1;
                }
                const Acc dz = e1 + times_t(ut[3], da[3], zero4());
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    da[0][v] = k[v].a * dz[v];
                    da[2][v] = k[v].b * dz[v];
                    n1[v] = k[v].f * dz[v];
                    n0[v] = k[v].e * e0[v];
                }
                n0 = times_t(ut[0], da[0], n0);
                const Acc s1t = times_t(ut[1], da[1], zero4());
                n0 += times_t(ut[2], da[2], s1t);
            }
            if (dxb) {
                Acc o0 = times_t(wt[0], da[0], zero4()), o1 = times_t(wt[1], da[1], zero4());
                o0 = times_t(wt[2], da[2], o0);
                o1 = times_t(wt[3], da[3], o1);
                if (g < 2 && at < end) {
                    float* o = dxb + (long long)at * d + 4 * g;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (4 * g + v < d) o[v] = o0[v] + o1[v];
                }
            }
            // ---- products over positions ----
            if constexpr (UP == 16) {
#pragma unroll
                for (int q = 0; q < 4; ++q) store4(S + q * 256 + r * 16 + 4 * g, da[q]);
                store4(S + ST + r * 16 + 4 * g, s0);
                if constexpr (CELL == LEM) store4(S + ST + 256 + r * 16 + 4 * g, zn);
#pragma unroll
                for (int s = 0; s < DS; ++s) S[XT + r * 16 + DS * g + s] = x[s];
            } else {
                const Acc t0 = g < 2 ? da[0] : da[1], t1 = g < 2 ? da[2] : da[3];
                store4(S + r * 16 + 4 * g, t0);
                store4(S + 256 + r * 16 + 4 * g, t1);
                if (g < 2) {
                    store4(S + ST + r * 16 + 4 * g, s0);
                    if constexpr (CELL == LEM) store4(S + ST + 256 + r * 16 + 4 * g, zn);
                }
#pragma unroll
                for (int s = 0; s < DS; ++s) S[ST + r * 16 + 8 + DS * g + s] = x[s];
                aW[0] += t0;
                aW[1] += t1;
            }
            wave_lds_fence();
            const float* q = S + g * 16 + r;   // row m of four: + 64 m
            float bs[4], bo[4];                // state, and UP = 16: input, UP = 8: the new z
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                bs[m] = q[64 * m + ST];
                bo[m] = UP == 16 ? q[64 * m + XT] : CELL == LEM ? q[64 * m + ST + 256] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < TILES; ++i) {
                Acc pU = zero4(), pW = zero4();
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const float t = q[64 * m + 256 * i];
                    pU = mfma(t, UP == 16 && CELL == LEM && i == 3 ? q[64 * m + ST + 256] : bs[m], pU);
                    if (UP == 16) pW = mfma(bo[m], t, pW);
                    else if (CELL == LEM && i == 1) pW = mfma(t, bo[m], pW);
                }
                __builtin_amdgcn_sched_barrier(0);   // (one block's products at a time: registers)
                aU[i] += pU;
                if (UP == 16) aW[i] += pW;
                else if (CELL == LEM && i == 1) aU[2] += pW;
            }
            wave_lds_fence();
        };
        // (a column that starts past the end has nothing to store: its positions are not below `end`)
        for (int t0 = 0; t0 < Lc; t0 += R) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int t = t0 + j, rel = a + Lc - 1 - t;
                const bool live = rel < end;
                Acc n0, n1;
                step(y0r[j], y1r[j], xr[j], rel + 1, n0, n1);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    e0[v] = live ? g0r[j][v] + n0[v] : 0.f;   // nothing follows the last position
                    e1[v] = live ? g1r[j][v] + n1[v] : 0.f;
                }
                ask(j, t + R);
            }
        }
        if (grp == 0) {   // the first position of the sequence
            const float* __restrict__ y0b = p.y0 ? p.y0 + (long long)b * ld : nullptr;
            const Acc s0 = y0b ? load_units<VEC>(y0b, j0, n) : zero4(), s1 = y0b ? load_units<VEC>(y0b + n, j0, n) : zero4();
            Acc n0, n1;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                e0[v] = r == 0 ? e0[v] : 0.f;
                e1[v] = r == 0 ? e1[v] : 0.f;
            }
            step(s0, s1, xr[0], r == 0 ? 0 : end, n0, n1);
            if (p.dy0 && r == 0) {
                float* o = p.dy0 + (long long)b * ld;
                if (UP == 16 || g < 2) store_units<false>(o, j0, n, n0);
                if (UP == 16 || g >= 2) store_units<false>(o + n, j0, n, n1);
            }
        }
    }

    // ---- the workgroup's row of dL/dtheta: W[4n,d] | U[4n,n] | b[4n] ----
    const int U0 = 4 * n * d, b0 = U0 + 4 * n * n, P = b0 + 4 * n;
    if constexpr (UP == 16) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = 4 * g + v;
                if (k < n && r < n) S[U0 + (q * n + k) * n + r] = aU[q][v];
                if (r < n) {   // row k of (dW | db)^T, column r
                    if (k < d && k < 8) S[(q * n + r) * d + k] = aW[q][v];
                    if (k == 8) S[b0 + q * n + r] = aW[q][v];
                }
            }
    } else {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const Acc sb = row_sums4(aW[t], r);
            const int q = 2 * t + (g >> 1);   // the block of this lane's rows
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = (4 * g + v) & 7;
                if (k >= n) continue;
                if (r < 8) {
                    if (r < n) S[U0 + (q * n + k) * n + r] = CELL == LEM && t == 1 && g >= 2 ? aU[2][v] : aU[t][v];
                } else if (r - 8 < d) {
                    S[(q * n + k) * d + r - 8] = aU[t][v];
                }
                if (r == 0) S[b0 + q * n + k] = sb[v];
            }
        }
    }
    __syncthreads();
    for (int q = tid; q < P; q += 256) p.partial[(long long)blockIdx.x * P + q] = (sT[0][q] + sT[1][q]) + (sT[2][q] + sT[3][q]);
}

template <int CELL, int UP, int DS, bool VEC>
hipError_t launch_v(const ChunkParams& p, hipStream_t s) {
    const dim3 units((unsigned)((long long)p.B * p.units)), groups((unsigned)chunk_rows(p));
    if (p.g) hipLaunchKernelGGL((cell_totals_kernel<CELL, UP, DS, VEC, true, false>), units, dim3(256), 0, s, p);
    else if (p.far) hipLaunchKernelGGL((cell_totals_kernel<CELL, UP, DS, VEC, false, true>), units, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((cell_totals_kernel<CELL, UP, DS, VEC, false, false>), units, dim3(256), 0, s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.g) hipLaunchKernelGGL((cell_dual_kernel<CELL, UP, DS, VEC>), groups, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((cell_walk_kernel<CELL, UP, DS, VEC>), groups, dim3(256), 0, s, p);
    return hipGetLastError();
}
template <int CELL, int UP, int DS>
hipError_t launch_d(const ChunkParams& p, hipStream_t s) {
    return p.cell_units % 4 == 0 ? launch_v<CELL, UP, DS, true>(p, s) : launch_v<CELL, UP, DS, false>(p, s);
}
template <int CELL>
hipError_t launch_cell(const ChunkParams& p, hipStream_t s) {
    if (p.cell_units <= 8) return p.d <= 4 ? launch_d<CELL, 8, 1>(p, s) : launch_d<CELL, 8, 2>(p, s);
    return p.d <= 4 ? launch_d<CELL, 16, 1>(p, s) : launch_d<CELL, 16, 2>(p, s);
}

}  // namespace

bool chunk_cells_supported(int dtype, int units, int d) { return dtype == 0 && units >= 1 && units <= 16 && d >= 1 && d <= 8; }

size_t chunk_cells_map_bytes(int units) { return chunk_map_bytes(units <= 8 ? 16 : 32); }

hipError_t launch_chunk_cells(bool lem, const ChunkParams& p, hipStream_t s) {
    if (!chunk_cells_supported(0, p.cell_units, p.d) || !chunk_params_valid(p)) return hipErrorInvalidValue;
    if (p.g ? !p.partial || !p.dtheta : !p.out) return hipErrorInvalidValue;
    const hipError_t e = lem ? launch_cell<LEM>(p, s) : launch_cell<LSTM>(p, s);
    if (e != hipSuccess || !p.g) return e;
    const long long n = p.cell_units;
    return launch_partial_reduce(0, p.partial, p.dtheta, 4 * n * p.d + 4 * n * n + 4 * n, (int)chunk_rows(p), s);
}

}  // namespace deer
