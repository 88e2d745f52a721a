// The GRU step and dual scan by chunks (chunk_gru.hip) at n = 64 in fp32.  A 64 x 64 running product and its factor are 128
// registers a lane for one wavefront, so four wavefronts share a position:
//   reduction: wavefront w keeps columns 16 w .. 16 w + 15 of the running product (16 registers) and assembles a quarter of
//     every factor (the rows of J whose gates it has evaluated) into LDS in operand order, double-buffered, one barrier a
//     position; all four read the whole factor (64 KB of LDS reads against 4 x 2,048 matrix-core cycles).
//   walk: wavefront w evaluates rows 16 w .. 16 w + 15 of all products; the column vectors cross LDS, one barrier a step.
// Bound: the reduction of a Newton step has its factors split in two fp16 numbers like that at n = 32 (chunk_gru.hip; wavefronts split the quarter that they
// assemble): 24 matrix instructions of 18 cycles a wavefront and position and about 110 vector instructions of 2.4, then the barrier and the LDS
// (one workgroup a compute unit at 5 x 9,973 positions: 2,000 cycles a position).  Far iterates and the dual scan, for the reason given
// there: 64 fp32 matrix instructions of 32 cycles.  Reduction at 5 x 9,973 positions, d = 7, with fp32 products / now: Newton step 303 / 185 us.
#include "chunk_common.h"
#include "split_f16.h"

namespace deer {

namespace {

constexpr int N = 64, NB = 4, MS = N * N + N;

// Gate operands of a wavefront (rows 16 w .. 16 w + 15)
template <int DS>
struct GateRows {
    Acc u[3][NB];
    float w[3][DS];
    Acc b[4];
};

template <int DS>
__device__ __forceinline__ void load_gate_rows(GateRows<DS>& o, const float* __restrict__ th, int d, int wave, int g, int r) {
    const float* __restrict__ U = th + 3 * N * d;
    const float* __restrict__ bias = U + 3 * N * N;
#pragma unroll
    for (int gate = 0; gate < 3; ++gate) {
        const int row = gate * N + 16 * wave + r;
#pragma unroll
        for (int K = 0; K < NB; ++K) o.u[gate][K] = load4(U + row * N + 16 * K + 4 * g);
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            const float v = th[row * d + min(DS * g + s, d - 1)];
            o.w[gate][s] = DS * g + s < d ? v : 0.f;
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) o.b[j] = load4(bias + j * N + 16 * wave + 4 * g);
}

// gates of this wavefront's rows at sixteen positions (columns); h: rows 16K + 4g + v of the state, hw: this wavefront's rows
template <int DS>
__device__ __forceinline__ void gates16(GruGates (&o)[4], const GateRows<DS>& k, const Acc (&h)[NB], const float (&x)[DS], Acc hw) {
    Acc ar = k.b[0], az = k.b[1], ac = k.b[2], aq = k.b[3];
#pragma unroll
    for (int K = 0; K < NB; ++K)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            ar = mfma(k.u[0][K][v], h[K][v], ar);
            az = mfma(k.u[1][K][v], h[K][v], az);
            aq = mfma(k.u[2][K][v], h[K][v], aq);
        }
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        ar = mfma(k.w[0][s], x[s], ar);
        az = mfma(k.w[1][s], x[s], az);
        ac = mfma(k.w[2][s], x[s], ac);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = gru_gates(ar[v], az[v], ac[v], aq[v], hw[v]);
}

template <int DS, bool REV, bool FAR>
__global__ __launch_bounds__(256, 2) void chunk_totals64_kernel(ChunkParams p) {
    // row factors of this wavefront's 16 rows; forward [kind][position][row], dual [position][row][kind]
    __shared__ __align__(16) float sF[4][4 * 16 * 16];
    __shared__ __align__(16) float sR[16 * N];            // forward: residual, dual: cotangent, [position][row]
    // factor in operand order, [block][lane]; split in two [column blocks / 2][row block][hi, lo][lane], in the same place
    __shared__ __align__(16) Acc sJ[2][NB * NB][64];
    __shared__ unsigned s_again[4];
    constexpr bool SPLIT = !FAR && !REV;
    if (step_closed(p.gate, FAR)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int b = (int)(blockIdx.x % (unsigned)p.B), unit = (int)(blockIdx.x / (unsigned)p.B);
    const int T = p.T, d = p.d, Lc = p.Lc, chunks = (T + Lc - 1) / Lc;
    const int first = unit * p.per_unit, nq = min(p.per_unit, chunks - first);   // chunks of this unit
    const float* __restrict__ yb = p.y + (long long)b * T * N;
    const float* __restrict__ xb = p.x + (long long)b * T * d;
    const float* __restrict__ y0b = p.y0 ? p.y0 + (long long)b * N : nullptr;
    const float* __restrict__ gb = REV ? p.g + (long long)b * T * N : nullptr;
    float* __restrict__ tot = p.tot + ((long long)b * chunks + first) * MS;
    float* __restrict__ sFw = sF[wave];

    const int lo = first * Lc, hi = min(T, (first + nq) * Lc);
    int top = hi;    // forward: one past the first position that is still to be reduced
    Acc h[NB], ow;   // state in front of each position, this wavefront's rows of the residual's other term
    float x[DS];
    auto request = [&](int blk) {
        int pos = (REV ? lo + 16 * blk : top - 16 * (blk + 1)) + r;
        pos = min(max(pos, lo), hi - 1);
        const float* hp = REV ? yb + (long long)pos * N : (pos > 0 ? yb + (long long)(pos - 1) * N : y0b);
#pragma unroll
        for (int K = 0; K < NB; ++K) h[K] = hp ? load4(hp + 16 * K + 4 * g) : zero4();
        ow = load4((REV ? gb : yb) + (long long)pos * N + 16 * wave + 4 * g);
        load_x<DS>(x, xb + (long long)(REV ? min(pos + 1, T - 1) : pos) * d, d, g);
    };
    request(0);
    GateRows<DS> gr;
    load_gate_rows<DS>(gr, p.theta, d, wave, g, r);
    // weights of the quarter of the factor this wavefront assembles.  forward (J^T): J[16 w + 4g + v][16 X + r], block (X, w);
    // dual (J): J[16 w + r][16 X + 4g + v], block (w, X) -- the gate operands themselves
    Acc ua[REV ? 1 : 3][NB];
    if constexpr (!REV) {
        const float* __restrict__ U = p.theta + 3 * N * d;
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int X = 0; X < NB; ++X)
#pragma unroll
                for (int v = 0; v < 4; ++v) ua[gate][X][v] = U[(gate * N + 16 * wave + 4 * g + v) * N + 16 * X + r];
    }
    float dsel[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) dsel[v] = (4 * g + v == r) ? 1.f : 0.f;

    Acc Q[NB];   // columns 16 w + r of the running product, rows 16 X + 4g + v
    float vec = 0.f;
    bool wide = !SPLIT, again = false;   // products of fp32 factors; a product of the other kind was not finite
    ColumnScale scale;
    auto reset = [&]() {
        vec = 0.f;
        scale.reset(!wide);
        const float unit_q = wide ? 1.f : (float)(1 << ColumnScale::kStart);
#pragma unroll
        for (int X = 0; X < NB; ++X)
#pragma unroll
            for (int v = 0; v < 4; ++v) Q[X][v] = X == wave ? dsel[v] * unit_q : 0.f;
    };
    auto parts = [&](int buf, int K2, int X, int part) { return reinterpret_cast<Half8*>(&sJ[buf][(K2 * NB + X) * 2 + part][0]); };

    auto assemble = [&](int buf, int c) {
        if constexpr (!REV) {
            const float* o = sFw + c * 16 + 4 * g;
            const Acc pz = load4(o), sr = load4(o + 256), st = load4(o + 512), z = load4(o + 768);
#pragma unroll
            for (int X = 0; X < NB; ++X) {
                Acc a;
                const float diag = X == wave ? 1.f : 0.f;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    a[v] = pz[v] * ua[1][X][v] + (sr[v] * ua[2][X][v] + (st[v] * ua[0][X][v] + diag * dsel[v] * z[v]));
                if (SPLIT && !wide) {
                    const Split4 s = split4(a);
                    reinterpret_cast<Half4*>(parts(buf, wave >> 1, X, 0) + lane)[wave & 1] = s.hi;
                    reinterpret_cast<Half4*>(parts(buf, wave >> 1, X, 1) + lane)[wave & 1] = s.lo;
                } else {
                    sJ[buf][X * NB + wave][lane] = a;
                }
            }
        } else {
            const Acc ff = load4(sFw + (c * 16 + r) * 4);
#pragma unroll
            for (int X = 0; X < NB; ++X) {
                Acc a;
                const float diag = X == wave ? 1.f : 0.f;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    a[v] = ff[0] * gr.u[1][X][v] + (ff[1] * gr.u[2][X][v] + (ff[2] * gr.u[0][X][v] + diag * dsel[v] * ff[3]));
                sJ[buf][wave * NB + X][lane] = a;
            }
        }
    };

    int q = REV ? 0 : nq - 1, kept = q;   // chunk being reduced; the same when all was last seen to be finite
    for (;;) {
        reset();
        int edge = REV ? min(T, (first + q + 1) * Lc) - 1 : (first + q) * Lc;   // the chunk's last position in traversal order
        const int blocks = (top - lo + 15) / 16;
        for (int blk = 0; blk < blocks; ++blk) {
            const int base = REV ? lo + 16 * blk : top - 16 * (blk + 1);
            if (SPLIT && !wide) {
                float m = 0.f, sum = 0.f;   // (sum: not a finite number if one of its terms is none)
#pragma unroll
                for (int X = 0; X < NB; ++X)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        m = fmaxf(m, fabsf(Q[X][v]));
                        sum += 0.f * Q[X][v];
                    }
                const float f = scale.next(max_groups(m));
#pragma unroll
                for (int X = 0; X < NB; ++X) Q[X] *= f;
                again |= __ballot(again || sum != 0.f) != 0ull;
                if (lane == 0) s_again[wave] = again;
            }
            {
                GruGates k[4];
                gates16<DS>(k, gr, h, x, wave == 0 ? h[0] : wave == 1 ? h[1] : wave == 2 ? h[2] : h[3]);
                Acc rv = ow;
                if constexpr (!REV) {
                    Acc fpz, fsr, fst, fz;
                    if constexpr (FAR) {
                        Acc hr = zero4(), hz = zero4(), hc = zero4();
#pragma unroll
                        for (int K = 0; K < NB; ++K)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                hr = mfma(gr.u[0][K][v], h[K][v], hr);
                                hz = mfma(gr.u[1][K][v], h[K][v], hz);
                                hc = mfma(gr.u[2][K][v], h[K][v], hc);
                            }
#pragma unroll
                        for (int v = 0; v < 4; ++v) rv[v] = gru_rhs(k[v], hr[v], hz[v], hc[v]);
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v) rv[v] = k[v].f - ow[v];
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) { fpz[v] = k[v].pz; fsr[v] = k[v].sr; fst[v] = k[v].st; fz[v] = k[v].z; }
                    float* o = sFw + r * 16 + 4 * g;
                    store4(o, fpz); store4(o + 256, fsr); store4(o + 512, fst); store4(o + 768, fz);
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) store4(sFw + (r * 16 + 4 * g + v) * 4, Acc{k[v].pz, k[v].sr, k[v].st, k[v].z});
                }
                store4(sR + r * N + 16 * wave + 4 * g, rv);
            }
            wave_lds_fence();
            const int c_lo = REV ? 0 : max(lo - base, 0), c_hi = REV ? min(hi - base, 16) : 16, cnt = c_hi - c_lo;
            assemble(0, REV ? c_lo : c_hi - 1);
            __syncthreads();
            if (SPLIT && !wide) {
                if ((s_again[0] | s_again[1] | s_again[2] | s_again[3]) != 0u) {   // (the same for the four wavefronts)
                    again = true;
                    break;
                }
                kept = q;
            }
            if (blk + 1 < blocks) request(blk + 1);
#pragma unroll 1
            for (int k = 0; k < cnt; ++k) {
                const int c = REV ? c_lo + k : c_hi - 1 - k;
                if (k + 1 < cnt) assemble((k + 1) & 1, REV ? c + 1 : c - 1);
                float sum_r = SPLIT ? 0.f : vec;
#pragma unroll
                for (int K = 0; K < NB; ++K) {
                    const Acc rv = load4(sR + c * N + 16 * K + 4 * g);
#pragma unroll
                    for (int v = 0; v < 4; ++v) sum_r += Q[K][v] * rv[v];
                }
                vec = SPLIT ? vec + sum_r * scale.down : sum_r;
                Acc Qn[NB];
#pragma unroll
                for (int X = 0; X < NB; ++X) Qn[X] = zero4();
                if (SPLIT && !wide) {
                    const Split8 B[2] = {split8(Q[0], Q[1]), split8(Q[2], Q[3])};
#pragma unroll
                    for (int K2 = 0; K2 < 2; ++K2) {
                        Half8 hi[NB];
#pragma unroll
                        for (int X = 0; X < NB; ++X) {
                            hi[X] = parts(k & 1, K2, X, 0)[lane];
                            Qn[X] = mfma16(parts(k & 1, K2, X, 1)[lane], B[K2].hi, Qn[X]);
                        }
#pragma unroll
                        for (int X = 0; X < NB; ++X) Qn[X] = mfma16(hi[X], B[K2].lo, Qn[X]);
#pragma unroll
                        for (int X = 0; X < NB; ++X) Qn[X] = mfma16(hi[X], B[K2].hi, Qn[X]);
                    }
                } else {
#pragma unroll
                    for (int K = 0; K < NB; ++K) {
                        Acc a[NB];
#pragma unroll
                        for (int X = 0; X < NB; ++X) a[X] = sJ[k & 1][X * NB + K][lane];
#pragma unroll
                        for (int v = 0; v < 4; ++v)
#pragma unroll
                            for (int X = 0; X < NB; ++X) Qn[X] = mfma(a[X][v], Q[K][v], Qn[X]);
                    }
                }
#pragma unroll
                for (int X = 0; X < NB; ++X) Q[X] = Qn[X];
                if (base + c == edge) {
                    // the chunk's map: M[16 w + r][16 X + 4g + v] = Q[X][v]
                    float* o = tot + (long long)q * MS;
                    float sum = 0.f;   // (not a finite number if one of its terms is none)
#pragma unroll
                    for (int X = 0; X < NB; ++X) {
                        if (SPLIT)
#pragma unroll
                            for (int v = 0; v < 4; ++v) sum += 0.f * Q[X][v];
                        Acc m = Q[X];
                        if (SPLIT)
#pragma unroll
                            for (int v = 0; v < 4; ++v) m[v] = __builtin_amdgcn_ldexpf(m[v], -scale.e);
                        store4(o + (16 * wave + r) * N + 16 * X + 4 * g, m);
                    }
                    again |= sum != 0.f;
                    const float s = sum_groups(vec);
                    if (g == 0) o[N * N + 16 * wave + r] = s;
                    reset();
                    q += REV ? 1 : -1;
                    edge = REV ? min(T, (first + q + 1) * Lc) - 1 : (first + q) * Lc;
                }
                __syncthreads();   // the next factor is complete, this one and (at the end of a block) the residuals are free
            }
        }
        if (wide) break;
        const bool bad = __ballot(again) != 0ull;
        if (lane == 0) s_again[wave] = bad;
        __syncthreads();
        if ((s_again[0] | s_again[1] | s_again[2] | s_again[3]) == 0u) break;   // (the same for the four wavefronts)
        wide = true;
        q = kept;
        top = min(T, (first + q + 1) * Lc);
        request(0);
    }

    // ---- the unit's map; none where no group follows ----
    const int pu = 16 / p.per_unit;
    if (REV ? unit < pu : unit >= (p.groups - 1) * pu) return;
    float* sx = sR;   // running vector, two copies
    Acc A[2][NB], Aw[NB];   // blocks of the next map: all rows of column block 0, this wavefront's rows
    float mv;
    auto map_at = [&](int i) { return tot + (long long)(REV ? nq - 1 - min(i, nq - 1) : min(i, nq - 1)) * MS; };
    auto ask = [&](const float* m) {
#pragma unroll
        for (int I = 0; I < NB; ++I) A[0][I] = load4(m + (16 * I + r) * N + 4 * g);
#pragma unroll
        for (int K = 0; K < NB; ++K) Aw[K] = load4(m + (16 * wave + r) * N + 16 * K + 4 * g);
        mv = m[N * N + 16 * wave + r];
    };
    ask(map_at(1));
    {
        const float* m = map_at(0);
#pragma unroll
        for (int K = 0; K < NB; ++K)
#pragma unroll
            for (int v = 0; v < 4; ++v) Q[K][v] = m[(16 * K + 4 * g + v) * N + 16 * wave + r];
        if (tid < N) sx[tid] = m[N * N + tid];
    }
    __syncthreads();
    for (int i = 1; i < nq; ++i) {
        const float* m = map_at(i);
        float s = 0.f;
#pragma unroll
        for (int K = 0; K < NB; ++K) {
            const Acc xk = load4(sx + ((i + 1) & 1) * N + 16 * K + 4 * g);
#pragma unroll
            for (int v = 0; v < 4; ++v) s += Aw[K][v] * xk[v];
        }
        s = sum_groups(s) + mv;
        if (g == 0) sx[(i & 1) * N + 16 * wave + r] = s;
        Acc Y[NB];
#pragma unroll
        for (int I = 0; I < NB; ++I) Y[I] = zero4();
#pragma unroll
        for (int K = 0; K < NB; ++K) {
            if (K + 1 < NB)
#pragma unroll
                for (int I = 0; I < NB; ++I) A[(K + 1) & 1][I] = load4(m + (16 * I + r) * N + 16 * (K + 1) + 4 * g);
            else
                ask(map_at(i + 1));
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int I = 0; I < NB; ++I) Y[I] = mfma(A[K & 1][I][v], Q[K][v], Y[I]);
        }
#pragma unroll
        for (int I = 0; I < NB; ++I) Q[I] = Y[I];
        __syncthreads();
    }
    float* o = p.sup + ((long long)b * p.units + unit) * MS;
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[(16 * I + 4 * g + v) * N + 16 * wave + r] = Q[I][v];
    if (tid < N) o[N * N + tid] = sx[((nq - 1) & 1) * N + tid];
}

// Step t of a chunk needs all rows of the state and of the correction (dual: of the state and of the three weighted
// cotangents) from the four wavefronts.
// SPLIT (not from far iterates): the products with the state and the correction have their factors split in two fp16 numbers, as in the walk at n = 32
// (chunk_gru.hip).  The wavefronts split their rows and hand the parts round; a column's scale needs the largest entry of all four, which takes
// a second barrier a step.  5 x 9,973 positions, d = 7: 142 us with fp32 products (102 instructions of 32 cycles a step and wavefront), now 120
// (6 of those and 42 of 18); 2-norm error of the trajectory against 64 bits 1.55e-7, now 1.48e-7 (n = 64).
template <int DS, bool REV, bool SPLIT>
__global__ __launch_bounds__(256, 2) void chunk_walk64_kernel(ChunkParams p) {
    constexpr int KINDS = REV ? 4 : 2;
    static_assert(!(SPLIT && REV), "");
    __shared__ float sM[2][4][16];   // largest entry of a column among a wavefront's rows: state, correction
    __shared__ __align__(16) Acc sX[2][KINDS][NB][64];   // [step parity][state, then correction or weighted cotangents][wavefront][lane]
    __shared__ __align__(16) float sx[2][N];
    __shared__ unsigned s_max[4];
    if (step_closed(p.gate, p.far != 0)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int b = (int)(blockIdx.x % (unsigned)p.B), grp = (int)(blockIdx.x / (unsigned)p.B);
    const int T = p.T, d = p.d, Lc = p.Lc, chunks = (T + Lc - 1) / Lc, nq = min(16, chunks - 16 * grp);
    // addresses relative to the group's first position, this wavefront's rows
    const long long first = (long long)b * T + (long long)16 * grp * Lc;
    const float* __restrict__ yb = p.y + first * N + 16 * wave + 4 * g;
    const float* __restrict__ xb = p.x + first * d;
    const float* __restrict__ gb = REV ? p.g + first * N + 16 * wave + 4 * g : nullptr;
    float* __restrict__ ob = p.out + first * N + 16 * wave + 4 * g;
    const int a = r * Lc, end = T - 16 * grp * Lc;
    auto row = [&](int rel) { return (unsigned)min(max(rel, 0), end - 1); };

    // requested R - 1 (dual: R) steps ahead; slots named by t mod R
    constexpr int R = 4;
    Acc yr[R], go[REV ? R : 1];
    float xr[R][DS];
    auto ask_y = [&](int j, int t) {
        const unsigned o = row(REV ? a + Lc - 1 - t : a + t) * N;
        yr[j] = load4(yb + o);
        if constexpr (REV) go[j] = load4(gb + o);
    };
    auto ask_x = [&](int j, int t) {
        const unsigned o = row(REV ? a + Lc - t : a + t) * (unsigned)d;
#pragma unroll
        for (int s = 0; s < DS; ++s) xr[j][s] = xb[o + min(DS * g + s, d - 1)];
    };
    if constexpr (!REV) {
        const bool start = a == 0 && grp == 0;
        const float* __restrict__ y0b = p.y0 ? p.y0 + (long long)b * N + 16 * wave + 4 * g : nullptr;
        const float* hp = start ? y0b : yb + (long long)(min(a, end) - 1) * N;
        yr[R - 1] = hp ? load4(hp) : zero4();
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (REV || j < R - 1) ask_y(j, j);
        ask_x(j, j);
    }
    GateRows<DS> gr;
    load_gate_rows<DS>(gr, p.theta, d, wave, g, r);
    Split8Weights us[SPLIT ? 3 : 1][2];   // parts of U_gate 2^eu with entries below 2^8
    int eu = 0;
    if constexpr (SPLIT) {
        float m = 0.f;
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int K = 0; K < NB; ++K)
#pragma unroll
                for (int v = 0; v < 4; ++v) m = fmaxf(m, fabsf(gr.u[gate][K][v]));
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
        eu = min(8 - exponent(max_groups(m)), 100);
        const float up = __builtin_amdgcn_ldexpf(1.f, eu);
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int q = 0; q < 2; ++q) us[gate][q] = split8_weights(gr.u[gate][2 * q] * up, gr.u[gate][2 * q + 1] * up);
    }
    Acc ut[REV ? 3 : 1][NB];   // dual: rows 16 w + r of U_gate^T
    if constexpr (REV) {
        const float* __restrict__ U = p.theta + 3 * N * d;
#pragma unroll
        for (int gate = 0; gate < 3; ++gate)
#pragma unroll
            for (int K = 0; K < NB; ++K)
#pragma unroll
                for (int v = 0; v < 4; ++v) ut[gate][K][v] = U[(gate * N + 16 * K + 4 * g + v) * N + 16 * wave + r];
    }

    // ---- carries: x <- M x + v over the units in front, then over the group's own chunks; a row of M per lane, a quarter
    // of the rows per wavefront, x in LDS ----
    Acc e = zero4();
    const bool far = !REV && p.far;
    {
        constexpr int PD = REV ? 2 : 4;
        const float y0v = far && p.y0 ? p.y0[(long long)b * N + lane] : 0.f;
        const bool zero = __ballot(y0v != 0.f) == 0;   // (the same for the four wavefronts)
        const int pu = 16 / p.per_unit;   // units of a group
        const float* __restrict__ own = p.tot + ((long long)b * chunks + 16 * grp) * MS;
        // the maps in front of the group: those of the units, and again those of the chunks if that overflowed (see fold_carries)
        const float* __restrict__ front = p.sup + (long long)b * p.units * MS;
        int maps = p.units, before = REV ? max(p.units - (grp + 1) * pu, 0) : grp * pu, steps = before + nq - 1;
        Acc A[PD][NB];
        float V[PD];
        auto request = [&](int j, int i) {
            i = min(i, steps - 1);
            const int k = i - before;
            const float* m = i < before ? front + (long long)(REV ? maps - 1 - i : i) * MS : own + (long long)(REV ? nq - 1 - k : k) * MS;
#pragma unroll
            for (int K = 0; K < NB; ++K) A[j][K] = load4(m + (16 * wave + r) * N + 16 * K + 4 * g);
            V[j] = m[N * N + 16 * wave + r];
        };
        for (int pass = 0;; ++pass) {
            if (steps > 0) {
#pragma unroll
                for (int j = 0; j < PD; ++j) request(j, j);
            }
            if (tid < N) sx[0][tid] = y0v;
            __syncthreads();
            for (int i0 = 0; i0 <= steps; i0 += PD) {
#pragma unroll
                for (int j = 0; j < PD; ++j) {
                    const int i = i0 + j;
                    if (i <= steps) {
                        const int k = i - before, qs = REV ? nq - 1 - k : k;
                        const Acc mine = load4(&sx[i & 1][16 * wave + 4 * g]);
                        e = (k >= 0 && r == qs) ? mine : e;
                        if (i < steps) {
                            float s = 0.f;
                            if (i > 0 || !zero) {   // in front of the sequence x is zero (unless y0 is not) and M is not looked at (it may have overflowed)
#pragma unroll
                                for (int K = 0; K < NB; ++K) {
                                    const Acc xk = load4(&sx[i & 1][16 * K + 4 * g]);
#pragma unroll
                                    for (int v = 0; v < 4; ++v) s += A[j][K][v] * xk[v];
                                }
                                s = sum_groups(s);
                            }
                            if (g == 0) sx[(i + 1) & 1][16 * wave + r] = s + V[j];
                            __syncthreads();
                        }
                    }
                    if (steps > 0) request(j, i + PD);
                }
            }
            if (pass > 0 || before == 0) break;   // (the same for the four wavefronts)
            float sum = 0.f;   // (not a finite number if one of its terms is none)
#pragma unroll
            for (int v = 0; v < 4; ++v) sum += 0.f * e[v];
            const unsigned long long bad = __ballot(sum != 0.f);
            if (lane == 0) s_max[wave] = bad ? 1u : 0u;
            __syncthreads();
            const bool again = (s_max[0] | s_max[1] | s_max[2] | s_max[3]) != 0u;
            __syncthreads();
            if (!again) break;
            maps = chunks;
            front = p.tot + (long long)b * chunks * MS;
            before = REV ? max(chunks - 16 * (grp + 1), 0) : 16 * grp;
            steps = before + nq - 1;
            e = zero4();
        }
    }

    Acc xv = zero4();   // forward: the new state in front of the position
    if constexpr (!REV) {
        xv = far ? e : yr[R - 1] + e;
        if (far) e = xv - yr[R - 1];
    }
    unsigned emax = 0u;   // largest |y_new - y| as raw bits (a NaN compares above everything)
    float down_h = 1.f, down_e = 1.f;
    // this wavefront's rows of the state and of the correction to all four (split: [hi, lo][column blocks / 2][lane], two wavefronts to a block of 16 bytes)
    auto publish = [&](int buf, const Acc& h, const Acc& c) {
        if constexpr (SPLIT) {
            float mh = 0.f, mc = 0.f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                mh = fmaxf(mh, fabsf(h[v]));
                mc = fmaxf(mc, fabsf(c[v]));
            }
            mh = max_groups(mh);
            mc = max_groups(mc);
            if (g == 0) {
                sM[0][wave][r] = mh;
                sM[1][wave][r] = mc;
            }
            __syncthreads();
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                mh = fmaxf(mh, sM[0][w][r]);
                mc = fmaxf(mc, sM[1][w][r]);
            }
            const int kh = min(13 - exponent(mh), 100), kc = min(13 - exponent(mc), 100);
            const Split4 hs = split4(h * __builtin_amdgcn_ldexpf(1.f, kh)), cs = split4(c * __builtin_amdgcn_ldexpf(1.f, kc));
            auto put = [&](int kind, int part, Half4 x) { reinterpret_cast<Half4*>(&sX[buf][kind][2 * part + (wave >> 1)][lane])[wave & 1] = x; };
            put(0, 0, hs.hi);
            put(0, 1, hs.lo);
            put(KINDS - 1, 0, cs.hi);
            put(KINDS - 1, 1, cs.lo);
            down_h = __builtin_amdgcn_ldexpf(1.f, -kh - eu);
            down_e = __builtin_amdgcn_ldexpf(1.f, -kc - eu);
        } else {
            sX[buf][0][wave][lane] = h;
            if constexpr (!REV) sX[buf][1][wave][lane] = c;
        }
        __syncthreads();
    };
    publish(0, yr[REV ? 0 : R - 1], e);
    for (int t0 = 0; t0 < Lc; t0 += R) {   // Lc is a multiple of four
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int t = t0 + j, rel = REV ? a + Lc - 1 - t : a + t;
            const bool live = rel < end;
            const int cur = j & 1, nxt = cur ^ 1;
            GruGates k[4];
            const Acc hw = yr[REV ? j : (j + R - 1) % R];
            Half8 eh[2], el[2];
            if constexpr (SPLIT) {
                Half8 hh[2], hl[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    hh[q] = __builtin_bit_cast(Half8, sX[cur][0][q][lane]);
                    hl[q] = __builtin_bit_cast(Half8, sX[cur][0][2 + q][lane]);
                    eh[q] = __builtin_bit_cast(Half8, sX[cur][KINDS - 1][q][lane]);
                    el[q] = __builtin_bit_cast(Half8, sX[cur][KINDS - 1][2 + q][lane]);
                }
                Acc a[4] = {gr.b[0], gr.b[1], gr.b[3], gr.b[2]};   // r, z, the candidate's hidden part, its input part
#pragma unroll
                for (int gate = 0; gate < 3; ++gate) {
                    Acc t = zero4();
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const Half8 small = split_small(hh[q]);
                        t = mfma16(us[gate][q].rest, small, t);
                        t = mfma16(us[gate][q].lo, small, t);
                        t = mfma16(us[gate][q].hi, hl[q], t);
                    }
#pragma unroll
                    for (int q = 0; q < 2; ++q) t = mfma16(us[gate][q].hi, hh[q], t);
                    a[gate] += t * down_h;
                }
#pragma unroll
                for (int s = 0; s < DS; ++s) {
                    a[0] = mfma(gr.w[0][s], xr[j][s], a[0]);
                    a[1] = mfma(gr.w[1][s], xr[j][s], a[1]);
                    a[3] = mfma(gr.w[2][s], xr[j][s], a[3]);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) k[v] = gru_gates(a[0][v], a[1][v], a[3][v], a[2][v], hw[v]);
            } else {
                Acc h[NB];
#pragma unroll
                for (int K = 0; K < NB; ++K) h[K] = sX[cur][0][K][lane];
                gates16<DS>(k, gr, h, xr[j], hw);
            }
            Acc y;
            if constexpr (!REV) {
                Acc er = zero4(), ez = zero4(), ec = zero4();
                if constexpr (SPLIT) {
                    auto correction = [&](int gate) {
                        Acc t = zero4();
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            t = mfma16(us[gate][q].lo, split_small(eh[q]), t);
                            t = mfma16(us[gate][q].hi, el[q], t);
                        }
#pragma unroll
                        for (int q = 0; q < 2; ++q) t = mfma16(us[gate][q].hi, eh[q], t);
                        return t * down_e;
                    };
                    er = correction(0);
                    ez = correction(1);
                    ec = correction(2);
                } else
#pragma unroll
                for (int K = 0; K < NB; ++K) {
                    const Acc ek = sX[cur][1][K][lane];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        er = mfma(gr.u[0][K][v], ek[v], er);
                        ez = mfma(gr.u[1][K][v], ek[v], ez);
                        ec = mfma(gr.u[2][K][v], ek[v], ec);
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) y[v] = k[v].c + (k[v].z * (xv[v] - k[v].c) + (k[v].pz * ez[v] + (k[v].sr * ec[v] + k[v].st * er[v])));
                const unsigned mask = live ? 0x7fffffffu : 0u;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    xv[v] = y[v];
                    e[v] = y[v] - yr[j][v];
                    emax = max(emax, __float_as_uint(e[v]) & mask);
                }
                publish(nxt, yr[j], e);
            } else {
                // lambda_pos = g_pos + J_{pos+1}^T lambda_{pos+1}
                Acc lz, lc, lr;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    lz[v] = k[v].pz * e[v];
                    lc[v] = k[v].sr * e[v];
                    lr[v] = k[v].st * e[v];
                    y[v] = k[v].z * e[v];
                }
                sX[nxt][0][wave][lane] = yr[(j + 1) % R];
                sX[cur][1][wave][lane] = lz;
                sX[cur][2][wave][lane] = lc;
                sX[cur][3][wave][lane] = lr;
                __syncthreads();
                Acc s[2][3];   // (by halves of the contraction: every instruction rounds at the size of its partial sum)
#pragma unroll
                for (int i = 0; i < 6; ++i) s[i / 3][i % 3] = zero4();
#pragma unroll
                for (int K = 0; K < NB; ++K) {
                    const Acc kz = sX[cur][1][K][lane], kc = sX[cur][2][K][lane], kr = sX[cur][3][K][lane];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        s[K >> 1][0] = mfma(ut[REV ? 1 : 0][K][v], kz[v], s[K >> 1][0]);
                        s[K >> 1][1] = mfma(ut[REV ? 2 : 0][K][v], kc[v], s[K >> 1][1]);
                        s[K >> 1][2] = mfma(ut[0][K][v], kr[v], s[K >> 1][2]);
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    y[v] = go[REV ? j : 0][v] + (y[v] + ((s[0][0][v] + s[1][0][v]) + ((s[0][1][v] + s[1][1][v]) + (s[0][2][v] + s[1][2][v]))));
                    e[v] = live ? y[v] : 0.f;   // nothing follows the last time
                }
            }
            if (live) store4(ob + (unsigned)(rel * N), y);
            if constexpr (!REV) ask_y((j + R - 1) % R, t - 1 + R);
            else ask_y(j, t + R);
            ask_x(j, t + R);
        }
    }
    if (!REV && p.err) {
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

template <int DS, bool REV>
hipError_t launch_ds(const ChunkParams& p, hipStream_t s) {
    const dim3 units((unsigned)((long long)p.B * p.units));
    if (!REV && p.far) hipLaunchKernelGGL((chunk_totals64_kernel<DS, REV, !REV>), units, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((chunk_totals64_kernel<DS, REV, false>), units, dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 groups((unsigned)((long long)p.B * p.groups));
    if (!REV && !p.far) hipLaunchKernelGGL((chunk_walk64_kernel<DS, REV, !REV>), groups, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((chunk_walk64_kernel<DS, REV, false>), groups, dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_chunk_gru64(const ChunkParams& p, hipStream_t s) {
    const bool rev = p.g != nullptr;
    if (p.d <= 4) return rev ? launch_ds<1, true>(p, s) : launch_ds<1, false>(p, s);
    if (p.d <= 8) return rev ? launch_ds<2, true>(p, s) : launch_ds<2, false>(p, s);
    return rev ? launch_ds<4, true>(p, s) : launch_ds<4, false>(p, s);
}

}  // namespace deer
