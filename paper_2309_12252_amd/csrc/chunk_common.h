// Pieces of the kernels that work by chunks (chunk_gru.hip, chunk_gru64.hip, chunk_cells.hip): matrix-core layout, sums over lanes,
// and the two operations on the maps of chunks and groups.
#pragma once
#include "deer_common.h"

namespace deer {
namespace {

using Acc = float __attribute__((ext_vector_type(4)));

__device__ __forceinline__ Acc mfma(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ Acc zero4() { return Acc{0.f, 0.f, 0.f, 0.f}; }

__device__ __forceinline__ Acc load4(const float* __restrict__ p) { return *reinterpret_cast<const Acc*>(p); }

__device__ __forceinline__ void store4(float* p, Acc v) { *reinterpret_cast<Acc*>(p) = v; }

// sum over the four lane groups (lanes r, r + 16, r + 32, r + 48), in every lane
__device__ __forceinline__ float sum_groups(float x) {
    unsigned u = __float_as_uint(x);
    const auto q = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float s = __uint_as_float(q[0]) + __uint_as_float(q[1]);
    u = __float_as_uint(s);
    const auto w = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(w[0]) + __uint_as_float(w[1]);
}

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}

// Four sums over the 16 lanes of a row, all four in every lane.  Lanes trade the values they do not keep (with the neighbour,
// then with the other pair of the quad), two rotations add the quads, the quad then hands its four totals round.
__device__ __forceinline__ Acc row_sums4(Acc q, int r) {
    const bool odd = r & 1, upper = r & 2;
    const float u0 = (odd ? q[1] : q[0]) + dpp<0xB1>(odd ? q[0] : q[1]);   // quad_perm 1,0,3,2
    const float u1 = (odd ? q[3] : q[2]) + dpp<0xB1>(odd ? q[2] : q[3]);
    float w = (upper ? u1 : u0) + dpp<0x4E>(upper ? u0 : u1);              // quad_perm 2,3,0,1
    w += dpp<0x124>(w);                                                    // row_ror 4
    w += dpp<0x128>(w);                                                    // row_ror 8
    return Acc{dpp<0x00>(w), dpp<0x55>(w), dpp<0xAA>(w), dpp<0xFF>(w)};
}

// the LDS slice of a wavefront is written and read by its own lanes only: LDS operations of a wavefront complete in order,
// the fence keeps the compiler from moving them
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct GruGates {
    float f, pz, sr, st, z, sc, c;
};

// gates of one row from the pre-activations ar, az, the candidate's input part ac and its hidden part q
__device__ __forceinline__ GruGates gru_gates(float ar, float az, float ac, float q, float h) {
    GruGates o;
    const float rg = feed_sigmoid(ar);
    o.z = feed_sigmoid(az);
    const float c = feed_tanh(ac + rg * q);
    const float zc = 1.0f - o.z;
    const float dh = h - c;
    o.c = c;
    o.f = c + o.z * dh;
    o.pz = dh * o.z * zc;
    o.sc = zc * (1.0f - c * c);
    o.sr = o.sc * rg;
    o.st = o.sr * q * (1.0f - rg);
    return o;
}

// Input operand of one position: lane group g takes columns DS g .. DS g + DS - 1 (past d: a valid entry; its weight is zero)
template <int DS>
__device__ __forceinline__ void load_x(float* o, const float* __restrict__ xrow, int d, int g) {
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        const int k = DS * g + s;
        o[s] = xrow[k < d ? k : d - 1];
    }
}

// A Newton iterate can be huge where the next one is small again (the LEM passes through 1e27 and more on ordinary inputs): a correction
// to it is then known to 1e-7 of its size only and the next iterate with it.  After a step of more than kFarStep (and from a caller's guess) the
// maps and carries therefore stand for the iterate itself, as in the single-pass scan: the right-hand side is f - J h with the products that cancel
// left out, and the recurrence starts from y0.  The caller says so (`far`); launches enqueued before such a step was known return at
// once, and the caller enqueues them again.  (A branch inside the reduction instead of a kernel of its own cost 3 to 8 % of a solve.)
__device__ __forceinline__ bool step_closed(const Gate& g, bool far) {
    if (!g.prev_err) return false;
    const float e = *reinterpret_cast<const float*>(g.prev_err);
    return (double)e <= g.tol || (!far && !(e <= kFarStep));
}

// f - J h of one row; hr, hz, hc: U_gate h
__device__ __forceinline__ float gru_rhs(const GruGates& k, float hr, float hz, float hc) {
    return (k.c - k.z * k.c) - (k.pz * hz + (k.sr * hc + k.st * hr));
}

template <int N> constexpr int map_size() { return N * N + N; }

// The map of a unit: the maps of its nq chunks composed in the order they apply (dual: the last chunk first).  Wavefront w <
// n / 16 takes columns 16 w .. 16 w + 15, wavefront n / 16 the vector.
template <int N, bool REV>
__device__ __forceinline__ void compose_unit(const float* __restrict__ tot, float* __restrict__ o, int nq, int wave, int g, int r) {
    constexpr int NB = N / 16, MS = map_size<N>();
    const bool is_vec = wave == NB;
    constexpr int PD = N == 16 ? 4 : 2;   // maps requested ahead
    Acc X[NB], A[PD][NB][NB], V[PD][NB];
    auto ask = [&](int j, int i) {
        i = min(i, nq - 1);
        const float* c = tot + (long long)(REV ? nq - 1 - i : i) * MS;
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            V[j][I] = is_vec ? load4(c + N * N + 16 * I + 4 * g) : zero4();
#pragma unroll
            for (int K = 0; K < NB; ++K) A[j][I][K] = load4(c + (16 * I + r) * N + 16 * K + 4 * g);
        }
    };
    const float* m = tot + (long long)(REV ? nq - 1 : 0) * MS;
#pragma unroll
    for (int K = 0; K < NB; ++K) {
        if (is_vec) X[K] = load4(m + N * N + 16 * K + 4 * g);
        else
#pragma unroll
            for (int v = 0; v < 4; ++v) X[K][v] = m[(16 * K + 4 * g + v) * N + 16 * wave + r];
    }
#pragma unroll
    for (int j = 0; j < PD; ++j) ask(j, 1 + j);
    for (int i0 = 1; i0 < nq; i0 += PD) {
#pragma unroll
        for (int j = 0; j < PD; ++j) {
            if (i0 + j < nq) {
                Acc Y[NB];
#pragma unroll
                for (int I = 0; I < NB; ++I) Y[I] = V[j][I];
#pragma unroll
                for (int K = 0; K < NB; ++K)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int I = 0; I < NB; ++I) Y[I] = mfma(A[j][I][K][v], X[K][v], Y[I]);
#pragma unroll
                for (int I = 0; I < NB; ++I) X[I] = Y[I];
            }
            ask(j, i0 + j + PD);
        }
    }
#pragma unroll
    for (int I = 0; I < NB; ++I) {
        if (is_vec) {
            if (r == 0) store4(o + N * N + 16 * I + 4 * g, X[I]);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) o[(16 * I + 4 * g + v) * N + 16 * wave + r] = X[I][v];
        }
    }
}

// x <- M x + v over the maps of the units in front of the group, then over those of the group's own chunks, whose carries are the columns
// of e.  A chain of small products with a vector: on the vector ALUs, because a matrix instruction would use one of its
// sixteen columns (512 cycles a step at n = 32 against about 200).  Even steps take x as operand B holds it (16K + 4g + v) and
// add over the lane groups, which leaves row 16I + r in lane r; odd steps start from there, multiply columns and add
// over the lanes of a row, which leaves the operand order again: no step moves x between lanes.  The maps are requested PD
// steps ahead (a step is shorter than a trip to the last-level cache).
// The map of a unit spans up to 16 chunks and can overflow where the map of no chunk does (an iterate far from the solution whose
// Jacobians expand); applied to a small or zero x it gives an infinity or a NaN that the chunks one by one would not give.  Such a value
// stays in x to the end, so the carries tell: they are then folded again from the chunks' maps alone.
// Of a far iterate x is the state itself and starts at start(row) = y0.
template <int N, bool REV, typename Start>
__device__ __forceinline__ void fold_carries(const ChunkParams& p, int b, int grp, int nq, int g, int r, Acc (&e)[N / 16], bool far, Start start) {
    constexpr int NB = N / 16, MS = map_size<N>(), PD = N == 16 ? 4 : 2;   // even
    Acc A[PD][NB][NB], V[PD][NB];
    Acc xk[NB];      // x[16K + 4g + v]
    float xr[NB];    // x[16K + r]
    const int pu = 16 / p.per_unit;   // units of a group
    const int chunks = (p.T + p.Lc - 1) / p.Lc;
    const float* __restrict__ own = p.tot + ((long long)b * chunks + 16 * grp) * MS;
    // the maps in front of the group: those of the units, in the second pass those of the chunks
    const float* __restrict__ front = p.sup + (long long)b * p.units * MS;
    int maps = p.units, before = REV ? max(p.units - (grp + 1) * pu, 0) : grp * pu, steps = before + nq - 1;
    auto request = [&](int j, int i) {
        i = min(i, steps - 1);
        const int k = i - before;
        const float* m = i < before ? front + (long long)(REV ? maps - 1 - i : i) * MS : own + (long long)(REV ? nq - 1 - k : k) * MS;
#pragma unroll
        for (int I = 0; I < NB; ++I) {
            if (j & 1) {
                V[j][I] = load4(m + N * N + 16 * I + 4 * g);
#pragma unroll
                for (int K = 0; K < NB; ++K)
#pragma unroll
                    for (int v = 0; v < 4; ++v) A[j][I][K][v] = m[(16 * I + 4 * g + v) * N + 16 * K + r];
            } else {
                V[j][I][0] = m[N * N + 16 * I + r];
#pragma unroll
                for (int K = 0; K < NB; ++K) A[j][I][K] = load4(m + (16 * I + r) * N + 16 * K + 4 * g);
            }
        }
    };
    // the carry in front of step i belongs to chunk i - before
    auto select = [&](int i, bool rows) {
        const int k = i - before, q = REV ? nq - 1 - k : k;
        if (k < 0) return;
#pragma unroll
        for (int K = 0; K < NB; ++K) {
            Acc c = xk[K];
            if (rows)
#pragma unroll
                for (int v = 0; v < 4; ++v) c[v] = __shfl(xr[K], 4 * g + v);
            e[K] = r == q ? c : e[K];
        }
    };
    bool zero = true;   // in front of the sequence x is zero (unless y0 is not) and M is not looked at (it may have overflowed)
    auto step = [&](int j, int i) {
        select(i, j & 1);
        if (j & 1) {
#pragma unroll
            for (int I = 0; I < NB; ++I) {
                Acc q = zero4();
#pragma unroll
                for (int K = 0; K < NB; ++K)
#pragma unroll
                    for (int v = 0; v < 4; ++v) q[v] += A[j][I][K][v] * xr[K];
                xk[I] = V[j][I] + row_sums4(q, r);
            }
        } else {
            float y[NB];
#pragma unroll
            for (int I = 0; I < NB; ++I) {
                float q[2] = {0.f, 0.f};
#pragma unroll
                for (int K = 0; K < NB; ++K)
#pragma unroll
                    for (int v = 0; v < 4; ++v) q[v & 1] += A[j][I][K][v] * xk[K][v];
                y[I] = V[j][I][0] + (i > 0 || !zero ? sum_groups(q[0] + q[1]) : 0.f);
            }
#pragma unroll
            for (int I = 0; I < NB; ++I) xr[I] = y[I];
        }
    };
    for (int pass = 0;; ++pass) {
#pragma unroll
        for (int K = 0; K < NB; ++K) {
            xk[K] = e[K] = zero4();
            xr[K] = 0.f;
        }
        if (!REV && far) {
            bool any = false;
#pragma unroll
            for (int K = 0; K < NB; ++K)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    xk[K][v] = start(16 * K + 4 * g + v);
                    any |= xk[K][v] != 0.f;
                }
            zero = __ballot(any) == 0;
        }
        if (steps > 0) {
#pragma unroll
            for (int j = 0; j < PD; ++j) request(j, j);
            int i = 0;
            for (; i + PD <= steps; i += PD) {
#pragma unroll
                for (int j = 0; j < PD; ++j) {
                    step(j, i + j);
                    request(j, i + j + PD);
                }
            }
#pragma unroll
            for (int j = 0; j < PD - 1; ++j)
                if (i + j < steps) step(j, i + j);
        }
        select(steps, steps & 1);
        if (pass > 0 || before == 0) return;
        float sum = 0.f;   // (not a finite number if one of its terms is none)
#pragma unroll
        for (int K = 0; K < NB; ++K)
#pragma unroll
            for (int v = 0; v < 4; ++v) sum += 0.f * e[K][v];
        if (!__ballot(sum != 0.f)) return;
        maps = chunks;
        front = p.tot + (long long)b * chunks * MS;
        before = REV ? max(maps - 16 * (grp + 1), 0) : 16 * grp;
        steps = before + nq - 1;
    }
}

}  // namespace
}  // namespace deer
