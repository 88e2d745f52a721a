// Newton step and gradient of the GRU with 8 channels in fp32 by chunks, plain (n = 8) and multi-head with strides: the reduction of
// every chunk to one affine map, the fold of the maps and the walk of sixteen chunks side by side, as for the larger
// states (chunk_gru.hip), with a matrix-core layout of its own (Sec. 3.1 eq. 3 and 5, Sec. 3.1.1 eq. 7, Sec. 4.4, App. B.4).
//
// Columns.  A column is one chunk of Lc positions of one recurrence (a head's r-th strided sequence of a batch entry; a plain GRU has
// one per batch entry); sixteen columns of one head form a group, a wavefront's work.  Recurrences of 16 chunks and more own
// whole groups, shorter ones (1, 2, 4 or 8 chunks) share one: a recurrence of one chunk needs no map at all, its walk is the whole step.
//
// Layout.  Sixteen rows of a 16x16x4 tile hold two gates of eight rows: row 4a + 2h + i is gate h of state row 2a + i.  The accumulator
// of lane (g = lane / 16, r = lane % 16) then has both gates of the state rows 2g, 2g + 1 of column r, and exactly these two rows are
// the B operand of the next product if the v-th instruction of a contraction takes the columns 2g + v: nothing moves between lanes
// in the walk.  In the reduction the same tile multiplies two chunks at once: its rows hold the two chunks' Jacobians, its columns
// eight columns of either running product, and the two diagonal blocks are kept by one select per register.  The sixteen chunks of a
// group are reduced side by side, eight independent products; the row factors reach the lanes that assemble J through LDS.
//
// Bound: issue (fp32 matrix instructions of 32 cycles and the vector ALU).  The single-pass scan with the cell inside composes every
// pair by cross-lane multiply-adds and spends half of a tile's life in the tree over its wavefronts and the look-back; for the strided
// recurrences of at most one chunk it still builds and composes all Jacobians, which a step by chunks never forms.
//
// Rows of 32 bytes of one head share 128-byte lines with those of three others, whose strides bring them there at other times; a large solve
// runs on copies [B,heads,T,.] (head_rows, time_rows): the walk at 64 x 1,024 x 32 heads, 8 levels, 101 us, on copies 64.
#include "chunk_common.h"

namespace deer {

namespace {

constexpr int N = 8;
constexpr int MS8 = 72;   // a map: 8 x 8 row-major, then the vector
using F2 = float __attribute__((ext_vector_type(2), aligned(4)));   // (the callers' rows need no more than their scalars' alignment)

// what lane (g, r) works on: column r of the wavefront's group
struct Column {
    int head, level, gi, gpr;   // (uniform) head, its stride level, group within its recurrence, groups per recurrence
    int a, lim;                 // first position, one past the last that exists (0: no such chunk)
    int shift;                  // log2 of the stride
    long long row;              // row of the first time index
    int b, r0;
};

__device__ __forceinline__ Column column_of(const Chunk8Params& p, int id, int r) {
    Column c;
    int k = 0;
    while (k + 1 < p.levels && id >= p.lv[k + 1].first) ++k;
    const Chunk8Level& lv = p.lv[k];
    const int rel = id - lv.first, m = rel / lv.groups, grp = rel - m * lv.groups;
    c.level = k;
    c.head = k + p.levels * m;
    c.shift = k;
    c.gpr = lv.Cc >= 16 ? lv.Cc / 16 : 1;
    c.gi = grp % c.gpr;
    const int col = grp * 16 + r, rec = col / lv.Cc, chunk = col - rec * lv.Cc;
    const int s = 1 << k, nrec = min(s, p.T);
    const int b = rec / nrec, r0 = rec - b * nrec, len = (p.T - r0 + s - 1) >> k;
    c.a = chunk * lv.Lc;
    c.lim = (b < p.B && c.a < len) ? len : 0;
    c.b = min(b, p.B - 1);
    c.r0 = r0;
    c.row = (long long)c.b * p.T * p.H + (long long)r0 * p.time_rows + (long long)c.head * p.head_rows;
    return c;
}

// the cell's operands of one head
template <int DS>
struct Cell8 {
    float uA[2], uB[2], wA[DS], wB[DS];
    Acc bA, bB;
};

template <int DS>
__device__ __forceinline__ void load_cell(Cell8<DS>& w, const float* __restrict__ th, int d, int g, int r) {
    const float* __restrict__ U = th + 3 * N * d;
    const float* __restrict__ bias = U + 3 * N * N;
    const int i = 2 * (r >> 2) + (r & 1), hi = (r >> 1) & 1;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int k = 2 * g + v;
        w.uA[v] = U[(hi * N + i) * N + k];
        const float c = U[(2 * N + i) * N + k];
        w.uB[v] = hi ? 0.f : c;
        w.bA[v] = bias[k];
        w.bA[2 + v] = bias[N + k];
        w.bB[v] = bias[3 * N + k];
        w.bB[2 + v] = bias[2 * N + k];
    }
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        const int k = DS * g + s, kc = min(k, d - 1);
        const float a = th[(hi * N + i) * d + kc], c = th[(2 * N + i) * d + kc];
        w.wA[s] = k < d ? a : 0.f;
        w.wB[s] = k < d && hi ? c : 0.f;
    }
}

template <int DS>
__device__ __forceinline__ void cell_gates(GruGates (&o)[2], const Cell8<DS>& w, const float (&h)[2], const float (&x)[DS]) {
    Acc A = w.bA, Bc = w.bB;
#pragma unroll
    for (int s = 0; s < DS; ++s) {
        A = mfma(w.wA[s], x[s], A);
        Bc = mfma(w.wB[s], x[s], Bc);
    }
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        A = mfma(w.uA[v], h[v], A);
        Bc = mfma(w.uB[v], h[v], Bc);
    }
#pragma unroll
    for (int v = 0; v < 2; ++v) o[v] = gru_gates(A[v], A[2 + v], Bc[2 + v], Bc[v], h[v]);
}

// rows 2g, 2g + 1 of a state vector
__device__ __forceinline__ void load_rows(float (&o)[2], const float* __restrict__ p, int g) {
    const F2 v = *reinterpret_cast<const F2*>(p + 2 * g);
    o[0] = v[0];
    o[1] = v[1];
}

// ------------------------------------------------------------------------------------------------------------------
// Maps of the chunks (see chunk_totals_kernel of chunk_gru.hip for the two directions).
// ------------------------------------------------------------------------------------------------------------------
template <int DS, bool REV, bool FAR>
__global__ __launch_bounds__(256, 2) void chunk8_totals_kernel(Chunk8Params p) {
    // per wavefront: row factors [chunk][row][p_z, s_r, s_t, z] and vectors [chunk][row]; at the end the sixteen maps
    __shared__ __align__(16) float sF[4][16 * MS8];
    if (step_closed(p.gate, FAR)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int id = (int)(blockIdx.x * 4u) + wave;
    if (id >= p.map_groups) return;
    const Column c = column_of(p, id, r);
    const int Lc = p.lv[c.level].Lc, d = p.d;
    const float* __restrict__ yb = p.y + c.row * N;
    const float* __restrict__ xb = p.x + c.row * d;
    const float* __restrict__ gb = REV ? p.g + c.row * N : nullptr;
    const float* __restrict__ y0b = p.y0 ? p.y0 + ((long long)c.b * p.H + c.head) * N : nullptr;
    const unsigned sy = (unsigned)(p.time_rows * N) << c.shift, sx = (unsigned)(p.time_rows * d) << c.shift;
    const float* __restrict__ th = p.theta + (long long)c.head * p.P;
    float* __restrict__ F = sF[wave];
    float* __restrict__ V = F + 16 * 32;

    constexpr int R = 4;
    float yr[R][2], gr[REV ? R : 1][2], xr[R][DS];
    const int last = max(c.lim, 1) - 1;
    auto ask = [&](int j, int t) {
        // forward: position a + Lc - 1 - t, the state in front of it and its input; dual: position a + t, its state and cotangent and the
        // input of the position after it
        const int pos = REV ? c.a + t : c.a + Lc - 1 - t;
        const int py = min(REV ? pos : pos - 1, last), px = min(max(REV ? pos + 1 : pos, 0), last);
        if (!REV && py < 0) {
            if (y0b) load_rows(yr[j], y0b, g);
            else yr[j][0] = yr[j][1] = 0.f;
        } else {
            load_rows(yr[j], yb + (unsigned)max(py, 0) * sy, g);
        }
        if constexpr (REV) load_rows(gr[j], gb + (unsigned)py * sy, g);
#pragma unroll
        for (int s = 0; s < DS; ++s) xr[j][s] = xb[(unsigned)px * sx + (unsigned)min(DS * g + s, d - 1)];
    };
    float o[2] = {0.f, 0.f};
    if constexpr (!REV) load_rows(o, yb + (unsigned)min(c.a + Lc - 1, last) * sy, g);
#pragma unroll
    for (int j = 0; j < R; ++j) ask(j, j);

    Cell8<DS> w;
    load_cell(w, th, d, g, r);
    // weights of the assembly.  Lane (g, m): rows 2g, 2g + 1 of J's column i(m) (forward, operand of J^T) or columns 2g, 2g + 1 of J's row i(m)
    // (dual), of chunk 2 pair + which(m)
    const int im = 2 * (r >> 2) + (r & 1), which = (r >> 1) & 1;
    float ja[3][2], dz[2];
    {
        const float* __restrict__ U = th + 3 * N * d;
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int k = 2 * g + v, row = REV ? im : k, col = REV ? k : im;
#pragma unroll
            for (int gate = 0; gate < 3; ++gate) ja[gate][v] = U[(gate * N + row) * N + col];
            dz[v] = k == im ? 1.f : 0.f;
        }
    }
    const bool left = r < 8;
    float Q[8][2], vec[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        vec[q] = 0.f;
#pragma unroll
        for (int v = 0; v < 2; ++v) Q[q][v] = (2 * g + v == (r & 7)) ? 1.f : 0.f;
    }

    for (int t0 = 0; t0 < Lc; t0 += R) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int t = t0 + j, pos = REV ? c.a + t : c.a + Lc - 1 - t;
            const bool live = pos < c.lim;
            GruGates k[2];
            cell_gates(k, w, yr[j], xr[j]);
            F2 res;
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                // positions that do not exist leave the map alone
                const Acc f = live ? Acc{k[v].pz, k[v].sr, k[v].st, k[v].z} : Acc{0.f, 0.f, 0.f, 1.f};
                store4(F + r * 32 + (2 * g + v) * 4, f);
                res[v] = live ? (REV ? gr[REV ? j : 0][v] : k[v].f - o[v]) : 0.f;
                if constexpr (!REV) o[v] = yr[j][v];
            }
            if constexpr (FAR) {
                Acc hA = zero4(), hB = zero4();   // U h
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    hA = mfma(w.uA[v], yr[j][v], hA);
                    hB = mfma(w.uB[v], yr[j][v], hB);
                }
#pragma unroll
                for (int v = 0; v < 2; ++v) res[v] = live ? gru_rhs(k[v], hA[v], hA[2 + v], hB[v]) : 0.f;
            }
            *reinterpret_cast<F2*>(V + r * 8 + 2 * g) = res;
            ask(j, t + R);
            wave_lds_fence();
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float* f = F + (2 * q + which) * 32;
                float a[2];
                if constexpr (!REV) {
                    const Acc f0 = load4(f + 8 * g), f1 = load4(f + 8 * g + 4);
                    a[0] = f0[0] * ja[1][0] + (f0[1] * ja[2][0] + (f0[2] * ja[0][0] + f0[3] * dz[0]));
                    a[1] = f1[0] * ja[1][1] + (f1[1] * ja[2][1] + (f1[2] * ja[0][1] + f1[3] * dz[1]));
                } else {
                    const Acc f0 = load4(f + 4 * im);
#pragma unroll
                    for (int v = 0; v < 2; ++v) a[v] = f0[0] * ja[1][v] + (f0[1] * ja[2][v] + (f0[2] * ja[0][v] + f0[3] * dz[v]));
                }
                const float* rv = V + (2 * q + (r >> 3)) * 8 + 2 * g;
                vec[q] += Q[q][0] * rv[0] + Q[q][1] * rv[1];
                Acc D = mfma(a[0], Q[q][0], zero4());
                D = mfma(a[1], Q[q][1], D);
                Q[q][0] = left ? D[0] : D[2];
                Q[q][1] = left ? D[1] : D[3];
            }
            wave_lds_fence();
        }
    }

    // the maps leave row-major: M[r & 7][2g + v] = Q[v] of chunk 2 pair + r / 8
    float* __restrict__ tot = p.tot + (long long)id * 16 * MS8;
    const bool compose = c.gpr > 1 && (REV ? c.gi > 0 : c.gi < c.gpr - 1);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int m = (2 * q + (r >> 3)) * MS8, at = m + (r & 7) * 8 + 2 * g;
        const F2 v2 = {Q[q][0], Q[q][1]};
        const float s = sum_groups(vec[q]);
        *reinterpret_cast<F2*>(tot + at) = v2;
        if (g == 0) tot[m + 64 + (r & 7)] = s;
        if (compose) {
            *reinterpret_cast<F2*>(F + at) = v2;
            if (g == 0) F[m + 64 + (r & 7)] = s;
        }
    }
    if (!compose) return;
    // the group's map: sixteen maps composed in the order they apply (columns 0 to 7 the matrix, column 8 the vector)
    wave_lds_fence();
    float X[2];
    {
        const float* m = F + (REV ? 15 : 0) * MS8;
#pragma unroll
        for (int v = 0; v < 2; ++v) X[v] = r < 8 ? m[(2 * g + v) * 8 + r] : (r == 8 ? m[64 + 2 * g + v] : 0.f);
    }
#pragma unroll
    for (int i = 1; i < 16; ++i) {
        const float* m = F + (REV ? 15 - i : i) * MS8;
        Acc D = zero4();
#pragma unroll
        for (int v = 0; v < 2; ++v) D[v] = r == 8 ? m[64 + 2 * g + v] : 0.f;
#pragma unroll
        for (int v = 0; v < 2; ++v) D = mfma(which ? 0.f : m[im * 8 + 2 * g + v], X[v], D);
        X[0] = D[0];
        X[1] = D[1];
    }
    float* __restrict__ sup = p.sup + (long long)id * MS8;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        if (r < 8) sup[(2 * g + v) * 8 + r] = X[v];
        else if (r == 8) sup[64 + 2 * g + v] = X[v];
    }
}

// ------------------------------------------------------------------------------------------------------------------
// The walk.  x <- M x + v over the maps of the groups in front and then over the group's own, every column of the tile holding the same
// x; each column keeps the x in front of its chunk.
// ------------------------------------------------------------------------------------------------------------------
template <bool REV>
__device__ __forceinline__ void fold8(const Chunk8Params& p, const Column& c, int id, int Cc, unsigned live, int g, int r, float (&e)[2], bool far) {
    constexpr int PD = 4;
    const int own = min(Cc, 16);
    int maps = c.gpr, before = REV ? c.gpr - 1 - c.gi : c.gi, steps = before + 15;
    const int im = 2 * (r >> 2) + (r & 1), which = (r >> 1) & 1;
    // the maps in front of the group: those of the groups, and again those of the chunks if that overflowed (see fold_carries)
    const float* __restrict__ front = p.sup + (long long)(id - c.gi) * MS8;
    const float* __restrict__ tot = p.tot + (long long)id * 16 * MS8;
    F2 A[PD], V[PD];
    auto request = [&](int j, int i) {
        i = min(i, steps - 1);
        const int q = i - before;
        const float* m = i < before ? front + (long long)(REV ? maps - 1 - i : i) * MS8 : tot + (REV ? 15 - q : q) * MS8;
        A[j] = *reinterpret_cast<const F2*>(m + im * 8 + 2 * g);
        V[j] = *reinterpret_cast<const F2*>(m + 64 + 2 * g);
    };
    float x[2] = {0.f, 0.f};
    bool fresh = true;   // nothing in front: x is zero and M is not looked at (it may have overflowed)
    // of a far iterate x starts at the y0 of the recurrence that column q belongs to
    float start[2] = {0.f, 0.f};
    if (!REV && far && p.y0) load_rows(start, p.y0 + ((long long)c.b * p.H + c.head) * N, g);
    auto begin = [&](int q) {
        x[0] = x[1] = 0.f;
        fresh = true;
        if (!REV && far) {
            x[0] = __shfl(start[0], 16 * g + q);
            x[1] = __shfl(start[1], 16 * g + q);
            fresh = __ballot(x[0] != 0.f || x[1] != 0.f) == 0;
        }
    };
    auto keep = [&](int i) {
        const int k = i - before, q = REV ? 15 - k : k;
        if (k < 0) return;
        if (k % own == 0 && (Cc < 16 || before == 0)) begin(q);
        e[0] = r == q ? x[0] : e[0];
        e[1] = r == q ? x[1] : e[1];
    };
    auto step = [&](int j, int i) {
        keep(i);
        const int k = i - before;
        if (REV && k >= 0 && fresh && !((live >> (15 - k)) & 1u)) return;   // no such chunk
        Acc D = {V[j][0], V[j][1], 0.f, 0.f};
        if (!fresh) {
            D = mfma(which ? 0.f : A[j][0], x[0], D);
            D = mfma(which ? 0.f : A[j][1], x[1], D);
        }
        x[0] = D[0];
        x[1] = D[1];
        fresh = false;
    };
    for (int pass = 0;; ++pass) {
        begin(0);
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
        keep(steps);
        if (pass > 0 || before == 0 || !__ballot(0.f * e[0] + 0.f * e[1] != 0.f)) return;
        maps = 16 * c.gpr;
        front = p.tot + (long long)(id - c.gi) * 16 * MS8;
        before *= 16;
        steps = before + 15;
        e[0] = e[1] = 0.f;
    }
}

template <int DS, bool FAR>
__global__ __launch_bounds__(256, 3) void chunk8_walk_kernel(Chunk8Params p) {
    __shared__ unsigned s_max[4];
    if (step_closed(p.gate, FAR)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int id = (int)(blockIdx.x * 4u) + wave;   // (the number of groups is a multiple of four)
    unsigned emax = 0u;   // largest |y_new - y| as raw bits (a NaN compares above everything)
    const Column c = column_of(p, id, r);
    if (__ballot(c.lim > 0)) {
        const int Lc = p.lv[c.level].Lc, d = p.d;
        const float* __restrict__ yb = p.y + c.row * N;
        const float* __restrict__ xb = p.x + c.row * d;
        float* __restrict__ ob = p.out + c.row * N;
        const unsigned sy = (unsigned)(p.time_rows * N) << c.shift, sx = (unsigned)(p.time_rows * d) << c.shift;
        const int last = max(c.lim, 1) - 1;

        // slot t mod R holds y at the position (the state in front of the next one) and the input of the cell the step evaluates
        constexpr int R = 4;
        float yr[R][2], xr[R][DS];
        auto ask_y = [&](int j, int t) { load_rows(yr[j], yb + (unsigned)min(c.a + t, last) * sy, g); };
        auto ask_x = [&](int j, int t) {
            const unsigned pos = (unsigned)min(c.a + t, last);
#pragma unroll
            for (int s = 0; s < DS; ++s) xr[j][s] = xb[pos * sx + (unsigned)min(DS * g + s, d - 1)];
        };
        if (c.a > 0) load_rows(yr[R - 1], yb + (unsigned)min(c.a - 1, last) * sy, g);
        else if (p.y0) load_rows(yr[R - 1], p.y0 + ((long long)c.b * p.H + c.head) * N, g);
        else yr[R - 1][0] = yr[R - 1][1] = 0.f;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (j < R - 1) ask_y(j, j);
            ask_x(j, j);
        }

        Cell8<DS> w;
        load_cell(w, p.theta + (long long)c.head * p.P, d, g, r);
        float e[2] = {0.f, 0.f};   // correction of the state in front of the position
        if (p.lv[c.level].C > 1) fold8<false>(p, c, id, p.lv[c.level].Cc, (unsigned)__ballot(c.lim > 0) & 0xffffu, g, r, e, FAR);
        float xn[2] = {0.f, 0.f};   // of a far iterate: the new state in front of the position
        if constexpr (FAR)
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                xn[v] = p.lv[c.level].C > 1 ? e[v] : yr[R - 1][v];   // (a recurrence of one chunk: y0)
                e[v] = xn[v] - yr[R - 1][v];
            }

        for (int t0 = 0; t0 < Lc; t0 += R) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int t = t0 + j, pos = c.a + t;
                const bool live = pos < c.lim;
                GruGates k[2];
                cell_gates(k, w, yr[(j + R - 1) % R], xr[j]);
                Acc eA = mfma(w.uA[0], e[0], zero4()), eB = mfma(w.uB[0], e[0], zero4());
                eA = mfma(w.uA[1], e[1], eA);
                eB = mfma(w.uB[1], e[1], eB);
                float y[2];
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    if constexpr (FAR) y[v] = k[v].c + (k[v].z * (xn[v] - k[v].c) + (k[v].pz * eA[2 + v] + (k[v].sr * eB[v] + k[v].st * eA[v])));
                    else y[v] = k[v].f + (k[v].z * e[v] + (k[v].pz * eA[2 + v] + (k[v].sr * eB[v] + k[v].st * eA[v])));
                }
                if (live) *reinterpret_cast<F2*>(ob + (unsigned)pos * sy + 2 * g) = F2{y[0], y[1]};
                const unsigned mask = live ? 0x7fffffffu : 0u;
#pragma unroll
                for (int v = 0; v < 2; ++v) {
                    if constexpr (FAR) xn[v] = y[v];
                    e[v] = y[v] - yr[j][v];
                    emax = max(emax, __float_as_uint(e[v]) & mask);
                }
                ask_y((j + R - 1) % R, t - 1 + R);
                ask_x(j, t + R);
            }
        }
    }
    if (p.err) {
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
// The dual walk with the vector-Jacobian product inside.  lambda_i = g_i + J_{i+1}^T lambda_{i+1} needs the gates of position i + 1 and their
// cotangents, which are all that dL/dx, dL/dtheta and (at the first position) dL/dy0 are made of: the cotangent lambda never reaches
// memory and no gate is computed twice.  A step of a column evaluates the cell at the position behind the one it solves for; one
// more step per first chunk takes the first position.  W^T d comes out of the same products as U^T d (the upper two rows of each
// lane group's four).  dL/dU and dL/dW have the columns on the contraction index: the cotangents and (h | x) cross a slice of LDS that
// is private to the wavefront.  The four wavefronts of a workgroup belong to one head; their sums leave as one row.
// A step's sixteen columns are added up by themselves and then to the sums (relative error of dL/dtheta, 32 heads x 1,024 steps x 8: 3.1e-7 with one
// accumulator over 16 Lc positions, now 2.0e-7), and J^T lambda is added up from zero, z lambda last (dL/dy0 2.4e-7, now 2.0e-7).
// ------------------------------------------------------------------------------------------------------------------
template <int DS>
__global__ __launch_bounds__(256, 2) void chunk8_dual_kernel(Chunk8Params p) {
    // per wavefront, [column][16]: (dar, daz) and (dq, dac) two rows of each at a time, (h | x)
    __shared__ __align__(16) float sT[4][3 * 256];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
    const int id = (int)(blockIdx.x * 4u) + wave;
    const Column c = column_of(p, id, r);
    const int d = p.d;
    float* __restrict__ S = sT[wave];
    Acc gA = zero4(), gB = zero4();              // [dU_r, dU_z | dW_r, dW_z] and [dU_c | dW_c] in accumulator layout
    Acc bA = zero4(), bB = zero4();              // bias sums of this column: (dar, daz), (dq, dac)
    if (__ballot(c.lim > 0)) {
        const int Lc = p.lv[c.level].Lc;
        const float* __restrict__ yb = p.y + c.row * N;
        const float* __restrict__ xb = p.x + c.row * d;
        const float* __restrict__ gb = p.g + c.row * N;
        float* __restrict__ dxb = p.dx ? p.dx + c.row * d : nullptr;
        const unsigned sy = (unsigned)(p.time_rows * N) << c.shift, sx = (unsigned)(p.time_rows * d) << c.shift;
        const float* __restrict__ th = p.theta + (long long)c.head * p.P;
        const int last = max(c.lim, 1) - 1;

        // slot t mod R: y and g at position a + Lc - 1 - t, the input of the position behind it
        constexpr int R = 4;
        float yr[R][2], gr[R][2], xr[R][DS];
        auto ask = [&](int j, int t) {
            const unsigned pos = (unsigned)min(max(c.a + Lc - 1 - t, 0), last), px = (unsigned)min(max(c.a + Lc - t, 0), last);
            load_rows(yr[j], yb + pos * sy, g);
            load_rows(gr[j], gb + pos * sy, g);
#pragma unroll
            for (int s = 0; s < DS; ++s) xr[j][s] = xb[px * sx + (unsigned)min(DS * g + s, d - 1)];
        };
#pragma unroll
        for (int j = 0; j < R; ++j) ask(j, j);

        Cell8<DS> w;
        load_cell(w, th, d, g, r);
        // transposed weights: rows of U^T (lower two of each four) and of W^T
        float tr[2], tz[2], tq[2], tc[2];
        {
            const float* __restrict__ U = th + 3 * N * d;
            const int im = 2 * (r >> 2) + (r & 1), hi = (r >> 1) & 1, xc = min(im, d - 1);
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const int k = 2 * g + v;
                const float wr = th[k * d + xc], wz = th[(N + k) * d + xc], wc = th[(2 * N + k) * d + xc];
                const float ur = U[k * N + im], uz = U[(N + k) * N + im], uc = U[(2 * N + k) * N + im];
                const bool in = im < d;
                tr[v] = hi ? (in ? wr : 0.f) : ur;
                tz[v] = hi ? (in ? wz : 0.f) : uz;
                tq[v] = hi ? 0.f : uc;
                tc[v] = hi && in ? wc : 0.f;
            }
        }
        float e[2] = {0.f, 0.f};   // lambda at the position the step evaluates
        if (p.lv[c.level].C > 1) fold8<true>(p, c, id, p.lv[c.level].Cc, (unsigned)__ballot(c.lim > 0) & 0xffffu, g, r, e, false);
        if (DS == 1 && g == 0) store4(S + 512 + r * 16 + 12, zero4());   // (columns of x that no lane writes)

        // one step at position `at` = pos + 1 with state h in front of it; returns J^T lambda
        auto step = [&](const float (&h)[2], const float (&x)[DS], int at, float (&o)[2]) {
            GruGates k[2];
            cell_gates(k, w, h, x);
            Acc cA, cB;
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                cA[v] = k[v].st * e[v];
                cA[2 + v] = k[v].pz * e[v];
                cB[v] = k[v].sr * e[v];
                cB[2 + v] = k[v].sc * e[v];
            }
            store4(S + r * 16 + 4 * g, cA);
            store4(S + 256 + r * 16 + 4 * g, cB);
            *reinterpret_cast<F2*>(S + 512 + r * 16 + 2 * g) = F2{h[0], h[1]};
#pragma unroll
            for (int s = 0; s < DS; ++s) S[512 + r * 16 + 8 + DS * g + s] = x[s];
            bA += cA;
            bB += cB;
            const float ze[2] = {k[0].z * e[0], k[1].z * e[1]};
            Acc D0 = zero4(), D1 = zero4();
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                D0 = mfma(tz[v], cA[2 + v], D0);
                D1 = mfma(tr[v], cA[v], D1);
            }
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                D0 = mfma(tq[v], cB[v], D0);
                D1 = mfma(tc[v], cB[2 + v], D1);
            }
            wave_lds_fence();
            Acc pA = zero4(), pB = zero4();
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const float* q = S + (4 * m + g) * 16 + r;
                pA = mfma(q[0], q[512], pA);
                pB = mfma(q[256], q[512], pB);
            }
            gA += pA;
            gB += pB;
            wave_lds_fence();
            if (dxb && at < c.lim) {
                float* q = dxb + (unsigned)at * sx + 2 * g;
                if (2 * g + 1 < d) *reinterpret_cast<F2*>(q) = F2{D0[2] + D1[2], D0[3] + D1[3]};
                else if (2 * g < d) q[0] = D0[2] + D1[2];
            }
            o[0] = ze[0] + (D0[0] + D1[0]);
            o[1] = ze[1] + (D0[1] + D1[1]);
        };
        float o[2];
        for (int t0 = 0; t0 < Lc; t0 += R) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int t = t0 + j, pos = c.a + Lc - 1 - t;
                const bool live = pos < c.lim;
                step(yr[j], xr[j], pos + 1, o);
#pragma unroll
                for (int v = 0; v < 2; ++v) e[v] = live ? gr[j][v] + o[v] : 0.f;   // nothing follows the last position
                ask(j, t + R);
            }
        }
        // the first position (chunks further on are done: the chunk in front took their first position)
        const bool start = c.a == 0 && c.lim > 0;
        if (__ballot(start)) {
            float h[2];
            const long long at = (long long)c.b * p.H + c.head;
            if (p.y0) load_rows(h, p.y0 + at * N, g);
            else h[0] = h[1] = 0.f;
#pragma unroll
            for (int v = 0; v < 2; ++v) e[v] = start ? e[v] : 0.f;
            step(h, xr[0], start ? 0 : c.lim, o);
            if (start && p.dy0) *reinterpret_cast<F2*>(p.dy0 + ((at << (p.levels - 1)) + c.r0) * N + 2 * g) = F2{o[0], o[1]};
        }
    }

    // ---- the workgroup's row of dL/dtheta: W[3n,d] | U[3n,n] | b[3n] | b_hc[n] ----
    const int P = (int)p.P, U0 = 3 * N * d, b0 = U0 + 3 * N * N;
    __syncthreads();
    float* __restrict__ row = &sT[0][0] + wave * 512;   // P <= 416
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int k = 2 * g + v;
        if (r < 8) {
            row[U0 + k * N + r] = gA[v];
            row[U0 + (N + k) * N + r] = gA[2 + v];
            row[U0 + (2 * N + k) * N + r] = gB[v];
        } else if (r - 8 < d) {
            row[k * d + r - 8] = gA[v];
            row[(N + k) * d + r - 8] = gA[2 + v];
            row[(2 * N + k) * d + r - 8] = gB[2 + v];
        }
    }
    bA = row_sums4(bA, r);
    bB = row_sums4(bB, r);
    if (r == 0) {
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int k = 2 * g + v;
            row[b0 + k] = bA[v];
            row[b0 + N + k] = bA[2 + v];
            row[b0 + 2 * N + k] = bB[2 + v];
            row[b0 + 3 * N + k] = bB[v];
        }
    }
    __syncthreads();
    for (int q = tid; q < P; q += 256)
        p.partial[(long long)blockIdx.x * P + q] = (sT[0][q] + (&sT[0][0])[512 + q]) + ((&sT[0][0])[1024 + q] + (&sT[0][0])[1536 + q]);
}

// Transposed copies of x and of the iterates: rows of R scalars, heads and times change places.  A thread takes consecutive scalars of what is contiguous
// on the caller's side ([B,T,H,R]); on the other one a row's pieces of lines meet in the L2.
template <int V, bool BACK>
__global__ __launch_bounds__(256) void heads_transpose_kernel(const float* __restrict__ src, float* __restrict__ dst, int T, int H, int R) {
    using F = float __attribute__((ext_vector_type(V)));
    const int words = H * R / V, per = (T + 31) / 32, b = (int)(blockIdx.x / (unsigned)per), t0 = 32 * (int)(blockIdx.x % (unsigned)per), rows = min(32, T - t0);
    for (int q = threadIdx.x; q < rows * words; q += 256) {
        const int t = t0 + q / words, w = q % words, h = w / (R / V), r = w % (R / V);
        const long long user = ((long long)b * T + t) * words + w, mine = (((long long)b * H + h) * T + t) * (R / V) + r;
        if constexpr (BACK) reinterpret_cast<F*>(dst)[user] = reinterpret_cast<const F*>(src)[mine];
        else reinterpret_cast<F*>(dst)[mine] = reinterpret_cast<const F*>(src)[user];
    }
}

// dL/dtheta of a head: the rows of its workgroups in a fixed order (16 strided sums per parameter, then these in order)
__global__ __launch_bounds__(256) void chunk8_reduce_kernel(Chunk8Params p) {
    __shared__ float part[16][17];
    const int ql = threadIdx.x & 15, s = threadIdx.x >> 4, h = (int)blockIdx.y;
    const int P = (int)p.P, q = (int)blockIdx.x * 16 + ql;
    const Chunk8Level& lv = p.lv[h % p.levels];
    const int rows = lv.groups / 4;
    const float* __restrict__ src = p.partial + ((long long)lv.first / 4 + (long long)(h / p.levels) * rows) * P + min(q, P - 1);
    float acc = 0.f;
    int k = s;
    for (; k + 7 * 16 < rows; k += 8 * 16) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(long long)(k + 16 * u) * P];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; k < rows; k += 16) acc += src[(long long)k * P];
    part[s][ql] = acc;
    __syncthreads();
    if (s == 0 && q < P) {
        float o = part[0][ql];
#pragma unroll
        for (int u = 1; u < 16; ++u) o += part[u][ql];
        p.dtheta[(long long)h * P + q] = o;
    }
}

template <int DS>
hipError_t launch8(const Chunk8Params& p, hipStream_t s) {
    const dim3 maps((unsigned)((p.map_groups + 3) / 4)), all((unsigned)(p.groups / 4));
    if (p.g) {
        if (p.map_groups > 0) hipLaunchKernelGGL((chunk8_totals_kernel<DS, true, false>), maps, dim3(256), 0, s, p);
        hipLaunchKernelGGL((chunk8_dual_kernel<DS>), all, dim3(256), 0, s, p);
        hipLaunchKernelGGL(chunk8_reduce_kernel, dim3((unsigned)((p.P + 15) / 16), (unsigned)p.H), dim3(256), 0, s, p);
    } else {
        if (p.map_groups > 0 && p.far) hipLaunchKernelGGL((chunk8_totals_kernel<DS, false, true>), maps, dim3(256), 0, s, p);
        else if (p.map_groups > 0) hipLaunchKernelGGL((chunk8_totals_kernel<DS, false, false>), maps, dim3(256), 0, s, p);
        if (p.far) hipLaunchKernelGGL((chunk8_walk_kernel<DS, true>), all, dim3(256), 0, s, p);
        else hipLaunchKernelGGL((chunk8_walk_kernel<DS, false>), all, dim3(256), 0, s, p);
    }
    return hipGetLastError();
}

}  // namespace

bool chunk_gru8_supported(int dtype, int n, int d, int T, int H) {
    // (positions of a recurrence are addressed by 32-bit scalar offsets)
    return dtype == 0 && n == N && d >= 1 && d <= 8 && (long long)T * H * 8 < (1LL << 31);
}

void chunk_gru8_layout(Chunk8Params& p, int L) {
    p.groups = p.map_groups = 0;
    for (int k = 0; k < p.levels; ++k) {
        Chunk8Level& lv = p.lv[k];
        const long long s = 1LL << k, len = (p.T + s - 1) / s, nrec = s < p.T ? s : p.T;
        const int heads = k < p.H ? (p.H - k + p.levels - 1) / p.levels : 0;
        long long C = (len + L - 1) / L;
        if (C < 16) while (C & (C - 1)) ++C;   // 1, 2, 4 or 8 chunks share a group of sixteen columns
        lv.Lc = (int)(((len + C - 1) / C + 3) / 4 * 4);
        lv.C = (int)((len + lv.Lc - 1) / lv.Lc);
        lv.Cc = C < 16 ? (int)C : (lv.C + 15) / 16 * 16;
        lv.groups = (int)((p.B * nrec * lv.Cc + 63) / 64 * 4);   // whole workgroups of four per head
        lv.first = p.groups;
        p.groups += heads * lv.groups;
        if (lv.C > 1) p.map_groups = p.groups;   // (the length of a recurrence falls with the level)
    }
}

hipError_t launch_chunk_gru8(const Chunk8Params& p, hipStream_t s) {
    if (!chunk_gru8_supported(0, N, p.d, p.T, p.H) || p.groups < 4 || p.groups % 4 != 0 || p.levels < 1 || p.levels > 8) return hipErrorInvalidValue;
    if (p.g ? !p.partial || !p.dtheta : !p.out) return hipErrorInvalidValue;
    return p.d <= 4 ? launch8<1>(p, s) : launch8<2>(p, s);
}

hipError_t launch_heads_transpose(const void* src, void* dst, int B, int T, int H, int R, bool back, hipStream_t s) {
    const float* in = reinterpret_cast<const float*>(src);
    float* out = reinterpret_cast<float*>(dst);
    const dim3 grid((unsigned)((long long)B * ((T + 31) / 32)));   // (one dimension: the second one ends at 65,535)
    // (the caller's arrays need no more than their scalars' alignment)
    const bool wide = R % 4 == 0 && (reinterpret_cast<uintptr_t>(src) & 15) == 0 && (reinterpret_cast<uintptr_t>(dst) & 15) == 0;
    if (wide && back) hipLaunchKernelGGL((heads_transpose_kernel<4, true>), grid, dim3(256), 0, s, in, out, T, H, R);
    else if (wide) hipLaunchKernelGGL((heads_transpose_kernel<4, false>), grid, dim3(256), 0, s, in, out, T, H, R);
    else if (back) hipLaunchKernelGGL((heads_transpose_kernel<1, true>), grid, dim3(256), 0, s, in, out, T, H, R);
    else hipLaunchKernelGGL((heads_transpose_kernel<1, false>), grid, dim3(256), 0, s, in, out, T, H, R);
    return hipGetLastError();
}

}  // namespace deer
