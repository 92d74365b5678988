// Forward contraction d[e][r] = sum_q A[e][q] B[r][q] (A = G v, B = G; upper tiles, split-K) on
// operands that pass through registers on their way to LDS: FP32 operands that are split into three
// BF16 parts there, 16-bit operands whose A side carries node weights.
#pragma once

#include <algorithm>

#include "rb_internal.h"
#include "rb_mfma.h"

namespace rb_fwd {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// Workgroup tile FB x FB, four waves of 64 x 64 complex; two workgroups per CU, so that one stages
// while the other multiplies. A stage holds, for the 128 rows of A and those of B, the operand
// type's FRAGS fragments per 32 rows, each 32 rows x 16 K in lane order (a KiB) with its two
// K halves FH bytes apart: the loaders' 8- and 16-byte pieces of a few rows then fall on distinct
// banks, and a fragment read touches every bank once. Four fragments leave room for two stages a
// workgroup (76 KiB), so that it also stages while it multiplies; six (57 KiB) do not.
constexpr int FB = 128, FTHREADS = 256;
constexpr int FH = 576, FF = 1216;         // bytes between halves, between fragments

// Upper-triangular tile index -> (tm, tn) with tm <= tn.
__device__ __forceinline__ void upper_tile(int idx, int T, int &tm, int &tn) {
    int r = 0, rem = idx;
    while (rem >= T - r) {
        rem -= T - r;
        ++r;
    }
    tm = r;
    tn = r + rem;
}

struct Shape {
    int n, K, nT, tiles, kchunk, splitk;  // kchunk: stages per K chunk
};

// K chunks of the kernel: a multiple of 8 (each XCD takes whole chunks, so that a chunk's columns
// of G come from HBM once), around 1024 workgroups, with the least time by rounds of two workgroups
// per CU. Fewer, longer chunks would round more (512 transducers, 152 053 nodes, FP32 operands:
// error 1.1e-7 with 48 chunks, 8.3e-8 with 96 in the same time); chunks of less than four stages
// are all start and end. want > 0: that many (a tuned configuration).
constexpr int SPLITK_FEW = 64;  // chunks tried on rings with many tiles
inline int splitk_base(int tiles) { return std::max(8, 1024 / tiles / 8 * 8); }
inline int splitk_most(int tiles) {
    return std::max(SPLITK_FEW, splitk_base(tiles) + splitk_base(tiles) / 4 / 8 * 8);
}
inline Shape make_shape(int n, int K, int bk, int n_cu, int want) {
    Shape s{};
    s.n = n;
    s.K = K;
    s.nT = (n + FB - 1) / FB;
    s.tiles = s.nT * (s.nT + 1) / 2;
    const int stages = (K + bk - 1) / bk, slots = std::max(1, n_cu / 8 * 2);
    if (want > 0) {
        s.splitk = std::min(want, stages);
    } else {
        const int k0 = std::max(8, std::min(splitk_base(s.tiles), stages / 4 / 8 * 8));
        long best = 0;
        for (int k = k0; k <= splitk_most(s.tiles); k += 8) {
            const long rounds = ((long)s.tiles * k / 8 + slots - 1) / slots;
            const long cost = rounds * ((stages + k - 1) / k + 4);
            if (k > k0 && stages / k < 4) break;
            if (!best || cost < best) {
                best = cost;
                s.splitk = k;
            }
        }
    }
    s.kchunk = (stages + s.splitk - 1) / s.splitk;
    s.splitk = (stages + s.kchunk - 1) / s.kchunk;
    return s;
}

// Workgroups are dealt to the 8 XCDs round-robin. Chunk c goes to XCD c mod 8, whole; where there
// are fewer chunks than XCDs (a tuned configuration, few nodes) tiles and chunks are dealt one by
// one instead, so that no XCD stays without (2048 transducers, 30 000 nodes, FP32: one chunk 21.1
// -> 6.2 ms, two 11.2 -> 4.1).
inline unsigned grid_of(const Shape &s) {
    return (unsigned)(s.tiles * (s.splitk < 8 ? s.splitk : (s.splitk + 7) / 8 * 8));
}

// Op: the operand type (see rb_gemm.hip, rb_lowp.hip). A thread stages a quarter of a stage's K
// for two rows of each side; Op::load fetches it, Op::put converts and stores it, Op::multiply
// runs a stage's MFMAs from a wave's fragments.
template <class Op>
__global__ void __launch_bounds__(FTHREADS, 2) forward_reg_kernel(const Op op, const Shape s,
                                                                  float2 *__restrict__ dpart) {
    constexpr int TILE = Op::FRAGS * FF, SIDE = (FB / 32) * TILE;  // bytes of 32 rows, of a side
    constexpr bool TWO = Op::FRAGS <= 4;
    __shared__ __attribute__((aligned(64))) char st0[2 * SIDE];
    __shared__ __attribute__((aligned(64))) char st1[TWO ? 2 * SIDE : 64];
    if (op.skip()) return;  // decided before this launch: the same for every workgroup
    const bool few = s.splitk < 8;
    const int kq = few ? blockIdx.x : blockIdx.x >> 3;
    const int split = few ? kq / s.tiles : (kq / s.tiles) * 8 + (blockIdx.x & 7);
    if (split >= s.splitk) return;
    int tm, tn;
    upper_tile(kq % s.tiles, s.nT, tm, tn);
    const int row0 = tm * FB, col0 = tn * FB;
    const int kbeg = split * s.kchunk * Op::BK, kend = min(s.K, kbeg + s.kchunk * Op::BK);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int q = tid & 3, r = tid >> 2;  // staged quarter, rows r and r + 64 of both sides

    floatx16 acc_re[2][2], acc_im[2][2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                acc_re[mt][nt][i] = 0.f;
                acc_im[mt][nt][i] = 0.f;
            }

    typename Op::Rows rows;
    op.rows(rows, s.n, s.K, row0 + r, col0 + r, q);
    typename Op::Raw raw;
    auto put = [&](char *st) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int at = ((r + 64 * u) >> 5) * TILE + (r & 31) * 16;
            op.put_a(raw, rows, u, q, st + at);
            op.put_b(raw, rows, u, q, st + SIDE + at);
        }
    };
    // rows or columns past n, and in a diagonal tile a wave below the diagonal, have no output
    const int wr = row0 + wm * 64, wc = col0 + wn * 64;
    const bool active = wr < s.n && wc < s.n && wr <= wc;
    auto multiply = [&](const char *st) {
        if (active)
            op.multiply(st + wm * 2 * TILE + (lane >> 5) * FH + (lane & 31) * 16,
                        st + SIDE + wn * 2 * TILE + (lane >> 5) * FH + (lane & 31) * 16, acc_re,
                        acc_im);
    };
    // one stage multiplied while the next is converted into the other buffer and the one after
    // it is being loaded
    auto step = [&](char *cur, char *nxt, int k0) {
        if (k0 + Op::BK < kend) put(nxt);
        if (k0 + 2 * Op::BK < kend) op.load(raw, rows, k0 + 2 * Op::BK + q * Op::Q, kend);
        __builtin_amdgcn_sched_barrier(0);
        multiply(cur);
        __syncthreads();
    };
    if constexpr (TWO) {
        op.load(raw, rows, kbeg + q * Op::Q, kend);
        put(st0);
        if (kbeg + Op::BK < kend) op.load(raw, rows, kbeg + Op::BK + q * Op::Q, kend);
        __syncthreads();
        for (int k0 = kbeg; k0 < kend; k0 += 2 * Op::BK) {
            step(st0, st1, k0);
            if (k0 + Op::BK < kend) step(st1, st0, k0 + Op::BK);
        }
    } else {
        // one stage, and no loads in flight while it is multiplied (their registers would be
        // spilled there): the CU's other workgroup multiplies while this one waits
        for (int k0 = kbeg; k0 < kend; k0 += Op::BK) {
            op.load(raw, rows, k0 + q * Op::Q, kend);
            __syncthreads();  // the stage has been read
            put(st0);
            __syncthreads();
            multiply(st0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    op.finish(rows);
    float2 *out = dpart + (size_t)split * s.n * s.n;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int gc = col0 + wn * 64 + nt * 32 + (lane & 31);
        if (gc >= s.n) continue;
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int gr = row0 + wm * 64 + mt * 32 + mfma_row(lane, i);
                if (gr <= gc)
                    out[(size_t)gr * s.n + gc] = make_float2(acc_re[mt][nt][i], acc_im[mt][nt][i]);
            }
    }
}

// d[e][r] = d[r][e] = mul / (rows[e] rows[r]) sum over the K chunks of the partial at e <= r; both
// entries come from the same sum, so d is exactly symmetric. A workgroup takes an 8 x 8 tile of
// the upper triangle, four threads per entry summing every fourth chunk (fixed order). mul
// (nullable): mul[1]^mul_pow; rows (nullable): powers of two. Check undoes what scales remain and
// sees every entry.
constexpr int RT = 8;
template <class Check>
__global__ void __launch_bounds__(256) reduce_kernel(const float2 *__restrict__ dpart, int n,
                                                     int splitk,
                                                     const float *__restrict__ mul, int mul_pow,
                                                     const float *__restrict__ rows,
                                                     const Check check, float2 *__restrict__ d) {
    __shared__ float2 red[4][RT][RT + 1];
    if (check.skip()) return;
    int te, tr;
    {   // tile of the upper triangle, counted by columns
        const int b = blockIdx.x;
        tr = (int)((sqrtf(8.f * (float)b + 1.f) - 1.f) * 0.5f);
        while (tr * (tr + 1) / 2 > b) --tr;
        while ((tr + 1) * (tr + 2) / 2 <= b) ++tr;
        te = b - tr * (tr + 1) / 2;
    }
    const int part = threadIdx.x >> 6, i = (threadIdx.x >> 3) & 7, j = threadIdx.x & 7;
    const int e = te * RT + i, r = tr * RT + j;
    float sr = 0.f, si = 0.f;
    if (e <= r && r < n) {
        const float2 *src = dpart + (size_t)e * n + r;
        const size_t nn = (size_t)n * n;
#pragma unroll 8
        for (int s = part; s < splitk; s += 4) {
            const float2 v = src[s * nn];
            sr += v.x;
            si += v.y;
        }
    }
    red[part][i][j] = make_float2(sr, si);
    __syncthreads();
    // threads 0-63 the tile's rows, 64-127 its columns (the mirrored entries)
    if (part > 1) return;
    const int a = part == 0 ? i : j, b = part == 0 ? j : i;
    const int ge = te * RT + a, gr = tr * RT + b;
    if (ge > gr || gr >= n || (part == 1 && ge == gr)) return;
    float2 v;
    v.x = (red[0][a][b].x + red[1][a][b].x) + (red[2][a][b].x + red[3][a][b].x);
    v.y = (red[0][a][b].y + red[1][a][b].y) + (red[2][a][b].y + red[3][a][b].y);
    // one factor: with large weights the sum times theirs alone can leave FP32's range
    float f = mul ? mul[1] : 1.f;
    if (mul_pow == 2) f *= f;
    if (rows) f /= rows[ge] * rows[gr];
    v = make_float2(v.x * f, v.y * f);
    v = check.unscale(v);
    check.see(ge, gr, v);
    if (part == 0) d[(size_t)ge * n + gr] = v;
    else d[(size_t)gr * n + ge] = v;
}

struct NoCheck {
    __device__ bool skip() const { return false; }
    __device__ float2 unscale(float2 v) const { return v; }
    __device__ void see(int, int, float2) const {}
};

inline unsigned reduce_grid(int n) {
    const unsigned nt = (unsigned)((n + RT - 1) / RT);
    return nt * (nt + 1) / 2;
}

}  // namespace rb_fwd
