// Complex GEMMs of the Born operator on FP32 operands (gfx950 matrix cores).
//
// Forward (Eqs. perturb1, derivative): d[e][r] = sum_q G[e][q] v[q] G[r][q] with
// v = w delta. Both operands are K-contiguous ([row][q]); d is symmetric (reciprocity), so
// only tiles with tile(e) <= tile(r) are computed. K = number of mask nodes is long, so the
// K range is split across workgroups (split-K) into FP32 partial tiles that a second kernel
// sums in a fixed order (deterministic) and mirrors.
//
// Row-reduced NN GEMM (Eq. functional-gradient with Q = 1, Eq. sound_speed_update2):
// for each component c, Y_c = R B_c with R [n][n] and B_c [n][n_mask]; the epilogue
// multiplies Y_c by the same operand at the output position (E_c[e][q] = B_c[e][q]) and
// sums over the rows e of the tile, giving per-column partial sums (re, im) per row block.
//
// Split operands. The FP32 matrix instructions run at 1/16 of the 16-bit rate. Both contractions
// take an FP32 value as the sum of three BF16 values, each the rounded error of the ones before
// it: 8 + 8 + 8 bits hold FP32's 24 exactly, with FP32's exponents, whatever else its row or column
// holds. Of a product's nine terms the six of up to 2^-16 are formed (BF16 MFMAs, exact
// products, FP32 accumulators); the other three come to at most 2^-24 of it. The contraction runs
// at 6/16 of the FP32 instructions' cost. An infinity or NaN of an operand (or a value that
// BF16's rounding takes past the largest) makes the sums it enters not finite, and a value
// below 2^-100, whose last part could leave the normal range, is noticed as it is split: either way
// the FP32 kernel after the split one recomputes everything, which returns at once otherwise.
#include "rb_internal.h"
#include "rb_mfma.h"
#include "rb_fwd.h"

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ floatx16 mfma32(float a, float b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

constexpr int RR_BM = 256, RR_BN = 64, RR_BK = 16;

// The row-reduced products are bilinear forms x^T R x (the same operand E = B on both
// sides), which see only the symmetric part Rs = (R + R^T) / 2. With row and column blocks
// of bm transducers, x^T Rs x = sum_I x_I^T Rs_II x_I + 2 sum_{J > I} x_I^T Rs_IJ x_J, so
// the operand is the block upper triangle R' = Rs on diagonal blocks, R + R^T above them, 0
// below, and row block I contracts over columns from its own block on.
template <int bm>
__device__ __forceinline__ float2 sym_upper(const float2 *__restrict__ R, int n, int row, int col) {
    const int bi = row / bm, bj = col / bm;
    if (row >= n || col >= n || bj < bi) return make_float2(0.f, 0.f);
    const float2 a = R[(size_t)row * n + col], b = R[(size_t)col * n + row];
    const float f = bj == bi ? 0.5f : 1.0f;
    return make_float2(f * (a.x + b.x), f * (a.y + b.y));
}

// Split operands --------------------------------------------------------------------------
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ floatx16 mfma_bf16(bf16x8 a, bf16x8 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 negate(bf16x8 x) {
    return __builtin_bit_cast(bf16x8, __builtin_bit_cast(uintx4, x) ^ 0x80008000u);
}

// Three BF16 parts of a pair of values, each packed in a word; least: the smallest magnitude of a
// value seen that is not zero, as its bits doubled less one.
constexpr int PARTS = 6;  // (re, im) x three parts
__device__ __forceinline__ void split_pair(float a, float b, uint32_t &least, uint32_t &w0,
                                           uint32_t &w1, uint32_t &w2) {
    least = min(least, min((__float_as_uint(a) << 1) - 1u, (__float_as_uint(b) << 1) - 1u));
    auto part = [&](uint32_t &w) {
        const bf16x2 h = {(__bf16)a, (__bf16)b};
        w = __builtin_bit_cast(uint32_t, h);
        a -= __uint_as_float(w << 16);
        b -= __uint_as_float(w & 0xffff0000u);
    };
    part(w0);
    part(w1);
    part(w2);
}
constexpr uint32_t SPLIT_TINY = (27u << 24) - 1u;  // 2^-100

// A stage's 16 K of a wave: two row tiles and two column tiles, PARTS fragments of FRAG bytes
// each, at pa and pb. The stage's products are summed on their own and added to the accumulators
// once: a dozen MFMAs that each rounded the long sum would leave more error than FP32's
// instructions, this leaves less. Fragments are read as they are needed (the columns' twice, LDS
// has the time): more of them at once than there are registers for.
template <int FRAG>
__device__ __forceinline__ void split_multiply(const char *pa, const char *pb,
                                               floatx16 (&acc_re)[2][2],
                                               floatx16 (&acc_im)[2][2]) {
    auto frag = [](const char *p, int tile, int part) {
        return *reinterpret_cast<const bf16x8 *>(p + (tile * PARTS + part) * FRAG);
    };
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        bf16x8 a[PARTS];
#pragma unroll
        for (int pl = 0; pl < PARTS; ++pl) a[pl] = frag(pa, mt, pl);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            floatx16 re, im;
#pragma unroll
            for (int i = 0; i < 16; ++i) re[i] = im[i] = 0.f;
            // part j of the columns with the rows' parts i, i + j <= 2, the smallest first
#pragma unroll
            for (int j = 2; j >= 0; --j) {
                const bf16x8 br = frag(pb, nt, j), bi = frag(pb, nt, 3 + j), bn = negate(bi);
#pragma unroll
                for (int i = 2 - j; i >= 0; --i) {
                    re = mfma_bf16(a[i], br, re);
                    im = mfma_bf16(a[i], bi, im);
                    re = mfma_bf16(a[3 + i], bn, re);
                    im = mfma_bf16(a[3 + i], br, im);
                }
            }
            acc_re[mt][nt] += re;
            acc_im[mt][nt] += im;
        }
        asm volatile("" ::: "memory");
    }
}

// State of a split contraction in device memory. plain: set before it (a value of R below 2^-100,
// weights that are not finite); bad: set by it (a value of another operand below 2^-100, sums that
// are not finite). Either makes the FP32 kernels after it recompute the result. rs: exponent of the
// forward's scaled weights.
struct SplitHead {
    int plain, bad, rs, pad;
};

// R' on its way into the row-reduced product: fragments of 32 rows x 16 K as one lane-ordered KiB
// (lane l: row l & 31, K 8 (l >> 5) .. + 7), [K / 16][row / 32][part], so that a row slab's K step
// is contiguous and a fragment read touches every LDS bank once.
constexpr int SR_FRAG = 512;  // values of a fragment
constexpr int SR_BM = RR_BM, SR_BN = 128, SR_BK = 16, SR_THREADS = 512;
constexpr int SR_WM = 64;  // rows of a wave, the block of R's triangle
constexpr int SR_A = (SR_BM / 32) * PARTS * SR_FRAG, SR_B = (SR_BN / 32) * PARTS * SR_FRAG;
inline __host__ __device__ int split_rows(int n) { return (n + SR_WM - 1) / SR_WM * SR_WM; }
inline size_t split_residual_bytes(int n) {
    return (size_t)split_rows(n) * rb_lp_pad(n) * (PARTS * 2);
}

// R' in parts, zero past n: np columns, split_rows(n) rows. A workgroup covers 32 rows x 64
// columns. head: cleared before.
__global__ void __launch_bounds__(256) split_residual_kernel(const float2 *__restrict__ R, int n,
                                                             int np, SplitHead *__restrict__ head,
                                                             __bf16 *__restrict__ Rf) {
    const int row = blockIdx.y * 32 + (threadIdx.x & 31);
    const int c0 = blockIdx.x * 64 + (threadIdx.x >> 5) * 8;
    if (c0 >= np) return;
    uint32_t w[PARTS][4], least = ~0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float2 a = sym_upper<SR_WM>(R, n, row, c0 + 2 * k);
        const float2 b = sym_upper<SR_WM>(R, n, row, c0 + 2 * k + 1);
        split_pair(a.x, b.x, least, w[0][k], w[1][k], w[2][k]);
        split_pair(a.y, b.y, least, w[3][k], w[4][k], w[5][k]);
    }
    if (least < SPLIT_TINY) head->plain = 1;
    const size_t frag = ((size_t)(c0 / SR_BK) * gridDim.y + blockIdx.y) * PARTS;
    __bf16 *dst = Rf + frag * SR_FRAG + ((c0 >> 3) & 1) * 256 + (threadIdx.x & 31) * 8;
#pragma unroll
    for (int pl = 0; pl < PARTS; ++pl)
        *reinterpret_cast<uint4 *>(dst + pl * SR_FRAG) =
            make_uint4(w[pl][0], w[pl][1], w[pl][2], w[pl][3]);
}

// The row-reduced products on split operands. Bound by the matrix pipes: 24 BF16 MFMAs of
// 32x32x16 per complex 32x32 tile and 16 K values, twice the MFMAs per staged byte of the
// 16-bit form, so the same workgroup (256 rows x 128 columns, eight waves of 64 x 64, two per
// SIMD) leaves LDS at about a third of its rate; a K step's MFMAs take a wave 3000 cycles, so
// one step ahead is far enough (two LDS stages of 72 KiB). R' comes in fragment order straight into
// LDS. B stays as the caller keeps it (FP32, complex, [row][column]): a lane takes one column of 8
// consecutive rows (512-byte runs per wave), which is a fragment's 8 K values, splits them in
// registers (about 12 instructions a pair) and writes six 16-byte pieces to LDS. Waves 0-3 and 4-7
// stage alternate K steps, so that a wave's loads are in flight for two steps. R's triangle has
// blocks of 64, a wave's rows: a wave skips the K blocks left of its own, which the FP32 kernel's
// 256-row blocks multiply as zeros. No operand is written to memory in split form: converting once
// in a pass of its own would move 47 GB more at 1024 transducers and 636160 nodes, where the
// back-projection takes 42.5 ms (1.2 PFLOP/s of MFMAs; the FP32 kernel 128.9 ms); its error against
// FP64 sums is 2.4e-7 over 1024 transducers, 2.0e-7 over 301 (6.3e-7, 3.3e-7; random operands).
__global__ void __launch_bounds__(SR_THREADS) rowred_split_kernel(
    const __bf16 *__restrict__ Rf, const float2 *__restrict__ B, int n, int np, int n_cols,
    int n_comp, int conj_b, int mblocks, int nblocks, SplitHead *__restrict__ head,
    float *__restrict__ parts) {
    // R' and B of two K steps, in arrays of their own: the compiler then sees that neither
    // the stores of B nor the reads of one step depend on loads in flight into another
    __shared__ __attribute__((aligned(1024))) __bf16 a0[SR_A], a1[SR_A];
    __shared__ __attribute__((aligned(1024))) __bf16 b0[SR_B], b1[SR_B];
    __shared__ float red[2][4][SR_BN];
    __shared__ int stop;
    if (head->plain) return;  // written before this launch

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;      // 4 x 2 waves of 64 x 64
    const int grp = wave >> 2, half = (wave >> 1) & 1;  // staging: K step parity, half of a step
    const int scol = (wave & 1) * 64 + lane;      // staged column of the tile
    const float bsign = conj_b ? -1.f : 1.f;
    const int ntile = split_rows(n) / 32, KT = np / SR_BK;
    const __amdgpu_buffer_rsrc_t ra = plane_rsrc(Rf, (size_t)ntile * 32 * np * (PARTS * 2));
    uint32_t least = ~0u;  // of all this lane staged

    // Persistent, one workgroup per CU; items and XCD ranges as in the FP32 kernel. K runs from
    // the last block down, so that the epilogue finds its diagonal block of B in L2.
    const int n_pairs = (mblocks + 1) / 2, n_items = nblocks * n_pairs;
    const int L = gridDim.x >> 3, xcd = blockIdx.x & 7;
    const int per = (((n_items + 7) / 8) + 1) & ~1;
    for (int it = blockIdx.x >> 3; it < per; it += L) {
        const int item = xcd * per + it;
        if (item >= n_items) break;
        const int nb = item / n_pairs, pr = item - nb * n_pairs;
        const int col0 = nb * SR_BN;
        for (int hf = 0; hf < 2; ++hf) {
            const int mb = hf == 0 ? pr : mblocks - 1 - pr;
            if (hf == 1 && mb == pr) break;  // middle slab of an odd count
            const int row0 = mb * SR_BM;
            const int steps = KT - row0 / SR_BK;
            float cs_re[2] = {0.f, 0.f}, cs_im[2] = {0.f, 0.f};
            // this wave's rows meet K from their own block of R' on; nothing of rows past n
            const int wrow = row0 + wm * SR_WM;
            const int wsteps = wrow < n ? KT - wrow / SR_BK : 0;
            const uint32_t ccol = (uint32_t)min(col0 + scol, n_cols - 1);
            float2 raw[8];
            // step i of the loop is K step KT - 1 - i; rows past n meet zeros of R'
            auto load_b = [&](const float2 *Bc, int i) {
                const int k0 = (KT - 1 - i) * SR_BK + half * 8;
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    raw[u] = (Bc + (size_t)min(k0 + u, n - 1) * n_cols)[ccol];
            };
            auto put_b = [&](__bf16 *st) {
                uint32_t w[PARTS][4];
                // the values are used from here on (the signs were applied where they are loaded,
                // which waited for the loads)
#pragma unroll
                for (int u = 0; u < 8; ++u) asm volatile("" : "+v"(raw[u].x), "+v"(raw[u].y));
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    split_pair(raw[2 * u].x, raw[2 * u + 1].x, least, w[0][u], w[1][u], w[2][u]);
                    split_pair(raw[2 * u].y * bsign, raw[2 * u + 1].y * bsign, least, w[3][u],
                               w[4][u], w[5][u]);
                }
                __bf16 *dst = st + (scol >> 5) * PARTS * SR_FRAG + half * 256 + (scol & 31) * 8;
#pragma unroll
                for (int pl = 0; pl < PARTS; ++pl)
                    *reinterpret_cast<uint4 *>(dst + pl * SR_FRAG) =
                        make_uint4(w[pl][0], w[pl][1], w[pl][2], w[pl][3]);
            };
            auto fetch_a = [&](int i, __bf16 *st) {
                const uint32_t kb = (uint32_t)((KT - 1 - i) * ntile + mb * (SR_BM / 32)) *
                                    (PARTS * SR_FRAG * 2);
#pragma unroll
                for (int u = 0; u < PARTS; ++u)
                    load_lds16(ra, st + (wave + 8 * u) * SR_FRAG, lane * 16,
                               kb + (uint32_t)(wave + 8 * u) * (SR_FRAG * 2));
            };
            // the first loads of a component: R' of a step, B of this wave's first
            auto begin = [&](const float2 *Bc) {
                fetch_a(0, a0);
                __builtin_amdgcn_sched_barrier(0);
                if (grp == 0 || steps > 1) load_b(Bc, grp);
                __builtin_amdgcn_sched_barrier(0);
            };
            begin(B);

            for (int c = 0; c < n_comp; ++c) {
                const float2 *Bc = B + (size_t)c * n * n_cols;
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
                auto multiply = [&](const __bf16 *sa, const __bf16 *sb) {
                    split_multiply<SR_FRAG * 2>(
                        reinterpret_cast<const char *>(sa + wm * 2 * PARTS * SR_FRAG + lane * 8),
                        reinterpret_cast<const char *>(sb + wn * 2 * PARTS * SR_FRAG + lane * 8),
                        acc_re, acc_im);
                };
                // A step whose successors are in flight. R' of step i + 1 is fetched here; the
                // waves that stage then store B of that step and load B of step i + 3 (8 loads,
                // younger than R'), the others' youngest loads are R' itself.
                auto step = [&](__bf16 *ca, __bf16 *cb, __bf16 *nb_, __bf16 *na, int i) {
                    const bool stage = ((grp ^ i) & 1) != 0;
                    fetch_a(i + 1, na);
                    __builtin_amdgcn_sched_barrier(0);
                    if (stage) put_b(nb_);
                    __builtin_amdgcn_sched_barrier(0);
                    if (i < wsteps) multiply(ca, cb);
                    __builtin_amdgcn_sched_barrier(0);
                    if (stage) {
                        load_b(Bc, i + 3);
                        lr_sync<8>();
                    } else {
                        lr_sync<0>();
                    }
                };
                // a step near the end: nothing is left in flight
                auto last = [&](__bf16 *ca, __bf16 *cb, __bf16 *nb_, __bf16 *na, int i) {
                    if (i + 1 < steps) fetch_a(i + 1, na);
                    if (((grp ^ i) & 1) != 0) {
                        if (i + 1 < steps) put_b(nb_);
                        if (i + 3 < steps) load_b(Bc, i + 3);
                    }
                    if (i < wsteps) multiply(ca, cb);
                    lr_sync<0>();
                };
                if (grp == 0) {
                    put_b(b0);
                    if (steps > 2) load_b(Bc, 2);
                }
                // R' of step 0 is older than each wave's 8 loads of B
                if (steps > 2) lr_sync<8>();
                else lr_sync<0>();
                int i = 0;
                for (; i + 4 < steps; i += 2) {
                    step(a0, b0, b1, a1, i);
                    step(a1, b1, b0, a0, i + 1);
                }
                for (; i < steps; i += 2) {
                    last(a0, b0, b1, a1, i);
                    if (i + 1 < steps) last(a1, b1, b0, a0, i + 1);
                }
                // every wave is past its reads: the next component's first loads run under
                // the epilogue
                if (c + 1 < n_comp) begin(Bc + (size_t)n * n_cols);
                // epilogue: sum over the rows of E_c[e][q] Y_c[e][q] (Y zero past n), 16 loads in
                // flight. The asm keeps its 64 addresses from being formed before the
                // K loop and spilled.
                int rbase = wrow, cbase = col0 + wn * 64 + (lane & 31);
                asm volatile("" : "+s"(rbase), "+v"(cbase));
                if (wsteps > 0) {
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt) {
                        const uint32_t gc = (uint32_t)min(cbase + nt * 32, n_cols - 1);
#pragma unroll
                        for (int mt = 0; mt < 2; ++mt) {
                            float2 ev[16];
#pragma unroll
                            for (int k = 0; k < 16; ++k) {
                                // rows br (lanes 0-31) and br + 4, clamped to the last row
                                const int br = rbase + mt * 32 + (k >> 2) * 8 + (k & 3);
                                const uint32_t up = br + 4 < n ? 4u * (uint32_t)n_cols : 0u;
                                ev[k] = (Bc + (size_t)min(br, n - 1) * n_cols)
                                    [(lane >> 5) * up + gc];
                            }
#pragma unroll
                            for (int k = 0; k < 16; ++k) {
                                const float er = ev[k].x, ei = ev[k].y * bsign;
                                const float yr = acc_re[mt][nt][k], yi = acc_im[mt][nt][k];
                                cs_re[nt] += er * yr - ei * yi;
                                cs_im[nt] += er * yi + ei * yr;
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
            }
            // combine the two lane halves, then the four waves of a column
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                cs_re[nt] += __shfl_xor(cs_re[nt], 32);
                cs_im[nt] += __shfl_xor(cs_im[nt], 32);
                if (lane < 32) {
                    red[0][wm][wn * 64 + nt * 32 + lane] = cs_re[nt];
                    red[1][wm][wn * 64 + nt * 32 + lane] = cs_im[nt];
                }
            }
            __syncthreads();
            if (tid < SR_BN && col0 + tid < n_cols) {
                const int gc = col0 + tid;
                const float sr = (red[0][0][tid] + red[0][1][tid]) +
                                 (red[0][2][tid] + red[0][3][tid]);
                const float si = (red[1][0][tid] + red[1][1][tid]) +
                                 (red[1][2][tid] + red[1][3][tid]);
                parts[(size_t)mb * n_cols + gc] = sr;
                parts[(size_t)(mblocks + mb) * n_cols + gc] = si;
                if (!isfinite(sr) || !isfinite(si)) head->bad = 1;
            }
            if (least < SPLIT_TINY) head->bad = 1;
            // a call that is turned down ends here (a look past this XCD's caches)
            if (tid == 0)
                stop = __hip_atomic_load(&head->bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();  // red[] and the stages are reused by the next slab
            if (stop) return;
        }
    }
}

// R' for the FP32 kernel, [n][n]: blocks of RR_BM.
__global__ void __launch_bounds__(256) sym_upper_kernel(const float2 *__restrict__ R, int n,
                                                        const SplitHead *__restrict__ head,
                                                        float2 *__restrict__ Rs) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if ((head && !head->plain && !head->bad) || i >= (size_t)n * n) return;
    const int row = (int)(i / n);
    Rs[i] = sym_upper<RR_BM>(R, n, row, (int)(i - (size_t)row * n));
}

// The FP32 form, for what the split form turns down (head: the split contraction before it,
// NULL to run in any case). R: R' from sym_upper_kernel (formed here, in every K step of every
// column block, it took 12.1 ms instead of 8.3 at 1024 transducers and 40 000 nodes).
// parts: [2][mblocks][n_cols] (re plane, then im plane).
__global__ void __launch_bounds__(256) rowred_kernel(const float2 *__restrict__ R,
                                                     const float2 *__restrict__ B, int n,
                                                     int n_cols, int n_comp, int conj_b,
                                                     int mblocks, int nblocks,
                                                     const SplitHead *__restrict__ head,
                                                     float *__restrict__ parts) {
    __shared__ float a_re[RR_BK][RR_BM], a_im[RR_BK][RR_BM];
    __shared__ float b_re[RR_BK][RR_BN], b_im[RR_BK][RR_BN];
    __shared__ float red[2][4][RR_BN];
    if (head && !head->plain && !head->bad) return;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float bsign = conj_b ? -1.f : 1.f;
    // Persistent: one workgroup per CU walks a static list of items, each one column block
    // and a pair of row blocks (i, mblocks - 1 - i) whose contractions (from the diagonal
    // block on) together span mblocks + 1 blocks, so every item costs the same. Each XCD
    // walks a contiguous range of items.
    const int n_pairs = (mblocks + 1) / 2, n_items = nblocks * n_pairs;
    const int L = gridDim.x >> 3, xcd = blockIdx.x & 7;
    const int per = (((n_items + 7) / 8) + 1) & ~1;
    for (int k = blockIdx.x >> 3; k < per; k += L) {
        const int item = xcd * per + k;
        if (item >= n_items) break;
        const int nb = item / n_pairs, pr = item - nb * n_pairs;
        for (int half = 0; half < 2; ++half) {
            const int mb = half == 0 ? pr : mblocks - 1 - pr;
            if (half == 1 && mb == pr) break;  // middle block of an odd count

            const int row0 = mb * RR_BM, col0 = nb * RR_BN;

            float cs_re[2] = {0.f, 0.f}, cs_im[2] = {0.f, 0.f};  // per n-tile column sums

            for (int c = 0; c < n_comp; ++c) {
                const float2 *Bc = B + (size_t)c * n * n_cols;
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
                for (int k0 = row0; k0 < n; k0 += RR_BK) {  // R' is zero left of the diagonal block
                    // A tile: row (row0 + tid), 16 consecutive k of R'
                    {
                        int gr = row0 + tid;
                        const float2 *src = R + (size_t)gr * n + k0;
#pragma unroll
                        for (int kk = 0; kk < RR_BK; ++kk) {
                            float2 v = make_float2(0.f, 0.f);
                            if (gr < n && k0 + kk < n) v = src[kk];
                            a_re[kk][tid] = v.x;
                            a_im[kk][tid] = v.y;
                        }
                    }
                    // B tile: 16 rows (k) x 64 columns; each thread 4 consecutive columns
                    {
                        int kk = tid >> 4, cc = (tid & 15) * 4;
                        int gk = k0 + kk;
                        const float2 *src = Bc + (size_t)gk * n_cols + col0 + cc;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            float2 v = make_float2(0.f, 0.f);
                            if (gk < n && col0 + cc + u < n_cols) v = src[u];
                            b_re[kk][cc + u] = v.x;
                            b_im[kk][cc + u] = bsign * v.y;
                        }
                    }
                    __syncthreads();
#pragma unroll
                    for (int kp = 0; kp < RR_BK / 2; ++kp) {
                        int k = 2 * kp + (lane >> 5);
                        float ar[2], ai[2], nai[2], br[2], bi[2];
#pragma unroll
                        for (int mt = 0; mt < 2; ++mt) {
                            int m = wave * 64 + mt * 32 + (lane & 31);
                            ar[mt] = a_re[k][m];
                            ai[mt] = a_im[k][m];
                            nai[mt] = -ai[mt];
                        }
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt) {
                            int cn = nt * 32 + (lane & 31);
                            br[nt] = b_re[k][cn];
                            bi[nt] = b_im[k][cn];
                        }
#pragma unroll
                        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                            for (int nt = 0; nt < 2; ++nt) {
                                acc_re[mt][nt] = mfma32(ar[mt], br[nt], acc_re[mt][nt]);
                                acc_re[mt][nt] = mfma32(nai[mt], bi[nt], acc_re[mt][nt]);
                                acc_im[mt][nt] = mfma32(ar[mt], bi[nt], acc_im[mt][nt]);
                                acc_im[mt][nt] = mfma32(ai[mt], br[nt], acc_im[mt][nt]);
                            }
                    }
                    __syncthreads();
                }
                // epilogue: sum over the rows of E_c[e][q] Y_c[e][q]
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    int gc = col0 + nt * 32 + (lane & 31);
                    if (gc >= n_cols) continue;
#pragma unroll
                    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            int gr = row0 + wave * 64 + mt * 32 + mfma_row(lane, i);
                            if (gr < n) {
                                float2 ev = Bc[(size_t)gr * n_cols + gc];
                                float er = ev.x, ei = bsign * ev.y;
                                float yr = acc_re[mt][nt][i], yi = acc_im[mt][nt][i];
                                cs_re[nt] += er * yr - ei * yi;
                                cs_im[nt] += er * yi + ei * yr;
                            }
                        }
                }
            }
            // combine the two lane halves (rows 4..7 of each group of 8), then the four waves
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                cs_re[nt] += __shfl_xor(cs_re[nt], 32);
                cs_im[nt] += __shfl_xor(cs_im[nt], 32);
                if (lane < 32) {
                    red[0][wave][nt * 32 + lane] = cs_re[nt];
                    red[1][wave][nt * 32 + lane] = cs_im[nt];
                }
            }
            __syncthreads();
            if (tid < RR_BN) {
                int gc = col0 + tid;
                if (gc < n_cols) {
                    float sr = red[0][0][tid] + red[0][1][tid] + red[0][2][tid] + red[0][3][tid];
                    float si = red[1][0][tid] + red[1][1][tid] + red[1][2][tid] + red[1][3][tid];
                    parts[(size_t)mb * n_cols + gc] = sr;
                    parts[(size_t)(mblocks + mb) * n_cols + gc] = si;
                }
            }
            __syncthreads();  // red[] and the LDS tiles are reused by the next block
        }
    }
}

constexpr int FW_B = 128, FW_BK = 16;
using rb_fwd::upper_tile;

// Forward on split operands ------------------------------------------------------------------
// Largest |Re|, |Im| of v = w delta, as bits: one partial maximum per workgroup.
constexpr int FS_PARTS = 64;
__global__ void __launch_bounds__(256) weight_max_kernel(int K, const float2 *__restrict__ w,
                                                         const float *__restrict__ delta,
                                                         uint32_t *__restrict__ vmax) {
    __shared__ uint32_t red[4];
    uint32_t m = 0;
    for (int k = blockIdx.x * 256 + threadIdx.x; k < K; k += FS_PARTS * 256) {
        const float dl = delta[k];
        m = max(m, max(__float_as_uint(w[k].x * dl) & 0x7fffffffu,
                       __float_as_uint(w[k].y * dl) & 0x7fffffffu));
    }
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) vmax[blockIdx.x] = max(max(red[0], red[1]), max(red[2], red[3]));
}

// v = w delta (rounded as a product of FP32 values) times the power of two that brings its largest
// part to [2^(VTOP-1), 2^VTOP), and the head (K = 0: that alone). Where delta falls off towards
// nothing (the tail of a Gaussian), G v keeps clear of 2^-100 with it, down to v's smallest
// subnormal; sums of 2^20 terms stay finite up to |G| = 2^13.
constexpr int VTOP = 80;
__global__ void __launch_bounds__(256) weight_scale_kernel(int K, const float2 *__restrict__ w,
                                                           const float *__restrict__ delta,
                                                           const uint32_t *__restrict__ vmax,
                                                           float2 *__restrict__ v,
                                                           SplitHead *__restrict__ head) {
    uint32_t m = 0;
    if (K > 0)
        for (int i = 0; i < FS_PARTS; ++i) m = max(m, vmax[i]);
    const bool finite = m < 0x7f800000u;
    int xv = 0;
    if (finite && m > 0) {
        (void)frexpf(__uint_as_float(m), &xv);
        xv = VTOP - xv;
    }
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0) *head = SplitHead{finite ? 0 : 1, 0, xv, 0};
    if (i < K) {
        const float2 wv = w[i];
        const float dl = delta[i];
        v[i] = make_float2(ldexpf(wv.x * dl, xv), ldexpf(wv.y * dl, xv));
    }
}

// FP32 rows G [n][K] (complex) for rb_fwd::forward_reg_kernel: a stage is 16 K as fragments
// (three parts of re, of im); WEIGHTS: the A side is G v. A lane's quarter of a stage is 32
// consecutive bytes of a row. Bound by the matrix pipes: 512 transducers and 152 053 nodes with
// weights take 1.01 ms (1.1 PFLOP/s of MFMAs) where the FP32 kernel took 2.41 ms, and the error
// against FP64 sums is 9.6e-8 (3.9e-7).
template <bool WEIGHTS>
struct SplitFwd {
    static constexpr int BK = 16, Q = 4, FRAGS = PARTS;
    const float2 *G, *v;
    SplitHead *head;
    typedef float f4 __attribute__((ext_vector_type(4), aligned(8)));
    struct Raw {
        f4 a[2][2], b[2][2], w[2];
    };
    struct Rows {
        const float2 *a[2], *b[2];
        uint32_t least;
    };
    __device__ bool skip() const { return head->plain; }
    __device__ void rows(Rows &o, int n, int K, int ra, int rb, int) const {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            o.a[u] = G + (size_t)min(ra + 64 * u, n - 1) * K;
            o.b[u] = G + (size_t)min(rb + 64 * u, n - 1) * K;
        }
        o.least = ~0u;
    }
    // four consecutive values of a row, zero from kend on
    static __device__ __forceinline__ void get(const float2 *row, int k, int kend, f4 (&x)[2]) {
        if (k + 4 <= kend) {
            x[0] = *reinterpret_cast<const f4 *>(row + k);
            x[1] = *reinterpret_cast<const f4 *>(row + k + 2);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float2 z = k + i < kend ? row[k + i] : make_float2(0.f, 0.f);
                x[i >> 1][2 * (i & 1)] = z.x;
                x[i >> 1][2 * (i & 1) + 1] = z.y;
            }
        }
    }
    __device__ __forceinline__ void load(Raw &x, const Rows &o, int k, int kend) const {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            get(o.a[u], k, kend, x.a[u]);
            get(o.b[u], k, kend, x.b[u]);
        }
        if constexpr (WEIGHTS) get(v, k, kend, x.w);
    }
    static __device__ __forceinline__ void put(const f4 (&x)[2], int q, uint32_t &least,
                                               char *dst) {
        uint32_t w[PARTS][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            split_pair(x[i][0], x[i][2], least, w[0][i], w[1][i], w[2][i]);
            split_pair(x[i][1], x[i][3], least, w[3][i], w[4][i], w[5][i]);
        }
        dst += (q >> 1) * rb_fwd::FH + (q & 1) * 8;
#pragma unroll
        for (int pl = 0; pl < PARTS; ++pl)
            *reinterpret_cast<uint2 *>(dst + pl * rb_fwd::FF) = make_uint2(w[pl][0], w[pl][1]);
    }
    __device__ __forceinline__ void put_a(const Raw &x, Rows &o, int u, int q, char *dst) const {
        if constexpr (WEIGHTS) {
            f4 y[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int h = 0; h < 4; h += 2) {
                    const float gx = x.a[u][i][h], gy = x.a[u][i][h + 1];
                    const float vx = x.w[i][h], vy = x.w[i][h + 1];
                    y[i][h] = gx * vx - gy * vy;
                    y[i][h + 1] = gx * vy + gy * vx;
                }
            put(y, q, o.least, dst);
        } else {
            put(x.a[u], q, o.least, dst);
        }
    }
    __device__ __forceinline__ void put_b(const Raw &x, Rows &o, int u, int q, char *dst) const {
        put(x.b[u], q, o.least, dst);
    }
    __device__ __forceinline__ void multiply(const char *pa, const char *pb,
                                             floatx16 (&acc_re)[2][2],
                                             floatx16 (&acc_im)[2][2]) const {
        split_multiply<rb_fwd::FF>(pa, pb, acc_re, acc_im);
    }
    __device__ void finish(const Rows &o) const {
        if (o.least < SPLIT_TINY) head->bad = 1;
    }
};

// The reduction's look at a split result.
struct SplitCheck {
    SplitHead *head;
    __device__ bool skip() const { return head->plain; }
    __device__ float2 unscale(float2 v) const {  // the weights' power of two
        return make_float2(ldexpf(v.x, -head->rs), ldexpf(v.y, -head->rs));
    }
    __device__ void see(int, int, float2 v) const {
        if (!isfinite(v.x) || !isfinite(v.y)) head->bad = 1;
    }
};
// The reduction after the FP32 kernel: only where that ran.
struct PlainCheck {
    const SplitHead *head;
    __device__ bool skip() const { return head && !head->plain && !head->bad; }
    __device__ float2 unscale(float2 v) const { return v; }
    __device__ void see(int, int, float2) const {}
};

// The FP32 form, for what the split form turns down (head NULL: in any case). dpart:
// [splitk][n][n] complex partial sums (only upper tiles written).
__global__ void __launch_bounds__(256) forward_kernel(const float2 *__restrict__ G,
                                                      const float2 *__restrict__ w,
                                                      const float *__restrict__ delta, int n,
                                                      int K, int T, int kchunk,
                                                      const SplitHead *__restrict__ head,
                                                      float2 *__restrict__ dpart) {
    __shared__ float a_re[FW_BK][FW_B], a_im[FW_BK][FW_B];
    __shared__ float b_re[FW_BK][FW_B], b_im[FW_BK][FW_B];
    if (head && !head->plain && !head->bad) return;
    int tm, tn;
    upper_tile(blockIdx.x, T, tm, tn);
    const int split = blockIdx.y;
    const int kbeg = split * kchunk, kend = min(K, kbeg + kchunk);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int row0 = tm * FW_B, col0 = tn * FW_B;

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

    const int lr = tid >> 1, kh = (tid & 1) * 8;  // loader: row, first k of 8
    for (int k0 = kbeg; k0 < kend; k0 += FW_BK) {
        {
            int gr = row0 + lr;
            const float2 *src = G + (size_t)gr * K + k0 + kh;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                int gk = k0 + kh + u;
                float2 g = make_float2(0.f, 0.f);
                if (gr < n && gk < kend) {
                    float2 gv = src[u];
                    if (w) {  // v = w delta (absent: the operand already carries it)
                        float2 wv = w[gk];
                        float dl = delta[gk];
                        float vr = wv.x * dl, vi = wv.y * dl;
                        g = make_float2(gv.x * vr - gv.y * vi, gv.x * vi + gv.y * vr);
                    } else {
                        g = gv;
                    }
                }
                a_re[kh + u][lr] = g.x;
                a_im[kh + u][lr] = g.y;
            }
        }
        {
            int gr = col0 + lr;
            const float2 *src = G + (size_t)gr * K + k0 + kh;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                int gk = k0 + kh + u;
                float2 g = make_float2(0.f, 0.f);
                if (gr < n && gk < kend) g = src[u];
                b_re[kh + u][lr] = g.x;
                b_im[kh + u][lr] = g.y;
            }
        }
        __syncthreads();
#pragma unroll
        for (int kp = 0; kp < FW_BK / 2; ++kp) {
            int k = 2 * kp + (lane >> 5);
            float ar[2], ai[2], nai[2], br[2], bi[2];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                int m = wm * 64 + mt * 32 + (lane & 31);
                ar[mt] = a_re[k][m];
                ai[mt] = a_im[k][m];
                nai[mt] = -ai[mt];
            }
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                int cn = wn * 64 + nt * 32 + (lane & 31);
                br[nt] = b_re[k][cn];
                bi[nt] = b_im[k][cn];
            }
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) {
                    acc_re[mt][nt] = mfma32(ar[mt], br[nt], acc_re[mt][nt]);
                    acc_re[mt][nt] = mfma32(nai[mt], bi[nt], acc_re[mt][nt]);
                    acc_im[mt][nt] = mfma32(ar[mt], bi[nt], acc_im[mt][nt]);
                    acc_im[mt][nt] = mfma32(ai[mt], br[nt], acc_im[mt][nt]);
                }
        }
        __syncthreads();
    }
    float2 *out = dpart + (size_t)split * n * n;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            int gc = col0 + wn * 64 + nt * 32 + (lane & 31);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                int gr = row0 + wm * 64 + mt * 32 + mfma_row(lane, i);
                if (gr < n && gc < n)
                    out[(size_t)gr * n + gc] = make_float2(acc_re[mt][nt][i], acc_im[mt][nt][i]);
            }
        }
}

}  // namespace

int rb_rowred_mblocks(int n) { return (n + RR_BM - 1) / RR_BM; }

// R's fragments fit one buffer descriptor, and a lane's offset of four rows of B 32 bits.
static bool rowred_split_fits(int n, int n_mask) {
    return split_residual_bytes(n) <= (size_t)0xfffffff0u && n_mask <= 1 << 26;
}

// R in parts and the head; R' for the FP32 kernel in the place of the parts, which are done with by
// then (alone where there are none).
size_t rb_rowred_ws_bytes(int n) {
    return rowred_split_fits(n, 1)
               ? rb_align(split_residual_bytes(n)) + rb_align(sizeof(SplitHead))
               : rb_align((size_t)n * n * sizeof(float2));
}

// Split operands where the scratch holds R's; else (and for values that the split form turns
// down) the FP32 kernel. That alone also where a CU's column blocks take three of its K steps at
// most: the split form has two launches more (us, FP32 / split: 4000 nodes, back-projections of 16
// transducers 30.6 / 39.4, of 17 44.8 / 39.1, adjoints of 32 21.3 / 24.5, of 48 30.1 / 29.3, of 49
// 41.8 / 30.2; 40 000 nodes, back-projection of 16 79 / 69, adjoint of 16 32.1 / 35.7, of 17 46.3 /
// 35.4).
rb_status rb_launch_rowred(rb_ctx *ctx, int n, int n_mask, const float *R, const float *B,
                           int n_comp, int conj_b, void *scratch, size_t scratch_bytes,
                           float *parts, int *mblocks_out) {
    const int mblocks = rb_rowred_mblocks(n);
    const int grid = std::max(8, ctx->n_cu / 8 * 8);  // one workgroup per CU (persistent)
    const int np = rb_lp_pad(n);
    const size_t nn = (size_t)n * n;
    if (scratch_bytes < nn * sizeof(float2))
        return rb_fail(ctx, RB_EINVAL, "no room for the symmetric residual");
    SplitHead *head = nullptr;
    rb_prof_begin(ctx, ST_BACKPROJECT);
    const int nblocks = (n_mask + RR_BN - 1) / RR_BN;
    const long ksteps = (n + RR_BK - 1) / RR_BK, rounds = (nblocks + grid - 1) / grid;
    const bool brief = n_comp * ksteps * rounds <= 3;
    if (!brief && rowred_split_fits(n, n_mask) && scratch_bytes >= rb_rowred_ws_bytes(n)) {
        __bf16 *Rf = static_cast<__bf16 *>(scratch);
        head = reinterpret_cast<SplitHead *>(static_cast<char *>(scratch) +
                                             rb_align(split_residual_bytes(n)));
        RB_TRY(rb_launch_fill_i32(ctx, reinterpret_cast<int32_t *>(head), sizeof(SplitHead) / 4,
                                  0));
        hipLaunchKernelGGL(split_residual_kernel, dim3((np + 63) / 64, split_rows(n) / 32),
                           dim3(256), 0, ctx->stream, (const float2 *)R, n, np, head, Rf);
        RB_CHECK_LAUNCH(ctx);
        hipLaunchKernelGGL(rowred_split_kernel, dim3(grid), dim3(SR_THREADS), 0, ctx->stream, Rf,
                           (const float2 *)B, n, np, n_mask, n_comp, conj_b, mblocks,
                           (n_mask + SR_BN - 1) / SR_BN, head, parts);
        RB_CHECK_LAUNCH(ctx);
    }
    float2 *Rs = static_cast<float2 *>(scratch);
    hipLaunchKernelGGL(sym_upper_kernel, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0,
                       ctx->stream, (const float2 *)R, n, head, Rs);
    RB_CHECK_LAUNCH(ctx);
    hipLaunchKernelGGL(rowred_kernel, dim3(grid), dim3(256), 0, ctx->stream, Rs,
                       (const float2 *)B, n, n_mask, n_comp, conj_b, mblocks,
                       nblocks, head, parts);
    RB_CHECK_LAUNCH(ctx);
    rb_prof_end(ctx);
    if (mblocks_out) *mblocks_out = mblocks;
    return RB_OK;
}

int rb_forward_default_splitk(int n, int n_mask, int n_cu) {
    return rb_fwd::make_shape(n, n_mask, FW_BK, n_cu, 0).splitk;
}

// Workspace of the FP32 forward: partial sums, the scaled weights and their partial maxima, the
// head.
static size_t forward_bytes(int n, int K, int splitk) {
    return rb_align((size_t)splitk * n * n * sizeof(float2)) +
           rb_align((size_t)K * sizeof(float2)) + rb_align(FS_PARTS * sizeof(uint32_t)) +
           rb_align(sizeof(SplitHead));
}

size_t rb_forward_ws_bytes(int n, int n_mask) {
    const int T = (n + FW_B - 1) / FW_B;
    return forward_bytes(n, n_mask,
                         std::max(RB_TUNE_SPLITK_MAX, rb_fwd::splitk_most(T * (T + 1) / 2)));
}

// Split operands; the FP32 kernel after them for what they turn down. That alone where the nodes
// are few: the split form has up to four launches more, and its eight K chunks write eight partial
// sums (us without weights, FP32 / split: 300 transducers, 32 nodes 17.2 / 19.6, 33 22.2 / 19.1;
// 1500 transducers, 128 nodes 50.1 / 62.0, 256 83.4 / 69.0; 2000, 128 81.0 / 89.6, 192 97.8 /
// 89.1).
rb_status rb_launch_forward(rb_ctx *ctx, const rb_green *gr, const float *w, const float *delta,
                            float *d, const float *gscale) {
    const int n = gr->n, K = gr->n_mask;
    const rb_tuning *t = rb_tuned(ctx, n, K, RB_F32);
    const bool brief = K <= (n > 1024 ? 160 : 32);
    const int want = t ? t->fwd_splitk : brief ? std::max(1, (K + FW_BK - 1) / FW_BK / 4) : 0;
    const rb_fwd::Shape s = rb_fwd::make_shape(n, K, FW_BK, ctx->n_cu, want);
    ctx->ws.used = 0;
    RB_TRY(rb_arena_reserve(ctx, &ctx->ws, forward_bytes(n, K, s.splitk)));
    float2 *dpart = rb_carve<float2>(&ctx->ws, (size_t)s.splitk * n * n);
    float2 *v = rb_carve<float2>(&ctx->ws, K);
    uint32_t *vmax = rb_carve<uint32_t>(&ctx->ws, FS_PARTS);
    SplitHead *head = brief ? nullptr : rb_carve<SplitHead>(&ctx->ws, 1);
    const float2 *G = (const float2 *)gr->G, *wp = (const float2 *)w;
    const unsigned reduce_grid = rb_fwd::reduce_grid(n);
    auto launch = [&](auto op) {
        hipLaunchKernelGGL(rb_fwd::forward_reg_kernel<decltype(op)>, dim3(rb_fwd::grid_of(s)),
                           dim3(rb_fwd::FTHREADS), 0, ctx->stream, op, s, dpart);
    };
    rb_prof_begin(ctx, ST_FORWARD);
    if (!brief) {
        if (w) {
            hipLaunchKernelGGL(weight_max_kernel, dim3(FS_PARTS), dim3(256), 0, ctx->stream, K, wp,
                               delta, vmax);
            RB_CHECK_LAUNCH(ctx);
        }
        const int kw = w ? K : 0;
        hipLaunchKernelGGL(weight_scale_kernel, dim3(kw ? (kw + 255) / 256 : 1), dim3(256), 0,
                           ctx->stream, kw, wp, delta, vmax, v, head);
        RB_CHECK_LAUNCH(ctx);
        if (w) launch(SplitFwd<true>{G, v, head});
        else launch(SplitFwd<false>{G, v, head});
        RB_CHECK_LAUNCH(ctx);
        rb_prof_end(ctx);
        rb_prof_begin(ctx, ST_FORWARD_REDUCE);
        // the operand may carry sqrt(v) gscale[0]
        hipLaunchKernelGGL(rb_fwd::reduce_kernel<SplitCheck>, dim3(reduce_grid), dim3(256), 0,
                           ctx->stream, dpart, n, s.splitk, gscale, 2, (const float *)nullptr,
                           SplitCheck{head}, (float2 *)d);
        RB_CHECK_LAUNCH(ctx);
    }
    hipLaunchKernelGGL(forward_kernel, dim3(s.tiles, s.splitk), dim3(256), 0, ctx->stream, G, wp,
                       delta, n, K, s.nT, s.kchunk * FW_BK, head, dpart);
    RB_CHECK_LAUNCH(ctx);
    if (brief) {
        rb_prof_end(ctx);
        rb_prof_begin(ctx, ST_FORWARD_REDUCE);
    }
    hipLaunchKernelGGL(rb_fwd::reduce_kernel<PlainCheck>, dim3(reduce_grid), dim3(256), 0,
                       ctx->stream, dpart, n, s.splitk, gscale, 2, (const float *)nullptr,
                       PlainCheck{head}, (float2 *)d);
    RB_CHECK_LAUNCH(ctx);
    rb_prof_end(ctx);
    return RB_OK;
}
