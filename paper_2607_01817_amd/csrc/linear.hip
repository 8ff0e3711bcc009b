// Projection GEMM for gfx950 (MI355X), bf16 MFMA with fp32 accumulation:
//   Y[m][n] = sum_k X[m][k] W[n][k]       X [M][K], W [N][K], Y [M][N]
// i.e. Y = X W^T with the weight stored [out][in].  It is the QKV projection
// before the split along heads and the output projection after the
// concatenation (Alg. 1, the main-stream steps around the chunk loop).
//
// Two epilogues.  The plain one stores Y.  The QKV one splits Y's columns
// n = z H d + h d + e into three [M][H][d] tensors (z = 0, 1, 2: queries, keys,
// values) and rotates the query and key pairs (e, e + 1), e even, by the rotary
// position embedding of token m on its latent grid (RoFormer's rotation; the
// pairs of a head vector form consecutive groups, each turning with one grid
// axis), in fp32 before the rounding to the storage type: the split along
// heads and the position embedding fused into the producing kernel.
//
// Work decomposition
//   * one workgroup computes a BM (m) x BN (n) tile of Y: 256 x 256 with 8
//     waves where that fills the CUs, down to 64 x 64 with 4 (pick_tile); the
//     waves share it as WM x WN rectangles of 32 x 32 MFMA tiles.  Whatever
//     the tile, every element sums its products in the order of k, so all
//     tiles give the same bits;
//   * both operands are K-contiguous rows, which is the operand layout of
//     v_mfma_f32_32x32x16_bf16 (8 consecutive k per lane), so neither needs a
//     transpose: the MFMA computes Y^T tiles, D[n][m] = sum_k W[n][k] X[m][k],
//     with W rows as the A operand and X rows as the B operand.  Each lane
//     then holds one row m and, per 32 x 32 tile, 4 runs of 4 consecutive
//     columns n: whole rotation pairs; the output goes through LDS so that
//     it leaves as 16-byte stores covering whole row segments;
//   * k advances in stages of 128 bytes per row (64 columns of bf16, 32 of
//     fp32), which go from global memory straight into one of ST LDS buffers
//     (buffer_load_dwordx4 ... lds) a stage or more ahead; fp32 operands are
//     rounded to bf16 when they are read from LDS;
//   * one barrier per stage, placed where the operands of the stage's last
//     k-step are already in registers: it frees that stage's buffer and hands
//     over the next one, and the MFMAs behind it need neither.  Before, the
//     operand reads followed the barrier and the blocks passed through
//     registers: 8192 x 8192 x 8192 took 925 us (1188 TFLOP/s), 56160 x 1920 x
//     5120 1056, 56160 x 5120 x 640 406; now 797, 942 and
//     352.  What bounds it now: the power limit (1.7 GHz with the matrix
//     cores 78 % busy on 8192 x 8192 x 4096, 396 us; an MFMA loop with the
//     same LDS reads on random operands reaches 1710 TFLOP/s), and on short
//     reductions of outputs that the last-level cache does not hold the
//     writes: 40000 x 4096 x 192 takes 111 us, 107 before, 40000 x 4008 x
//     192, whose rows begin inside cache lines, 126 and 107;
//   * tiles are ordered in groups of 8 row tiles (all column tiles of a group
//     before the next group); workgroups are persistent, each round of the
//     grid takes the next G tiles of that order, and the 8 XCDs each take a
//     contiguous range of a round, so the 32 workgroups resident on an XCD
//     share 8 X panels and 4 W panels through its L2;
//   * a workgroup's tiles form one stream of stages, so the next tile's first
//     stages load during the current tile's last ones and its epilogue.
//
// Tails: rows past M or N are read through buffer resources bounded by the
// last row, so they read as zeros; rows past M and columns past N are not
// stored.  K must be a multiple of 64 and N of 8 (checked by the caller).
#include <type_traits>

#include "attention_tiles.h"
#include "hcms_internal.h"
#include "linear_tiles.h"

namespace hcms {
namespace {

using namespace tiles;

typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kGroupM = 8;               // row tiles per group of the tile order

// One workgroup's tile: BM rows of X by BN rows of W, WM x WN waves, ST stages
// of LDS.  A stage holds 128 bytes of every row: kBK columns.
template <int BM_, int BN_, int WM_, int WN_, int ST_, int PER_CU_>
struct Tile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, ST = ST_, PER_CU = PER_CU_;
    static constexpr int W = WM * WN, THREADS = 64 * W;
    static constexpr int MT = BM / WM / 32, NT = BN / WN / 32;   // 32 x 32 tiles per wave
    static constexpr int XL = BM / 8 / W, WL = BN / 8 / W;       // loads per wave and stage
    static constexpr int STAGE_B = (BM + BN) * 128;
    static constexpr int OUT_B = 4096;                           // output staging per wave
    static constexpr int LDS_B = ST * STAGE_B + W * OUT_B;
    static_assert(XL * 8 * W == BM && WL * 8 * W == BN && W % 2 == 0, "whole loads per wave");
    static_assert(LDS_B * PER_CU <= 160 * 1024 && ST >= 2, "LDS of a CU");
};

// Arguments of the QKV epilogue: destinations, and the rotation (table NULL:
// no rotation).  table holds (cos, sin) pairs; axis a, coordinate c, pair i'
// of the axis's group is entry tab_off[a] + c * pairs[a] + i'.
template <typename T>
struct QkvOut {
    T *dst[3];
    const float *table;
    int H, d;
    RopeAxes ax;
};
template <typename T>
using QkvArgs = __attribute__((address_space(4))) const QkvOut<T>;

// Resource over [base, base + min(bytes, 2^32 - 1)).
__device__ inline __amdgpu_buffer_rsrc_t span_rsrc(const void *base, int64_t bytes) {
    const int64_t n = bytes < 0 ? 0 : (bytes > 0xFFFFFFFFll ? 0xFFFFFFFFll : bytes);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0,
                                             static_cast<int>(static_cast<uint32_t>(n)), 0x00020000);
}

// Output of one wave's MT x NT tiles at rows mb .., columns nb .. of Y.  Lane
// (li, g) holds token mb + 32 mt + li and, per 32 x 32 tile, runs of 4
// consecutive features 8 rb + 4 g.  Runs of 8 bytes, 32 rows apart, coalesce
// badly, so the wave passes its part through a private 4 KiB of LDS, 32 tokens
// by 128 bytes at a time, and stores whole 128-byte row segments, 16 bytes per
// lane.  Chunk c of staged row r sits at position c ^ (r % 8).
template <typename T, bool QKV, typename C>
__device__ inline void store_tile(f32x16 (&acc)[C::NT][C::MT], char *stage, T *y, QkvArgs<T> *qp,
                                  int mb, int nb, int M, int N, int lane) {
    constexpr int MT = C::MT, NT = C::NT;
    constexpr int kSeg = sizeof(T) == 2 ? (NT % 2 == 0 ? 2 : 1) : 1;   // 32-column tiles per segment
    constexpr int kChunks = kSeg * 32 * sizeof(T) / 16;                // 16-byte chunks per staged row
    constexpr int kRows = 64 / kChunks;                                // rows per store instruction
    const int li = lane & 31, g = lane >> 5;
    const int hd = qp->H * qp->d;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        int tab_row[kRopeMaxAxes] = {};
        // The head element of the next 8 aligned columns.  Opaque, so that the
        // compiler steps it instead of keeping all of a row's in registers.
        int e8 = 0, n8 = 0;
        if constexpr (QKV) {
            n8 = nb;
            asm volatile("" : "+s"(n8));
            e8 = n8 % qp->d;
            // Per grid axis, the table entry of pair 0 of the axis at the
            // token's coordinate.
            if (qp->table != nullptr) {
                int rest = min(mb + mt * 32 + li, M - 1);
                for (int a = qp->ax.n_axes - 1; a >= 0; --a) {
                    const int cc = rest % qp->ax.grid[a];
                    rest /= qp->ax.grid[a];
                    tab_row[a] = qp->ax.tab_off[a] + cc * qp->ax.pairs[a] - qp->ax.pair_start[a];
                }
            }
        }
#pragma unroll
        for (int sg = 0; sg < NT / kSeg; ++sg) {
#pragma unroll
            for (int h = 0; h < kSeg; ++h)
#pragma unroll
                for (int rb = 0; rb < 4; ++rb) {
                    const f32x16 &t = acc[sg * kSeg + h][mt];
                    f32x4 v = {t[rb * 4 + 0], t[rb * 4 + 1], t[rb * 4 + 2], t[rb * 4 + 3]};
                    if constexpr (QKV) {
                        // Features of 8 aligned columns share q / k / v and
                        // head (N, H d and d are multiples of 8), the same
                        // for the whole wave.
                        if (qp->table != nullptr && n8 < 2 * hd) {
                            const int e = e8 + g * 4;
#pragma unroll
                            for (int q2 = 0; q2 < 2; ++q2) {
                                const int p = e / 2 + q2;
                                int row = tab_row[0];
#pragma unroll
                                for (int a = 1; a < kRopeMaxAxes; ++a)
                                    if (a < qp->ax.n_axes && p >= qp->ax.pair_start[a]) row = tab_row[a];
                                const f32x2 cs = *reinterpret_cast<const f32x2 *>(qp->table + 2 * (row + p));
                                const float x0 = v[2 * q2], x1 = v[2 * q2 + 1];
                                v[2 * q2] = __builtin_fmaf(x0, cs[0], -(x1 * cs[1]));
                                v[2 * q2 + 1] = __builtin_fmaf(x0, cs[1], x1 * cs[0]);
                            }
                        }
                        n8 += 8;
                        e8 = e8 + 8 == qp->d ? 0 : e8 + 8;
                        asm volatile("" : "+s"(n8), "+s"(e8));
                    }
                    if constexpr (sizeof(T) == 2) {
                        const int c = h * 4 + rb;
                        *reinterpret_cast<bf16x4 *>(stage + li * kChunks * 16 +
                                                    ((c ^ (li & (kChunks - 1))) << 4) + g * 8) =
                            __builtin_convertvector(v, bf16x4);
                    } else {
                        const int c = rb * 2 + g;
                        *reinterpret_cast<f32x4 *>(stage + li * kChunks * 16 + ((c ^ (li & (kChunks - 1))) << 4)) = v;
                    }
                }
            // The lane's chunk of each staged row: 16 / sizeof(T) features.
            const int ch = lane & (kChunks - 1);
            const int n = nb + sg * kSeg * 32 + ch * (16 / static_cast<int>(sizeof(T)));
            T *col;
            int64_t ld;
            if constexpr (QKV) {
                const int z = n >= 2 * hd ? 2 : n >= hd ? 1 : 0;
                col = qp->dst[z] + (n - z * hd);
                ld = hd;
            } else {
                col = y + n;
                ld = N;
            }
            u32x4 o[32 / kRows];
#pragma unroll
            for (int q = 0; q < 32 / kRows; ++q) {
                const int row = q * kRows + lane / kChunks;
                o[q] = *reinterpret_cast<const u32x4 *>(stage + row * kChunks * 16 + ((ch ^ (row & (kChunks - 1))) << 4));
            }
#pragma unroll
            for (int q = 0; q < 32 / kRows; ++q) {
                const int mm = mb + mt * 32 + q * kRows + lane / kChunks;
                if (mm < M && n < N) *reinterpret_cast<u32x4 *>(col + static_cast<int64_t>(mm) * ld) = o[q];
            }
        }
    }
}

// Operand of k-step ks, 8 consecutive k of one row, from a staged row (128
// bytes, 16-byte chunk c at position c ^ swizzle); `off` is the lane's offset
// of k-step 0.  fp32 in LDS takes two chunks and is rounded to bf16.
__device__ inline bf16x8 operand(const char *p, unsigned off, int ks, const __bf16 *) {
    return *reinterpret_cast<const bf16x8 *>(p + (off ^ (ks << 5)));
}
__device__ inline bf16x8 operand(const char *p, unsigned off, int ks, const float *) {
    const f32x4 a = *reinterpret_cast<const f32x4 *>(p + (off ^ (ks << 6)));
    const f32x4 b = *reinterpret_cast<const f32x4 *>(p + (off ^ (ks << 6) ^ 16));
    const f32x8 x = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_convertvector(x, bf16x8);
}

template <typename T, bool QKV, typename C>
__global__ __launch_bounds__(C::THREADS, C::PER_CU *C::W / 4) void linear_kernel(
    QkvOut<T> qo, const T *__restrict__ x, const T *__restrict__ w, T *__restrict__ y, int M, int N,
    int K, int tiles_m, int tiles_n) {
    constexpr int MT = C::MT, NT = C::NT, ST = C::ST, W = C::W;
    // fp32 storage on the tiles with two stages: through registers, rounded
    // to bf16 on the way into LDS, so that a stage holds 64 columns and twice
    // as many bytes are in flight as the buffers could take; from HBM, whose
    // latency a stage of 32 columns does not cover, 4096 x 4096 x 8192 took
    // 471 us without it.
    constexpr bool kReg = sizeof(T) == 4 && ST == 2;
    using L = std::conditional_t<kReg, __bf16, T>;   // element type in LDS
    constexpr int kBK = 128 / sizeof(L);   // columns per stage
    constexpr int KS = kBK / 16;           // MFMA k-steps per stage
    constexpr int LPW = C::XL + C::WL;     // loads per wave and stage
    constexpr int kHalf = kReg ? LPW : (LPW + 1) / 2;   // of them right behind the barrier
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS_B];

    const int G = gridDim.x, b = blockIdx.x;
    const int xcd = b & 7, per = G >> 3, rem = G & 7;
    const int slot = xcd * per + min(xcd, rem) + (b >> 3);
    const int n_tiles = tiles_m * tiles_n;
    if (slot >= n_tiles) return;
    const int n_mine = (n_tiles - 1 - slot) / G + 1;
    auto origin = [&](int r, int &m0, int &n0) {
        const int L = r * G + slot;
        const int group = L / (kGroupM * tiles_n);
        const int first_m = group * kGroupM;
        const int gm = min(tiles_m - first_m, kGroupM);
        const int in_group = L - group * kGroupM * tiles_n;
        m0 = (first_m + in_group % gm) * C::BM;
        n0 = (in_group / gm) * C::BN;
    };

    const unsigned row_bytes = static_cast<unsigned>(K) * sizeof(T);
    auto x_rsrc = [&](int m0) {
        return span_rsrc(x + static_cast<int64_t>(m0) * K, static_cast<int64_t>(M - m0) * row_bytes);
    };
    auto w_rsrc = [&](int n0) {
        return span_rsrc(w + static_cast<int64_t>(n0) * K, static_cast<int64_t>(N - n0) * row_bytes);
    };

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, g = lane >> 5;
    const int wm = wave / C::WN, wn = wave % C::WN;

    // Load i of a wave brings rows 8 (i W + wave) + lane / 8 of the stage's X
    // rows (then of its W rows), 16 bytes per lane; the lane at position
    // lane % 8 of its row fetches chunk (lane % 8) ^ swizzle(row), swizzle(r) =
    // (r / 2) % 8, so that 16 rows of one chunk lie in 16 different groups of
    // 4 banks.
    const unsigned voff = (8 * wave + (lane >> 3)) * row_bytes +
                          (((lane & 7) ^ ((4 * wave + (lane >> 4)) & 7)) << (kReg ? 5 : 4));
    const unsigned pass_bytes = 8 * W * row_bytes;
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>(lds));

    // The stages of the workgroup's tiles form one stream.  A stage past its
    // end is loaded through empty resources: zeros into a buffer that nobody
    // reads, so that every step issues the same number of loads.
    const int nkb = K / kBK;   // K is a multiple of 64
    int ld_r = 0, ld_kb = 0;
    int lm0, ln0;
    origin(0, lm0, ln0);
    __amdgpu_buffer_rsrc_t lxs = x_rsrc(lm0), lws = w_rsrc(ln0);
    // kReg: the fp32 values of the lane's chunk of every load, and their way
    // into LDS.
    f32x4 raw[kReg ? LPW : 1][2];
    auto store_raw = [&](int buf) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const f32x8 v = __builtin_shufflevector(raw[i][0], raw[i][1], 0, 1, 2, 3, 4, 5, 6, 7);
            *reinterpret_cast<bf16x8 *>(lds + buf * C::STAGE_B + (i * W + wave) * 1024 + lane * 16) =
                __builtin_convertvector(v, bf16x8);
        }
    };
    auto load_one = [&](int i, int buf) {
        if constexpr (kReg) {
            const __amdgpu_buffer_rsrc_t rs = i < C::XL ? lxs : lws;
            const unsigned so = ld_kb * 256 + (i < C::XL ? i : i - C::XL) * pass_bytes;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                raw[i][h] = __builtin_bit_cast(
                    f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 16 * h, so, 0));
            return;
        }
        const unsigned dst = lds0 + buf * C::STAGE_B + (i * W + wave) * 1024;
        const unsigned soff = ld_kb * 128;
        if (i < C::XL) load_lds(dst, lxs, voff, soff + i * pass_bytes);
        else load_lds(dst, lws, voff, soff + (i - C::XL) * pass_bytes);
    };
    auto advance = [&]() {
        if (++ld_kb < nkb) return;
        ld_kb = 0;
        if (++ld_r < n_mine) {
            origin(ld_r, lm0, ln0);
            lxs = x_rsrc(lm0);
            lws = w_rsrc(ln0);
        } else {
            lxs = span_rsrc(x, 0);
            lws = span_rsrc(w, 0);
        }
    };

    const unsigned rd = li * 128 + (((sizeof(L) == 2 ? g : 2 * g) ^ ((li >> 1) & 7)) << 4);
    const char *const xrd = lds + wm * MT * 32 * 128;
    const char *const wrd = lds + C::BM * 128 + wn * NT * 32 * 128;

    f32x16 acc[NT][MT];
    bf16x8 a[2][NT], bx[2][MT];
    auto read_ops = [&](int set, int ks, int buf) {
        const int base = buf * C::STAGE_B;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
            a[set][nt] = operand(wrd + base + nt * 32 * 128, rd, ks, static_cast<const L *>(nullptr));
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            bx[set][mt] = operand(xrd + base + mt * 32 * 128, rd, ks, static_cast<const L *>(nullptr));
    };
    auto mfma = [&](int set, int i) {
        const int nt = i / MT, mt = i % MT;
        acc[nt][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[set][nt], bx[set][mt], acc[nt][mt], 0, 0, 0);
    };

#pragma unroll
    for (int st = 0; st < ST; ++st) {
        const int n = st < ST - 1 ? LPW : kHalf;
#pragma unroll
        for (int i = 0; i < LPW; ++i)
            if (i < n) load_one(i, st);
        if constexpr (kReg)
            if (st < ST - 1) store_raw(st);
        if (st < ST - 1) advance();
    }
    if constexpr (!kReg) wait_vm<(ST - 2) * LPW + kHalf>();
    __syncthreads();
    read_ops(0, 0, 0);

    // MFMAs of operand set `set` with the loads l0 .. l1 - 1 into `into`.
    auto phase = [&](int set, int l0, int l1, int into) {
        constexpr int kMf = NT * MT;
#pragma unroll
        for (int i = 0; i < kMf; ++i) {
            mfma(set, i);
#pragma unroll
            for (int l = 0; l < LPW; ++l)
                if (l >= l0 && l < l1 && (l - l0) * kMf / (l1 - l0) == i) load_one(l, into);
            if (l0 < l1) __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int buf = 0, prev = ST - 1;
    for (int r = 0; r < n_mine; ++r) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = f32x16{};
        // End the scalar loads of the code before the loop: one that could
        // still be pending would turn the counted waits for the operand reads
        // of the first k-step into waits for all of them (simm16: lgkmcnt 0,
        // the others open).
        __builtin_amdgcn_s_waitcnt(0xC07F);
        for (int kb = 0; kb < nkb; ++kb) {
            // All but the stage's last k-step, each beside the operand reads
            // of the next; the first also issues the second half of the loads
            // into the buffer that the step before freed (all of them right
            // behind the barrier cost 2-3 %, thirds over three k-steps gained
            // nothing more).
#pragma unroll
            for (int ks = 0; ks + 1 < KS; ++ks) {
                read_ops((ks + 1) & 1, ks + 1, buf);
                __builtin_amdgcn_sched_barrier(0);
                phase(ks & 1, ks == 0 ? kHalf : LPW, LPW, prev);
                if (ks == 0) advance();
            }
            if constexpr (kReg) store_raw(prev);
            // The last k-step's operands are in registers: past this barrier
            // the stage's buffer is free and the next stage is in LDS, so the
            // last MFMAs run beside the first loads into the one and the first
            // operand reads of the other, and the matrix cores do not wait for
            // LDS after the barrier.
            if constexpr (!kReg) wait_vm<(ST - 2) * LPW>();
            __syncthreads();
            const int next = buf + 1 == ST ? 0 : buf + 1;
            read_ops(KS & 1, 0, next);
            __builtin_amdgcn_sched_barrier(0);
            phase((KS - 1) & 1, 0, kHalf, buf);
            prev = buf;
            buf = next;
        }
        static_assert(KS % 2 == 0, "the first k-step's operands are in set 0");
        int m0, n0;
        origin(r, m0, n0);
        // The QKV arguments are read from the kernel arguments here (qo is
        // the first), so that they hold no registers in the k-loop.
        QkvArgs<T> *qo_args = (QkvArgs<T> *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(qo_args));
        store_tile<T, QKV, C>(acc, lds + ST * C::STAGE_B + wave * C::OUT_B, y, qo_args, m0 + wm * MT * 32,
                              n0 + wn * NT * 32, M, N, lane);
    }
    wait_vm<0>();   // no load into LDS is pending when the workgroup ends
}

// Rotation table: entry e of axis a (tab_off[a] <= e < tab_off[a] + grid[a] *
// pairs[a]) is (cos, sin) of c * base^(-i' / pairs[a]), c = (e - tab_off[a]) /
// pairs[a], i' = (e - tab_off[a]) % pairs[a]; computed in fp64, rounded to fp32.
__global__ __launch_bounds__(256) void rope_table_kernel(float *table, RopeAxes ax, double base,
                                                         int total) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    int a = 0;
    while (a + 1 < ax.n_axes && e >= ax.tab_off[a + 1]) ++a;
    const int rel = e - ax.tab_off[a];
    const int c = rel / ax.pairs[a], ip = rel % ax.pairs[a];
    const double ang = static_cast<double>(c) *
                       pow(base, -static_cast<double>(ip) / static_cast<double>(ax.pairs[a]));
    table[2 * e] = static_cast<float>(cos(ang));
    table[2 * e + 1] = static_cast<float>(sin(ang));
}

template <typename T, bool QKV, typename C>
hipError_t launch_tile(const T *x, const T *w, T *y, int M, int N, int K, const QkvOut<T> &qo,
                       int n_cu, hipStream_t stream) {
    const int tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    const int64_t tiles = static_cast<int64_t>(tiles_m) * tiles_n;
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    // Persistent workgroups, whose tiles stream without a pipeline refill: on
    // 56160 x 1920 x 5120 923 us against 973 with one workgroup per tile, with
    // K = 640 and N = 5120 345 against 370.  Two workgroups per CU overlap
    // each other's refills and lose more to the fixed shares (8192 x 8192 x
    // 4096 907 against 764), except when the reduction is short.
    const int64_t slots = static_cast<int64_t>(n_cu) * C::PER_CU;
    const bool persist = tiles > slots && (C::PER_CU == 1 || K <= 1024);
    const int64_t blocks = persist ? slots : tiles;
    if (blocks < 1) return hipErrorInvalidValue;
    linear_kernel<T, QKV, C><<<static_cast<unsigned>(blocks), C::THREADS, 0, stream>>>(
        qo, x, w, y, M, N, K, tiles_m, tiles_n);
    return hipGetLastError();
}

// The tiles in the order of kTiles.
using TileA = Tile<256, 256, 4, 2, 2, 1>;
using TileB = Tile<192, 256, 2, 4, 2, 1>;
using TileC = Tile<256, 192, 4, 2, 2, 1>;
using TileD = Tile<128, 128, 4, 2, 4, 1>;
using TileE = Tile<64, 128, 2, 2, 4, 1>;
using TileF = Tile<64, 64, 2, 2, 4, 2>;
template <typename C>
constexpr bool costs_of(const TileCost &c) {
    return c.bm == C::BM && c.bn == C::BN && c.per_cu == C::PER_CU;
}
static_assert(costs_of<TileA>(kTiles[0]) && costs_of<TileB>(kTiles[1]) && costs_of<TileC>(kTiles[2]) &&
              costs_of<TileD>(kTiles[3]) && costs_of<TileE>(kTiles[4]) && costs_of<TileF>(kTiles[5]));

template <typename T, bool QKV>
hipError_t launch_typed(const void *x, const void *w, void *y, int M, int N, int K,
                        const QkvOut<T> &qo, hipStream_t stream) {
    int device = 0, n_cu = 0;
    hipError_t e = hipGetDevice(&device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return e;
    if (n_cu < 1) return hipErrorInvalidValue;
    auto run = [&](auto tile) {
        using C = decltype(tile);
        return launch_tile<T, QKV, C>(static_cast<const T *>(x), static_cast<const T *>(w),
                                      static_cast<T *>(y), M, N, K, qo, n_cu, stream);
    };
    switch (linear_tile(M, N, K, sizeof(T), QKV, n_cu)) {
        case 0:
            if constexpr (!(QKV && sizeof(T) == 4)) return run(TileA{});
            else break;
        case 1: return run(TileB{});
        case 2: return run(TileC{});
        case 3: return run(TileD{});
        case 4: return run(TileE{});
        case 5: return run(TileF{});
    }
    return hipErrorInvalidValue;
}

template <typename T>
QkvOut<T> qkv_out(void *q, void *k, void *v, const float *table, const RopeAxes &ax, int H, int d) {
    QkvOut<T> o{};
    o.dst[0] = static_cast<T *>(q);
    o.dst[1] = static_cast<T *>(k);
    o.dst[2] = static_cast<T *>(v);
    o.table = table;
    o.H = H;
    o.d = d;
    o.ax = ax;
    return o;
}

}  // namespace

int linear_k_multiple() { return 64; }

hipError_t launch_linear(const void *x, const void *w, void *y, int M, int N, int K, int dtype,
                         hipStream_t stream) {
    if (M == 0 || N == 0) return hipSuccess;
    if (dtype == 0) return launch_typed<__bf16, false>(x, w, y, M, N, K, QkvOut<__bf16>{}, stream);
    if (dtype == 1) return launch_typed<float, false>(x, w, y, M, N, K, QkvOut<float>{}, stream);
    return hipErrorInvalidValue;
}

hipError_t launch_qkv_projection(const void *x, const void *w, void *q, void *k, void *v,
                                 const float *table, const RopeAxes &ax, int S, int D, int H, int d,
                                 int dtype, hipStream_t stream) {
    if (S == 0) return hipSuccess;
    const int N = 3 * H * d;
    if (dtype == 0)
        return launch_typed<__bf16, true>(x, w, nullptr, S, N, D,
                                          qkv_out<__bf16>(q, k, v, table, ax, H, d), stream);
    if (dtype == 1)
        return launch_typed<float, true>(x, w, nullptr, S, N, D,
                                         qkv_out<float>(q, k, v, table, ax, H, d), stream);
    return hipErrorInvalidValue;
}

hipError_t launch_rope_table(float *table, const RopeAxes &ax, double base, hipStream_t stream) {
    const int last = ax.n_axes - 1;
    const int total = ax.tab_off[last] + ax.grid[last] * ax.pairs[last];
    if (total == 0) return hipSuccess;
    rope_table_kernel<<<(total + 255) / 256, 256, 0, stream>>>(table, ax, base, total);
    return hipGetLastError();
}

}  // namespace hcms
