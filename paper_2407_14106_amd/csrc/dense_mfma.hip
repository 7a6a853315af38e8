// Full softmax attention for bf16 features on the matrix cores: the
// interleaved fully-connected layer of §3.2 (every node attends to every node,
// Eq. (1) of §2.1), forward and backward, streaming over the keys with no
// n x n buffer.
//
// Design (CDNA4, wave64, v_mfma_f32_32x32x16_bf16):
//   - A workgroup owns the rows of 2 to 8 wavefronts of one head, 32 or (large
//     forwards) 64 rows each, so every operand fragment read from LDS feeds one
//     or two products; where a layer has few such blocks for the chip, a second
//     set of wavefronts takes half of the partners (FullShape).  The partner rows
//     stream through LDS in 64-row stages, double buffered: the next stage is
//     loaded straight into LDS while the current one is multiplied, with one
//     barrier per stage.
//   - Scores are formed transposed (partners x owned rows), so each lane holds
//     one owned row and 16 of its partners; per-row statistics need one
//     v_permlane32_swap between the half-waves.  The probabilities (or dS)
//     become the next product's B operand straight from the accumulators; the
//     A operand of that product (V^T, K^T, dO^T, Q^T) is read from the
//     row-major copy by transposing LDS reads.
//   - The forward's running maximum is lazy: the accumulators are rescaled only
//     when weights reach 2^8, so weights stay below 256 and the result is
//     unchanged.
//   - D_i = <dO_i, O_i> from the given O: every full-layer weight is O(1/n),
//     so no cancellation-prone sum over partners is needed.
//   - Workgroups are remapped so that each XCD works on one range of
//     (head, row block) pairs and shares that head's K and V in its L2.
//   - Measured at 65,536 x 8 x 64: forward 10.5 -> 8.6 ms (1,020 TFLOP/s, a large
//     bf16 matrix product reaches about 1,130 here), backward 34.0 -> 28.6 ms (the
//     seven products it forms run at 1,080 TFLOP/s); at 3,001 x 8 x 64 86 -> 41 and
//     205 -> 110 us.
#include "tile_attn.h"

namespace gt {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kStage = 64;               // partner rows per LDS stage
constexpr float kNegInf = -__builtin_huge_valf();
constexpr float kLazy = 8.f;             // lazy-max slack, exp2 domain

__device__ __forceinline__ int crow(int i, int lane) { return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3); }

// A compile-time flag passed as a value (generic lambdas take it as auto).
template <bool B>
struct Flag {
    static constexpr bool value = B;
};

__device__ __forceinline__ f32x16_t zero16() {
    f32x16_t z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}

__device__ __forceinline__ f32x16_t mma(bf16x8_t a, bf16x8_t b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The value of x held by the partner lane (lane ^ 32) combined with x.
__device__ __forceinline__ float pair_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Accumulator elements 8*half .. +7 as a bf16 B operand.
__device__ __forceinline__ bf16x8_t acc_b16(const f32x16_t& c, int half) {
    bf16x8_t o;
#pragma unroll
    for (int t = 0; t < 8; ++t) o[t] = (__bf16)c[8 * half + t];
    return o;
}

// B operand fragments of one owned row (global memory): features
// 16c + 8(lane/32) .. +7 for c < D/16; zero for rows >= n.
template <int D>
struct Frag {
    bf16x8_t v[D / 16];
    __device__ __forceinline__ void load(const uint16_t* X, int64_t row, int64_t n, int H, int h, int lane) {
        const int64_t src = row < n ? row : n - 1;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            uint4 x = *reinterpret_cast<const uint4*>(X + (src * H + h) * D + 16 * c + 8 * (lane >> 5));
            if (row >= n) x = make_uint4(0, 0, 0, 0);
            v[c] = __builtin_bit_cast(bf16x8_t, x);
        }
    }
    // this lane's share of <this, o>
    __device__ __forceinline__ float dot(const Frag& o) const {
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < D / 16; ++c)
#pragma unroll
            for (int t = 0; t < 8; ++t) s = fmaf(float(v[c][t]), float(o.v[c][t]), s);
        return s;
    }
};

// Make the exp2-domain scale positive, so that a score masked with -inf stays
// -inf when scaled: a negative scale negates the owned rows (exact in bf16), a
// zero scale becomes 1 on rows of zeros.
template <int D, int NB>
__device__ __forceinline__ void positive_scale(Frag<D> (&q)[NB], float& sl2) {
    if (!(sl2 <= 0.f)) return;
    const uint32_t keep = sl2 < 0.f ? ~0u : 0u, flip = sl2 < 0.f ? 0x80008000u : 0u;
    sl2 = sl2 < 0.f ? -sl2 : 1.f;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            uint4 x = __builtin_bit_cast(uint4, q[b].v[c]);
            x = make_uint4((x.x & keep) ^ flip, (x.y & keep) ^ flip, (x.z & keep) ^ flip, (x.w & keep) ^ flip);
            q[b].v[c] = __builtin_bit_cast(bf16x8_t, x);
        }
}

// --------------------------------------------------------- staged operands
// Partner rows are staged 64 at a time by loads that write LDS directly (no
// registers, no stores), one row-major copy of each operand, double buffered:
// the next stage's loads are issued before the current one is multiplied.  A
// row's 16-byte pieces are permuted by the row number (the loads place lane i
// at byte 16 i, so a lane picks the piece it fetches), which spreads the same
// piece of neighbouring rows over all LDS banks.  The row operand of a product
// is read as it lies; the transposed operand (features x partners) by
// ds_read_b64_tr_b16, which turns a 4 partners x 16 features block round.
template <int D>
struct Tile {
    static constexpr int kPieces = D / 8;                  // 16-byte pieces per row
    static constexpr int kElems = kStage * D;              // one staged operand
    static constexpr int kLoads = kElems * 2 / 1024;       // 1 KiB wavefront loads per operand
    __device__ __forceinline__ static int turn(int r) { return D == 64 ? r & 7 : (r >> 1) & 3; }

    // This wavefront's share of a stage of X[:, h, :], rows base .. base + 63
    // (rows past the end repeat the last one).
    template <int WAVES>
    __device__ __forceinline__ static void fetch(uint16_t* s, const uint16_t* __restrict__ X, int64_t base, int64_t n,
                                                 int H, int h, int wave, int lane) {
#pragma unroll
        for (int q0 = 0; q0 < kLoads; q0 += WAVES) {
            const int q = q0 + wave;
            if (q >= kLoads) break;  // uniform
            const int at = q * 64 + lane, r = at / kPieces, c = (at % kPieces) ^ turn(r);
            const int64_t left = n - 1 - base;
            const int row = r < left ? r : int(left);
            const uint16_t* src = X + (base * H + h) * D + int64_t(row * H) * D + 8 * c;
            __builtin_amdgcn_global_load_lds(
                reinterpret_cast<const __attribute__((address_space(1))) uint32_t*>(reinterpret_cast<uintptr_t>(src)),
                reinterpret_cast<__attribute__((address_space(3))) uint32_t*>(
                    reinterpret_cast<uintptr_t>(s + q * 512)),
                16, 0, 0);
        }
    }
    // Zero the rows past the end of a staged operand, for the same reason as drop_past_end; the whole workgroup, once
    // the stage is in LDS.  (The tiles' column pass has no use for it: its weights come in two parts, whose products
    // with an infinity cancel to NaN.)
    template <int THREADS>
    __device__ __forceinline__ static void zero_past_end(uint16_t* s, int64_t base, int64_t n) {
        if (__builtin_expect(base + kStage <= n, 1)) return;
        const int rows = n > base ? int(n - base) : 0;
        for (int q = rows * kPieces + int(threadIdx.x); q < kStage * kPieces; q += THREADS)
            *reinterpret_cast<uint4*>(s + 8 * q) = make_uint4(0, 0, 0, 0);
        __syncthreads();
    }
    // Row operand: row r, features 16 c + 8 (lane / 32) .. + 7.
    __device__ __forceinline__ static bf16x8_t rows(const uint16_t* s, int r, int c, int lane) {
        return __builtin_bit_cast(
            bf16x8_t, *reinterpret_cast<const uint4*>(s + r * D + 8 * ((2 * c + (lane >> 5)) ^ turn(r))));
    }
    // Transposed operand: feature 32 db + lane % 32; partners base + 4 (lane / 32) + {0..3} and base + 8 + 4 (lane
    // / 32) + {0..3}, the partner order of an accumulator-layout B operand (acc_b16).
    __device__ __forceinline__ static bf16x8_t cols(const uint16_t* s, int db, int base, int lane) {
        typedef short s16x4_t __attribute__((ext_vector_type(4)));
        const int k = 4 * (lane >> 5) + ((lane & 15) >> 2);
        const int c = (4 * db + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ turn(k);
        const uint16_t* p = s + (base + k) * D + 8 * c + 4 * (lane & 1);
        // turn(k + 8) = turn(k)
        const s16x4_t x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            reinterpret_cast<__attribute__((address_space(3))) s16x4_t*>(reinterpret_cast<uintptr_t>(p)));
        const s16x4_t y = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            reinterpret_cast<__attribute__((address_space(3))) s16x4_t*>(reinterpret_cast<uintptr_t>(p + 8 * D)));
        typedef short s16x8_t __attribute__((ext_vector_type(8)));
        return __builtin_bit_cast(bf16x8_t, s16x8_t{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]});
    }
};

// Zero what a transposed operand (features x the 32 partners of a block, Tile::cols at 0 and 16) holds of partners past
// the end: the staged rows there repeat the last node, and their zero weights times an infinity would be NaN.  Only a
// ragged last stage needs it (and the masks), so the forward and the column pass of the full layer have that stage
// apart from the loop (a branch in the loop cost a step of 16,384 x 8 x 32 2.3%; apart, within 0.5%).
template <int D>
__device__ __forceinline__ void drop_past_end(bf16x8_t (&a)[D / 32][2], int64_t first, int64_t n, int lane) {
    const int left = int(n - first) - 4 * (lane >> 5);
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int t = 0; t < 8; ++t)
            if (16 * half + 8 * (t / 4) + t % 4 >= left)
#pragma unroll
                for (int db = 0; db < D / 32; ++db) a[db][half][t] = (__bf16)0.f;
}

// The stage fetched last is in LDS for every wavefront, and every wavefront is done with the one before.
__device__ __forceinline__ void stage_done() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// Workgroup -> (head, first owned row); false for the padding of the grid.
template <int ROWS>
__device__ __forceinline__ bool wg_coords(int64_t n, int H, int& h, int64_t& row0) {
    const int64_t blocks = cdiv(n, ROWS);
    const int64_t b = xcd_block(blockIdx.x, gridDim.x);
    if (b >= blocks * H) return false;
    h = int(b / blocks);
    row0 = (b % blocks) * ROWS;
    return true;
}
template <int ROWS>
inline unsigned full_grid(int64_t n, int H) { return xcd_grid(cdiv(n, ROWS) * H); }

__device__ __forceinline__ f32x16_t splat16(float x) {
    f32x16_t z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = x;
    return z;
}

// Accumulators (features x owned rows) times `f` as bf16, one owned row's 8-byte pieces per lane.
template <int D>
__device__ __forceinline__ void store_acc(uint16_t* o, const f32x16_t (&a)[D / 32], float f, int lane) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            *reinterpret_cast<uint2*>(o + 32 * db + 8 * j + 4 * (lane >> 5)) =
                make_uint2(pack_bf16x2(a[db][4 * j] * f, a[db][4 * j + 1] * f),
                           pack_bf16x2(a[db][4 * j + 2] * f, a[db][4 * j + 3] * f));
}

// Where the partners of a stage are shared by KS = 2 sets of wavefronts: add
// the second set's accumulators to the first's (false for the second set).
template <int KS, int WAVES, int N>
__device__ __forceinline__ bool add_shares(f32x16_t* a, int part) {
    if constexpr (KS == 2) {
        __shared__ float s_x[N * 16][WAVES * kWave];
        const int at = int(threadIdx.x) % (WAVES * kWave);
        if (part == 1)
#pragma unroll
            for (int k = 0; k < N; ++k)
#pragma unroll
                for (int i = 0; i < 16; ++i) s_x[16 * k + i][at] = a[k][i];
        __syncthreads();
        if (part == 0)
#pragma unroll
            for (int k = 0; k < N; ++k)
#pragma unroll
                for (int i = 0; i < 16; ++i) a[k][i] += s_x[16 * k + i][at];
    }
    return part == 0;
}

// ------------------------------------------------------------------ forward
// The running reference m of a row is checked after the fact: a block's weights
// exp2(s - m) are summed anyway, and only where a lane's sum of 16 exceeds 2^8 (or is
// not a number, as from the first block's m = -inf) are the block's scores
// formed again, the true maximum taken and the accumulators rescaled.  Weights
// stay below 2^8 as with a maximum taken first, without its 16 vector
// operations a block.

template <int D, int NB, int WAVES, int KS>
__global__ __launch_bounds__(WAVES * KS * kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_full_fwd(
    int64_t n, int H, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    float sl2, uint16_t* __restrict__ O, float* __restrict__ LSE) {
    using Tl = Tile<D>;
    // one variable per buffer: the compiler then knows that a stage's reads do
    // not touch the buffer being filled, and does not wait for its loads
    __shared__ __attribute__((aligned(16))) uint16_t sK0[Tl::kElems], sK1[Tl::kElems];
    __shared__ __attribute__((aligned(16))) uint16_t sV0[Tl::kElems], sV1[Tl::kElems];
    int h;
    int64_t row0;
    if (!wg_coords<32 * NB * WAVES>(n, H, h, row0)) return;
    const int lane = lane_id(), wave = uniform(int(threadIdx.x) / kWave);
    const int part = KS == 1 ? 0 : wave / WAVES;  // which of a stage's KS shares of the partners
    const int64_t q0 = row0 + (wave - part * WAVES) * 32 * NB;
    Tl::template fetch<WAVES * KS>(sK0, K, 0, n, H, h, wave, lane);
    Tl::template fetch<WAVES * KS>(sV0, V, 0, n, H, h, wave, lane);
    Frag<D> qf[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) qf[b].load(Q, q0 + 32 * b + (lane & 31), n, H, h, lane);
    positive_scale<D, NB>(qf, sl2);
    f32x16_t acc[NB][D / 32];
    float m[NB], l[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int db = 0; db < D / 32; ++db) acc[b][db] = zero16();
        m[b] = kNegInf;
        l[b] = 0.f;
    }
    stage_done();
    const int64_t stages = cdiv(n, kStage);
    auto stage = [&](int64_t t, auto ragged, const uint16_t* cK, const uint16_t* cV, uint16_t* nK, uint16_t* nV) {
        const int64_t kbase = t * kStage;
        if (!ragged.value && t + 1 < stages) {
            Tl::template fetch<WAVES * KS>(nK, K, kbase + kStage, n, H, h, wave, lane);
            Tl::template fetch<WAVES * KS>(nV, V, kbase + kStage, n, H, h, wave, lane);
        }
#pragma unroll
        for (int kx = 0; kx < kStage / 32 / KS; ++kx) {
            const int kb = kx + part * (kStage / 32 / KS);
            const int64_t key0 = kbase + 32 * kb;
            if (ragged.value && KS > 1 && key0 >= n) break;  // no partner left for this share (its maximum may still be -inf)
            f32x16_t s[NB];
            auto scores = [&] {
#pragma unroll
                for (int b = 0; b < NB; ++b) s[b] = zero16();
#pragma unroll
                for (int c = 0; c < D / 16; ++c) {
                    const bf16x8_t a = Tl::rows(cK, 32 * kb + (lane & 31), c, lane);
#pragma unroll
                    for (int b = 0; b < NB; ++b) s[b] = mma(a, qf[b].v[c], s[b]);
                }
                if constexpr (ragged.value) {  // partners >= n take no weight
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (key0 + crow(i, lane) >= n)
#pragma unroll
                            for (int b = 0; b < NB; ++b) s[b][i] = kNegInf;
                }
            };
            float ls[NB];
            auto weights = [&] {  // s becomes the weights, ls this lane's sums of them
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    float x[2] = {0.f, 0.f};
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float p = ex2(fmaf(s[b][i], sl2, -m[b]));
                        s[b][i] = p;
                        x[i & 1] += p;
                    }
                    ls[b] = x[0] + x[1];
                }
            };
            scores();
            bf16x8_t vt[D / 32][2];
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int half = 0; half < 2; ++half) vt[db][half] = Tl::cols(cV, db, 32 * kb + 16 * half, lane);
            if constexpr (ragged.value) drop_past_end<D>(vt, key0, n, lane);
            __builtin_amdgcn_sched_barrier(0);
            weights();
            bool high = false;
#pragma unroll
            for (int b = 0; b < NB; ++b) high |= !(ls[b] <= 256.f);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(high) != 0, 0)) {
                scores();
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    float mx = s[b][0];
#pragma unroll
                    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[b][i]);
                    const float mn = fmaxf(m[b], pair_max(mx) * sl2);
                    const float alpha = ex2(m[b] - mn);
                    l[b] *= alpha;
#pragma unroll
                    for (int db = 0; db < D / 32; ++db)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[b][db][i] *= alpha;
                    m[b] = mn;
                }
                weights();
            }
            bf16x8_t pb[NB][2];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                l[b] += ls[b];
                pb[b][0] = acc_b16(s[b], 0);
                pb[b][1] = acc_b16(s[b], 1);
            }
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const bf16x8_t a = vt[db][half];
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b][db] = mma(a, pb[b][half], acc[b][db]);
                }
        }
        stage_done();
    };
    const int64_t whole = n / kStage;
    for (int64_t t = 0; t < whole; t += 2) {
        stage(t, Flag<false>{}, sK0, sV0, sK1, sV1);
        if (t + 1 < whole) stage(t + 1, Flag<false>{}, sK1, sV1, sK0, sV0);
    }
    if (whole < stages) stage(whole, Flag<true>{}, whole & 1 ? sK1 : sK0, whole & 1 ? sV1 : sV0, sK0, sV0);
    if constexpr (KS == 2) {  // the second share's states to the first's wavefronts
        __shared__ float s_x[NB * (16 * (D / 32) + 2)][WAVES * kWave];
        const int at = int(threadIdx.x) % (WAVES * kWave);
        if (part == 1) {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                float(*x)[WAVES * kWave] = s_x + b * (16 * (D / 32) + 2);
                x[0][at] = m[b];
                x[1][at] = l[b];
#pragma unroll
                for (int db = 0; db < D / 32; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) x[2 + 16 * db + i][at] = acc[b][db][i];
            }
        }
        __syncthreads();
        if (part == 1) return;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float(*x)[WAVES * kWave] = s_x + b * (16 * (D / 32) + 2);
            // a share without partners (n <= 32) leaves m = -inf and l = 0
            const float mo = x[0][at], mn = fmaxf(m[b], mo);
            const float w0 = ex2(m[b] - mn), w1 = ex2(mo - mn);
            m[b] = mn;
            l[b] = fmaf(x[1][at], w1, l[b] * w0);
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[b][db][i] = fmaf(x[2 + 16 * db + i][at], w1, acc[b][db][i] * w0);
        }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t q = q0 + 32 * b + (lane & 31);
        const float lt = pair_sum(l[b]);
        if (q >= n) continue;
        const float inv = lt > 0.f ? 1.f / lt : 0.f;
        if (lane < 32) LSE[q * H + h] = lt > 0.f ? (m[b] + __log2f(lt)) * kLn2 : kNegInf;
        store_acc<D>(O + (q * H + h) * D, acc[b], inv, lane);
    }
}

// ---------------------------------------------------------------- dQ (rows)
// dQ_i = scale sum_j P_ij (dP_ij - D_i) K_j with dP_ij = <dO_i, V_j>; also
// writes D_i for the column pass.  The dP products start from -D_i, so their
// sum is dP - D with no subtraction.

template <int D, int NB, int WAVES, int KS>
__global__ __launch_bounds__(WAVES * KS * kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_full_dq(
    int64_t n, int H, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    const uint16_t* __restrict__ O, const uint16_t* __restrict__ dO, const float* __restrict__ LSE, float sl2,
    float scale, uint16_t* __restrict__ dQ, float* __restrict__ Dv) {
    using Tl = Tile<D>;
    // one variable per buffer: the compiler then knows that a stage's reads do
    // not touch the buffer being filled, and does not wait for its loads
    __shared__ __attribute__((aligned(16))) uint16_t sK0[Tl::kElems], sK1[Tl::kElems];
    __shared__ __attribute__((aligned(16))) uint16_t sV0[Tl::kElems], sV1[Tl::kElems];
    int h;
    int64_t row0;
    if (!wg_coords<32 * NB * WAVES>(n, H, h, row0)) return;
    const int lane = lane_id(), wave = uniform(int(threadIdx.x) / kWave);
    const int part = KS == 1 ? 0 : wave / WAVES;  // which of a stage's KS shares of the partners
    const int64_t q0 = row0 + (wave - part * WAVES) * 32 * NB;
    Tl::template fetch<WAVES * KS>(sK0, K, 0, n, H, h, wave, lane);
    Tl::template fetch<WAVES * KS>(sV0, V, 0, n, H, h, wave, lane);
    Frag<D> qf[NB], gf[NB];
    float lse2[NB];
    f32x16_t nD[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t q = q0 + 32 * b + (lane & 31);
        qf[b].load(Q, q, n, H, h, lane);
        gf[b].load(dO, q, n, H, h, lane);
        Frag<D> of;
        of.load(O, q, n, H, h, lane);
        const float Dq = pair_sum(gf[b].dot(of));
        lse2[b] = q < n ? LSE[q * H + h] * kLog2e : 0.f;
        if (q < n && lane < 32) Dv[q * H + h] = Dq;
        nD[b] = splat16(-Dq);
    }
    f32x16_t acc[NB][D / 32];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int db = 0; db < D / 32; ++db) acc[b][db] = zero16();
    stage_done();
    const int64_t stages = cdiv(n, kStage);
    auto stage = [&](int64_t t, const uint16_t* cK, const uint16_t* cV, uint16_t* nK, uint16_t* nV) {
        const int64_t kbase = t * kStage;
        if (t + 1 < stages) {
            Tl::template fetch<WAVES * KS>(nK, K, kbase + kStage, n, H, h, wave, lane);
            Tl::template fetch<WAVES * KS>(nV, V, kbase + kStage, n, H, h, wave, lane);
        }
#pragma unroll
        for (int kx = 0; kx < kStage / 32 / KS; ++kx) {
            const int kb = kx + part * (kStage / 32 / KS);
            f32x16_t s[NB], dp[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                s[b] = zero16();
                dp[b] = nD[b];
            }
#pragma unroll
            for (int c = 0; c < D / 16; ++c) {
                const bf16x8_t a = Tl::rows(cK, 32 * kb + (lane & 31), c, lane);
                const bf16x8_t v = Tl::rows(cV, 32 * kb + (lane & 31), c, lane);
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    s[b] = mma(a, qf[b].v[c], s[b]);
                    dp[b] = mma(v, gf[b].v[c], dp[b]);
                }
            }
            const int64_t key0 = kbase + 32 * kb;
            if (__builtin_expect(key0 + 32 > n, 0)) {  // ragged last block: no dS for partners >= n
                // kept as a branch (the empty asm stops the compiler from turning
                // it into selects on every block)
                asm volatile("" ::: "memory");
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (key0 + crow(i, lane) >= n)
#pragma unroll
                        for (int b = 0; b < NB; ++b) dp[b][i] = 0.f;
            }
            bf16x8_t kt[D / 32][2];
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int half = 0; half < 2; ++half) kt[db][half] = Tl::cols(cK, db, 32 * kb + 16 * half, lane);
            __builtin_amdgcn_sched_barrier(0);
            bf16x8_t db16[NB][2];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
#pragma unroll
                for (int i = 0; i < 16; ++i) s[b][i] = ex2(fmaf(s[b][i], sl2, -lse2[b])) * dp[b][i];
                db16[b][0] = acc_b16(s[b], 0);
                db16[b][1] = acc_b16(s[b], 1);
            }
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const bf16x8_t a = kt[db][half];
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b][db] = mma(a, db16[b][half], acc[b][db]);
                }
        }
        stage_done();
    };
    for (int64_t t = 0; t < stages; t += 2) {
        stage(t, sK0, sV0, sK1, sV1);
        if (t + 1 < stages) stage(t + 1, sK1, sV1, sK0, sV0);
    }
    if (!add_shares<KS, WAVES, NB * (D / 32)>(&acc[0][0], part)) return;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t q = q0 + 32 * b + (lane & 31);
        if (q < n) store_acc<D>(dQ + (q * H + h) * D, acc[b], scale, lane);
    }
}

// ----------------------------------------------------------- dK, dV (cols)
// dK_j = scale sum_i P_ij (dP_ij - D_i) Q_i and dV_j = sum_i P_ij dO_i, with
// the wavefront owning 32 NB keys and the queries streaming through LDS; the dP
// products start from the queries' -D_i.

template <int D, int NB, int WAVES, int KS>
__global__ __launch_bounds__(WAVES * KS * kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_full_dkdv(
    int64_t n, int H, const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    const uint16_t* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ Dv, float sl2,
    float scale, uint16_t* __restrict__ dK, uint16_t* __restrict__ dV) {
    using Tl = Tile<D>;
    // one variable per buffer: the compiler then knows that a stage's reads do
    // not touch the buffer being filled, and does not wait for its loads
    __shared__ __attribute__((aligned(16))) uint16_t sQ0[Tl::kElems], sQ1[Tl::kElems];
    __shared__ __attribute__((aligned(16))) uint16_t sG0[Tl::kElems], sG1[Tl::kElems];
    __shared__ __attribute__((aligned(16))) float sL0[kStage], sL1[kStage];
    __shared__ __attribute__((aligned(16))) float sD0[kStage], sD1[kStage];
    int h;
    int64_t row0;
    if (!wg_coords<32 * NB * WAVES>(n, H, h, row0)) return;
    const int lane = lane_id(), wave = uniform(int(threadIdx.x) / kWave);
    const int part = KS == 1 ? 0 : wave / WAVES;  // which of a stage's KS shares of the queries
    const int64_t k0 = row0 + (wave - part * WAVES) * 32 * NB;
    // LSE (exp2 domain) and -D of the stage's queries, loaded a stage ahead by the
    // first wavefront and stored at the stage's end; queries >= n get
    // LSE = +inf so that their weights are exactly zero.
    float rl = 0.f, rd = 0.f;
    auto load_rows = [&](int64_t base) {
        if (wave == 0) {
            const int64_t qn = base + lane;
            rl = qn < n ? LSE[qn * H + h] * kLog2e : __builtin_huge_valf();
            rd = qn < n ? -Dv[qn * H + h] : 0.f;
        }
    };
    auto store_rows = [&](float* toL, float* toD) {
        if (wave == 0) {
            toL[lane] = rl;
            toD[lane] = rd;
        }
    };
    load_rows(0);
    Tl::template fetch<WAVES * KS>(sQ0, Q, 0, n, H, h, wave, lane);
    Tl::template fetch<WAVES * KS>(sG0, dO, 0, n, H, h, wave, lane);
    Frag<D> kf[NB], vf[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        kf[b].load(K, k0 + 32 * b + (lane & 31), n, H, h, lane);
        vf[b].load(V, k0 + 32 * b + (lane & 31), n, H, h, lane);
    }
    f32x16_t dk[NB][D / 32], dv[NB][D / 32];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int db = 0; db < D / 32; ++db) dk[b][db] = dv[b][db] = zero16();
    store_rows(sL0, sD0);
    stage_done();
    const int64_t stages = cdiv(n, kStage);
    auto stage = [&](int64_t t, auto ragged, const uint16_t* cQ, const uint16_t* cG, uint16_t* nQ, uint16_t* nG,
                     const float* cL, const float* cD, float* nL, float* nD) {
        const int64_t qbase = t * kStage;
        if (!ragged.value && t + 1 < stages) {
            load_rows(qbase + kStage);
            Tl::template fetch<WAVES * KS>(nQ, Q, qbase + kStage, n, H, h, wave, lane);
            Tl::template fetch<WAVES * KS>(nG, dO, qbase + kStage, n, H, h, wave, lane);
        }
#pragma unroll
        for (int kx = 0; kx < kStage / 32 / KS; ++kx) {
            const int qb = kx + part * (kStage / 32 / KS);
            // rows of accumulator element i: 32 qb + 8 (i/4) + 4 (lane/32) + i%4
            f32x16_t s[NB], dp[NB], mD;
            float Lr[16];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 32 * qb + 8 * j + 4 * (lane >> 5);
                const float4 lv = *reinterpret_cast<const float4*>(&cL[r]);
                const float4 dv4 = *reinterpret_cast<const float4*>(&cD[r]);
                Lr[4 * j] = lv.x, Lr[4 * j + 1] = lv.y, Lr[4 * j + 2] = lv.z, Lr[4 * j + 3] = lv.w;
                mD[4 * j] = dv4.x, mD[4 * j + 1] = dv4.y, mD[4 * j + 2] = dv4.z, mD[4 * j + 3] = dv4.w;
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                s[b] = zero16();
                dp[b] = mD;
            }
#pragma unroll
            for (int c = 0; c < D / 16; ++c) {
                const bf16x8_t a = Tl::rows(cQ, 32 * qb + (lane & 31), c, lane);
                const bf16x8_t g = Tl::rows(cG, 32 * qb + (lane & 31), c, lane);
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    s[b] = mma(a, kf[b].v[c], s[b]);
                    dp[b] = mma(g, vf[b].v[c], dp[b]);
                }
            }
            bf16x8_t gt_[D / 32][2], qt_[D / 32][2];
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    gt_[db][half] = Tl::cols(cG, db, 32 * qb + 16 * half, lane);
                    qt_[db][half] = Tl::cols(cQ, db, 32 * qb + 16 * half, lane);
                }
            if constexpr (ragged.value) drop_past_end<D>(gt_, qbase + 32 * qb, n, lane);
            __builtin_amdgcn_sched_barrier(0);
            bf16x8_t pb[NB][2], sb[NB][2];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    s[b][i] = ex2(fmaf(s[b][i], sl2, -Lr[i]));
                    dp[b][i] *= s[b][i];
                }
                pb[b][0] = acc_b16(s[b], 0);
                pb[b][1] = acc_b16(s[b], 1);
                sb[b][0] = acc_b16(dp[b], 0);
                sb[b][1] = acc_b16(dp[b], 1);
            }
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const bf16x8_t g = gt_[db][half];
                    const bf16x8_t a = qt_[db][half];
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        dv[b][db] = mma(g, pb[b][half], dv[b][db]);
                        dk[b][db] = mma(a, sb[b][half], dk[b][db]);
                    }
                }
        }
        if (!ragged.value && t + 1 < stages) store_rows(nL, nD);
        stage_done();
    };
    const int64_t whole = n / kStage;
    for (int64_t t = 0; t < whole; t += 2) {
        stage(t, Flag<false>{}, sQ0, sG0, sQ1, sG1, sL0, sD0, sL1, sD1);
        if (t + 1 < whole) stage(t + 1, Flag<false>{}, sQ1, sG1, sQ0, sG0, sL1, sD1, sL0, sD0);
    }
    if (whole < stages) {
        const bool odd = whole & 1;
        stage(whole, Flag<true>{}, odd ? sQ1 : sQ0, odd ? sG1 : sG0, sQ0, sG0, odd ? sL1 : sL0, odd ? sD1 : sD0, sL0, sD0);
    }
    if constexpr (KS > 1) {
        add_shares<KS, WAVES, NB * (D / 32)>(&dk[0][0], part);
        __syncthreads();
        if (!add_shares<KS, WAVES, NB * (D / 32)>(&dv[0][0], part)) return;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t key = k0 + 32 * b + (lane & 31);
        if (key >= n) continue;
        store_acc<D>(dK + (key * H + h) * D, dk[b], scale, lane);
        store_acc<D>(dV + (key * H + h) * D, dv[b], 1.f, lane);
    }
}

// ------------------------------------------------------------ dense tiles
// Sparse layers: the dense tiles of the plan (§3.4), computed whole on the
// matrix cores with the tile's bit mask deciding which pairs are edges.  The
// row-owned kernels walk a tile row's dense tiles, the column-owned kernel a
// tile column's (in chunks of tiles); a workgroup has T/32 wavefronts of 32
// owned rows (one MFMA block each, kTileNB) and stages the partners 64 at a
// time.  Each kernel leaves fp32
// partial sums per (node, head) for the edge kernels, which add the remainder
// edges and finish every row and column.  A row may have no edge in a tile:
// its weights are exactly zero (masked scores are -inf, and an all-masked
// running maximum is treated as 0 in the exponent).

// Mask words of one owned row for one tile: bit c of word w <=> key 32 w + c.
template <int T>
__device__ __forceinline__ void load_mask_row(uint32_t (&mw)[T / 32], const uint32_t* __restrict__ row) {
    if constexpr (T == 128) {
        const uint4 v = *reinterpret_cast<const uint4*>(row);
        mw[0] = v.x, mw[1] = v.y, mw[2] = v.z, mw[3] = v.w;
    } else {
        const uint2 v = *reinterpret_cast<const uint2*>(row);
        mw[0] = v.x, mw[1] = v.y;
    }
}

// ---- chunks of the dense tiles of each tile row (column)

// Workgroup b -> tile row (column) I, its list range [t0, t1) and the output
// slot (-1: the partial state of the row; else an extra slot); false for the
// surplus of the grid.
__device__ __forceinline__ bool tile_chunk(const TileChunks& ck, const int64_t* __restrict__ ptr, int64_t R,
                                           int64_t b, int64_t& I, int64_t& t0, int64_t& t1, int64_t& slot) {
    if (b >= ck.chunk_off[R]) return false;
    int64_t lo = 0, hi = R;  // the last I with chunk_off[I] <= b
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (ck.chunk_off[mid] <= b) lo = mid;
        else hi = mid;
    }
    I = lo;
    const int64_t j = b - ck.chunk_off[lo];
    t0 = ptr[lo] + j * ck.CH;
    t1 = t0 + ck.CH < ptr[lo + 1] ? t0 + ck.CH : ptr[lo + 1];
    slot = j == 0 ? -1 : ck.extra_off[lo] + j - 1;
    return true;
}

// Output row of node q (tile row I) for a chunk writing `slot`.
__device__ __forceinline__ int64_t out_row(int64_t q, int64_t I, int64_t slot, int T) {
    return slot < 0 ? q : slot * T + (q - I * T);
}

// The plan in one workgroup (a tile plan has at most 16,384 tile rows).
// Wavefront w owns the 64 ROUNDS rows from 64 ROUNDS w, in rounds of 64
// consecutive rows (one per lane), so every load and store is coalesced: the
// wavefront totals give each wavefront its base, then each round's wavefront
// scan, plus the running total of the rounds before it, gives every row its chunk
// offset, extra-slot offset and place in the list of rows with extra slots.
// ROUNDS fits the plan (16 rounds for any plan: 512 tile rows 10.5 us, with one
// round 5.0; 7,600 tile rows 17, with 8 rounds 11).
constexpr int kPlanThreads = 1024;
constexpr int kPlanWaves = kPlanThreads / kWave;
constexpr int64_t kPlanMaxRows = 16384;

// Inclusive wavefront sum scan on DPP moves (no LDS round trips): shifts by
// 1, 2, 4 and 8 lanes scan each 16-lane row; broadcasting lane 15 into rows 1
// and 3, then lane 31 into rows 2 and 3, adds the totals of the rows before.
// Lanes a move does not reach take 0 (the `old` operand).
template <int Ctrl, int RowMask>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(x), Ctrl, RowMask, 0xF, false));
}
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t x) {
    x += dpp_u32<0x111, 0xF>(x);  // row_shr:1
    x += dpp_u32<0x112, 0xF>(x);  // row_shr:2
    x += dpp_u32<0x114, 0xF>(x);  // row_shr:4
    x += dpp_u32<0x118, 0xF>(x);  // row_shr:8
    x += dpp_u32<0x142, 0xA>(x);  // row_bcast:15 into rows 1, 3
    x += dpp_u32<0x143, 0xC>(x);  // row_bcast:31 into rows 2, 3
    return x;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, kWave);
    return x;
}

template <int ROUNDS>
__global__ __launch_bounds__(kPlanThreads) void k_tile_chunk_plan1(int64_t R, const int64_t* __restrict__ ptr,
                                                                   int CH, int64_t* __restrict__ chunk_off,
                                                                   int64_t* __restrict__ extra_off,
                                                                   int32_t* __restrict__ merge_rows,
                                                                   uint32_t* __restrict__ merge_cnt) {
    // Counts fit in 32 bits: at most R <= 16,384 tiles per row and R rows.
    __shared__ uint32_t s_w[3][kPlanWaves];
    const int t = threadIdx.x, w = t / kWave, lane = lane_id();
    const int64_t base = int64_t(w) * (ROUNDS * kWave);
    uint32_t k[ROUNDS];  // chunks of row base + 64 j + lane
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int64_t I = base + kWave * j + lane;
        k[j] = I < R ? (uint32_t(ptr[I + 1] - ptr[I]) + uint32_t(CH) - 1u) / uint32_t(CH) : 0u;
    }
    uint32_t c = 0, e = 0, m = 0;
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        c += k[j];
        e += k[j] > 1u ? k[j] - 1u : 0u;
        m += k[j] > 1u ? 1u : 0u;
    }
    c = wave_sum_u32(c);
    e = wave_sum_u32(e);
    m = wave_sum_u32(m);
    if (lane == 0) {
        s_w[0][w] = c;
        s_w[1][w] = e;
        s_w[2][w] = m;
    }
    __syncthreads();
    uint32_t bc = 0, be = 0, bm = 0, tc = 0, te = 0, tm = 0;
#pragma unroll 1
    for (int x = 0; x < kPlanWaves; ++x) {
        if (x < w) {
            bc += s_w[0][x];
            be += s_w[1][x];
            bm += s_w[2][x];
        }
        tc += s_w[0][x];
        te += s_w[1][x];
        tm += s_w[2][x];
    }
#pragma unroll
    for (int j = 0; j < ROUNDS; ++j) {
        const int64_t I = base + kWave * j + lane;
        const uint32_t xe = k[j] > 1u ? k[j] - 1u : 0u, xm = k[j] > 1u ? 1u : 0u;
        const uint32_t ic = wave_incl_scan_u32(k[j]), ie = wave_incl_scan_u32(xe), im = wave_incl_scan_u32(xm);
        if (I < R) {
            chunk_off[I] = int64_t(bc + ic - k[j]);
            extra_off[I] = int64_t(be + ie - xe);
            if (xm) merge_rows[bm + im - 1u] = int32_t(I);
        }
        bc += uint32_t(__builtin_amdgcn_readlane(int(ic), kWave - 1));
        be += uint32_t(__builtin_amdgcn_readlane(int(ie), kWave - 1));
        bm += uint32_t(__builtin_amdgcn_readlane(int(im), kWave - 1));
    }
    if (t == 0) {
        chunk_off[R] = int64_t(tc);
        extra_off[R] = int64_t(te);
        *merge_cnt = tm;
    }
}

gt_status tile_chunk_plan(const gt_tiles* p, const int64_t* ptr, const TileChunks& ck, hipStream_t s) {
    const int64_t R = p->n_row_tiles;
    if (R > kPlanMaxRows) return fail(GT_ERR_UNSUPPORTED, "dense tiles: more than 16384 tile rows");
#define GT_CHUNK_PLAN(ROUNDS)                                                                                  \
    k_tile_chunk_plan1<ROUNDS><<<1, kPlanThreads, 0, s>>>(R, ptr, ck.CH, ck.chunk_off, ck.extra_off, ck.merge_rows, \
                                                          ck.merge_cnt)
    if (R <= kPlanThreads) GT_CHUNK_PLAN(1);
    else if (R <= 4 * kPlanThreads) GT_CHUNK_PLAN(4);
    else if (R <= 8 * kPlanThreads) GT_CHUNK_PLAN(8);
    else GT_CHUNK_PLAN(16);
#undef GT_CHUNK_PLAN
    static_assert(kPlanMaxRows == 16 * kPlanThreads, "16 rounds hold any plan");
    GT_LAUNCH_CHECK("tile_chunk_plan");
    return GT_OK;
}

// Fold the extra slots of each tile row into its partial state.  A workgroup
// takes kMergeRows<D> rows of one (tile row, head), D / 4 consecutive lanes per
// row, one float4 each, so every slot row is read as whole cache lines.
constexpr int kMergeThreads = 256;
constexpr int kTileNB = 1;  // 32-row blocks per wavefront in the dense-tile kernels
template <int D>
constexpr int kMergeRows = kMergeThreads / (D / 4);

inline dim3 merge_grid(const TileChunks& ck, int H, int T, int D) {
    return dim3(unsigned(ck.max_merge), unsigned(H), unsigned(T / (kMergeThreads / (D / 4))));
}

// ... the forward's online-softmax states (m, l, acc) ...
template <int D, int T>
__global__ __launch_bounds__(kMergeThreads) void k_tiles_merge_fwd(int64_t n, int H, TileChunks ck,
                                                                   float* __restrict__ pm, float* __restrict__ pl,
                                                                   float* __restrict__ pacc) {
    if (blockIdx.x >= *ck.merge_cnt) return;
    const int64_t I = ck.merge_rows[blockIdx.x];
    const int h = blockIdx.y;
    const int64_t e0 = ck.extra_off[I], e1 = ck.extra_off[I + 1];
    const int lr = blockIdx.z * kMergeRows<D> + threadIdx.x / (D / 4);
    const int f = 4 * (threadIdx.x % (D / 4));
    const int64_t q = I * T + lr;
    if (q >= n) return;
    const int64_t row = q * H + h;
    const float m0 = pm[row];
    float M = m0;
    for (int64_t e = e0; e < e1; ++e) M = fmaxf(M, ck.m[(e * T + lr) * H + h]);
    if (M == -__builtin_huge_valf()) return;  // no dense-tile edge in any chunk
    const float w0 = m0 == -__builtin_huge_valf() ? 0.f : ex2(m0 - M);
    float lsum = pl[row] * w0;
    float4* out = reinterpret_cast<float4*>(pacc + row * D + f);
    float4 acc = *out;
    acc.x *= w0;
    acc.y *= w0;
    acc.z *= w0;
    acc.w *= w0;
#pragma unroll 2
    for (int64_t e = e0; e < e1; ++e) {
        const int64_t xr = (e * T + lr) * H + h;
        const float me = ck.m[xr];
        if (me == -__builtin_huge_valf()) continue;
        const float w = ex2(me - M);
        lsum += ck.l[xr] * w;
        const float4 x = *reinterpret_cast<const float4*>(ck.acc + xr * D + f);
        acc.x += x.x * w;
        acc.y += x.y * w;
        acc.z += x.z * w;
        acc.w += x.w * w;
    }
    *out = acc;
    if (f == 0) {
        pm[row] = M;
        pl[row] = lsum;
    }
}

// ... and plain sums (the backward's A, B, D and dK, dV).
template <int D, int T>
__global__ __launch_bounds__(kMergeThreads) void k_tiles_merge_sum(int64_t n, int H, TileChunks ck,
                                                                   float* __restrict__ a, float* __restrict__ b,
                                                                   float* __restrict__ m) {
    if (blockIdx.x >= *ck.merge_cnt) return;
    const int64_t I = ck.merge_rows[blockIdx.x];
    const int h = blockIdx.y;
    const int64_t e0 = ck.extra_off[I], e1 = ck.extra_off[I + 1];
    const int lr = blockIdx.z * kMergeRows<D> + threadIdx.x / (D / 4);
    const int f = 4 * (threadIdx.x % (D / 4));
    const int64_t q = I * T + lr;
    if (q >= n) return;
    const int64_t row = q * H + h;
    float4* pa = reinterpret_cast<float4*>(a + row * D + f);
    float4* pb = b ? reinterpret_cast<float4*>(b + row * D + f) : nullptr;
    float4 sa = *pa, sb = pb ? *pb : make_float4(0.f, 0.f, 0.f, 0.f);
    float sm = (m && f == 0) ? m[row] : 0.f;
#pragma unroll 2
    for (int64_t e = e0; e < e1; ++e) {
        const int64_t xr = (e * T + lr) * H + h;
        const float4 x = *reinterpret_cast<const float4*>(ck.acc + xr * D + f);
        sa.x += x.x;
        sa.y += x.y;
        sa.z += x.z;
        sa.w += x.w;
        if (pb) {
            const float4 y = *reinterpret_cast<const float4*>(ck.acc2 + xr * D + f);
            sb.x += y.x;
            sb.y += y.y;
            sb.z += y.z;
            sb.w += y.w;
        }
        if (m && f == 0) sm += ck.m[xr];
    }
    *pa = sa;
    if (pb) *pb = sb;
    if (m && f == 0) m[row] = sm;
}

// NB 32-row blocks per wavefront (2: every K and V fragment read from LDS
// feeds two products; 1: half the registers, twice the wavefronts).  The
// tiles are launched with NB = 1 (kTileNB): a chunk holds only a few tiles, so
// the kernels are latency-bound and more resident wavefronts pay more than
// the operand reuse.  Wavefronts per SIMD: forward 4 at d = 32, 3 at d = 64; dQ
// and dK/dV 3 at d = 32, 2 at d = 64.  Measured on 65,536 nodes, 8 heads, tiles from
// 5% on (us, backward of the layer): d = 32 at 2 wavefronts 406, at 3 371; with a
// bias dK/dV at 1 wavefront in a SIMD 4120 (d = 64) and 3870 (d = 32), at 2 and 3
// 3650 and 3320.  A stage's cells of the bias are addressed from a uniform base,
// with one offset a lane: an address a cell is what took the registers (256 and 186
// AGPRs).
template <int D, int T, int NB, bool kBias = false>
__global__ __launch_bounds__(T * 2 / NB) __attribute__((amdgpu_waves_per_eu(D >= 64 ? 3 : 4))) void k_tiles_fwd(
    int64_t n, int H, const int64_t* __restrict__ tile_rowptr,
                                                 const int32_t* __restrict__ tile_col,
                                                 const uint32_t* __restrict__ tile_mask,
                                                 const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                                                 const uint16_t* __restrict__ V, float sl2, float* __restrict__ pm,
                                                 float* __restrict__ pl, float* __restrict__ pacc, int64_t R,
                                                 TileChunks ck, TileBias tb) {
    constexpr int W = T / 32;
    using Tl = Tile<D>;
    constexpr int kWaves = T / (32 * NB);
    __shared__ __attribute__((aligned(16))) uint16_t sK0[Tl::kElems], sK1[Tl::kElems];
    __shared__ __attribute__((aligned(16))) uint16_t sV0[Tl::kElems], sV1[Tl::kElems];
    const int h = blockIdx.y;
    int64_t I, t0, t1, slot;
    if (!tile_chunk(ck, tile_rowptr, R, blockIdx.x, I, t0, t1, slot)) return;
    if (slot >= 0) {
        pm = ck.m;
        pl = ck.l;
        pacc = ck.acc;
    }
    const int lane = lane_id(), wave = uniform(int(threadIdx.x) / kWave);
    const int ql0 = (threadIdx.x / kWave) * 32 * NB;  // first owned row inside the tile row
    const int64_t q0 = int64_t(I) * T + ql0;
    Frag<D> qf[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) qf[b].load(Q, q0 + 32 * b + (lane & 31), n, H, h, lane);
    positive_scale<D, NB>(qf, sl2);
    f32x16_t acc[NB][D / 32];
    float m[NB], l[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int db = 0; db < D / 32; ++db) acc[b][db] = zero16();
        m[b] = kNegInf;
        l[b] = 0.f;
    }
    // Stages run over the chunk's dense tiles, T/64 per tile; a stage's rows (and
    // a tile's mask words) are on their way while the one before is multiplied.
    constexpr int NSG = T / kStage;
    const int64_t stages = (t1 - t0) * NSG;
    uint32_t mw[NB][W], mwn[NB][W];
    int cols = 0;  // tile columns of 64 tiles, one per lane
    int64_t kcol = 0;
    auto prefetch = [&](int64_t g, uint16_t* nK, uint16_t* nV) {
        const int64_t j = g / NSG, k = t0 + j;
        if (g % NSG == 0) {
            if (j % kWave == 0) cols = k + lane < t1 ? tile_col[k + lane] : 0;
            kcol = int64_t(__builtin_amdgcn_readlane(cols, int(j % kWave))) * T;
#pragma unroll
            for (int b = 0; b < NB; ++b)
                load_mask_row<T>(mwn[b], tile_mask + (k * T + ql0 + 32 * b + (lane & 31)) * W);
        }
        Tl::template fetch<kWaves>(nK, K, kcol + kStage * (g % NSG), n, H, h, wave, lane);
        Tl::template fetch<kWaves>(nV, V, kcol + kStage * (g % NSG), n, H, h, wave, lane);
    };
    auto stage = [&](int64_t g, const uint16_t* cK, uint16_t* cV, uint16_t* nK, uint16_t* nV) {
        const int st = int(g % NSG);
        Tl::template zero_past_end<kWaves * kWave>(cV, kcol + kStage * st, n);
        if (st == 0)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int w = 0; w < W; ++w) mw[b][w] = mwn[b][w];
        if (g + 1 < stages) prefetch(g + 1, nK, nV);
#pragma unroll
        for (int kb = 0; kb < kStage / 32; ++kb) {
            f32x16_t s[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) s[b] = zero16();
#pragma unroll
            for (int c = 0; c < D / 16; ++c) {
                const bf16x8_t a = Tl::rows(cK, 32 * kb + (lane & 31), c, lane);
#pragma unroll
                for (int b = 0; b < NB; ++b) s[b] = mma(a, qf[b].v[c], s[b]);
            }
            bool grow = false;
            float mt[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint32_t w = mw[b][2 * st + kb];
                if constexpr (kBias) {
                    // scores in the exp2 domain with the bias added: s sl2 + b log2 e
                    const float* cell = tb.b + TileBias::at(t0 + g / NSG, H, h, T, 32 * (NB * wave + b),
                                                            kStage * st + 32 * kb);
                    const int xl = (lane & 31) * T + 4 * (lane >> 5);
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        // the per-tile bias is -inf off the edges, so it masks the cell itself: no test and
                        // no branch, which keeps the wait states of the accumulator reads that follow
                        const float bb = (cell + (8 * (i >> 2) + (i & 3)))[xl];
                        s[b][i] = fmaf(s[b][i], sl2, bb * kLog2e);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (!((w >> crow(i, lane)) & 1u)) s[b][i] = kNegInf;
                }
                float mx = s[b][0];
#pragma unroll
                for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[b][i]);
                mt[b] = kBias ? pair_max(mx) : pair_max(mx) * sl2;
                grow |= mt[b] > m[b] + kLazy;
            }
            if (__builtin_amdgcn_ballot_w64(grow)) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const float mn = fmaxf(m[b], mt[b]);
                    if (mn == kNegInf) continue;
                    const float alpha = ex2(m[b] - mn);
                    l[b] *= alpha;
#pragma unroll
                    for (int db = 0; db < D / 32; ++db)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[b][db][i] *= alpha;
                    m[b] = mn;
                }
            }
            bf16x8_t pb[NB][2];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const float mm = m[b] == kNegInf ? 0.f : m[b];
                float ls = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float p = kBias ? ex2(s[b][i] - mm) : ex2(fmaf(s[b][i], sl2, -mm));
                    s[b][i] = p;
                    ls += p;
                }
                l[b] += ls;
                pb[b][0] = acc_b16(s[b], 0);
                pb[b][1] = acc_b16(s[b], 1);
            }
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const bf16x8_t a = Tl::cols(cV, db, 32 * kb + 16 * half, lane);
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b][db] = mma(a, pb[b][half], acc[b][db]);
                }
        }
        stage_done();
    };
    prefetch(0, sK0, sV0);
    stage_done();
#pragma unroll 1
    for (int64_t g = 0; g < stages; g += 2) {
        stage(g, sK0, sV0, sK1, sV1);
        if (g + 1 < stages) stage(g + 1, sK1, sV1, sK0, sV0);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t q = q0 + 32 * b + (lane & 31);
        const float lt = pair_sum(l[b]);
        if (q >= n) continue;
        const int64_t orow = out_row(q, I, slot, T);
        if (lane < 32) {
            pm[orow * H + h] = m[b];
            pl[orow * H + h] = lt;
        }
        float* o = pacc + (orow * H + h) * D;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x16_t& a = acc[b][db];
                *reinterpret_cast<float4*>(o + 32 * db + 8 * j + 4 * (lane >> 5)) =
                    make_float4(a[4 * j], a[4 * j + 1], a[4 * j + 2], a[4 * j + 3]);
            }
    }
}

// Weights w as bf16 hi + lo parts (about 16 mantissa bits): B operands of
// two products whose sum keeps the fp32 weight, for sums of many large
// weights and for the A - D B difference of the row pass.
__device__ __forceinline__ void split_b16(const f32x16_t& w, int half, bf16x8_t& hi, bf16x8_t& lo) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        hi[t] = (__bf16)w[8 * half + t];
        lo[t] = (__bf16)(w[8 * half + t] - float(hi[t]));
    }
}

// Row pass over the dense tiles: A = sum P dP K, B = sum P K and the D sum
// sum P dP of every owned row (the edge kernels form dQ = scale (A - D B)).
template <int D, int T, int NB, bool kBias = false>
__global__ __launch_bounds__(T * 2 / NB) __attribute__((amdgpu_waves_per_eu(NB > 1 ? 1 : D < 64 ? 3 : 2))) void k_tiles_dq(
    int64_t n, int H, const int64_t* __restrict__ tile_rowptr,
                                                const int32_t* __restrict__ tile_col,
                                                const uint32_t* __restrict__ tile_mask,
                                                const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                                                const uint16_t* __restrict__ V, const uint16_t* __restrict__ dO,
                                                const float* __restrict__ LSE, float sl2, float* __restrict__ pa,
                                                float* __restrict__ pb, float* __restrict__ pd, int64_t R,
                                                TileChunks ck, TileBias tb) {
    constexpr int W = T / 32;
    using Tl = Tile<D>;
    constexpr int kWaves = T / (32 * NB);
    __shared__ __attribute__((aligned(16))) uint16_t sK0[Tl::kElems], sK1[Tl::kElems];
    __shared__ __attribute__((aligned(16))) uint16_t sV0[Tl::kElems], sV1[Tl::kElems];
    const int h = blockIdx.y;
    int64_t I, t0, t1, slot;
    if (!tile_chunk(ck, tile_rowptr, R, blockIdx.x, I, t0, t1, slot)) return;
    if (slot >= 0) {
        pa = ck.acc;
        pb = ck.acc2;
        pd = ck.m;
    }
    const int lane = lane_id(), wave = uniform(int(threadIdx.x) / kWave);
    const int ql0 = (threadIdx.x / kWave) * 32 * NB;
    const int64_t q0 = int64_t(I) * T + ql0;
    Frag<D> qf[NB], gf[NB];
    float lse2[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t q = q0 + 32 * b + (lane & 31);
        qf[b].load(Q, q, n, H, h, lane);
        gf[b].load(dO, q, n, H, h, lane);
        lse2[b] = q < n ? LSE[q * H + h] * kLog2e : 0.f;
    }
    f32x16_t accA[NB][D / 32], accB[NB][D / 32];
    float dsum[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int db = 0; db < D / 32; ++db) accA[b][db] = accB[b][db] = zero16();
        dsum[b] = 0.f;
    }
    // Stages run over the chunk's dense tiles, T/64 per tile; a stage's rows (and
    // a tile's mask words) are on their way while the one before is multiplied.
    constexpr int NSG = T / kStage;
    const int64_t stages = (t1 - t0) * NSG;
    uint32_t mw[NB][W], mwn[NB][W];
    int cols = 0;  // tile columns of 64 tiles, one per lane
    int64_t kcol = 0;
    auto prefetch = [&](int64_t g, uint16_t* nK, uint16_t* nV) {
        const int64_t j = g / NSG, k = t0 + j;
        if (g % NSG == 0) {
            if (j % kWave == 0) cols = k + lane < t1 ? tile_col[k + lane] : 0;
            kcol = int64_t(__builtin_amdgcn_readlane(cols, int(j % kWave))) * T;
#pragma unroll
            for (int b = 0; b < NB; ++b)
                load_mask_row<T>(mwn[b], tile_mask + (k * T + ql0 + 32 * b + (lane & 31)) * W);
        }
        Tl::template fetch<kWaves>(nK, K, kcol + kStage * (g % NSG), n, H, h, wave, lane);
        Tl::template fetch<kWaves>(nV, V, kcol + kStage * (g % NSG), n, H, h, wave, lane);
    };
    auto stage = [&](int64_t g, const uint16_t* cK, const uint16_t* cV, uint16_t* nK, uint16_t* nV) {
        const int st = int(g % NSG);
        if (st == 0)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int w = 0; w < W; ++w) mw[b][w] = mwn[b][w];
        if (g + 1 < stages) prefetch(g + 1, nK, nV);
#pragma unroll
        for (int kb = 0; kb < kStage / 32; ++kb) {
            f32x16_t s[NB], dp[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) s[b] = dp[b] = zero16();
#pragma unroll
            for (int c = 0; c < D / 16; ++c) {
                const bf16x8_t a = Tl::rows(cK, 32 * kb + (lane & 31), c, lane);
#pragma unroll
                for (int b = 0; b < NB; ++b) s[b] = mma(a, qf[b].v[c], s[b]);
                const bf16x8_t v = Tl::rows(cV, 32 * kb + (lane & 31), c, lane);
#pragma unroll
                for (int b = 0; b < NB; ++b) dp[b] = mma(v, gf[b].v[c], dp[b]);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const uint32_t w = mw[b][2 * st + kb];
                const float* cell = nullptr;
                const int xl = (lane & 31) * T + 4 * (lane >> 5);
                if constexpr (kBias)
                    cell = tb.b + TileBias::at(t0 + g / NSG, H, h, T, 32 * (NB * wave + b), kStage * st + 32 * kb);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    float p;
                    if constexpr (kBias) {
                        const float bb = (cell + (8 * (i >> 2) + (i & 3)))[xl];
                        p = ex2(fmaf(s[b][i], sl2, bb * kLog2e - lse2[b]));  // 0 off the edges (bias -inf)
                    } else {
                        p = (w >> crow(i, lane)) & 1u ? ex2(fmaf(s[b][i], sl2, -lse2[b])) : 0.f;
                    }
                    s[b][i] = p;
                    dp[b][i] *= p;
                    dsum[b] += dp[b][i];
                }
            }
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const bf16x8_t a = Tl::cols(cK, db, 32 * kb + 16 * half, lane);
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        bf16x8_t hi, lo;
                        split_b16(dp[b], half, hi, lo);
                        accA[b][db] = mma(a, lo, mma(a, hi, accA[b][db]));
                        split_b16(s[b], half, hi, lo);
                        accB[b][db] = mma(a, lo, mma(a, hi, accB[b][db]));
                    }
                }
        }
        stage_done();
    };
    prefetch(0, sK0, sV0);
    stage_done();
#pragma unroll 1
    for (int64_t g = 0; g < stages; g += 2) {
        stage(g, sK0, sV0, sK1, sV1);
        if (g + 1 < stages) stage(g + 1, sK1, sV1, sK0, sV0);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t q = q0 + 32 * b + (lane & 31);
        const float ds = pair_sum(dsum[b]);
        if (q >= n) continue;
        const int64_t orow = out_row(q, I, slot, T);
        if (lane < 32) pd[orow * H + h] = ds;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int f = 32 * db + 8 * j + 4 * (lane >> 5);
                const f32x16_t& x = accA[b][db];
                const f32x16_t& y = accB[b][db];
                *reinterpret_cast<float4*>(pa + (orow * H + h) * D + f) =
                    make_float4(x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3]);
                *reinterpret_cast<float4*>(pb + (orow * H + h) * D + f) =
                    make_float4(y[4 * j], y[4 * j + 1], y[4 * j + 2], y[4 * j + 3]);
            }
    }
}

// One butterfly step of a 32 x 32 bit-matrix transpose held one row per lane
// in each half of the wavefront: the lanes with bit J set trade the low J bits
// of each 2J-bit group for their partner's high J bits (ds_swizzle in bitmask
// mode, xor J within 32 lanes).
template <int J>
__device__ __forceinline__ uint32_t bit_transpose_step(uint32_t w, int lane) {
    constexpr uint32_t lo = J == 16 ? 0x0000FFFFu : J == 8 ? 0x00FF00FFu : J == 4 ? 0x0F0F0F0Fu : J == 2 ? 0x33333333u
                                                                                                           : 0x55555555u;
    const uint32_t t = uint32_t(__builtin_amdgcn_ds_swizzle(int(w), (J << 10) | 0x1F));
    return (lane & J) ? (w & ~lo) | ((t & ~lo) >> J) : (w & lo) | ((t & lo) << J);
}

// Transpose of the 64 x 32 bit matrix whose row r is lane r's word: on return
// bit r of lane c's word (either half: both get the same 64 bits) is entry
// (r, c % 32).
__device__ __forceinline__ uint64_t bit_transpose_64x32(uint32_t w, int lane) {
    w = bit_transpose_step<16>(w, lane);
    w = bit_transpose_step<8>(w, lane);
    w = bit_transpose_step<4>(w, lane);
    w = bit_transpose_step<2>(w, lane);
    w = bit_transpose_step<1>(w, lane);
    const uint32_t other = __shfl_xor(w, 32, kWave);
    return lane < 32 ? uint64_t(w) | (uint64_t(other) << 32) : uint64_t(other) | (uint64_t(w) << 32);
}

// Column pass over the dense tiles: unscaled dK and dV sums of every owned key.
// The stage's masks are transposed so that each lane holds, for its key, one
// 64-bit word over the stage's 64 queries.
template <int D, int T, int NB, bool kBias = false>
__global__ __launch_bounds__(T * 2 / NB) __attribute__((amdgpu_waves_per_eu(NB > 1 ? 1 : D < 64 ? 3 : 2))) void k_tiles_dkdv(
    int64_t n, int H, int64_t n_row_tiles,
                                                  const int64_t* __restrict__ tileT_ptr,
                                                  const int32_t* __restrict__ tileT_idx,
                                                  const int64_t* __restrict__ tile_rowptr,
                                                  const uint32_t* __restrict__ tile_mask,
                                                  const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K,
                                                  const uint16_t* __restrict__ V, const uint16_t* __restrict__ dO,
                                                  const float* __restrict__ LSE, const float* __restrict__ Dv,
                                                  float sl2, float* __restrict__ pdk, float* __restrict__ pdv,
                                                  TileChunks ck, TileBias tb) {
    constexpr int W = T / 32;
    using Tl = Tile<D>;
    constexpr int kWaves = T / (32 * NB);
    __shared__ __attribute__((aligned(16))) uint16_t sQ0[Tl::kElems], sQ1[Tl::kElems];
    __shared__ __attribute__((aligned(16))) uint16_t sG0[Tl::kElems], sG1[Tl::kElems];
    __shared__ __attribute__((aligned(16))) float sL0[kStage], sL1[kStage];
    __shared__ __attribute__((aligned(16))) float sD0[kStage], sD1[kStage];
    const int h = blockIdx.y;
    int64_t J, u0, u1, slot;
    if (!tile_chunk(ck, tileT_ptr, n_row_tiles, blockIdx.x, J, u0, u1, slot)) return;
    if (slot >= 0) {
        pdk = ck.acc;
        pdv = ck.acc2;
    }
    const int lane = lane_id(), wave = uniform(int(threadIdx.x) / kWave);
    const int kl0 = (threadIdx.x / kWave) * 32 * NB;  // first owned key inside the tile column
    const int64_t k0 = int64_t(J) * T + kl0;
    Frag<D> kf[NB], vf[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        kf[b].load(K, k0 + 32 * b + (lane & 31), n, H, h, lane);
        vf[b].load(V, k0 + 32 * b + (lane & 31), n, H, h, lane);
    }
    f32x16_t dk[NB][D / 32], dv[NB][D / 32];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int db = 0; db < D / 32; ++db) dk[b][db] = dv[b][db] = zero16();
    constexpr int NSG = T / kStage;
    const int64_t stages = (u1 - u0) * NSG;
    uint32_t mword[NB];  // the next stage's: this lane's row, mask words of the wavefront's key blocks
    float2 stat = make_float2(0.f, 0.f);  // the next stage's: LSE (exp2 domain) and D of its query `lane`
    int tiles = 0, trow = 0;  // 64 tiles of the column and their tile rows, one per lane
    int64_t tn = 0, tk = 0;   // the next stage's tile, the stage's
    auto prefetch = [&](int64_t g, uint16_t* nQ, uint16_t* nG) {
        const int64_t j = g / NSG;
        if (g % NSG == 0 && j % kWave == 0) {
            tiles = u0 + j + lane < u1 ? tileT_idx[u0 + j + lane] : 0;
            int64_t lo = 0, hi = n_row_tiles;  // tile row of the tile: the last I with tile_rowptr[I] <= it
            while (hi - lo > 1) {
                const int64_t mid = (lo + hi) >> 1;
                if (tile_rowptr[mid] <= tiles) lo = mid;
                else hi = mid;
            }
            trow = int(lo);
        }
        tn = __builtin_amdgcn_readlane(tiles, int(j % kWave));
        const int st = int(g % NSG);
        const int64_t qbase = int64_t(__builtin_amdgcn_readlane(trow, int(j % kWave))) * T + kStage * st;
#pragma unroll
        for (int b = 0; b < NB; ++b) mword[b] = tile_mask[(tn * T + kStage * st + lane) * W + (kl0 / 32 + b)];
        if (wave == 0) {
            stat = make_float2(__builtin_huge_valf(), 0.f);  // queries >= n take no weight
            const int64_t qn = qbase + lane;
            if (qn < n) stat = make_float2(LSE[qn * H + h] * kLog2e, Dv[qn * H + h]);
        }
        Tl::template fetch<kWaves>(nQ, Q, qbase, n, H, h, wave, lane);
        Tl::template fetch<kWaves>(nG, dO, qbase, n, H, h, wave, lane);
    };
    // transposed masks: bit r of mt[b] <=> query r of the stage attends to key k0 + 32 b + lane % 32
    uint64_t mt[NB];
    auto stage = [&](int64_t g, const uint16_t* cQ, const uint16_t* cG, const float* cL, const float* cD,
                     uint16_t* nQ, uint16_t* nG, float* nL, float* nD) {
#pragma unroll
        for (int b = 0; b < NB; ++b) mt[b] = bit_transpose_64x32(mword[b], lane);
        tk = tn;
        if (g + 1 < stages) prefetch(g + 1, nQ, nG);
#pragma unroll
        for (int qb = 0; qb < kStage / 32; ++qb) {
            f32x16_t s[NB], dp[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) s[b] = dp[b] = zero16();
#pragma unroll
            for (int c = 0; c < D / 16; ++c) {
                const bf16x8_t a = Tl::rows(cQ, 32 * qb + (lane & 31), c, lane);
#pragma unroll
                for (int b = 0; b < NB; ++b) s[b] = mma(a, kf[b].v[c], s[b]);
                const bf16x8_t g8 = Tl::rows(cG, 32 * qb + (lane & 31), c, lane);
#pragma unroll
                for (int b = 0; b < NB; ++b) dp[b] = mma(g8, vf[b].v[c], dp[b]);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                float4 lv, d4;  // read where used: all 32 held spilled 12 registers at d = 32 (385 us)
                const uint32_t w = uint32_t(mt[b] >> (32 * qb));
                int64_t x0 = 0;
                const int xl = 4 * (lane >> 5) * T + (lane & 31);
                if constexpr (kBias)
                    x0 = TileBias::at(tk, H, h, T, kStage * int(g % NSG) + 32 * qb, 32 * (NB * wave + b));
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int r4 = 32 * qb + 8 * (i >> 2) + 4 * (lane >> 5);
                    if (i % 4 == 0) {
                        lv = *reinterpret_cast<const float4*>(&cL[r4]);
                        d4 = *reinterpret_cast<const float4*>(&cD[r4]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    const float Li = i % 4 == 0 ? lv.x : i % 4 == 1 ? lv.y : i % 4 == 2 ? lv.z : lv.w;
                    const float Di = i % 4 == 0 ? d4.x : i % 4 == 1 ? d4.y : i % 4 == 2 ? d4.z : d4.w;
                    const bool on = (w >> crow(i, lane)) & 1u;
                    float p = 0.f;
                    if constexpr (kBias) {
                        const int64_t x = x0 + (8 * (i >> 2) + (i & 3)) * T;
                        p = ex2(fmaf(s[b][i], sl2, (tb.b + x)[xl] * kLog2e - Li));  // 0 off the edges (bias -inf)
                        s[b][i] = p * (dp[b][i] - Di);
                        (tb.db + x)[xl] = s[b][i];  // every cell (0 off the edges), so no branch is needed
                    } else {
                        p = on ? ex2(fmaf(s[b][i], sl2, -Li)) : 0.f;
                        s[b][i] = p * (dp[b][i] - Di);
                    }
                    dp[b][i] = p;
                }
            }
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const bf16x8_t g8 = Tl::cols(cG, db, 32 * qb + 16 * half, lane);
                    const bf16x8_t a = Tl::cols(cQ, db, 32 * qb + 16 * half, lane);
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        bf16x8_t hi16, lo16;
                        split_b16(dp[b], half, hi16, lo16);
                        dv[b][db] = mma(g8, lo16, mma(g8, hi16, dv[b][db]));
                        split_b16(s[b], half, hi16, lo16);
                        dk[b][db] = mma(a, lo16, mma(a, hi16, dk[b][db]));
                    }
                }
        }
        if (wave == 0) {
            nL[lane] = stat.x;
            nD[lane] = stat.y;
        }
        stage_done();
    };
    prefetch(0, sQ0, sG0);
    if (wave == 0) {
        sL0[lane] = stat.x;
        sD0[lane] = stat.y;
    }
    stage_done();
#pragma unroll 1
    for (int64_t g = 0; g < stages; g += 2) {
        stage(g, sQ0, sG0, sL0, sD0, sQ1, sG1, sL1, sD1);
        if (g + 1 < stages) stage(g + 1, sQ1, sG1, sL1, sD1, sQ0, sG0, sL0, sD0);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int64_t key = k0 + 32 * b + (lane & 31);
        if (key >= n) continue;
        const int64_t orow = out_row(key, J, slot, T);
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int f = 32 * db + 8 * j + 4 * (lane >> 5);
                const f32x16_t& x = dk[b][db];
                const f32x16_t& y = dv[b][db];
                *reinterpret_cast<float4*>(pdk + (orow * H + h) * D + f) =
                    make_float4(x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3]);
                *reinterpret_cast<float4*>(pdv + (orow * H + h) * D + f) =
                    make_float4(y[4 * j], y[4 * j + 1], y[4 * j + 2], y[4 * j + 3]);
            }
    }
}

}  // namespace

// How the full layer is cut, by the (head, 128 rows) blocks it has for the 256
// CUs.  W wavefronts of NB 32-row blocks share a workgroup's rows; with KS = 2 a
// second set of wavefronts takes half of every stage's partners.  Measured at
// d = 64 (forward / backward, us), W x NB x KS:
//   1,000 x 4 (32 blocks):   2x1x2 15 / 37    4x1x2 17 / 44     4x1x1 20 / 54
//   3,001 x 8 (192 blocks):  2x1x2 46 / 119   4x1x2 41 / 110    4x1x1 51 / 145
//   6,000 x 8 (376 blocks):  2x1x2 115 / 386  4x1x2 140 / 386   4x1x1 136 / 385   8x1x1 - / 348   2x2x2 126 / -
//   16,384 x 8 (1,024):      2x1x2 766 / 2179 4x2x1 600 / -     8x1x1 - / 1808
enum class FullShape { narrow, shared, some, many };
inline FullShape full_shape(int64_t n, int H) {
    const int64_t blocks = cdiv(n, 128) * H;
    return blocks <= 128 ? FullShape::narrow
           : blocks <= 256 ? FullShape::shared
           : blocks <= 512 ? FullShape::some
                           : FullShape::many;
}

template <int D>
gt_status full_fwd_bf16(int64_t n, int H, const uint16_t* Q, const uint16_t* K, const uint16_t* V, float sl2,
                        uint16_t* O, float* LSE, hipStream_t s) {
    if (n <= 0) return GT_OK;
    const FullShape f = full_shape(n, H);
#define GT_FULL_FWD(NB, W, KS) \
    k_full_fwd<D, NB, W, KS><<<full_grid<32 * NB * W>(n, H), W * KS * kWave, 0, s>>>(n, H, Q, K, V, sl2, O, LSE)
    if (f == FullShape::narrow) GT_FULL_FWD(1, 2, 2);
    else if (f == FullShape::shared) GT_FULL_FWD(1, 4, 2);
    else if (f == FullShape::some) GT_FULL_FWD(1, 2, 2);
    else GT_FULL_FWD(2, 4, 1);
#undef GT_FULL_FWD
    GT_LAUNCH_CHECK("full_fwd_bf16");
    return GT_OK;
}

template <int D>
gt_status full_bwd_bf16(int64_t n, int H, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                        const uint16_t* O, const uint16_t* dO, const float* LSE, float sl2, float scale,
                        uint16_t* dQ, uint16_t* dK, uint16_t* dV, float* Dv, hipStream_t s) {
    if (n <= 0) return GT_OK;
    const FullShape f = full_shape(n, H);
#define GT_FULL_BWD(W, KS)                                                                                       \
    do {                                                                                                         \
        k_full_dq<D, 1, W, KS><<<full_grid<32 * W>(n, H), W * KS * kWave, 0, s>>>(n, H, Q, K, V, O, dO, LSE, sl2, \
                                                                                  scale, dQ, Dv);                \
        GT_LAUNCH_CHECK("full_bwd_bf16 dq");                                                                     \
        k_full_dkdv<D, 1, W, KS><<<full_grid<32 * W>(n, H), W * KS * kWave, 0, s>>>(n, H, Q, K, V, dO, LSE, Dv,  \
                                                                                    sl2, scale, dK, dV);         \
    } while (0)
    if (f == FullShape::narrow) GT_FULL_BWD(2, 2);
    else if (f == FullShape::shared) GT_FULL_BWD(4, 2);
    else GT_FULL_BWD(8, 1);
#undef GT_FULL_BWD
    GT_LAUNCH_CHECK("full_bwd_bf16 dkdv");
    return GT_OK;
}


#define GT_TILES_T(CALL)                                                          \
    do {                                                                          \
        if (p->T == 128) {                                                        \
            constexpr int TT = 128;                                               \
            CALL;                                                                 \
        } else if (p->T == 64) {                                                  \
            constexpr int TT = 64;                                                \
            CALL;                                                                 \
        } else {                                                                  \
            return fail(GT_ERR_UNSUPPORTED, "dense tiles: T must be 64 or 128");  \
        }                                                                         \
    } while (0)

template <int D>
gt_status tiles_fwd_bf16(const gt_tiles* p, int H, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                         float sl2, TilePartials tp, TileBias tb, hipStream_t s) {
    gt_status st = tile_chunk_plan(p, p->tile_rowptr, tp.ck, s);
    if (st != GT_OK) return st;
    const dim3 grid(unsigned(tp.ck.max_chunks), unsigned(H));
    constexpr int NB = kTileNB;
    if (tb.b)
        GT_TILES_T((k_tiles_fwd<D, TT, NB, true><<<grid, TT * 2 / NB, 0, s>>>(
            p->n, H, p->tile_rowptr, p->tile_col, p->tile_mask, Q, K, V, sl2, tp.m, tp.l, tp.acc, p->n_row_tiles,
            tp.ck, tb)));
    else
        GT_TILES_T((k_tiles_fwd<D, TT, NB><<<grid, TT * 2 / NB, 0, s>>>(p->n, H, p->tile_rowptr, p->tile_col,
                                                                        p->tile_mask, Q, K, V, sl2, tp.m, tp.l,
                                                                        tp.acc, p->n_row_tiles, tp.ck, tb)));
    GT_LAUNCH_CHECK("tiles_fwd_bf16");
    GT_TILES_T((k_tiles_merge_fwd<D, TT><<<merge_grid(tp.ck, H, TT, D), kMergeThreads, 0, s>>>(
        p->n, H, tp.ck, tp.m, tp.l, tp.acc)));
    GT_LAUNCH_CHECK("tiles_merge_fwd_bf16");
    return GT_OK;
}

template <int D>
gt_status tiles_dq_bf16(const gt_tiles* p, int H, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                        const uint16_t* dO, const float* LSE, float sl2, TilePartials dq, TileBias tb,
                        hipStream_t s) {
    gt_status st = tile_chunk_plan(p, p->tile_rowptr, dq.ck, s);
    if (st != GT_OK) return st;
    const dim3 grid(unsigned(dq.ck.max_chunks), unsigned(H));
    constexpr int NB = kTileNB;
    if (tb.b)
        GT_TILES_T((k_tiles_dq<D, TT, NB, true><<<grid, TT * 2 / NB, 0, s>>>(
            p->n, H, p->tile_rowptr, p->tile_col, p->tile_mask, Q, K, V, dO, LSE, sl2, dq.acc, dq.acc2, dq.m,
            p->n_row_tiles, dq.ck, tb)));
    else
        GT_TILES_T((k_tiles_dq<D, TT, NB><<<grid, TT * 2 / NB, 0, s>>>(p->n, H, p->tile_rowptr, p->tile_col,
                                                                       p->tile_mask, Q, K, V, dO, LSE, sl2, dq.acc,
                                                                       dq.acc2, dq.m, p->n_row_tiles, dq.ck, tb)));
    GT_LAUNCH_CHECK("tiles_dq_bf16");
    GT_TILES_T((k_tiles_merge_sum<D, TT><<<merge_grid(dq.ck, H, TT, D), kMergeThreads, 0, s>>>(
        p->n, H, dq.ck, dq.acc, dq.acc2, dq.m)));
    GT_LAUNCH_CHECK("tiles_merge_dq_bf16");
    return GT_OK;
}

template <int D>
gt_status tiles_dkdv_bf16(const gt_tiles* p, int H, const uint16_t* Q, const uint16_t* K, const uint16_t* V,
                          const uint16_t* dO, const float* LSE, const float* Dv, float sl2, TilePartials dk,
                          TilePartials dv, TileBias tb, hipStream_t s) {
    gt_status st = tile_chunk_plan(p, p->tileT_ptr, dk.ck, s);
    if (st != GT_OK) return st;
    const dim3 grid(unsigned(dk.ck.max_chunks), unsigned(H));
    constexpr int NB = kTileNB;
    if (tb.b)
        GT_TILES_T((k_tiles_dkdv<D, TT, NB, true><<<grid, TT * 2 / NB, 0, s>>>(
            p->n, H, p->n_row_tiles, p->tileT_ptr, p->tileT_idx, p->tile_rowptr, p->tile_mask, Q, K, V, dO, LSE, Dv,
            sl2, dk.acc, dv.acc, dk.ck, tb)));
    else
        GT_TILES_T((k_tiles_dkdv<D, TT, NB><<<grid, TT * 2 / NB, 0, s>>>(p->n, H, p->n_row_tiles, p->tileT_ptr,
                                                                         p->tileT_idx, p->tile_rowptr, p->tile_mask,
                                                                         Q, K, V, dO, LSE, Dv, sl2, dk.acc, dv.acc,
                                                                         dk.ck, tb)));
    GT_LAUNCH_CHECK("tiles_dkdv_bf16");
    GT_TILES_T((k_tiles_merge_sum<D, TT><<<merge_grid(dk.ck, H, TT, D), kMergeThreads, 0, s>>>(
        p->n, H, dk.ck, dk.acc, dv.acc, nullptr)));
    GT_LAUNCH_CHECK("tiles_merge_dkdv_bf16");
    return GT_OK;
}

#define GT_TILES_INST(D)                                                                                        \
    template gt_status tiles_fwd_bf16<D>(const gt_tiles*, int, const uint16_t*, const uint16_t*, const uint16_t*, \
                                         float, TilePartials, TileBias, hipStream_t);                           \
    template gt_status tiles_dq_bf16<D>(const gt_tiles*, int, const uint16_t*, const uint16_t*, const uint16_t*,  \
                                        const uint16_t*, const float*, float, TilePartials, TileBias,           \
                                        hipStream_t);                                                           \
    template gt_status tiles_dkdv_bf16<D>(const gt_tiles*, int, const uint16_t*, const uint16_t*,                \
                                          const uint16_t*, const uint16_t*, const float*, const float*, float,  \
                                          TilePartials, TilePartials, TileBias, hipStream_t);
GT_TILES_INST(32)
GT_TILES_INST(64)

template gt_status full_fwd_bf16<32>(int64_t, int, const uint16_t*, const uint16_t*, const uint16_t*, float,
                                     uint16_t*, float*, hipStream_t);
template gt_status full_fwd_bf16<64>(int64_t, int, const uint16_t*, const uint16_t*, const uint16_t*, float,
                                     uint16_t*, float*, hipStream_t);
template gt_status full_bwd_bf16<32>(int64_t, int, const uint16_t*, const uint16_t*, const uint16_t*,
                                     const uint16_t*, const uint16_t*, const float*, float, float, uint16_t*,
                                     uint16_t*, uint16_t*, float*, hipStream_t);
template gt_status full_bwd_bf16<64>(int64_t, int, const uint16_t*, const uint16_t*, const uint16_t*,
                                     const uint16_t*, const uint16_t*, const float*, float, float, uint16_t*,
                                     uint16_t*, uint16_t*, float*, hipStream_t);

}  // namespace gt
