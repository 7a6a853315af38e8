// Neighbourhood softmax attention (§3.2, local topology-induced pattern) on the
// remainder edges of a tile plan, forward and backward, plus the two entry
// points that also run the dense-tile kernels (tile_attn.hip).
//
// Edge kernels ("rows" and "cols"): a wavefront serves 64 / (H * d/F) nodes at
// once, each (node, head) owned by d/F lanes that hold F features (32 bytes of
// bf16) of it.  The node's own vectors stay in registers while the lanes walk
// its edge list, gathering the neighbours' slices.  Scores use the paper's
// scaled dot product in the exp2 domain; the forward keeps an online max / sum
// per (node, head), so nothing per edge is ever written to memory.
//
// Nodes with more than GT_LONG_ROW remainder edges are cut into runs, each
// walked like a short row in the same launch, and merged afterwards.
//
// The backward never uses atomics: dQ is gathered per row over the CSR, dK and
// dV per column over the remainder's transpose.
#include "attn_common.h"
#include "prim.h"
#include "tile_attn.h"

namespace gt {
namespace {

constexpr int kThreads = 256;
constexpr float kNegInf = -__builtin_huge_valf();

// The passes are bound by the rate of the row gathers through L2 and L1: over
// 1M nodes of 8 x 32 bf16 features and 31 edges a node of a clustered graph the
// gathers alone take 1.58 ms (gt_gather_probe), and in a copy of that probe with
// each node's own row read and a result row written 1.76 ms (100K nodes of 8 x 64,
// 17 edges: 0.150 and 0.206).  The forward takes two
// edges at a time with nothing in flight meanwhile, at 6 wavefronts per SIMD:
// 1.88 ms (0.225), no slower than with rows in flight at 4 (1.87; with pairs in
// flight 2.0, the registers spill).  The row pass holds 4 wavefronts, so it keeps
// the rows of the next kAheadRows edges in flight while one is used: 1.90 ms
// (0.251) against 2.42 (0.32) with none and 2.10 (0.285) when every quad waited for
// its ids.  The column pass takes two edges at a time with none in flight:
// 2.14 ms (0.304); with 2 in flight 2.22, its row statistics take the registers.
constexpr int kAheadRows = 2;
template <typename T, int D, int H>
constexpr int kLaneBytes = EdgeCfg<T, D, H>::F * int(sizeof(T));
// Wavefronts per SIMD the row pass is compiled for (2 where a lane holds 64
// bytes of a row; the backward with a bias takes one less).
template <typename T, int D, int H>
constexpr int kEdgeWaves = kLaneBytes<T, D, H> > 32 ? 2 : 4;

template <typename T, int D, int H>
struct Lanes {
    using C = EdgeCfg<T, D, H>;
    int slot, h, part;
    __device__ __forceinline__ explicit Lanes(int t) {
        slot = t / C::G;
        h = (t / C::L) % H;
        part = t % C::L;
    }
    __device__ __forceinline__ int64_t off(int64_t node) const { return (node * H + h) * D + part * C::RUN; }
};

// Per-edge additive bias (the graph encoding added to the scaled product,
// §2.1 Eq. (3); it shares the attention's sparse layout, §3.3): fp32
// [nnz, H] indexed by the edge's position in the input CSR of the plan.  A
// remainder edge's input position is sp_pos[remainder position] (the same
// position when the plan has no dense tile and no sp_pos).  The column pass
// finds an in-edge's input position through csc_pos and writes dB = dS there.
// The dense tiles take the bias laid out per tile (tile).
struct EdgeBias {
    const float* b = nullptr;  // null: no bias on the remainder edges
    const int32_t* sp_pos = nullptr;
    const int32_t* csc_pos = nullptr;
    float* db = nullptr;
    TileBias tile;
    // bias of remainder position pos, head h, in the exp2 domain
    __device__ __forceinline__ float at(int64_t pos, int H, int h) const {
        return b[(sp_pos ? int64_t(sp_pos[pos]) : pos) * H + h] * kLog2e;
    }
    // bias of input-CSR position e, head h, in the exp2 domain
    __device__ __forceinline__ float at_input(int64_t e, int H, int h) const { return b[e * H + h] * kLog2e; }
};

// F fp32 accumulators of one (node, head) slice.
template <int F>
struct Acc {
    float v[F];
    __device__ __forceinline__ Acc() {
#pragma unroll
        for (int i = 0; i < F; ++i) v[i] = 0.f;
    }
};

// A running maximum starts at the lowest finite value, which no finite score
// is below, so that a missing edge (score -inf) weighs exp2(-inf - m) = 0 with
// no test.
constexpr float kMinRef = -3.402823466e38f;

// Online-softmax state of one (node, head) slice.
template <int F>
struct Online {
    float m = kMinRef;  // running max, log2 domain
    float l = 0.f;      // running sum of exp2(s - m)
    float acc[F];       // running sum of exp2(s - m) * v
    __device__ __forceinline__ Online() {
#pragma unroll
        for (int i = 0; i < F; ++i) acc[i] = 0.f;
    }
};

// A lane's F fp32 values of a [n, H, D] array.
template <int F, int RUN, int STR>
__device__ __forceinline__ void load_f32_slice(float (&dst)[F], const float* src) {
#pragma unroll
    for (int i = 0; i < F; i += 4) {
        const float4 v = *reinterpret_cast<const float4*>(src + (i / RUN) * STR + i % RUN);
        dst[i] = v.x;
        dst[i + 1] = v.y;
        dst[i + 2] = v.z;
        dst[i + 3] = v.w;
    }
}

template <int F, int RUN, int STR>
__device__ __forceinline__ void store_f32_slice(float* dst, const float (&v)[F]) {
#pragma unroll
    for (int i = 0; i < F; i += 4)
        *reinterpret_cast<float4*>(dst + (i / RUN) * STR + i % RUN) = make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
}

template <typename T, int D, int H>
__device__ __forceinline__ void load_fwd_partial(Online<EdgeCfg<T, D, H>::F>& st, const TilePartials& tp, int64_t node,
                                                 int h, int64_t off) {
    using C = EdgeCfg<T, D, H>;
    st.m = fmaxf(tp.m[node * H + h], kMinRef);
    st.l = tp.l[node * H + h];
    load_f32_slice<C::F, C::RUN, C::STR>(st.acc, tp.acc + off);
}

// The running max is a lazy reference: it moves only when a score exceeds it
// by more than 2^8 (in the exp2 domain), so the accumulator is rescaled
// rarely; weights stay below 2^8 and the result is unchanged.
constexpr float kRescale = 8.f;

// One partner row of each of two arrays, as gathered.
template <typename T, int D, int H>
struct Rows {
    SliceOf<T, D, H> a, b;  // bf16: 16 registers
    __device__ __forceinline__ void load(const T* __restrict__ A, const T* __restrict__ B, int64_t off) {
        a.load(A + off);
        b.load(B + off);
    }
};

// Two edges for the forward state.  j0/j1 are always valid node ids (callers
// substitute a valid id for missing edges); ok0/ok1 say which of the two are
// edges.
template <typename T, int D, int H>
__device__ __forceinline__ void fwd_step(Online<EdgeCfg<T, D, H>::F>& st, const SliceOf<T, D, H>& q,
                                         const T* __restrict__ K, const T* __restrict__ V, int64_t j0, int64_t j1,
                                         bool ok0, bool ok1, const Lanes<T, D, H>& ln, float sl2, float b0 = 0.f,
                                         float b1 = 0.f) {
    using C = EdgeCfg<T, D, H>;
    Rows<T, D, H> x0, x1;
    x0.load(K, V, ln.off(j0));
    x1.load(K, V, ln.off(j1));
    float s0 = fmaf(group_sum<C::L>(q.dot(x0.a)), sl2, b0);
    float s1 = fmaf(group_sum<C::L>(q.dot(x1.a)), sl2, b1);
    s0 = ok0 ? s0 : kNegInf;
    s1 = ok1 ? s1 : kNegInf;
    const float mb = fmaxf(s0, s1);
    const bool grow = mb > st.m + kRescale;
    if (__builtin_amdgcn_ballot_w64(grow)) {  // wave-uniform; alpha is exactly 1 where the maximum stays
        const float mn = grow ? mb : st.m;
        const float alpha = ex2(st.m - mn);
        st.l *= alpha;
#pragma unroll
        for (int i = 0; i < C::F; ++i) st.acc[i] *= alpha;
        st.m = mn;
    }
    const float p0 = ex2(s0 - st.m);
    const float p1 = ex2(s1 - st.m);
    st.l += p0 + p1;
    if constexpr (sizeof(T) == 2) {
        const uint32_t w = pack_bf16x2(p0, p1);
        x0.b.axpy_w(st.acc, w & 0xFFFFu, w << 16);
        x1.b.axpy_w(st.acc, w >> 16, w & 0xFFFF0000u);
    } else {
#pragma unroll
        for (int i = 0; i < C::F; ++i) st.acc[i] = fmaf(p1, x1.b.f(i), fmaf(p0, x0.b.f(i), st.acc[i]));
    }
}

// The ids of a row's edges, held by the row's G lanes: lane l of the group has
// edges t0 + l (and t0 + G + l where a group is small) of the chunk at t0, one
// coalesced load for the whole chunk, so a chunk can be loaded while the one
// before it is worked on.  An edge's id then goes to the group by a lane
// permute.  (Loading each quad's ids in every lane made each wavefront wait
// for the ids before it could issue the quad's gathers.)
template <int G>
struct EdgeIds {
    static constexpr int R = G < 16 ? 2 : 1;
    static constexpr int kChunk = R * G;
    int v[R];
    // Past the row's end the last edge is repeated; `first` may be read there.
    __device__ __forceinline__ void load(const int32_t* __restrict__ first, int last, int t0, int l) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = t0 + r * G + l;
            v[r] = first[e < last ? e : last];
        }
    }
    // Value of chunk entry u (u0 + a lane's own du, u0 uniform and u0 + du on one side of G).
    __device__ __forceinline__ int pick(int u0, int du, int group4) const {
        int x = v[0];
        if constexpr (R == 2) x = u0 < G ? v[0] : v[1];
        return __builtin_amdgcn_ds_bpermute(group4 + 4 * ((u0 + du) & (G - 1)), x);
    }
    __device__ __forceinline__ int pick(int u, int group4) const {
        if constexpr (G == kWave) return __builtin_amdgcn_readlane(v[0], u);
        return pick(u, 0, group4);
    }
};

// The edge list of one lane group: `deg` ids at cl + a.  Every lane of the
// wavefront takes part in a walk, dmax (uniform) edges long: past its own end
// a group repeats its last edge, and a group without edges reads some row of
// the list, whose weight is 0 but whose values may be infinite, so the caller
// resets what such a group has summed.
template <int G>
struct EdgeList {
    const int32_t* first;
    int deg, last, l, group4;
    __device__ __forceinline__ EdgeList(const int32_t* __restrict__ cl, int64_t len, int64_t a, int deg_, int lane)
        : deg(deg_), last(deg_ > 0 ? deg_ - 1 : 0), l(lane & (G - 1)), group4(4 * (lane & ~(G - 1))) {
        if (deg_ <= 0) a = a < len ? a : len - 1;  // read only where dmax > 0, so len > 0
        first = cl + a;
    }
    __device__ __forceinline__ void ids(EdgeIds<G>& x, int t0) const { x.load(first, last, t0, l); }
    // One edge at a time, the rows of the next DEP edges in flight while one is
    // used: load(x, j) issues an edge's gathers, use(x, t, k) takes edge t (an edge
    // if t < deg; k, a constant, is t mod DEP).
    template <int DEP, class X, class Load, class Use>
    __device__ __forceinline__ void walk_ahead(int dmax, Load load, Use use) const {
        using Ids = EdgeIds<G>;
        constexpr int CH = Ids::kChunk;
        static_assert(CH % DEP == 0, "a block of edges does not straddle chunks");
        if (dmax <= 0) return;
        Ids cur, nxt;
        ids(cur, 0);
        X x[DEP];
        int id[DEP];
        auto pick = [&](const Ids& from, int u) {
#pragma unroll
            for (int k = 0; k < DEP; ++k) id[k] = from.pick(u + k, group4);
        };
        pick(cur, 0);
#pragma unroll
        for (int k = 0; k < DEP; ++k) load(x[k], id[k]);
        for (int t0 = 0; t0 < dmax; t0 += CH) {
            nxt = cur;
            if (t0 + CH < dmax) ids(nxt, t0 + CH);
            const int m = dmax - t0 < CH ? dmax - t0 : CH;
            int u = 0;
            // whole blocks followed by whole blocks: no branch around a load, so that
            // the compiler counts the loads in flight instead of waiting for them all;
            // the next ids by a branch, so that only a chunk's last block waits for nxt
            for (; u < m && t0 + u + 2 * DEP <= dmax; u += DEP) {
                if (u + DEP < CH) pick(cur, u + DEP);
                else pick(nxt, 0);
#pragma unroll
                for (int k = 0; k < DEP; ++k) {
                    use(x[k], t0 + u + k, k);
                    load(x[k], id[k]);
                }
            }
            for (; u < m; u += DEP) {
                if (t0 + u + DEP < dmax) {
                    if (u + DEP < CH) pick(cur, u + DEP);
                    else pick(nxt, 0);
                }
#pragma unroll
                for (int k = 0; k < DEP; ++k) {
                    const int t = t0 + u + k;
                    if (t < dmax) {
                        use(x[k], t, k);
                        if (t + DEP < dmax) load(x[k], id[k]);
                    }
                }
            }
            cur = nxt;
        }
    }
    // Two edges at a time: step(j0, j1, t, ok0, ok1) takes edges t and t + 1.
    template <class Step>
    __device__ __forceinline__ void walk(int dmax, Step step) const {
        using Ids = EdgeIds<G>;
        if (dmax <= 0) return;
        Ids cur, nxt;
        ids(cur, 0);
        for (int t0 = 0; t0 < dmax; t0 += Ids::kChunk) {
            nxt = cur;
            if (t0 + Ids::kChunk < dmax) ids(nxt, t0 + Ids::kChunk);
            const int m = dmax - t0 < Ids::kChunk ? dmax - t0 : Ids::kChunk;
            for (int u = 0; u < m; u += 2) {
                const int t = t0 + u;
                step(cur.pick(u, group4), cur.pick(u + 1, group4), t, t < deg, t + 1 < deg);
            }
            cur = nxt;
        }
    }
};

// The value of lane k (0 or 1) of each L-lane group, in every lane of the group.
template <int L, int k>
__device__ __forceinline__ float group_bcast(float x) {
    const int v = __float_as_int(x);
    if constexpr (L == 2) return __int_as_float(__builtin_amdgcn_mov_dpp(v, k ? 0xF5 : 0xA0, 0xF, 0xF, true));
    const int q = __builtin_amdgcn_mov_dpp(v, k ? 0x55 : 0x00, 0xF, 0xF, true);  // in each quad
    if constexpr (L == 4) return __int_as_float(q);
    return __int_as_float(__builtin_amdgcn_update_dpp(q, q, 0x114, 0xF, 0xA, false));  // row_shr:4 into the odd quads
}

// The value of the first lane of each G-lane group (one node's lanes), in
// every lane of the group.
template <int G>
__device__ __forceinline__ int group_first(int x) {
    if constexpr (G == 1) return x;
    else if constexpr (G == 2) return __builtin_amdgcn_mov_dpp(x, 0xA0, 0xF, 0xF, false);  // quad_perm 0,0,2,2
    else if constexpr (G == 4) return __builtin_amdgcn_mov_dpp(x, 0x00, 0xF, 0xF, false);  // quad_perm 0,0,0,0
    else if constexpr (G == 16) return __builtin_amdgcn_mov_dpp(x, 0x150, 0xF, 0xF, false);  // row_newbcast:0
    else if constexpr (G == 64) return __builtin_amdgcn_readfirstlane(x);
    else return __shfl(x, lane_id() & ~(G - 1), kWave);
}

// Bias (exp2 domain) of a row's edge t at remainder offset a; 0 where the edge
// is missing.  One lane of each (node, head) group reads it.
template <typename LN>
__device__ __forceinline__ float bias_one(const EdgeBias& eb, int64_t a, int t, bool ok, int H, const LN& ln) {
    float x = 0.f;
    if (ln.part == 0 && ok) x = eb.at(a + t, H, ln.h);
    return group_bcast<LN::C::L, 0>(x);
}

// The bias of four edges of each of a wavefront's nodes moves through LDS, so
// that a lane reads one vector (kPer floats, all of one edge, of the quad's
// block of 4 H floats) instead of one float per edge, each group's block at
// `s`.  The wavefront alone uses its block, and its LDS operations take effect
// in program order, so no barrier is needed.
template <typename T, int D, int H>
struct BiasStage {
    using C = EdgeCfg<T, D, H>;
    static constexpr int kPer = 4 * H >= C::G ? 4 * H / C::G : 1;
    static constexpr bool kOn = kPer <= H;
    static constexpr int kWaveFloats = C::NPW * 4 * H;
    // First float of this lane's share; lanes from 4 H on have none.
    __device__ __forceinline__ static int at(const Lanes<T, D, H>& ln) { return (ln.h * C::L + ln.part) * kPer; }
    __device__ __forceinline__ static bool mine(const Lanes<T, D, H>& ln) {
        return kPer * C::G <= 4 * H || at(ln) < 4 * H;
    }
};

template <int P>
__device__ __forceinline__ void ld_floats(float (&v)[P], const float* __restrict__ src) {
    if constexpr (P == 4) {
        const float4 x = *reinterpret_cast<const float4*>(src);
        v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
    } else if constexpr (P == 2) {
        const float2 x = *reinterpret_cast<const float2*>(src);
        v[0] = x.x, v[1] = x.y;
    } else {
        v[0] = *src;
    }
}
template <int P>
__device__ __forceinline__ void st_floats(float* __restrict__ dst, const float (&v)[P]) {
    if constexpr (P == 4) *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    else if constexpr (P == 2) *reinterpret_cast<float2*>(dst) = make_float2(v[0], v[1]);
    else *dst = v[0];
}

__device__ __forceinline__ void lds_order() {
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// This lane's share of the quad's bias block (kPer floats of the edge at input position pos); 0 where !on.
template <int P>
__device__ __forceinline__ void bias_share(float (&v)[P], const float* __restrict__ b, int64_t pos, int H, int e0,
                                           bool on) {
#pragma unroll
    for (int k = 0; k < P; ++k) v[k] = 0.f;
    if (on) ld_floats<P>(v, b + pos * H + e0 % H);
}

// The shares of a group through LDS: the bias (exp2 domain) of the quad's four
// edges for this lane's head.
template <typename T, int D, int H, int P>
__device__ __forceinline__ float4 bias_swap(const float (&v)[P], const Lanes<T, D, H>& ln, float* s) {
    using BS = BiasStage<T, D, H>;
    lds_order();
    if (BS::mine(ln))
#pragma unroll
        for (int k = 0; k < P; ++k) s[BS::at(ln) + k] = v[k];
    lds_order();
    float4 x = make_float4(s[ln.h], s[H + ln.h], s[2 * H + ln.h], s[3 * H + ln.h]);
    lds_order();
    x.x *= kLog2e, x.y *= kLog2e, x.z *= kLog2e, x.w *= kLog2e;
    return x;
}

// Write ds (this lane's head, a quad's four edges) to db: this lane's share, at the input position pos.
template <typename T, int D, int H>
__device__ __forceinline__ void db_quad(float* __restrict__ db, int64_t pos, bool on, float4 ds,
                                        const Lanes<T, D, H>& ln, float* s) {
    using BS = BiasStage<T, D, H>;
    constexpr int P = BS::kPer;
    lds_order();
    if (ln.part == 0) {
        s[ln.h] = ds.x;
        s[H + ln.h] = ds.y;
        s[2 * H + ln.h] = ds.z;
        s[3 * H + ln.h] = ds.w;
    }
    lds_order();
    if (on) {
        float v[P];
#pragma unroll
        for (int k = 0; k < P; ++k) v[k] = s[BS::at(ln) + k];
        st_floats<P>(db + pos * H + BS::at(ln) % H, v);
    }
    lds_order();
}

// EdgeList::walk for a bias kernel, four edges at a time, the bias exchanged
// in LDS when a quad starts; step(j0, j1, t, ok0, ok1, b0, b1) takes two edges,
// after(pos, on) runs once the quad's steps are done (the column pass writes
// dB there).  A lane needs the input position of one edge of each quad, the
// one its share belongs to: from the position list `pos` (read in chunks like
// the ids), or the list position a + t itself where pos is null.  Its share of
// the next quad is loaded a quad ahead.
template <typename T, int D, int H, class Step, class After>
__device__ __forceinline__ void walk_bias(const EdgeList<EdgeCfg<T, D, H>::G>& el, const int32_t* __restrict__ pos,
                                          int64_t a, int dmax, const float* __restrict__ b, const Lanes<T, D, H>& ln,
                                          float* s, Step step, After after) {
    using BS = BiasStage<T, D, H>;
    using Ids = EdgeIds<EdgeCfg<T, D, H>::G>;
    constexpr int P = BS::kPer, CH = Ids::kChunk;
    static_assert(CH % 4 == 0, "quads do not cross chunks");
    if (dmax <= 0) return;
    const int e0 = BS::at(ln), u = (e0 / H) & 3;
    const bool mine = BS::mine(ln);
    const int32_t* pfirst = pos ? pos + (el.deg > 0 ? a : 0) : nullptr;
    Ids cur, nxt, pcur, pnxt;
    el.ids(cur, 0);
    pcur = cur;
    if (pos) pcur.load(pfirst, el.last, 0, el.l);
    nxt = cur;
    pnxt = pcur;
    // this lane's edge of the quad at chunk offset c (uniform) of the chunk at t0
    auto at = [&](const Ids& p, int t0, int c) -> int64_t { return pos ? int64_t(p.pick(c, u, el.group4)) : a + t0 + c + u; };
    float v[P];
    int64_t p0 = at(pcur, 0, 0);
    bias_share<P>(v, b, p0, H, e0, mine && u < el.deg);
    for (int t0 = 0; t0 < dmax; t0 += CH) {
        const bool more = t0 + CH < dmax;
        if (more) {
            el.ids(nxt, t0 + CH);
            if (pos) pnxt.load(pfirst, el.last, t0 + CH, el.l);
        }
        const int m = dmax - t0 < CH ? dmax - t0 : CH;
        for (int c = 0; c < m; c += 4) {
            const int t = t0 + c;
            float vn[P];
#pragma unroll
            for (int k = 0; k < P; ++k) vn[k] = 0.f;
            int64_t p1 = p0;
            if (t + 4 < dmax) {  // the next quad's share
                p1 = c + 4 < CH ? at(pcur, t0, c + 4) : at(pnxt, t0 + CH, 0);
                bias_share<P>(vn, b, p1, H, e0, mine && t + 4 + u < el.deg);
            }
            const float4 x = bias_swap<T, D, H, P>(v, ln, s);
            step(cur.pick(c, el.group4), cur.pick(c + 1, el.group4), t, t < el.deg, t + 1 < el.deg, x.x, x.y);
            if (t + 2 < dmax)
                step(cur.pick(c + 2, el.group4), cur.pick(c + 3, el.group4), t + 2, t + 2 < el.deg, t + 3 < el.deg,
                     x.z, x.w);
            after(p0, mine && t + u < el.deg);
            p0 = p1;
#pragma unroll
            for (int k = 0; k < P; ++k) v[k] = vn[k];
        }
        cur = nxt;
        pcur = pnxt;
    }
}

// ------------------------------------------------------- work distribution
// Workgroups go to the 8 XCDs round-robin.  Each XCD walks contiguous runs of
// kXcdRows nodes (runs c, c + 8, c + 16, ...), so the partners of neighbouring
// rows share its L2, while a stretch of high-degree nodes, which a reordered
// power-law graph has at its start, is spread over all XCDs (with one eighth of
// the nodes per XCD the first one held 40% of the edges: forward and backward
// of 1M power-law nodes, 4 x 32, 5.9 ms; in runs, and the long rows' runs in the
// same launch, 3.0).  The runs per XCD divide the nodes evenly.
constexpr int64_t kXcdRows = 2048;
struct RowGrid {
    unsigned run = 1;   // workgroups per run
    unsigned grid = 8;  // workgroups in all
};
inline RowGrid row_grid(int64_t n, int64_t rows_per_block) {
    const int64_t blocks = cdiv(n, rows_per_block);
    const int64_t m = n / (kXcds * kXcdRows) > 1 ? n / (kXcds * kXcdRows) : 1;
    RowGrid g;
    g.run = unsigned(cdiv(blocks > 0 ? blocks : 1, kXcds * m));
    g.grid = unsigned(kXcds * m * g.run);
    return g;
}
__device__ __forceinline__ int64_t row_block(unsigned b, unsigned run) {
    const unsigned k = b / kXcds;
    return (int64_t(k / run) * kXcds + b % kXcds) * run + k % run;
}

// Remainder rows (columns) with more than GT_LONG_ROW edges, up to a row that
// attends to every node, are cut into runs: a run is walked by one lane group
// like a short row, in the same launch (the runs' workgroups first, the short
// rows fill the chip behind them), leaves its partial state, and one
// workgroup per long row merges its runs with the row's dense-tile partial.
// (A token row and column of 980K edges beside 1M short rows:
// chunks of 2,048 edges, a workgroup each, launched after the short rows took
// 0.20 ms a pass and their merge 0.13-0.23 ms; forward and backward 2.84 -> 2.34
// ms.  128 molecules and a token row of 3,137 edges: 155 -> 60 us, with one launch
// and a merge per pass instead of six.)
// A run holds kMinRun edges, more where the long rows' edges would give more
// runs than run_spread: a wavefront of them for each of the chip's 1,024 SIMDs,
// and 4,096 at least.  (1M power-law nodes, 4.6M edges in 4,000 long rows, forward
// / backward, us: 1 x 32 in 4,096 runs 590 / 1425, in 32,768 421 / 997, in 131,072
// 414 / 1027; 4 x 32 in 4,096 885 / 2095, at most 256 edges each 893 / 2113, in
// 32,768 897 / 2128.)  But no more than kMaxRun, the longest short row: a run's sums are
// serial fp32 chains.  (Moving the sums of longer runs to their partial state
// every 256 edges instead costs the short rows registers: 1M x 8 x 32 forward 1.87 ->
// 1.92 ms, and 1.90 where the runs' walk is apart from theirs.)  Past
// kMaxRuns runs (268M edges of long rows) the partial states, up to 8 KB each, would
// outgrow the features, so runs lengthen.
constexpr int kMinRun = 32;
constexpr int kMaxRun = GT_LONG_ROW;
constexpr int64_t kMaxRuns = int64_t(1) << 20;
constexpr int run_spread_bits(int H, int D) { return H * D >= 256 ? 12 : H * D >= 128 ? 13 : H * D >= 64 ? 14 : 15; }
constexpr int64_t run_spread(int H, int D) { return int64_t(1) << run_spread_bits(H, D); }
// Up to one wavefront of long rows, every lane group finds its run from the
// rows' lengths itself; beyond, the rows' first runs are listed before.
constexpr int64_t kPlanFree = kWave;

struct LongRows {
    const int32_t* list = nullptr;
    int64_t n = 0;
    const int64_t* ptr = nullptr;
    const int64_t* off = nullptr;  // [n + 2]: first run of each row, their number, the run length; null: none listed
    int spread_bits = 0;           // run_spread_bits of the features
};

// Edges of a run, `edges` being those of all long rows.
__device__ __forceinline__ int run_length(int64_t edges, int spread_bits) {
    int64_t c = (edges + (int64_t(1) << spread_bits) - 1) >> spread_bits;
    if (c > kMaxRun) c = cdiv(edges, kMaxRuns) > kMaxRun ? cdiv(edges, kMaxRuns) : kMaxRun;
    return c > kMinRun ? int((c + kMinRun - 1) / kMinRun * kMinRun) : kMinRun;
}
// At most so many runs beyond one per row: edges <= nnz over the run length.
inline int64_t run_bound(int64_t nnz, int64_t spread) {
    const int64_t a = nnz / kMinRun < spread ? nnz / kMinRun : spread;
    const int64_t b = nnz / kMaxRun < kMaxRuns ? nnz / kMaxRun : kMaxRuns;
    return a > b ? a : b;
}

// Every long row's runs, one row per lane (lr.n <= kPlanFree).
struct LaneRuns {
    int incl, cnt, len;  // runs up to and with this row, its own, the run length
    __device__ __forceinline__ explicit LaneRuns(const LongRows& lr) {
        const int lane = lane_id();
        int64_t deg = 0;
        if (lane < lr.n) {
            const int64_t i = lr.list[lane];
            deg = lr.ptr[i + 1] - lr.ptr[i];
        }
        len = run_length(wave_sum(deg), lr.spread_bits);
        cnt = int(cdiv(deg, len));
        incl = cnt;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int up = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += up;
        }
    }
};

// A run: its node and its edges at a, deg of them (-1 past the last run).
struct Run {
    int64_t a;
    int32_t i;
    int deg;
};
// Run v (each lane its own).  All lanes take part.
__device__ __forceinline__ Run run_at(const LongRows& lr, int64_t v) {
    int64_t r, first;
    int len;
    bool on;
    if (!lr.off) {
        const LaneRuns x(lr);
        on = v < __shfl(x.incl, kWave - 1, kWave);
        int k = 0;  // rows whose runs all lie before v
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1)
            if (__shfl(x.incl, k + o - 1, kWave) <= v) k += o;
        r = on ? k : 0;  // past the last run k would pass the list's end
        first = __shfl(x.incl - x.cnt, int(r), kWave);
        len = x.len;
    } else {
        on = v < lr.off[lr.n];
        int64_t lo = 0, hi = lr.n;  // the last r with off[r] <= v
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (lr.off[mid] <= v) lo = mid;
            else hi = mid;
        }
        r = lo;
        first = lr.off[lo];
        len = int(lr.off[lr.n + 1]);
    }
    const int32_t i = lr.list[r];
    const int64_t a = lr.ptr[i], e0 = on ? (v - first) * len : 0, left = lr.ptr[i + 1] - a - e0;
    return Run{a + e0, i, on ? (left < len ? int(left) : len) : -1};
}
// Runs [c0, c1) of list entry r (uniform).
__device__ __forceinline__ void run_range(const LongRows& lr, int64_t r, int64_t& c0, int64_t& c1) {
    if (!lr.off) {
        const LaneRuns x(lr);
        c1 = __shfl(x.incl, int(r), kWave);
        c0 = c1 - __shfl(x.cnt, int(r), kWave);
    } else {
        c0 = lr.off[r];
        c1 = lr.off[r + 1];
    }
}

// What one lane group of a rows (columns) kernel walks: a node's edges, or a
// run of a long row's; deg = -1 for nothing (a long row, or past the end).
struct Work {
    int64_t a;
    int32_t i, run;  // run: -1 for a node's own row
    int deg;
    // Workgroups below run_blocks take runs, rows_per_block of them each.
    __device__ __forceinline__ Work(int64_t n, const int64_t* __restrict__ ptr, const LongRows& lr,
                                    unsigned run_blocks, unsigned xcd_run, int rows_per_block, int slot) {
        if (blockIdx.x < run_blocks) {
            run = int32_t(blockIdx.x) * rows_per_block + slot;
            const Run r = run_at(lr, run);
            i = r.i;
            a = r.a;
            deg = r.deg;
            return;
        }
        run = -1;
        const int64_t node = row_block(blockIdx.x - run_blocks, xcd_run) * rows_per_block + slot;
        i = node < n ? int32_t(node) : 0;
        a = ptr[i];
        const int64_t dg = ptr[i + 1] - a;
        deg = node < n && dg <= GT_LONG_ROW ? int(dg) : -1;
    }
    __device__ __forceinline__ bool own() const { return run < 0 && deg >= 0; }
};

// The first runs of more than kPlanFree long rows: in one workgroup, which takes
// 2.2 us for every 1,024 rows, up to kPlanOne rows; beyond, the edges' total, the
// rows' runs and their scan take a launch or two each, 20 us in all (20,000 rows
// 45 us in one workgroup, 200,000 rows 430).
constexpr int kPlanThr = 1024;
constexpr int64_t kPlanOne = 8192;
constexpr int kPlanSums = 64;

__device__ __forceinline__ int64_t long_length(const LongRows& lr, int64_t r) {
    if (r >= lr.n) return 0;
    const int64_t i = lr.list[r];
    return lr.ptr[i + 1] - lr.ptr[i];
}

__global__ __launch_bounds__(kThreads) void k_long_total(LongRows lr, int64_t* __restrict__ sums) {
    __shared__ int64_t s_w[kThreads / kWave];
    const int t = threadIdx.x;
    int64_t sum = 0;
    for (int64_t r = blockIdx.x * int64_t(kThreads) + t; r < lr.n; r += int64_t(kPlanSums) * kThreads)
        sum += long_length(lr, r);
    sum = wave_sum(sum);
    if (t % kWave == 0) s_w[t / kWave] = sum;
    __syncthreads();
    if (t > 0) return;
    for (int k = 1; k < kThreads / kWave; ++k) sum += s_w[k];
    sums[blockIdx.x] = sum;
}

__global__ __launch_bounds__(kThreads) void k_long_counts(LongRows lr, const int64_t* __restrict__ sums,
                                                          int32_t* __restrict__ counts, int64_t* __restrict__ off) {
    static_assert(kPlanSums == kWave, "one sum a lane");
    const int len = run_length(wave_sum(sums[lane_id()]), lr.spread_bits);
    const int64_t r = blockIdx.x * int64_t(kThreads) + threadIdx.x;
    if (r < lr.n) counts[r] = int32_t(cdiv(long_length(lr, r), len));
    if (r == 0) off[lr.n + 1] = len;
}

__global__ __launch_bounds__(kPlanThr) void k_long_plan(LongRows lr, int64_t* __restrict__ off) {
    __shared__ int64_t s_w[kPlanThr / kWave];
    const int t = threadIdx.x, w = t / kWave, lane = lane_id();
    int64_t sum = 0;
    for (int64_t r = t; r < lr.n; r += kPlanThr) sum += long_length(lr, r);
    sum = wave_sum(sum);
    if (lane == 0) s_w[w] = sum;
    __syncthreads();
    int64_t total = 0;
    for (int k = 0; k < kPlanThr / kWave; ++k) total += s_w[k];
    const int len = run_length(total, lr.spread_bits);
    int64_t base = 0;
    for (int64_t r0 = 0; r0 < lr.n; r0 += kPlanThr) {
        const int64_t cnt = cdiv(long_length(lr, r0 + t), len);
        int64_t incl = cnt;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int64_t up = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += up;
        }
        __syncthreads();  // s_w has been read
        if (lane == kWave - 1) s_w[w] = incl;
        __syncthreads();
        int64_t before = base, all = 0;
        for (int k = 0; k < kPlanThr / kWave; ++k) {
            if (k < w) before += s_w[k];
            all += s_w[k];
        }
        if (r0 + t < lr.n) off[r0 + t] = before + incl - cnt;
        base += all;
    }
    if (t == 0) {
        off[lr.n] = base;
        off[lr.n + 1] = len;
    }
}

// Floats a run leaves (float4-aligned): the forward acc[H D], m[H], l[H]; the
// row pass a[H D], b[H D], d[H]; the column pass dk[H D], dv[H D].
constexpr int64_t pad4(int64_t x) { return (x + 3) & ~int64_t(3); }
constexpr int64_t fwd_run_floats(int H, int D) { return int64_t(H) * D + pad4(2 * H); }
constexpr int64_t row_run_floats(int H, int D) { return 2 * int64_t(H) * D + pad4(H); }
constexpr int64_t col_run_floats(int H, int D) { return 2 * int64_t(H) * D; }

constexpr int64_t kFoldBlocks = 4096;
struct LongPlan {
    int64_t* off = nullptr;  // [n_long + 2] where the runs are planned before
    int64_t* sums = nullptr; // [kPlanSums], counts [n_long] and a scan's scratch: over kPlanOne rows
    int32_t* counts = nullptr;
    ScanTmp scan;
    float* part = nullptr;   // [max_runs, floats per run]
    int64_t max_runs = 0;
    int fold = 1;            // parts a row's runs are folded into before the merge (1: not folded)
    unsigned blocks(int64_t rows_per_block) const {
        return max_runs > 0 ? xcd_grid(cdiv(max_runs, rows_per_block)) : 0;
    }
};

inline LongPlan long_plan_take(Ws& ws, int64_t n_long, int64_t nnz, int64_t spread, int64_t per_run) {
    LongPlan lp;
    if (n_long <= 0) return lp;
    const int64_t more = run_bound(nnz, spread), parts = kFoldBlocks / n_long;
    lp.max_runs = n_long + more;
    // few long rows may hold thousands of runs each: 64 workgroups a row fold
    // them first (more rows: fewer each, none from 2,048 rows on)
    if (more > 512) lp.fold = int(parts < 1 ? 1 : parts > 64 ? 64 : parts);
    if (n_long > kPlanFree) lp.off = ws.take<int64_t>(size_t(n_long + 2));
    if (n_long > kPlanOne) {
        lp.sums = ws.take<int64_t>(kPlanSums);
        lp.counts = ws.take<int32_t>(size_t(n_long));
        lp.scan.block_sums = ws.take<int64_t>(size_t(scan_tmp_elems(n_long)));
    }
    lp.part = ws.take<float>(size_t(lp.max_runs * per_run));
    return lp;
}

gt_status long_rows(const int32_t* list, int64_t n_long, const int64_t* ptr, int spread_bits, const LongPlan& lp,
                    LongRows& lr, hipStream_t s) {
    lr = LongRows{};
    if (n_long <= 0) return GT_OK;
    lr.list = list;
    lr.n = n_long;
    lr.ptr = ptr;
    lr.spread_bits = spread_bits;
    if (n_long > kPlanOne) {
        k_long_total<<<kPlanSums, kThreads, 0, s>>>(lr, lp.sums);
        GT_LAUNCH_CHECK("long_total");
        k_long_counts<<<unsigned(cdiv(n_long, kThreads)), kThreads, 0, s>>>(lr, lp.sums, lp.counts, lp.off);
        GT_LAUNCH_CHECK("long_counts");
        const gt_status st = exclusive_scan_i32(lp.counts, n_long, lp.off, lp.scan, s);
        if (st != GT_OK) return st;
    } else if (lp.off) {
        k_long_plan<<<1, kPlanThr, 0, s>>>(lr, lp.off);
        GT_LAUNCH_CHECK("long_plan");
    }
    lr.off = lp.off;
    return GT_OK;
}

// ------------------------------------------------------------------ forward

template <typename T, int D, int H, bool kBias>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(kBias || kLaneBytes<T, D, H> > 32 ? 1 : 6))) void k_fwd_rows(int64_t n, const int64_t* __restrict__ rp,
                                                       const int32_t* __restrict__ cl, int64_t len,
                                                       const T* __restrict__ Q,
                                                       const T* __restrict__ K, const T* __restrict__ V, float sl2,
                                                       T* __restrict__ O, float* __restrict__ LSE, TilePartials tp,
                                                       EdgeBias eb, unsigned xcd_run,
    LongRows lr, unsigned run_blocks, float* __restrict__ part) {
    using C = EdgeCfg<T, D, H>;
    const Lanes<T, D, H> ln(lane_id());
    constexpr int kRows = C::NPW * (kThreads / kWave);
    const Work w(n, rp, lr, run_blocks, xcd_run, kRows, int(threadIdx.x) / C::G);
    const int64_t i = w.i, a = w.a;
    const int deg = w.deg;
    const int dmax = uniform(wave_max(deg));
    const int64_t off = ln.off(i);
    SliceOf<T, D, H> q;
    q.load(Q + off);
    Online<C::F> st;
    auto begin = [&] {
        st = Online<C::F>();
        if (w.own() && tp.has_row(i)) load_fwd_partial<T, D, H>(st, tp, i, ln.h, off);
    };
    begin();
    const EdgeList<C::G> el(cl, len, a, deg, lane_id());
    using BS = BiasStage<T, D, H>;
    if constexpr (kBias && BS::kOn) {
        __shared__ float s_bias[kThreads / kWave][BS::kWaveFloats];
        float* sb = s_bias[threadIdx.x / kWave] + ln.slot * 4 * H;
        walk_bias<T, D, H>(
            el, eb.sp_pos, a, dmax, eb.b, ln, sb,
            [&](int64_t j0, int64_t j1, int, bool ok0, bool ok1, float b0, float b1) {
                fwd_step<T, D, H>(st, q, K, V, j0, j1, ok0, ok1, ln, sl2, b0, b1);
            },
            [](int64_t, bool) {});
    } else {
        el.walk(dmax, [&](int64_t j0, int64_t j1, int t, bool ok0, bool ok1) {
            float b0 = 0.f, b1 = 0.f;
            if constexpr (kBias) {
                b0 = bias_one(eb, a, t, ok0, H, ln);
                b1 = bias_one(eb, a, t + 1, ok1, H, ln);
            }
            fwd_step<T, D, H>(st, q, K, V, j0, j1, ok0, ok1, ln, sl2, b0, b1);
        });
    }
    if (deg <= 0) begin();
    if (w.run >= 0) {
        if (deg >= 0) {
            float* out = part + int64_t(w.run) * fwd_run_floats(H, D);
            store_f32_slice<C::F, C::RUN, C::STR>(out + ln.off(0), st.acc);
            if (ln.part == 0) {
                out[H * D + ln.h] = st.m;
                out[H * D + H + ln.h] = st.l;
            }
        }
    } else if (w.own()) {
        const float inv = st.l > 0.f ? 1.f / st.l : 0.f;
        store_slice<T, C::F, C::STR>(O + off, st.acc, inv);
        if (ln.part == 0) LSE[i * H + ln.h] = st.l > 0.f ? (st.m + __log2f(st.l)) * kLn2 : kNegInf;
    }
}

// ----------------------------------------------------------------- backward

// Row pass.  With D_i = sum_j P_ij dP_ij (which equals <dO_i, O_i> for the
// exact output O; the stored O is rounded to the feature dtype, so D is formed
// from the edges instead),
//   dQ_i = scale * sum_j P_ij (dP_ij - D_i) K_j = scale * (A_i - D_i B_i),
//   A_i = sum_j P_ij dP_ij K_j,  B_i = sum_j P_ij K_j,
// so one pass over the row yields A, B and D together.
template <int F>
struct RowSums {
    Acc<F> a, b;
    float d[2] = {0.f, 0.f};  // D over the even and the odd edges
};

template <typename T, int D, int H>
__device__ __forceinline__ void dq_step(RowSums<EdgeCfg<T, D, H>::F>& rs, const SliceOf<T, D, H>& q,
                                        const SliceOf<T, D, H>& g, float lse2, const Rows<T, D, H>& x, bool ok,
                                        int odd, float sl2, float bias = 0.f) {
    using C = EdgeCfg<T, D, H>;
    const float s = fmaf(group_sum<C::L>(q.dot(x.a)), sl2, bias);
    const float dp = group_sum<C::L>(g.dot(x.b));
    const float e = ex2(s - lse2);
    const float p = ok ? e : 0.f;
    const float w = p * dp;
    rs.d[odd] += w;
#pragma unroll
    for (int f = 0; f < C::F; ++f) {
        const float k = x.a.f(f);
        rs.a.v[f] = fmaf(w, k, rs.a.v[f]);
        rs.b.v[f] = fmaf(p, k, rs.b.v[f]);
    }
}

template <typename T, int D, int H>
__device__ __forceinline__ void load_row_partial(RowSums<EdgeCfg<T, D, H>::F>& rs, const TilePartials& tp,
                                                 int64_t node, int h, int64_t off) {
    using C = EdgeCfg<T, D, H>;
    load_f32_slice<C::F, C::RUN, C::STR>(rs.a.v, tp.acc + off);
    load_f32_slice<C::F, C::RUN, C::STR>(rs.b.v, tp.acc2 + off);
    rs.d[0] = tp.m[node * H + h];
}

template <typename T, int D, int H, bool kBias>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(kBias && kEdgeWaves<T, D, H> > 2 ? kEdgeWaves<T, D, H> - 1 : kEdgeWaves<T, D, H>))) void k_bwd_rows(int64_t n, const int64_t* __restrict__ rp,
                                                       const int32_t* __restrict__ cl, int64_t len,
                                                       const T* __restrict__ Q,
                                                       const T* __restrict__ K, const T* __restrict__ V,
                                                       const T* __restrict__ dO, const float* __restrict__ LSE,
                                                       float* __restrict__ Dv, float2* __restrict__ stat, float sl2,
                                                       float scale,
                                                       T* __restrict__ dQ, TilePartials tp, EdgeBias eb, unsigned xcd_run,
    LongRows lr, unsigned run_blocks, float* __restrict__ part) {
    using C = EdgeCfg<T, D, H>;
    const Lanes<T, D, H> ln(lane_id());
    constexpr int kRows = C::NPW * (kThreads / kWave);
    const Work w(n, rp, lr, run_blocks, xcd_run, kRows, int(threadIdx.x) / C::G);
    const int64_t i = w.i, a = w.a;
    const int deg = w.deg;
    const int dmax = uniform(wave_max(deg));
    const int64_t off = ln.off(i);
    SliceOf<T, D, H> q, g;
    q.load(Q + off);
    g.load(dO + off);
    const float lse2 = LSE[i * H + ln.h] * kLog2e;
    RowSums<C::F> rs;
    auto begin = [&] {
        rs = RowSums<C::F>();
        if (w.own() && tp.has_row(i)) load_row_partial<T, D, H>(rs, tp, i, ln.h, off);
    };
    begin();
    const EdgeList<C::G> el(cl, len, a, deg, lane_id());
    using BS = BiasStage<T, D, H>;
    if constexpr (kBias && BS::kOn) {
        __shared__ float s_bias[kThreads / kWave][BS::kWaveFloats];
        float* sb = s_bias[threadIdx.x / kWave] + ln.slot * 4 * H;
        walk_bias<T, D, H>(
            el, eb.sp_pos, a, dmax, eb.b, ln, sb,
            [&](int64_t j0, int64_t j1, int, bool ok0, bool ok1, float b0, float b1) {
                Rows<T, D, H> x0, x1;
                x0.load(K, V, ln.off(j0));
                x1.load(K, V, ln.off(j1));
                dq_step<T, D, H>(rs, q, g, lse2, x0, ok0, 0, sl2, b0);
                dq_step<T, D, H>(rs, q, g, lse2, x1, ok1, 1, sl2, b1);
            },
            [](int64_t, bool) {});
    } else {
        el.template walk_ahead<kAheadRows, Rows<T, D, H>>(
            dmax, [&](Rows<T, D, H>& x, int64_t jj) { x.load(K, V, ln.off(jj)); },
            [&](const Rows<T, D, H>& x, int t, int k) {
                const bool ok = t < el.deg;
                float b = 0.f;
                if constexpr (kBias) b = bias_one(eb, a, t, ok, H, ln);
                dq_step<T, D, H>(rs, q, g, lse2, x, ok, k & 1, sl2, b);
            });
    }
    if (deg <= 0) begin();
    if (w.run >= 0) {
        if (deg >= 0) {
            float* out = part + int64_t(w.run) * row_run_floats(H, D);
            store_f32_slice<C::F, C::RUN, C::STR>(out + ln.off(0), rs.a.v);
            store_f32_slice<C::F, C::RUN, C::STR>(out + H * D + ln.off(0), rs.b.v);
            if (ln.part == 0) out[2 * H * D + ln.h] = rs.d[0] + rs.d[1];
        }
    } else if (w.own()) {
        const float d = rs.d[0] + rs.d[1];
#pragma unroll
        for (int f = 0; f < C::F; ++f) rs.a.v[f] = fmaf(-d, rs.b.v[f], rs.a.v[f]);
        store_slice<T, C::F, C::STR>(dQ + off, rs.a.v, scale);
        if (ln.part == 0) {
            if (Dv) Dv[i * H + ln.h] = d;
            if (stat) stat[i * H + ln.h] = make_float2(lse2, d);
        }
    }
}

// Column pass: dK_j = scale * sum_i dS_ij Q_i, dV_j = sum_i P_ij dO_i over the in-edges of j.
// With a bias, c0/c1 are the two in-edges' CSC positions; the bias is read and
// dB = dS written at their CSR positions.
template <typename T, int D, int H, bool kBias = false>
__device__ __forceinline__ void dkv_step(Acc<EdgeCfg<T, D, H>::F>& dk, Acc<EdgeCfg<T, D, H>::F>& dv,
                                         const SliceOf<T, D, H>& k, const SliceOf<T, D, H>& v,
                                         const T* __restrict__ Q,
                                         const T* __restrict__ dO, const float2* __restrict__ stat, int64_t i0,
                                         int64_t i1, bool ok0, bool ok1, const Lanes<T, D, H>& ln, float sl2,
                                         const EdgeBias& eb = EdgeBias{}, int64_t c0 = 0, int64_t c1 = 0,
                                         float* staged = nullptr) {
    using C = EdgeCfg<T, D, H>;
    Rows<T, D, H> r0, r1;
    r0.load(Q, dO, ln.off(i0));
    r1.load(Q, dO, ln.off(i1));
    // lane 0 of each (node, head) group reads the first edge's pair, lane 1 the second's; both go to the group
    // by DPP (one load with all its lanes of use; two loads of one lane in two each: 2.18 against 2.13 ms at
    // 1M x 8 x 32, 31 edges a node)
    const float2 stt = stat[(ln.part & 1 ? i1 : i0) * H + ln.h];
    const float l0 = group_bcast<C::L, 0>(stt.x), D0 = group_bcast<C::L, 0>(stt.y);
    const float l1 = group_bcast<C::L, 1>(stt.x), D1 = group_bcast<C::L, 1>(stt.y);
    float s0 = group_sum<C::L>(r0.a.dot(k)) * sl2;
    float s1 = group_sum<C::L>(r1.a.dot(k)) * sl2;
    int64_t e0 = 0, e1 = 0;
    if (kBias && staged) {
        // staged: the bias came through LDS (staged[0..1]), dS goes back in staged[2..3]
        s0 += staged[0];
        s1 += staged[1];
    } else if constexpr (kBias) {
        // the node's first lane reads the CSR positions, one lane per head the bias
        int p0 = 0, p1 = 0;
        if ((lane_id() & (C::G - 1)) == 0) {
            p0 = ok0 ? eb.csc_pos[c0] : 0;
            p1 = ok1 ? eb.csc_pos[c1] : 0;
        }
        e0 = group_first<C::G>(p0);
        e1 = group_first<C::G>(p1);
        float y0 = 0.f, y1 = 0.f;
        if (ln.part == 0) {
            y0 = ok0 ? eb.at_input(e0, H, ln.h) : 0.f;
            y1 = ok1 ? eb.at_input(e1, H, ln.h) : 0.f;
        }
        s0 += group_bcast<C::L, 0>(y0);
        s1 += group_bcast<C::L, 0>(y1);
    }
    const float dp0 = group_sum<C::L>(r0.b.dot(v));
    const float dp1 = group_sum<C::L>(r1.b.dot(v));
    const float x0 = ex2(s0 - l0), x1 = ex2(s1 - l1);
    const float p0 = ok0 ? x0 : 0.f;
    const float p1 = ok1 ? x1 : 0.f;
    const float ds0 = p0 * (dp0 - D0);
    const float ds1 = p1 * (dp1 - D1);
    if (kBias && staged) {
        staged[2] = ok0 ? ds0 : 0.f;
        staged[3] = ok1 ? ds1 : 0.f;
    } else if constexpr (kBias) {
        if (ln.part == 0) {
            if (ok0) eb.db[e0 * H + ln.h] = ds0;
            if (ok1) eb.db[e1 * H + ln.h] = ds1;
        }
    }
#pragma unroll
    for (int f = 0; f < C::F; ++f) {
        dk.v[f] = fmaf(ds1, r1.a.f(f), fmaf(ds0, r0.a.f(f), dk.v[f]));
        dv.v[f] = fmaf(p1, r1.b.f(f), fmaf(p0, r0.b.f(f), dv.v[f]));
    }
}

template <typename T, int D, int H, bool kBias>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(kBias && kEdgeWaves<T, D, H> > 2 ? kEdgeWaves<T, D, H> - 1 : 1))) void k_bwd_cols(int64_t n, const int64_t* __restrict__ cp,
                                                       const int32_t* __restrict__ rw, int64_t len,
                                                       const T* __restrict__ Q,
                                                       const T* __restrict__ K, const T* __restrict__ V,
                                                       const T* __restrict__ dO, const float2* __restrict__ stat,
                                                       float sl2, float scale, T* __restrict__ dK,
                                                       T* __restrict__ dV, TilePartials tpk, TilePartials tpv,
                                                       EdgeBias eb, unsigned xcd_run,
    LongRows lr, unsigned run_blocks, float* __restrict__ part) {
    using C = EdgeCfg<T, D, H>;
    const Lanes<T, D, H> ln(lane_id());
    constexpr int kRows = C::NPW * (kThreads / kWave);
    const Work w(n, cp, lr, run_blocks, xcd_run, kRows, int(threadIdx.x) / C::G);
    const int64_t j = w.i, a = w.a;
    const int deg = w.deg;
    const int dmax = uniform(wave_max(deg));
    const int64_t off = ln.off(j);
    SliceOf<T, D, H> k, v;
    k.load(K + off);
    v.load(V + off);
    Acc<C::F> dk, dv;
    auto begin = [&] {
        dk = dv = Acc<C::F>();
        if (w.own() && tpk.has_col(j)) {
            load_f32_slice<C::F, C::RUN, C::STR>(dk.v, tpk.acc + off);
            load_f32_slice<C::F, C::RUN, C::STR>(dv.v, tpv.acc + off);
        }
    };
    begin();
    const EdgeList<C::G> el(rw, len, a, deg, lane_id());
    using BS = BiasStage<T, D, H>;
    if constexpr (kBias && BS::kOn) {
        __shared__ float s_bias[kThreads / kWave][BS::kWaveFloats];
        float* sb = s_bias[threadIdx.x / kWave] + ln.slot * 4 * H;
        float4 ds = make_float4(0.f, 0.f, 0.f, 0.f);
        walk_bias<T, D, H>(
            el, eb.csc_pos, a, dmax, eb.b, ln, sb,
            [&](int64_t i0, int64_t i1, int t, bool ok0, bool ok1, float b0, float b1) {
                float x[4] = {b0, b1, 0.f, 0.f};
                dkv_step<T, D, H, true>(dk, dv, k, v, Q, dO, stat, i0, i1, ok0, ok1, ln, sl2, eb, 0, 0, x);
                if (t & 2) ds.z = x[2], ds.w = x[3];
                else ds.x = x[2], ds.y = x[3], ds.z = 0.f, ds.w = 0.f;
            },
            [&](int64_t pos, bool on) { db_quad<T, D, H>(eb.db, pos, on, ds, ln, sb); });
    } else {
        el.walk(dmax, [&](int64_t i0, int64_t i1, int t, bool ok0, bool ok1) {
            dkv_step<T, D, H, kBias>(dk, dv, k, v, Q, dO, stat, i0, i1, ok0, ok1, ln, sl2, eb, a + t, a + t + 1);
        });
    }
    if (deg <= 0) begin();
    if (w.run >= 0) {
        if (deg >= 0) {
            float* out = part + int64_t(w.run) * col_run_floats(H, D);
            store_f32_slice<C::F, C::RUN, C::STR>(out + ln.off(0), dk.v);
            store_f32_slice<C::F, C::RUN, C::STR>(out + H * D + ln.off(0), dv.v);
        }
    } else if (w.own()) {
        store_slice<T, C::F, C::STR>(dK + off, dk.v, scale);
        store_slice<T, C::F, C::STR>(dV + off, dv.v, 1.f);
    }
}

// --------------------------------------------------- merge of the long rows
// Where a row may hold many runs, `parts` workgroups a row first fold them: each
// sums (the forward: merges) its share of the runs into the first of them.
// Then one workgroup per row: H D / 4 threads take four features of a run (or
// of a share's first run) each, NG groups of them every NG-th one, and the groups' sums
// are added in order in LDS.  All in a fixed order: results are reproducible.
template <int H, int D>
struct MergeCfg {
    static constexpr int Q4 = H * D / 4, NG = kThreads / Q4;
    static_assert(kThreads % Q4 == 0, "threads per run divide the workgroup");
};
__device__ __forceinline__ int64_t fold_share(int64_t runs, int parts) { return parts > 1 ? cdiv(runs, parts) : 1; }

template <typename T>
__device__ __forceinline__ void store4(T* __restrict__ p, float4 v) {
    if constexpr (sizeof(T) == 2)
        *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
    else
        *reinterpret_cast<float4*>(p) = v;
}
__device__ __forceinline__ float4 add4(float4 a, float4 b) {
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
// a wa + b wb
__device__ __forceinline__ float4 mix4(float4 a, float wa, float4 b, float wb) {
    return make_float4(fmaf(b.x, wb, a.x * wa), fmaf(b.y, wb, a.y * wa), fmaf(b.z, wb, a.z * wa),
                       fmaf(b.w, wb, a.w * wa));
}

template <int D, int H>
__global__ __launch_bounds__(kThreads) void k_fwd_fold(LongRows lr, int parts, float* __restrict__ part) {
    constexpr int64_t kF = fwd_run_floats(H, D);
    int64_t c0, c1;
    run_range(lr, blockIdx.x / parts, c0, c1);
    const int64_t share = fold_share(c1 - c0, parts);
    c0 += (blockIdx.x % parts) * share;
    c1 = c0 + share < c1 ? c0 + share : c1;
    const int q = threadIdx.x, h = 4 * q / D;
    if (q >= H * D / 4 || c1 - c0 < 2) return;
    float m = kMinRef, l = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int64_t c = c0; c < c1; ++c) {
        const float* pc = part + c * kF;
        const float4 v = *reinterpret_cast<const float4*>(pc + 4 * q);
        const float pm = pc[H * D + h], pl = pc[H * D + H + h];
        const float mn = fmaxf(m, pm), wa = ex2(m - mn), wb = ex2(pm - mn);
        o = mix4(o, wa, v, wb);
        l = fmaf(pl, wb, l * wa);
        m = mn;
    }
    // a head's m and l are read by the D / 4 lanes of one wavefront, which all
    // have read them when its first lane writes
    float* out = part + c0 * kF;
    *reinterpret_cast<float4*>(out + 4 * q) = o;
    if (4 * q % D == 0) {
        out[H * D + h] = m;
        out[H * D + H + h] = l;
    }
}

// F floats per run, summed.
template <int64_t F>
__global__ __launch_bounds__(kThreads) void k_sum_fold(LongRows lr, int parts, float* __restrict__ part) {
    int64_t c0, c1;
    run_range(lr, blockIdx.x / parts, c0, c1);
    const int64_t share = fold_share(c1 - c0, parts);
    c0 += (blockIdx.x % parts) * share;
    c1 = c0 + share < c1 ? c0 + share : c1;
    if (c1 - c0 < 2) return;
    for (int q = threadIdx.x; q < F / 4; q += kThreads) {
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
        for (int64_t c = c0; c < c1; ++c) o = add4(o, *reinterpret_cast<const float4*>(part + c * F + 4 * q));
        *reinterpret_cast<float4*>(part + c0 * F + 4 * q) = o;
    }
}

template <typename T, int D, int H>
__global__ __launch_bounds__(kThreads) void k_fwd_long_merge(LongRows lr, int parts, const float* __restrict__ part, TilePartials tp,
                                                       T* __restrict__ O, float* __restrict__ LSE) {
    using M = MergeCfg<H, D>;
    constexpr int64_t kF = fwd_run_floats(H, D);
    __shared__ float4 s_o[M::NG][M::Q4];
    __shared__ float s_m[M::NG][M::Q4], s_l[M::NG][M::Q4];
    const int64_t i = lr.list[blockIdx.x];
    int64_t c0, c1;
    run_range(lr, blockIdx.x, c0, c1);
    const int64_t step = fold_share(c1 - c0, parts);
    const int g = threadIdx.x / M::Q4, q = threadIdx.x % M::Q4, h = 4 * q / D;
    float m = kMinRef, l = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int64_t c = c0 + g * step; c < c1; c += M::NG * step) {
        const float* pc = part + c * kF;
        const float4 v = *reinterpret_cast<const float4*>(pc + 4 * q);
        const float pm = pc[H * D + h], pl = pc[H * D + H + h];
        const float mn = fmaxf(m, pm), wa = ex2(m - mn), wb = ex2(pm - mn);
        o = mix4(o, wa, v, wb);
        l = fmaf(pl, wb, l * wa);
        m = mn;
    }
    s_o[g][q] = o;
    s_m[g][q] = m;
    s_l[g][q] = l;
    __syncthreads();
    if (g != 0) return;
    const int64_t at = i * H * D + 4 * q;
    if (tp.has_row(i)) {
        m = fmaxf(tp.m[i * H + h], kMinRef);
        l = tp.l[i * H + h];
        o = *reinterpret_cast<const float4*>(tp.acc + at);
    } else {
        m = kMinRef;
        l = 0.f;
        o = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int k = 0; k < M::NG; ++k) {
        const float pm = s_m[k][q], mn = fmaxf(m, pm), wa = ex2(m - mn), wb = ex2(pm - mn);
        o = mix4(o, wa, s_o[k][q], wb);
        l = fmaf(s_l[k][q], wb, l * wa);
        m = mn;
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    store4(O + at, make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv));
    if (4 * q % D == 0) LSE[i * H + h] = l > 0.f ? (m + __log2f(l)) * kLn2 : kNegInf;
}

template <typename T, int D, int H>
__global__ __launch_bounds__(kThreads) void k_bwd_rows_long_merge(LongRows lr, int parts, const float* __restrict__ part,
                                                            TilePartials tp, const float* __restrict__ LSE,
                                                            float scale, T* __restrict__ dQ, float* __restrict__ Dv,
                                                            float2* __restrict__ stat) {
    using M = MergeCfg<H, D>;
    constexpr int64_t kF = row_run_floats(H, D);
    __shared__ float4 s_a[M::NG][M::Q4], s_b[M::NG][M::Q4];
    __shared__ float s_d[M::NG][M::Q4];
    const int64_t i = lr.list[blockIdx.x];
    int64_t c0, c1;
    run_range(lr, blockIdx.x, c0, c1);
    const int64_t step = fold_share(c1 - c0, parts);
    const int g = threadIdx.x / M::Q4, q = threadIdx.x % M::Q4, h = 4 * q / D;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    float d = 0.f;
#pragma unroll 4
    for (int64_t c = c0 + g * step; c < c1; c += M::NG * step) {
        const float* pc = part + c * kF;
        a = add4(a, *reinterpret_cast<const float4*>(pc + 4 * q));
        b = add4(b, *reinterpret_cast<const float4*>(pc + H * D + 4 * q));
        d += pc[2 * H * D + h];
    }
    s_a[g][q] = a;
    s_b[g][q] = b;
    s_d[g][q] = d;
    __syncthreads();
    if (g != 0) return;
    const int64_t at = i * H * D + 4 * q;
    if (tp.has_row(i)) {
        a = add4(a, *reinterpret_cast<const float4*>(tp.acc + at));
        b = add4(b, *reinterpret_cast<const float4*>(tp.acc2 + at));
        d += tp.m[i * H + h];
    }
    for (int k = 1; k < M::NG; ++k) {
        a = add4(a, s_a[k][q]);
        b = add4(b, s_b[k][q]);
        d += s_d[k][q];
    }
    store4(dQ + at, make_float4(fmaf(-d, b.x, a.x) * scale, fmaf(-d, b.y, a.y) * scale, fmaf(-d, b.z, a.z) * scale,
                                fmaf(-d, b.w, a.w) * scale));
    if (4 * q % D == 0) {
        if (Dv) Dv[i * H + h] = d;
        if (stat) stat[i * H + h] = make_float2(LSE[i * H + h] * kLog2e, d);
    }
}

template <typename T, int D, int H>
__global__ __launch_bounds__(kThreads) void k_bwd_cols_long_merge(LongRows lr, int parts, const float* __restrict__ part,
                                                            TilePartials tpk, TilePartials tpv, float scale,
                                                            T* __restrict__ dK, T* __restrict__ dV) {
    using M = MergeCfg<H, D>;
    constexpr int64_t kF = col_run_floats(H, D);
    __shared__ float4 s_k[M::NG][M::Q4], s_v[M::NG][M::Q4];
    const int64_t j = lr.list[blockIdx.x];
    int64_t c0, c1;
    run_range(lr, blockIdx.x, c0, c1);
    const int64_t step = fold_share(c1 - c0, parts);
    const int g = threadIdx.x / M::Q4, q = threadIdx.x % M::Q4;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
#pragma unroll 4
    for (int64_t c = c0 + g * step; c < c1; c += M::NG * step) {
        const float* pc = part + c * kF;
        a = add4(a, *reinterpret_cast<const float4*>(pc + 4 * q));
        b = add4(b, *reinterpret_cast<const float4*>(pc + H * D + 4 * q));
    }
    s_k[g][q] = a;
    s_v[g][q] = b;
    __syncthreads();
    if (g != 0) return;
    const int64_t at = j * H * D + 4 * q;
    if (tpk.has_col(j)) {
        a = add4(a, *reinterpret_cast<const float4*>(tpk.acc + at));
        b = add4(b, *reinterpret_cast<const float4*>(tpv.acc + at));
    }
    for (int k = 1; k < M::NG; ++k) {
        a = add4(a, s_k[k][q]);
        b = add4(b, s_v[k][q]);
    }
    store4(dK + at, make_float4(a.x * scale, a.y * scale, a.z * scale, a.w * scale));
    store4(dV + at, b);
}

// The column pass reads each in-edge's row statistics as one (LSE log2 e, D)
// pair: one 8-byte gather per edge instead of two 4-byte ones.
__global__ void k_pack_stats(int64_t m, const float* __restrict__ LSE, const float* __restrict__ Dv,
                             float2* __restrict__ out) {
    for (int64_t x = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; x < m; x += int64_t(gridDim.x) * blockDim.x)
        out[x] = make_float2(LSE[x] * kLog2e, Dv[x]);
}

// ------------------------------------------------------------ gather probe
// Measurement only: the forward edge kernel's data movement (every remainder
// edge of a row of at most GT_LONG_ROW edges reads its partner's two feature
// rows, same lanes, same edge walk) with no arithmetic but an XOR, so the rate
// the gather path allows for a plan can be timed beside the real kernels.
template <int F, int STR>
__device__ __forceinline__ uint32_t xor_words(const Slice<uint16_t, F, STR>& x) {
    uint32_t r = 0;
#pragma unroll
    for (int i = 0; i < F / 2; ++i) r ^= x.w[i];
    return r;
}
template <int F, int STR>
__device__ __forceinline__ uint32_t xor_words(const Slice<float, F, STR>& x) {
    uint32_t r = 0;
#pragma unroll
    for (int i = 0; i < F; ++i) r ^= __float_as_uint(x.w[i]);
    return r;
}

constexpr uint32_t kProbeSinkKey = 0x9E3779B9u;

template <typename T, int D, int H>
__global__ __launch_bounds__(kThreads) void k_gather_probe(int64_t n, const int64_t* __restrict__ rp,
                                                           const int32_t* __restrict__ cl, int64_t len,
                                                           const T* __restrict__ A, const T* __restrict__ B,
                                                           uint32_t* __restrict__ sink, unsigned run) {
    using C = EdgeCfg<T, D, H>;
    const Lanes<T, D, H> ln(lane_id());
    const int64_t wave = row_block(blockIdx.x, run) * (kThreads / kWave) + threadIdx.x / kWave;
    const int64_t i = wave * C::NPW + ln.slot;
    const bool live = i < n;
    const int64_t self = live ? i : 0;
    int64_t a = 0;
    int deg = 0;
    if (live) {
        a = rp[i];
        const int64_t dg = rp[i + 1] - a;
        deg = dg > GT_LONG_ROW ? -1 : int(dg);
    }
    const int dmax = uniform(wave_max(deg));
    uint32_t acc = 0;
    const EdgeList<C::G> el(cl, len, a, deg, lane_id());
    el.walk(dmax, [&](int64_t j0, int64_t j1, int, bool, bool) {
        Rows<T, D, H> x0, x1;
        x0.load(A, B, ln.off(j0));
        x1.load(A, B, ln.off(j1));
        acc ^= xor_words(x0.a) ^ xor_words(x1.a) ^ xor_words(x0.b) ^ xor_words(x1.b);
    });
    if (acc == kProbeSinkKey) sink[0] = acc;  // keeps the loads; practically never taken
}

template <typename T, int D, int H>
gt_status run_probe(const gt_tiles* p, const void* A, const void* B, uint32_t* sink, hipStream_t s) {
    using C = EdgeCfg<T, D, H>;
    if (p->n == 0) return GT_OK;
    const RowGrid rg = row_grid(p->n, C::NPW * (kThreads / kWave));
    k_gather_probe<T, D, H><<<rg.grid, kThreads, 0, s>>>(p->n, p->sp_rowptr, p->sp_col, p->nnz_sparse,
                                                         static_cast<const T*>(A), static_cast<const T*>(B), sink,
                                                         rg.run);
    GT_LAUNCH_CHECK("gather_probe");
    return GT_OK;
}

// ---------------------------------------------------------------- launchers

template <typename T, int D, int H, bool kBias>
gt_status run_fwd_t(const gt_tiles* p, const void* Q, const void* K, const void* V, float scale, void* O, float* LSE,
                    void* ws_ptr, EdgeBias eb, hipStream_t s) {
    using C = EdgeCfg<T, D, H>;
    const int64_t n = p->n;
    if (n == 0) return GT_OK;
    Ws ws(ws_ptr);
    ws.take<char>(256);
    TilePartials tp = tile_partials_fwd(ws, p, H, D);
    LongPlan lp = long_plan_take(ws, p->n_long_rows, p->nnz_sparse, run_spread(H, D), fwd_run_floats(H, D));
    const float sl2 = scale * kLog2e;
    gt_status st;
    if (p->n_dense > 0) {
        if ((st = tile_fwd<T, D, H>(p, static_cast<const T*>(Q), static_cast<const T*>(K),
                                    static_cast<const T*>(V), sl2, tp, eb.tile, s)) != GT_OK)
            return st;
    } else {
        tp = TilePartials{};
    }
    LongRows lr;
    if ((st = long_rows(p->long_rows, p->n_long_rows, p->sp_rowptr, run_spread_bits(H, D), lp, lr, s)) != GT_OK) return st;
    const RowGrid rg = row_grid(n, C::NPW * (kThreads / kWave));
    const unsigned runs = lp.blocks(C::NPW * (kThreads / kWave));
    k_fwd_rows<T, D, H, kBias><<<runs + rg.grid, kThreads, 0, s>>>(
        n, p->sp_rowptr, p->sp_col, p->nnz_sparse, static_cast<const T*>(Q), static_cast<const T*>(K),
        static_cast<const T*>(V), sl2, static_cast<T*>(O), LSE, tp, eb, rg.run, lr, runs, lp.part);
    GT_LAUNCH_CHECK("sparse_fwd_rows");
    if (p->n_long_rows > 0) {
        if (lp.fold > 1) {
            k_fwd_fold<D, H><<<unsigned(p->n_long_rows) * lp.fold, kThreads, 0, s>>>(lr, lp.fold, lp.part);
            GT_LAUNCH_CHECK("sparse_fwd_fold");
        }
        k_fwd_long_merge<T, D, H><<<unsigned(p->n_long_rows), kThreads, 0, s>>>(lr, lp.fold, lp.part, tp,
                                                                               static_cast<T*>(O), LSE);
        GT_LAUNCH_CHECK("sparse_fwd_long_merge");
    }
    return GT_OK;
}

template <typename T, int D, int H>
gt_status run_fwd(const gt_tiles* p, const void* Q, const void* K, const void* V, float scale, void* O, float* LSE,
                  void* ws_ptr, EdgeBias eb, hipStream_t s) {
    return eb.b ? run_fwd_t<T, D, H, true>(p, Q, K, V, scale, O, LSE, ws_ptr, eb, s)
                : run_fwd_t<T, D, H, false>(p, Q, K, V, scale, O, LSE, ws_ptr, eb, s);
}

template <typename T, int D, int H, bool kBias>
gt_status run_bwd_rows_t(const gt_tiles* p, const void* Q, const void* K, const void* V, const void* dO,
                         const float* LSE, float scale, void* dQ, float* Dv, float2* stat, void* ws_ptr,
                         EdgeBias eb, hipStream_t s) {
    using C = EdgeCfg<T, D, H>;
    const int64_t n = p->n;
    if (n == 0) return GT_OK;
    Ws ws(ws_ptr);
    ws.take<char>(256);
    TileBwdPartials tb = tile_partials_bwd(ws, p, H, D, true, false);
    LongPlan lp = long_plan_take(ws, p->n_long_rows, p->nnz_sparse, run_spread(H, D), row_run_floats(H, D));
    const float sl2 = scale * kLog2e;
    const T *q = static_cast<const T*>(Q), *k = static_cast<const T*>(K), *v = static_cast<const T*>(V);
    const T* g = static_cast<const T*>(dO);
    gt_status st;
    if (p->n_dense > 0) {
        if ((st = tile_bwd_dq<T, D, H>(p, q, k, v, g, LSE, sl2, tb.dq, eb.tile, s)) != GT_OK) return st;
    }
    LongRows lr;
    if ((st = long_rows(p->long_rows, p->n_long_rows, p->sp_rowptr, run_spread_bits(H, D), lp, lr, s)) != GT_OK) return st;
    const RowGrid rg = row_grid(n, C::NPW * (kThreads / kWave));
    const unsigned runs = lp.blocks(C::NPW * (kThreads / kWave));
    k_bwd_rows<T, D, H, kBias><<<runs + rg.grid, kThreads, 0, s>>>(
        n, p->sp_rowptr, p->sp_col, p->nnz_sparse, q, k, v, g, LSE, Dv, stat, sl2, scale, static_cast<T*>(dQ), tb.dq,
        eb, rg.run, lr, runs, lp.part);
    GT_LAUNCH_CHECK("sparse_bwd_rows");
    if (p->n_long_rows > 0) {
        if (lp.fold > 1) {
            k_sum_fold<row_run_floats(H, D)>
                <<<unsigned(p->n_long_rows) * lp.fold, kThreads, 0, s>>>(lr, lp.fold, lp.part);
            GT_LAUNCH_CHECK("sparse_bwd_rows_fold");
        }
        k_bwd_rows_long_merge<T, D, H><<<unsigned(p->n_long_rows), kThreads, 0, s>>>(
            lr, lp.fold, lp.part, tb.dq, LSE, scale, static_cast<T*>(dQ), Dv, stat);
        GT_LAUNCH_CHECK("sparse_bwd_rows_long_merge");
    }
    return GT_OK;
}

template <typename T, int D, int H>
gt_status run_bwd_rows(const gt_tiles* p, const void* Q, const void* K, const void* V, const void* dO,
                       const float* LSE, float scale, void* dQ, float* Dv, float2* stat, void* ws_ptr, EdgeBias eb,
                       hipStream_t s) {
    return eb.b ? run_bwd_rows_t<T, D, H, true>(p, Q, K, V, dO, LSE, scale, dQ, Dv, stat, ws_ptr, eb, s)
                : run_bwd_rows_t<T, D, H, false>(p, Q, K, V, dO, LSE, scale, dQ, Dv, stat, ws_ptr, eb, s);
}

template <typename T, int D, int H, bool kBias>
gt_status run_bwd_cols_t(const gt_tiles* p, const void* Q, const void* K, const void* V, const void* dO,
                         const float* LSE, const float* Dv, const float2* packed, float scale, void* dK, void* dV,
                         void* ws_ptr, EdgeBias eb, hipStream_t s) {
    using C = EdgeCfg<T, D, H>;
    const int64_t n = p->n;
    if (n == 0) return GT_OK;
    Ws ws(ws_ptr);
    ws.take<char>(256);
    TileBwdPartials tb = tile_partials_bwd(ws, p, H, D, false, true);
    LongPlan lp = long_plan_take(ws, p->n_long_cols, p->nnz_sparse, run_spread(H, D), col_run_floats(H, D));
    float2* stat = packed ? nullptr : ws.take<float2>(size_t(n) * H);
    const float sl2 = scale * kLog2e;
    const T *q = static_cast<const T*>(Q), *k = static_cast<const T*>(K), *v = static_cast<const T*>(V);
    const T* g = static_cast<const T*>(dO);
    gt_status st;
    if (p->n_dense > 0) {
        if ((st = tile_bwd_dkdv<T, D, H>(p, q, k, v, g, LSE, Dv, sl2, tb.dk, tb.dv, eb.tile, s)) != GT_OK)
            return st;
    }
    if (!packed) {
        k_pack_stats<<<grid_for(n * H, 256, 8192), 256, 0, s>>>(n * H, LSE, Dv, stat);
        GT_LAUNCH_CHECK("sparse_bwd_pack_stats");
    }
    LongRows lr;
    if ((st = long_rows(p->long_cols, p->n_long_cols, p->sp_colptr, run_spread_bits(H, D), lp, lr, s)) != GT_OK) return st;
    const RowGrid rg = row_grid(n, C::NPW * (kThreads / kWave));
    const unsigned runs = lp.blocks(C::NPW * (kThreads / kWave));
    k_bwd_cols<T, D, H, kBias><<<runs + rg.grid, kThreads, 0, s>>>(
        n, p->sp_colptr, p->sp_row, p->nnz_sparse, q, k, v, g, packed ? packed : stat, sl2, scale,
        static_cast<T*>(dK), static_cast<T*>(dV), tb.dk, tb.dv, eb, rg.run, lr, runs, lp.part);
    GT_LAUNCH_CHECK("sparse_bwd_cols");
    if (p->n_long_cols > 0) {
        if (lp.fold > 1) {
            k_sum_fold<col_run_floats(H, D)>
                <<<unsigned(p->n_long_cols) * lp.fold, kThreads, 0, s>>>(lr, lp.fold, lp.part);
            GT_LAUNCH_CHECK("sparse_bwd_cols_fold");
        }
        k_bwd_cols_long_merge<T, D, H><<<unsigned(p->n_long_cols), kThreads, 0, s>>>(
            lr, lp.fold, lp.part, tb.dk, tb.dv, scale, static_cast<T*>(dK), static_cast<T*>(dV));
        GT_LAUNCH_CHECK("sparse_bwd_cols_long_merge");
    }
    return GT_OK;
}

template <typename T, int D, int H>
gt_status run_bwd_cols(const gt_tiles* p, const void* Q, const void* K, const void* V, const void* dO,
                       const float* LSE, const float* Dv, const float2* packed, float scale, void* dK, void* dV,
                       void* ws_ptr, EdgeBias eb, hipStream_t s) {
    return eb.b ? run_bwd_cols_t<T, D, H, true>(p, Q, K, V, dO, LSE, Dv, packed, scale, dK, dV, ws_ptr, eb, s)
                : run_bwd_cols_t<T, D, H, false>(p, Q, K, V, dO, LSE, Dv, packed, scale, dK, dV, ws_ptr, eb, s);
}

template <typename T, int D, int H>
gt_status run_bwd(const gt_tiles* p, const void* Q, const void* K, const void* V, const void* dO, const float* LSE,
                  float scale, void* dQ, void* dK, void* dV, void* ws_ptr, EdgeBias eb, hipStream_t s) {
    if (p->n == 0) return GT_OK;
    // the row pass leaves the packed statistics the column pass reads; D alone
    // only where the tile kernels read it
    Ws ws(ws_ptr);
    float2* stat = ws.take<float2>(size_t(p->n) * H);
    float* Dv = p->n_dense > 0 ? ws.take<float>(size_t(p->n) * H) : nullptr;
    char* rest = ws.take<char>(1);
    gt_status st = run_bwd_rows<T, D, H>(p, Q, K, V, dO, LSE, scale, dQ, Dv, stat, rest, eb, s);
    if (st != GT_OK) return st;
    return run_bwd_cols<T, D, H>(p, Q, K, V, dO, LSE, Dv, stat, scale, dK, dV, rest, eb, s);
}

bool supported(int32_t H, int32_t d, gt_dtype dt) {
    return (d == 32 || d == 64) && (H == 1 || H == 2 || H == 4 || H == 8 || H == 16) && (dt == GT_F32 || dt == GT_BF16);
}

gt_status check_plan(const char* who, const gt_tiles* p) {
    if (!p) return fail(GT_ERR_INVALID_ARG, std::string(who) + ": null plan");
    if (p->n < 0 || p->n >= (int64_t(1) << 31) || (p->T != 64 && p->T != 128))
        return fail(GT_ERR_INVALID_ARG, std::string(who) + ": plan not built (n or T invalid)");
    if (p->n > 0 && (!p->sp_rowptr || !p->sp_colptr || !p->tile_rowptr || !p->tileT_ptr))
        return fail(GT_ERR_INVALID_ARG, std::string(who) + ": plan arrays missing");
    if ((p->nnz_sparse > 0 && (!p->sp_col || !p->sp_row)) || (p->n_long_rows > 0 && !p->long_rows) ||
        (p->n_long_cols > 0 && !p->long_cols) ||
        (p->n_dense > 0 && (!p->tile_col || !p->tile_mask || !p->tileT_idx)))
        return fail(GT_ERR_INVALID_ARG, std::string(who) + ": plan arrays missing");
    return GT_OK;
}

size_t fwd_ws(const gt_tiles* p, int32_t H, int32_t d) {
    Ws ws(nullptr);
    ws.take<char>(256);
    tile_partials_fwd(ws, p, H, d);
    long_plan_take(ws, p->n_long_rows, p->nnz_sparse, run_spread(H, d), fwd_run_floats(H, d));
    return ws.size();
}
size_t bwd_part_ws(const gt_tiles* p, int32_t H, int32_t d, bool rows, bool cols, bool with_stat = true) {
    Ws ws(nullptr);
    ws.take<char>(256);
    tile_partials_bwd(ws, p, H, d, rows, cols);
    if (rows) long_plan_take(ws, p->n_long_rows, p->nnz_sparse, run_spread(H, d), row_run_floats(H, d));
    if (cols) {
        long_plan_take(ws, p->n_long_cols, p->nnz_sparse, run_spread(H, d), col_run_floats(H, d));
        if (with_stat) ws.take<float2>(size_t(p->n > 0 ? p->n : 1) * H);
    }
    return ws.size();
}
size_t bwd_ws(const gt_tiles* p, int32_t H, int32_t d) {
    Ws ws(nullptr);
    ws.take<float2>(size_t(p->n > 0 ? p->n : 1) * H);
    if (p->n_dense > 0) ws.take<float>(size_t(p->n > 0 ? p->n : 1) * H);
    const size_t a = bwd_part_ws(p, H, d, true, false), b = bwd_part_ws(p, H, d, false, true, false);
    ws.take<char>(a > b ? a : b);
    return ws.size();
}

}  // namespace
}  // namespace gt

using namespace gt;

extern "C" size_t gt_sparse_attn_fwd_workspace_size(const gt_tiles* plan, int32_t H, int32_t d, gt_dtype dtype) {
    if (!plan || !supported(H, d, dtype)) return 0;
    return fwd_ws(plan, H, d);
}

extern "C" gt_status gt_sparse_attn_fwd(const gt_tiles* plan, int32_t H, int32_t d, gt_dtype dtype, const void* Q,
                                        const void* K, const void* V, float scale, void* O, float* LSE, void* ws,
                                        size_t ws_bytes, hipStream_t stream) {
    gt_status st = check_plan("gt_sparse_attn_fwd", plan);
    if (st != GT_OK) return st;
    if (!supported(H, d, dtype)) return fail(GT_ERR_UNSUPPORTED, "gt_sparse_attn_fwd: unsupported (H, d, dtype)");
    if (plan->n > 0 && (!Q || !K || !V || !O || !LSE || !ws))
        return fail(GT_ERR_INVALID_ARG, "gt_sparse_attn_fwd: null pointer");
    if (ws_bytes < fwd_ws(plan, H, d)) return fail(GT_ERR_WORKSPACE, "gt_sparse_attn_fwd: workspace too small");
    return GT_DISPATCH_ATTN(dtype, d, H, run_fwd, plan, Q, K, V, scale, O, LSE, ws, EdgeBias{}, stream);
}

extern "C" size_t gt_sparse_attn_bwd_workspace_size(const gt_tiles* plan, int32_t H, int32_t d, gt_dtype dtype) {
    if (!plan || !supported(H, d, dtype)) return 0;
    return bwd_ws(plan, H, d);
}

extern "C" size_t gt_sparse_attn_bwd_rows_workspace_size(const gt_tiles* plan, int32_t H, int32_t d,
                                                         gt_dtype dtype) {
    if (!plan || !supported(H, d, dtype)) return 0;
    return bwd_part_ws(plan, H, d, true, false);
}

extern "C" gt_status gt_sparse_attn_bwd_rows(const gt_tiles* plan, int32_t H, int32_t d, gt_dtype dtype,
                                             const void* Q, const void* K, const void* V, const void* dO,
                                             const float* LSE, float scale, void* dQ, float* Dstat, void* ws,
                                             size_t ws_bytes, hipStream_t stream) {
    gt_status st = check_plan("gt_sparse_attn_bwd_rows", plan);
    if (st != GT_OK) return st;
    if (!supported(H, d, dtype)) return fail(GT_ERR_UNSUPPORTED, "gt_sparse_attn_bwd_rows: unsupported (H, d, dtype)");
    if (plan->n > 0 && (!Q || !K || !V || !dO || !LSE || !dQ || !Dstat || !ws))
        return fail(GT_ERR_INVALID_ARG, "gt_sparse_attn_bwd_rows: null pointer");
    if (ws_bytes < bwd_part_ws(plan, H, d, true, false))
        return fail(GT_ERR_WORKSPACE, "gt_sparse_attn_bwd_rows: workspace too small");
    return GT_DISPATCH_ATTN(dtype, d, H, run_bwd_rows, plan, Q, K, V, dO, LSE, scale, dQ, Dstat,
                            static_cast<float2*>(nullptr), ws, EdgeBias{}, stream);
}

extern "C" size_t gt_sparse_attn_bwd_cols_workspace_size(const gt_tiles* plan, int32_t H, int32_t d,
                                                         gt_dtype dtype) {
    if (!plan || !supported(H, d, dtype)) return 0;
    return bwd_part_ws(plan, H, d, false, true);
}

extern "C" gt_status gt_sparse_attn_bwd_cols(const gt_tiles* plan, int32_t H, int32_t d, gt_dtype dtype,
                                             const void* Q, const void* K, const void* V, const void* dO,
                                             const float* LSE, const float* Dstat, float scale, void* dK, void* dV,
                                             void* ws, size_t ws_bytes, hipStream_t stream) {
    gt_status st = check_plan("gt_sparse_attn_bwd_cols", plan);
    if (st != GT_OK) return st;
    if (!supported(H, d, dtype)) return fail(GT_ERR_UNSUPPORTED, "gt_sparse_attn_bwd_cols: unsupported (H, d, dtype)");
    if (plan->n > 0 && (!Q || !K || !V || !dO || !LSE || !Dstat || !dK || !dV || !ws))
        return fail(GT_ERR_INVALID_ARG, "gt_sparse_attn_bwd_cols: null pointer");
    if (ws_bytes < bwd_part_ws(plan, H, d, false, true))
        return fail(GT_ERR_WORKSPACE, "gt_sparse_attn_bwd_cols: workspace too small");
    return GT_DISPATCH_ATTN(dtype, d, H, run_bwd_cols, plan, Q, K, V, dO, LSE, Dstat,
                            static_cast<const float2*>(nullptr), scale, dK, dV, ws, EdgeBias{}, stream);
}

extern "C" gt_status gt_sparse_attn_bwd(const gt_tiles* plan, int32_t H, int32_t d, gt_dtype dtype, const void* Q,
                                        const void* K, const void* V, const void* dO, const float* LSE, float scale,
                                        void* dQ, void* dK, void* dV, void* ws, size_t ws_bytes, hipStream_t stream) {
    gt_status st = check_plan("gt_sparse_attn_bwd", plan);
    if (st != GT_OK) return st;
    if (!supported(H, d, dtype)) return fail(GT_ERR_UNSUPPORTED, "gt_sparse_attn_bwd: unsupported (H, d, dtype)");
    if (plan->n > 0 && (!Q || !K || !V || !dO || !LSE || !dQ || !dK || !dV || !ws))
        return fail(GT_ERR_INVALID_ARG, "gt_sparse_attn_bwd: null pointer");
    if (ws_bytes < bwd_ws(plan, H, d)) return fail(GT_ERR_WORKSPACE, "gt_sparse_attn_bwd: workspace too small");
    return GT_DISPATCH_ATTN(dtype, d, H, run_bwd, plan, Q, K, V, dO, LSE, scale, dQ, dK, dV, ws, EdgeBias{}, stream);
}

// ------------------------------------------------------------ with a bias
// The bias is indexed by input-CSR position.  Remainder edges read it through
// sp_pos (forward, row pass) or csc_pos (column pass).  On a plan with dense
// tiles it is first laid out per tile in the workspace (TileBias: the tile
// kernels read it with the same cell indexing as their masks), and the column
// pass's tile dS are written back to dbias at the tile edges' positions.

namespace gt {
namespace {

int64_t tile_bias_elems(const gt_tiles* p, int32_t H) {
    return p->n_dense > 0 ? p->n_dense * int64_t(H) * p->T * p->T : 0;
}

// The cells of local row r, word w (32 columns) of dense tile k: each thread
// takes one (r, w), whose first edge position is tile_pos[k T + r] plus the
// edges of the row's earlier words.  kToTiles: bias -> per-tile layout (-inf
// off the edges, so the tile kernels need no mask test where they add it);
// else per-tile dS -> dbias at the edges' positions.
template <bool kToTiles>
__global__ __launch_bounds__(256) void k_tile_bias_move(int H, int T, const uint32_t* __restrict__ mask,
                                                        const int32_t* __restrict__ tile_pos,
                                                        const float* __restrict__ src, float* __restrict__ dst) {
    const int64_t k = blockIdx.x;
    const int h = blockIdx.y;
    const int W = T / 32;
    for (int x = threadIdx.x; x < T * W; x += blockDim.x) {
        const int r = x / W, w = x % W;
        const uint32_t* row = mask + (k * T + r) * W;
        int pre = 0;
        for (int u = 0; u < w; ++u) pre += __popc(row[u]);
        const uint32_t word = row[w];
        const int64_t p0 = int64_t(tile_pos[k * T + r]) + pre;
        const int64_t cell = TileBias::at(k, H, h, T, r, 32 * w);
        for (int bit = 0; bit < 32; ++bit) {
            const bool on = (word >> bit) & 1u;
            const int64_t e = p0 + __popc(word & ((1u << bit) - 1u));
            if (kToTiles) dst[cell + bit] = on ? src[e * H + h] : -__builtin_huge_valf();
            else if (on) dst[e * H + h] = src[cell + bit];
        }
    }
}

gt_status tile_bias_move(bool to_tiles, const gt_tiles* p, int32_t H, const float* src, float* dst, hipStream_t s) {
    if (p->n_dense <= 0) return GT_OK;
    const dim3 grid(unsigned(p->n_dense), unsigned(H));
    if (to_tiles) k_tile_bias_move<true><<<grid, 256, 0, s>>>(H, p->T, p->tile_mask, p->tile_pos, src, dst);
    else k_tile_bias_move<false><<<grid, 256, 0, s>>>(H, p->T, p->tile_mask, p->tile_pos, src, dst);
    GT_LAUNCH_CHECK("tile_bias_move");
    return GT_OK;
}

gt_status check_bias(const char* who, const gt_tiles* plan, const float* bias) {
    if (plan->nnz_sparse >= (int64_t(1) << 31))
        return fail(GT_ERR_INVALID_ARG, std::string(who) + ": more than 2^31 - 1 edges");
    if (plan->n_dense > 0 && ((plan->nnz_sparse > 0 && !plan->sp_pos) || !plan->tile_pos))
        return fail(GT_ERR_INVALID_ARG, std::string(who) + ": a plan with dense tiles needs sp_pos and tile_pos "
                                                            "(pass them to gt_build_tiles)");
    if ((plan->nnz_sparse > 0 || plan->n_dense > 0) && !bias)
        return fail(GT_ERR_INVALID_ARG, std::string(who) + ": null bias");
    return GT_OK;
}

size_t fwd_bias_ws(const gt_tiles* p, int32_t H, int32_t d) {
    Ws ws(nullptr);
    ws.take<char>(fwd_ws(p, H, d));
    ws.take<float>(size_t(tile_bias_elems(p, H)));
    return ws.size();
}
size_t bwd_bias_ws(const gt_tiles* p, int32_t H, int32_t d) {
    Ws ws(nullptr);
    ws.take<char>(bwd_ws(p, H, d));
    ws.take<float>(size_t(tile_bias_elems(p, H)));
    ws.take<float>(size_t(tile_bias_elems(p, H)));
    return ws.size();
}

}  // namespace
}  // namespace gt

extern "C" size_t gt_sparse_attn_fwd_bias_workspace_size(const gt_tiles* plan, int32_t H, int32_t d,
                                                         gt_dtype dtype) {
    if (!plan || !supported(H, d, dtype)) return 0;
    return fwd_bias_ws(plan, H, d);
}

extern "C" size_t gt_sparse_attn_bwd_bias_workspace_size(const gt_tiles* plan, int32_t H, int32_t d,
                                                         gt_dtype dtype) {
    if (!plan || !supported(H, d, dtype)) return 0;
    return bwd_bias_ws(plan, H, d);
}

extern "C" gt_status gt_sparse_attn_fwd_bias(const gt_tiles* plan, int32_t H, int32_t d, gt_dtype dtype,
                                             const void* Q, const void* K, const void* V, const float* bias,
                                             float scale, void* O, float* LSE, void* ws, size_t ws_bytes,
                                             hipStream_t stream) {
    gt_status st = check_plan("gt_sparse_attn_fwd_bias", plan);
    if (st != GT_OK) return st;
    if ((st = check_bias("gt_sparse_attn_fwd_bias", plan, bias)) != GT_OK) return st;
    if (!supported(H, d, dtype))
        return fail(GT_ERR_UNSUPPORTED, "gt_sparse_attn_fwd_bias: unsupported (H, d, dtype)");
    if (plan->n > 0 && (!Q || !K || !V || !O || !LSE || !ws))
        return fail(GT_ERR_INVALID_ARG, "gt_sparse_attn_fwd_bias: null pointer");
    if (ws_bytes < fwd_bias_ws(plan, H, d))
        return fail(GT_ERR_WORKSPACE, "gt_sparse_attn_fwd_bias: workspace too small");
    if (plan->n == 0) return GT_OK;
    Ws w(ws);
    void* main = w.take<char>(fwd_ws(plan, H, d));
    EdgeBias eb;
    if (plan->nnz_sparse > 0) {
        eb.b = bias;
        eb.sp_pos = plan->sp_pos;
    }
    if (plan->n_dense > 0) {
        float* bt = w.take<float>(size_t(tile_bias_elems(plan, H)));
        if ((st = tile_bias_move(true, plan, H, bias, bt, stream)) != GT_OK) return st;
        eb.tile.b = bt;
    }
    return GT_DISPATCH_ATTN(dtype, d, H, run_fwd, plan, Q, K, V, scale, O, LSE, main, eb, stream);
}

extern "C" gt_status gt_sparse_attn_bwd_bias(const gt_tiles* plan, const int32_t* csc_pos, int32_t H, int32_t d,
                                             gt_dtype dtype, const void* Q, const void* K, const void* V,
                                             const float* bias, const void* dO, const float* LSE, float scale,
                                             void* dQ, void* dK, void* dV, float* dbias, void* ws, size_t ws_bytes,
                                             hipStream_t stream) {
    gt_status st = check_plan("gt_sparse_attn_bwd_bias", plan);
    if (st != GT_OK) return st;
    if ((st = check_bias("gt_sparse_attn_bwd_bias", plan, bias)) != GT_OK) return st;
    if (!supported(H, d, dtype))
        return fail(GT_ERR_UNSUPPORTED, "gt_sparse_attn_bwd_bias: unsupported (H, d, dtype)");
    if (plan->n > 0 && (!Q || !K || !V || !dO || !LSE || !dQ || !dK || !dV || !ws))
        return fail(GT_ERR_INVALID_ARG, "gt_sparse_attn_bwd_bias: null pointer");
    if ((plan->nnz_sparse > 0 && !csc_pos) || ((plan->nnz_sparse > 0 || plan->n_dense > 0) && !dbias))
        return fail(GT_ERR_INVALID_ARG, "gt_sparse_attn_bwd_bias: null csc_pos or dbias");
    if (ws_bytes < bwd_bias_ws(plan, H, d))
        return fail(GT_ERR_WORKSPACE, "gt_sparse_attn_bwd_bias: workspace too small");
    if (plan->n == 0) return GT_OK;
    Ws w(ws);
    void* main = w.take<char>(bwd_ws(plan, H, d));
    EdgeBias eb;
    if (plan->nnz_sparse > 0) {
        eb.b = bias;
        eb.sp_pos = plan->sp_pos;
        eb.csc_pos = csc_pos;
        eb.db = dbias;
    }
    float* dbt = nullptr;
    if (plan->n_dense > 0) {
        float* bt = w.take<float>(size_t(tile_bias_elems(plan, H)));
        dbt = w.take<float>(size_t(tile_bias_elems(plan, H)));
        if ((st = tile_bias_move(true, plan, H, bias, bt, stream)) != GT_OK) return st;
        eb.tile.b = bt;
        eb.tile.db = dbt;
    }
    st = GT_DISPATCH_ATTN(dtype, d, H, run_bwd, plan, Q, K, V, dO, LSE, scale, dQ, dK, dV, main, eb, stream);
    if (st != GT_OK) return st;
    return dbt ? tile_bias_move(false, plan, H, dbt, dbias, stream) : GT_OK;
}

extern "C" gt_status gt_gather_probe(const gt_tiles* plan, int32_t H, int32_t d, gt_dtype dtype, const void* A,
                                     const void* B, uint32_t* sink, hipStream_t stream) {
    gt_status st = check_plan("gt_gather_probe", plan);
    if (st != GT_OK) return st;
    if (!supported(H, d, dtype)) return fail(GT_ERR_UNSUPPORTED, "gt_gather_probe: unsupported (H, d, dtype)");
    if (plan->n > 0 && (!A || !B || !sink)) return fail(GT_ERR_INVALID_ARG, "gt_gather_probe: null pointer");
    return GT_DISPATCH_ATTN(dtype, d, H, run_probe, plan, A, B, sink, stream);
}
