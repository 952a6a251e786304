// Resident CG: a whole sweep of the textbook recurrences in one launch.  The
// workgroups of an instance (its team) stay on their compute units for all
// iterations, keep the search direction's window and the iterate in LDS, the
// first blocks of every row in registers, and meet twice per iteration to
// exchange the partial sums of p.q and of (r.z, r.r).
//
// What bounds it: the two meetings, about 2 us each, the vector instructions
// of the product (about 34 a stored block) and, at the top of the range, the
// blocks that do not fit the registers.  Three launches per iteration (SpMV,
// update, direction) pay each launch's fill and drain, move every vector
// through memory between them and stream all blocks.  Per iteration, three
// launches -> resident, in solves of one sweep of 96 iterations with the solve's
// other work spread over them (FP16 blocks with block Jacobi, FP32 and FP64 with
// Jacobi), in us:
//   rows       256        2,560       33k         66k         131k        262k
//   FP16   12.7 ->  5.8  16.5 ->  6.7  18.1 ->  7.9  17.8 ->  9.4  22.0 -> 11.3  28.3 -> 14.0
//   FP32   13.9 ->  6.3  19.8 ->  7.6  21.4 ->  9.9  23.5 -> 12.2  27.9 -> 14.7  38.8 -> 23.3
//   FP64   13.7 ->  6.5  20.0 ->  8.2  23.2 -> 10.5  26.1 -> 12.9  34.7 -> 20.9  55.6 -> 37.8
// Where an iteration's time goes, of a frame of 262k rows in FP16 (15.9 us): 4.3
// product, 1.3 wait for the workgroup's slowest wavefront, 2-4 p.q meeting, 1
// update, 1.5 sums and stores, 3.5 (r.z, r.r) meeting, 1.8 direction.
//
// The sums are formed in exactly the order of the three-launch iteration at
// its default schedule (8-slice SpMV items, 2048-row vector items), so both
// give the same bits: a slice's p.q lanes are summed by the wavefront
// butterfly, eight slices in order make an SpMV item, thread t of 1024 adds
// items t, t + 1024, ...; the update's thread adds row t and row t + 1024 of
// its item, 16 wavefronts in order make a vector item.  The pair of 64-row
// slices (w, w + 16) of a 32-slice item is therefore the smallest unit of
// work; a workgroup owns 2, 4 or 8 consecutive pairs of one item.
//
// Memory shared between workgroups during the launch (the partial sums and
// the halo rows' z) goes through relaxed agent-scope atomics, which bypass
// the caches that are not coherent across the XCDs: no fence writes back or
// invalidates an L2.  A value is published after every wavefront of the
// workgroup has waited for its earlier stores (s_waitcnt vmcnt(0), then the
// workgroup barrier), so a workgroup that has seen it also finds those
// stores.  Slots hold EMPTY until written; each set of slots has two buffers,
// and the buffer of the next iteration is emptied at a point where every
// workgroup is known to have read it.  Every wait is bounded (
// PC_OPT_RESIDENT_POLLS); a workgroup that gives up marks the instance (flag 4)
// and leaves without writing its results, and so do the others in turn, except
// that workgroups which have the last meeting's values finish and write theirs;
// the solver then restarts the instance from what its iterate holds with the
// three launches.  Teams of
// more than one workgroup are launched cooperatively, so all of them are
// resident at once.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "pc_resident.h"
#include "pc_spmv.h"

namespace pc {

typedef unsigned long long u64;
constexpr u64 EMPTY = 0xfff7a5a5a5a5a5a5ull;   // a NaN that publish() never writes
constexpr int REPLICAS = 8;                    // copies of the slots: 256 workgroups polling one copy measured
                                               // 3.7-4.2 us per meeting, eight copies 2.8 us

__device__ __forceinline__ void agent_store(u64 *p, u64 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 agent_load(const u64 *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store_f(float *p, float v) {
    __hip_atomic_store((unsigned *)p, __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float agent_load_f(const float *p) {
    return __uint_as_float(__hip_atomic_load((const unsigned *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void agent_store_f(double *p, double v) {
    agent_store((u64 *)p, __builtin_bit_cast(u64, v));
}
__device__ __forceinline__ double agent_load_f(const double *p) {
    return __builtin_bit_cast(double, agent_load((const u64 *)p));
}
__device__ __forceinline__ u64 sum_bits(double v) {
    const u64 b = __builtin_bit_cast(u64, v);
    return b == EMPTY ? 0x7ff8000000000000ull : b;
}
// every earlier memory operation of this wavefront has completed
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

struct ResArgs {
    // solver layout (pc_spmv.h)
    const int *slice_vbase, *lane_row, *row_lane;
    const uint8_t *slot_cnt;
    const int16_t *jdel;   // block columns as offsets from the slice's first row, or (FAR) as rows of the window
    const void *jval;
    const double *mass;
    const double *vscale_inv;   // FP16 blocks: 1 / S of slice s at [2 s]
    int nv;
    // teams
    ResInst const *inst;
    const int4 *wg;        // instance, first pair, pairs, rank in the team
    const ResWin *win;     // block-column window of each workgroup
    const int *inst_win;   // largest window of each instance's workgroups
    int win_rows;          // LDS rows of the window
    int win_cap;           // instances with a wider window are left to the three-launch iteration
    int wg0;               // first workgroup of the launch
    PcgState *st;
    float *p;
    void *x, *r;           // iterate and residual (TV)
    const float *pre;      // preconditioner: 3 (Jacobi) or 6 (block Jacobi) per row
    void *exch;            // three planes of nv: z (block Jacobi, FP32) or r (Jacobi, TV)
    u64 *slots;
    int slot_n;            // slots of one buffer (p.q, then r.z and r.r)
    int slot_rep;          // distance between copies
    int slot_rz;           // first (r.z, r.r) slot
    int par, max_iters;
    int polls;             // of a wait, before it gives up
};

// One stored block of a lane as it lies in memory, with its column (row of
// the window, DIAG set for the row's own diagonal block): 5 registers for the
// 16-bit types, 10 for FP32, 19 for FP64.  load() reads lane l of a slot of
// width w whose values start at `seg` (uniform) and whose columns start at
// `cols`: scalar bases with 32-bit lane offsets.
constexpr unsigned DIAG = 0x8000u;
template <typename TB> struct RawBlock;
template <typename TB> struct RawHalf {
    uint4 a;
    unsigned b;   // value 8, column in the upper half
    __device__ __forceinline__ void load(const char *seg, int w, unsigned l) {
        a = *reinterpret_cast<const uint4 *>(seg + 16u * l);
        b = *reinterpret_cast<const uint16_t *>(seg + 16 * w + 2u * l);
    }
    __device__ __forceinline__ void set_col(unsigned c) { b = (b & 0xffffu) | c << 16; }
    __device__ __forceinline__ unsigned col() const { return b >> 16; }
    __device__ __forceinline__ void clear() { a = make_uint4(0u, 0u, 0u, 0u); b = 0u; }
    // to the compiler, new values: what is unpacked from kept blocks is not
    // carried through the iterations in registers of its own
    __device__ __forceinline__ void refresh() {
        asm volatile("" : "+v"(a.x), "+v"(a.y), "+v"(a.z), "+v"(a.w), "+v"(b));
    }
};
template <> struct RawBlock<f16_t> : RawHalf<f16_t> {
    __device__ __forceinline__ void get(float v[9]) const {
        v[0] = f16_to_f32(a.x & 0xffffu); v[1] = f16_to_f32(a.x >> 16);
        v[2] = f16_to_f32(a.y & 0xffffu); v[3] = f16_to_f32(a.y >> 16);
        v[4] = f16_to_f32(a.z & 0xffffu); v[5] = f16_to_f32(a.z >> 16);
        v[6] = f16_to_f32(a.w & 0xffffu); v[7] = f16_to_f32(a.w >> 16);
        v[8] = f16_to_f32(b & 0xffffu);
    }
};
template <> struct RawBlock<bf16_t> : RawHalf<bf16_t> {
    __device__ __forceinline__ void get(float v[9]) const {
        v[0] = __uint_as_float(a.x << 16); v[1] = __uint_as_float(a.x & 0xffff0000u);
        v[2] = __uint_as_float(a.y << 16); v[3] = __uint_as_float(a.y & 0xffff0000u);
        v[4] = __uint_as_float(a.z << 16); v[5] = __uint_as_float(a.z & 0xffff0000u);
        v[6] = __uint_as_float(a.w << 16); v[7] = __uint_as_float(a.w & 0xffff0000u);
        v[8] = __uint_as_float(b << 16);
    }
};
template <typename R> struct RawWide {
    R v9[9];
    unsigned c;
    __device__ __forceinline__ void load(const char *seg, int w, unsigned l) {
        constexpr int CE = 16 / (int)sizeof(R);
#pragma unroll
        for (int q = 0; q < 8 / CE; ++q) {
            const uint4 u = *reinterpret_cast<const uint4 *>(seg + 16 * q * w + 16u * l);
            if constexpr (CE == 4) {
                v9[4 * q] = __uint_as_float(u.x); v9[4 * q + 1] = __uint_as_float(u.y);
                v9[4 * q + 2] = __uint_as_float(u.z); v9[4 * q + 3] = __uint_as_float(u.w);
            } else {
                v9[2 * q] = join64(u.x, u.y);
                v9[2 * q + 1] = join64(u.z, u.w);
            }
        }
        v9[8] = *reinterpret_cast<const R *>(seg + 8 * (int)sizeof(R) * w + (unsigned)sizeof(R) * l);
    }
    __device__ __forceinline__ void set_col(unsigned col) { c = col; }
    __device__ __forceinline__ unsigned col() const { return c; }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int q = 0; q < 9; ++q) v9[q] = R(0);
    }
    __device__ __forceinline__ void refresh() {
#pragma unroll
        for (int q = 0; q < 9; ++q) asm volatile("" : "+v"(v9[q]));
        asm volatile("" : "+v"(c));
    }
    __device__ __forceinline__ void get(R v[9]) const {
#pragma unroll
        for (int q = 0; q < 9; ++q) v[q] = v9[q];
    }
};
template <> struct RawBlock<float> : RawWide<float> {};
template <> struct RawBlock<double> : RawWide<double> {};

// Slots per slice whose blocks stay in registers for the whole launch (K)
// and per group in flight of those that stream (U), by slices per wavefront
// (512 threads: 256 registers a thread; 256 threads: 512).  A regular
// triangulation has 12 stored blocks a row, 13 with the diagonal.  G: blocks
// applied between two reads of window rows.
template <typename TB, int NS, int NT> struct Keep;
template <int NS, int NT> struct Keep<f16_t, NS, NT> {
    static constexpr int K = NS == 1 ? 18 : 12, U = 2, G = 3;
};
template <int NS, int NT> struct Keep<bf16_t, NS, NT> : Keep<f16_t, NS, NT> {};
template <int NS, int NT> struct Keep<float, NS, NT> {
    static constexpr int K = NS == 1 ? 12 : 5, U = 2, G = 3;
};
template <int NS, int NT> struct Keep<double, NS, NT> {
    static constexpr int K = NT == 256 ? 14 : (NS == 1 ? 5 : 2), U = 1, G = 2;
};

// Vectors a workgroup keeps in LDS: the iterate, and with two slices per
// wavefront, whose blocks take the registers, the residual.
constexpr int res_vectors(int ns) { return ns; }

// Doubles of LDS that hold an exchange's values while they are summed in
// order: 256 chains of 8 (p.q) or 2 x 128 of 9 or 2 x 64 of 16, padded.
constexpr int RAW = 2304;

// Slots of a slice: lane k of `meta` holds slot k's count in bits 6..12 and
// its offset from the slice's first stored block above.
struct SliceSlots {
    unsigned meta;
    int base, n;
};

// Slot k's block of this lane.  Branch-free: lanes past the slot's count and
// slots past the slice's last load a valid neighbour and get the lane's own
// row as their column, so they contribute a product with x_i - x_i = 0.
template <typename TB>
__device__ __forceinline__ void load_slot(RawBlock<TB> &B, const ResArgs &A, const SliceSlots &S, int k, int lane,
                                          int shift, unsigned self) {
    const unsigned m = (unsigned)__builtin_amdgcn_readlane((int)S.meta, min(k, S.n - 1));
    const int c = (int)(m >> 6) & 127, off = S.base + (int)(m >> 13);
    const unsigned l = (unsigned)min(lane, c - 1);
    B.load((const char *)A.jval + (int64_t)off * (9 * (int)sizeof(TB)), slot_width(c), l);
    const int16_t d = *reinterpret_cast<const int16_t *>((const char *)A.jdel + 2 * (int64_t)off + 2u * l);
    unsigned col = (unsigned)(shift + (int)d);
    const bool act = lane < (k < S.n ? c : 0);
    B.set_col(act ? (col == self ? col | DIAG : col) : self);
}

// the block's row of the window
template <typename TB>
__device__ __forceinline__ float3 block_p(const RawBlock<TB> &B, const float4 *pw) {
    const float4 v = pw[B.col() & (DIAG - 1)];
    return make_float3(v.x, v.y, v.z);
}

// a += block (x_j - x_i), or block x_i for the diagonal block (j = i)
template <typename TB, typename A>
__device__ __forceinline__ void apply_block(const RawBlock<TB> &B, const float3 &pj, A x0, A x1, A x2, A &a0, A &a1,
                                            A &a2) {
    typename BlockIO<TB>::R v[9];
    B.get(v);
    const A f = (B.col() & DIAG) ? A(0) : A(-1);
    const A d0 = __builtin_fma(f, x0, (A)pj.x), d1 = __builtin_fma(f, x1, (A)pj.y), d2 = __builtin_fma(f, x2, (A)pj.z);
    a0 += dot3((A)v[0], d0, (A)v[1], d1, (A)v[2], d2);
    a1 += dot3((A)v[3], d0, (A)v[4], d1, (A)v[5], d2);
    a2 += dot3((A)v[6], d0, (A)v[7], d1, (A)v[8], d2);
}

// The lane's N published values: `at(c)` gives the slot of value c, or null
// where the lane has none (its value is 0).  Polls until all are there; false
// when the wait gave up (v is then not set).  The count runs down from a kernel
// argument and at least one poll is made: tested before the first, with v set to
// 0 on the way out, it cost 0.6 us an iteration of the small FP64 systems.
template <int N, typename F>
__device__ __forceinline__ bool poll(F at, int polls, double (&v)[N]) {
    u64 b[N];
    do {
#pragma unroll
        for (int c = 0; c < N; ++c) {
            const u64 *p = at(c);
            b[c] = 0ull;
            if (p) b[c] = agent_load(p);
        }
        bool all = true;
#pragma unroll
        for (int c = 0; c < N; ++c) all = all && b[c] != EMPTY;
        if (__all(all)) {
#pragma unroll
            for (int c = 0; c < N; ++c) v[c] = __builtin_bit_cast(double, b[c]);
            return true;
        }
    } while (--polls > 0);
    return false;
}

// Sum in order of L values that poll() left in LDS, by the lane of their
// chain (chains an odd number of doubles apart, so the lanes' reads spread
// over the banks).
template <int L>
__device__ __forceinline__ double chain_sum(const double *v) {
    double val[L], s = 0.0;
#pragma unroll
    for (int i = 0; i < L; ++i) val[i] = v[i];
#pragma unroll
    for (int i = 0; i < L; ++i) s += val[i];
    return s;
}

// NS: 64-row slices per wavefront.  NS = 1 (SPLIT): the two slices of a pair
// are on two wavefronts (w and w + pairs); NS = 2: one pair per wavefront.
// KIND: 0 Jacobi, 1 block Jacobi.  FAR: windows with far rows and placed
// columns (with contacts; a kernel of its own because the loop over the far
// rows cost the others 3% where it was skipped).
template <typename TB, typename TV, int NS, int NT, int KIND, bool FAR>
__global__ void __launch_bounds__(NT) k_pcg_resident(ResArgs A) {
    extern __shared__ float4 pwin[];
    constexpr bool SPLIT = NS == 1;
    constexpr int NPL = SPLIT ? NT / 128 : 8;   // pairs per workgroup
    constexpr int K = Keep<TB, NS, NT>::K, U = Keep<TB, NS, NT>::U, GR = Keep<TB, NS, NT>::G;
    // the iterate, and for the kernels that keep most blocks in registers the
    // residual too, in LDS behind the window: component c of slice j's row of
    // thread t at (c NS + j) NT + t
    constexpr bool RLDS = NS == 2;
    typedef typename SpmvAcc<TB>::T Acc;
    typedef typename std::conditional<KIND == 0, TV, float>::type TE;   // exchanged planes
    __shared__ double ssum[2][NPL];    // slice sums of p.q, [half][local pair]
    __shared__ double wsum[2][NPL + 8];   // pair sums of r.z and r.r
    __shared__ double P1[16], P2[2][4];    // wavefront sums
    __shared__ double2 pass[SPLIT ? NPL : 1][WAVE];
    __shared__ int bad;
    const int4 G = A.wg[A.wg0 + (int)blockIdx.x];
    const ResInst I = A.inst[G.x];
    if (A.inst_win[G.x] > A.win_cap) return;
    PcgState &T = A.st[G.x];
    if (T.done) return;   // written by the team's first workgroup at its end, after everyone has started
    const int par = A.par;
    double rz = T.rzp[par];
    const double thresh = T.thresh;
    const int maxit = T.maxit;
    int iters = T.iters, flags = 0;
    const int t0 = threadIdx.x, nt = blockDim.x;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE)), nw = nt / WAVE;
    const int np = G.z;
    const ResWin W = A.win[A.wg0 + (int)blockIdx.x];
    const int lo = W.lo, wn = W.n, hi = lo + wn, nfar = FAR ? W.bn + W.an : 0;   // near rows [lo, hi), then the far ones
    auto far_row = [&](int f) { return f < W.bn ? W.blo + f : W.alo + f - W.bn; };
    if (t0 == 0) bad = A.polls == 0;   // 0: give up at the first meeting
    for (int k = t0; k < wn + nfar; k += nt) pwin[k] = ld3(A.p, !FAR || k < wn ? lo + k : far_row(k - wn));
    // rows of this workgroup: [a0, a1) and [b0, b1); the other rows of its
    // window are its halo
    const int it0 = G.y / 16, w0 = G.y % 16, rend = I.row0 + I.nrows;
    const int a0 = min(rend, I.row0 + 2048 * it0 + 64 * w0), a1 = min(rend, a0 + 64 * np);
    const int b0 = min(rend, I.row0 + 2048 * it0 + 1024 + 64 * w0), b1 = min(rend, b0 + 64 * np);
    const int h0 = max(0, a0 - lo), h1 = max(0, min(b0, hi) - a1), h2 = max(0, hi - max(a1, b1));
    const int hb = max(a1, b1), nh = h0 + h1 + h2;

    // the wavefront's slices j: local pair, half; first row r0 (rend: none);
    // the lane's row in stored order, relative to the window (-1 none)
    int r0[NS], srel[NS];
    SliceSlots slots[NS];
    RawBlock<TB> keep[NS][K > 0 ? K : 1];
    TV rv_[RLDS ? 1 : NS][3], q[NS][3];
    TV *const X = (TV *)A.x, *const R = (TV *)A.r;
    TE *const E = (TE *)A.exch;
    TV *const LX = (TV *)(pwin + A.win_rows);
    TV *const LR = LX + 3 * NS * NT;
    double *const raw = (double *)(LX + 3 * NS * NT * res_vectors(NS));   // published values, RAW of them
    auto pair_of = [&](int j) { return SPLIT ? (w < np ? w : w - np) : w; };
    auto half_of = [&](int j) { return SPLIT ? (w < np ? 0 : 1) : j; };
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int lane = lane_id();
        const int pl = pair_of(j), pg = G.y + pl;
        const int sl = 32 * (pg / 16) + 16 * half_of(j) + pg % 16;
        const bool have = pl < np && sl < I.nsl && (!SPLIT || w < 2 * np);
        r0[j] = have ? I.row0 + 64 * sl : rend;
        srel[j] = -1;
        slots[j].meta = 0u;
        slots[j].base = slots[j].n = 0;
        const int row = r0[j] + lane;
        if (have) {
            const int s = I.slice0 + sl;
            const int srow = A.lane_row[s * WAVE + lane], cnt = (int)A.slot_cnt[s * WAVE + lane];
            srel[j] = srow >= 0 ? srow - lo : -1;
            slots[j].base = A.slice_vbase[s];
            slots[j].n = __popcll(__ballot(cnt > 0));
            slots[j].meta = (row < rend ? (unsigned)A.row_lane[row] : 0u) | (unsigned)cnt << 6 |
                            (unsigned)wave_excl_scan(slot_width(cnt)) << 13;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            keep[j][k].clear();
            keep[j][k].set_col((unsigned)max(srel[j], 0));
            if (slots[j].n > 0)
                load_slot<TB>(keep[j][k], A, slots[j], k, lane, FAR ? 0 : r0[j] - lo, (unsigned)max(srel[j], 0));
            __builtin_amdgcn_sched_barrier(0);
        }
        const bool in = row < rend;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            LX[(c * NS + j) * NT + t0] = in ? X[3 * row + c] : TV(0);
            const TV rc = in ? R[3 * row + c] : TV(0);
            if constexpr (RLDS)
                LR[(c * NS + j) * NT + t0] = rc;
            else
                rv_[j][c] = rc;
            q[j][c] = TV(0);
        }
    }
    // Published values.  A workgroup's values of a meeting are consecutive
    // slots, written by one store instruction of its first wavefront(s) with
    // each copy's values on consecutive lanes: written one by one by the
    // wavefronts that form them, 8 values a workgroup took 5.0 us per meeting
    // of 256 workgroups against 2.65 us.
    //   p.q: SPLIT: slices, at 2 pair + half; else 8-slice sums, at 2 (8-pair
    //        run) + half;
    //   r.z, r.r: SPLIT: pairs, at 2 pair + which; else the run that starts an
    //        item as one sum, the other's pairs (32 slots an item).
    const int vq = SPLIT ? 2 * I.k : 2;
    const int vr = SPLIT ? 2 * I.k : (w0 == 0 ? 2 : 16);
    const int cq = t0 % vq, cr = t0 % vr;
    const int dq = t0 < vq * REPLICAS ? t0 / vq * A.slot_rep + I.pq_off + G.w * vq + cq : -1;
    const int dr = t0 < vr * REPLICAS
                       ? t0 / vr * A.slot_rep + A.slot_rz + I.rz_off + (SPLIT ? G.w * vr : 32 * it0 + 2 * w0) + cr
                       : -1;
    const u64 *const mine = A.slots + (size_t)(blockIdx.x % REPLICAS) * A.slot_rep;
    wait_stores();
    __syncthreads();

    int done = 0;
    for (int it = 0;; ++it) {
        const int buf = (it & 1) * A.slot_n, nbuf = A.slot_n - buf;
        // the lane as a new value each iteration: no address formed from it is
        // carried through the loop in registers of its own
        int lane = lane_id();
        asm volatile("" : "+v"(lane));
        const int t = WAVE * w + lane;
#pragma unroll
        for (int j = 0; j < NS; ++j) asm volatile("" : "+v"(srel[j]));
        // every workgroup has read the previous iteration's p.q
        if (dq >= 0) agent_store(A.slots + dq + nbuf, EMPTY);
        // ---- q = A p, slice sums of p.q.  Blocks past the kept ones stream
        // from memory: while a group is applied the next one's loads are in
        // flight, over the end of a slice into the wavefront's next one.
        RawBlock<TB> cur[U];
        bool ahead = false;
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            __builtin_amdgcn_sched_barrier(0);   // one slice's loads at a time
            if (r0[j] >= rend) continue;         // uniform per wavefront
            const int self = max(srel[j], 0), n = slots[j].n;
            const float4 ps = pwin[self];
            const Acc x0 = ps.x, x1 = ps.y, x2 = ps.z;
            Acc s0 = 0, s1 = 0, s2 = 0;
            const double m = A.mass[lo + self];
            if (n > K && !ahead) {
#pragma unroll
                for (int u = 0; u < U; ++u) load_slot<TB>(cur[u], A, slots[j], K + u, lane, FAR ? 0 : r0[j] - lo, (unsigned)self);
            }
            // kept blocks, GR at a time; the next ones' rows of the window
            // are read while these are applied
            float3 pj[2][GR];
#pragma unroll
            for (int k = 0; k < K + GR; k += GR) {
                if (SPLIT && k >= n + GR) break;   // uniform
#pragma unroll
                for (int u = k; u < k + GR; ++u)
                    if (u < K) {
                        keep[j][u].refresh();
                        pj[k / GR & 1][u - k] = block_p(keep[j][u], pwin);
                    }
                __builtin_amdgcn_sched_barrier(0);
                if (k == 0) continue;
#pragma unroll
                for (int u = k - GR; u < k; ++u)
                    if (u < K)
                        apply_block<TB, Acc>(keep[j][u], pj[(k / GR & 1) ^ 1][u - k + GR], x0, x1, x2, s0, s1, s2);
                __builtin_amdgcn_sched_barrier(0);
            }
            constexpr int J1 = NS - 1;
            const int jn = j < J1 ? j + 1 : j;
            const bool cross = j < J1 && r0[jn] < rend && slots[jn].n > K;
            ahead = cross && n > K;
            for (int k = K; k < n; k += U) {
                RawBlock<TB> nxt[U];
                float3 ps4[U];
                const bool over = cross && k + U >= n;
                SliceSlots S = slots[j];
                S.meta = over ? slots[jn].meta : S.meta;
                S.base = over ? slots[jn].base : S.base;
                S.n = over ? slots[jn].n : S.n;
                const int sf = over ? max(srel[jn], 0) : self, rr = over ? r0[jn] : r0[j], kn = over ? K : k + U;
#pragma unroll
                for (int u = 0; u < U; ++u) load_slot<TB>(nxt[u], A, S, kn + u, lane, FAR ? 0 : rr - lo, (unsigned)sf);
#pragma unroll
                for (int u = 0; u < U; ++u) ps4[u] = block_p(cur[u], pwin);
#pragma unroll
                for (int u = 0; u < U; ++u) apply_block<TB, Acc>(cur[u], ps4[u], x0, x1, x2, s0, s1, s2);
#pragma unroll
                for (int u = 0; u < U; ++u) cur[u] = nxt[u];
            }
            double y0 = (double)s0, y1 = (double)s1, y2 = (double)s2;
            if constexpr (BlockIO<TB>::SCALED) {
                const double vi = A.vscale_inv[2 * (I.slice0 + (r0[j] - I.row0) / WAVE)];
                y0 *= vi; y1 *= vi; y2 *= vi;
            }
            const TV q0 = (TV)__builtin_fma(m, (double)x0, y0), q1 = (TV)__builtin_fma(m, (double)x1, y1),
                     q2 = (TV)__builtin_fma(m, (double)x2, y2);
            double pq = dot3((double)x0, (double)q0, (double)x1, (double)q1, (double)x2, (double)q2);
            if (srel[j] < 0) pq = 0.0;
            const double s64 = wave_sum(pq);
            if (lane == 0) ssum[half_of(j)][pair_of(j)] = s64;
            // natural row order for the vector updates
            const int perm = (int)(slots[j].meta & 63u);
            q[j][0] = __shfl(q0, perm, WAVE);
            q[j][1] = __shfl(q1, perm, WAVE);
            q[j][2] = __shfl(q2, perm, WAVE);
        }
        __syncthreads();
        if (dq >= 0) {
            double sum;
            if constexpr (SPLIT) {
                sum = ssum[cq & 1][cq / 2];
            } else {
                // an SpMV item: eight slices in order
                const int sl = 32 * it0 + 16 * cq + w0;
                double val[8];
                sum = 0.0;
#pragma unroll
                for (int i = 0; i < 8; ++i) val[i] = ssum[cq][i];
#pragma unroll
                for (int i = 0; i < 8; ++i) sum += sl + i < I.nsl ? val[i] : 0.0;
            }
            agent_store(A.slots + dq + buf, sum_bits(sum));
        }
        // preconditioner entries, in flight while the sums are exchanged
        float pre[NS][KIND == 0 ? 3 : 6];
        auto load_pre = [&](int j) {
            const int row = r0[j] + lane;
            if (row >= rend) return;
            if constexpr (KIND == 0) {
#pragma unroll
                for (int c = 0; c < 3; ++c) pre[j][c] = A.pre[3 * row + c];
            } else {
                const float2 *b = (const float2 *)(A.pre + 6 * (int64_t)row);
                const float2 u = b[0], v = b[1], z = b[2];
                pre[j][0] = u.x; pre[j][1] = u.y; pre[j][2] = v.x;
                pre[j][3] = v.y; pre[j][4] = z.x; pre[j][5] = z.y;
            }
        };
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < NS; ++j) load_pre(j);
        __builtin_amdgcn_sched_barrier(0);
        // ---- p.q of the instance
        double pq;
        if constexpr (SPLIT) {
            // chunk c of this wavefront: slices 64 (w + nw c) ..
            double v[4];
            if (!poll<4>(
                    [&](int c) {
                        const int s = 64 * (w + nw * c) + lane;
                        return s < I.nsl ? mine + buf + I.pq_off + 2 * (16 * (s / 32) + s % 16) + (s / 16 & 1) : nullptr;
                    },
                    A.polls, v))
                bad = 1;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int s = 64 * (w + nw * c) + lane;
                if (s < 8 * I.ngroups) raw[9 * (s / 8) + s % 8] = v[c];
            }
            __syncthreads();
            // lane: an SpMV item; wavefront: 64 of them
            if (64 * w < I.ngroups) {
                const double s = wave_sum(64 * w + lane < I.ngroups ? chain_sum<8>(raw + 9 * (64 * w + lane)) : 0.0);
                if (lane == 0) P1[w] = s;
            }
        } else {
            // thread t: SpMV item t
            double v[1];
            if (!poll<1>(
                    [&](int) {
                        return t < I.ngroups ? mine + buf + I.pq_off + ((t & ~3) | (t & 1) << 1 | (t >> 1 & 1)) : nullptr;
                    },
                    A.polls, v))
                bad = 1;
            if (64 * w < I.ngroups) {
                const double s = wave_sum(0.0 + v[0]);
                if (lane == 0) P1[w] = s;
            }
        }
        __syncthreads();
        pq = 0.0;
        for (int k = 0; 64 * k < I.ngroups; ++k) pq += P1[k];
        if (bad) {
            if (t == 0) {
                atomicOr(&T.flags, 4);
                T.done = 1;
            }
            return;
        }
        const double alpha = rz / pq;
        if (!(pq > 0.0) || !isfinite(alpha)) {
            flags |= isfinite(pq) ? 1 : 2;
            done = 1;
            break;
        }
        // every workgroup has read the previous iteration's r.z
        if (dr >= 0) agent_store(A.slots + dr + nbuf, EMPTY);
        // ---- r -= alpha q, z = P^-1 r, partial sums; x += alpha p
        float zf[NS][3];
        double arz = 0.0, arr = 0.0;
        // slice j's rows, and their part of the sums, which continue those of
        // the pair's first slice
        auto update_rows = [&](int j, double (&rk)[3], double (&zk)[3]) {
            const int row = r0[j] + lane;
            if (row >= rend) return;
            TV rv[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int l = (c * NS + j) * NT + t;
                rv[c] = (TV)__builtin_fma(-alpha, (double)q[j][c], (double)(RLDS ? LR[l] : rv_[RLDS ? 0 : j][c]));
                rk[c] = rv[c];
                if constexpr (RLDS)
                    LR[l] = rv[c];
                else
                    rv_[j][c] = rv[c];
            }
            if constexpr (KIND != 0) {
                block_times(pre[j], rk, zk[0], zk[1], zk[2]);
#pragma unroll
                for (int c = 0; c < 3; ++c) zf[j][c] = (float)zk[c];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if constexpr (KIND == 0)
                    agent_store_f(E + (size_t)c * A.nv + row, rv[c]);
                else
                    agent_store_f(E + (size_t)c * A.nv + row, zf[j][c]);
            }
            const float4 po = pwin[row - lo];
            const float pc[3] = {po.x, po.y, po.z};
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                TV &xc = LX[(c * NS + j) * NT + t];
                xc = (TV)__builtin_fma(alpha, (double)pc[c], (double)xc);
            }
        };
        auto add_rows = [&](int j, bool first, const double (&rk)[3], const double (&zk)[3], double &rzs, double &rrs) {
            if (r0[j] + lane >= rend) return;
            sum_rr(rrs, rk, first);
            if constexpr (KIND == 0)
                sum_rz_jacobi(rzs, rk, pre[j]);
            else
                rzs += dot3(rk[0], zk[0], rk[1], zk[1], rk[2], zk[2]);
        };
        if constexpr (SPLIT) {
            // the second slice's wavefront continues the first one's sums
            double rk[3], zk[3];
            update_rows(0, rk, zk);
            if (w < np) {
                add_rows(0, true, rk, zk, arz, arr);
                pass[w][lane] = make_double2(arz, arr);
            }
            __syncthreads();
            if (w >= np && w < 2 * np) {
                const double2 c = pass[w - np][lane];
                arz = c.x;
                arr = c.y;
                add_rows(0, false, rk, zk, arz, arr);
                const double s0 = wave_sum(arz), s1 = wave_sum(arr);
                if (lane == 0) {
                    wsum[0][w - np] = s0;
                    wsum[1][w - np] = s1;
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                double rk[3], zk[3];
                __builtin_amdgcn_sched_barrier(0);   // one slice's values at a time
                update_rows(j, rk, zk);
                add_rows(j, j == 0, rk, zk, arz, arr);
            }
            const double s0 = wave_sum(arz), s1 = wave_sum(arr);
            if (lane == 0) {
                wsum[0][w] = s0;
                wsum[1][w] = s1;
            }
        }
        wait_stores();
        __syncthreads();
        if (dr >= 0) {
            double sum;
            if constexpr (SPLIT) {
                sum = wsum[cr & 1][cr / 2];
            } else {
                // the item's first eight pairs in order, or one pair
                const int pl = cr / 2, nr = w0 == 0 ? min(8, np) : 1;
                double val[8];
                sum = 0.0;
#pragma unroll
                for (int i = 0; i < 8; ++i) val[i] = wsum[cr & 1][pl + i];
#pragma unroll
                for (int i = 0; i < 8; ++i) sum += i < nr ? val[i] : 0.0;
            }
            agent_store(A.slots + dr + buf, sum_bits(sum));
        }
        // ---- r.z and r.r of the instance
        // value e: SPLIT: pair e / 2; else (32 slots an item) the sum of the
        // item's first eight pairs, then each of the others
        constexpr int PER = SPLIT ? 32 : 18, ST = SPLIT ? 17 : 9, NC = SPLIT ? 4 : 5;
        double v[NC];
        const int ne = PER * I.nitems;
        if (!poll<NC>(
                [&](int c) {
                    const int e = t + nt * c, i = e / PER, k = e % PER;
                    const bool on = e < ne && (SPLIT ? 32 * i + k / 2 < I.nsl : k < 2 || 32 * i + 7 + k / 2 < I.nsl);
                    return on ? mine + buf + A.slot_rz + I.rz_off + 32 * i + (SPLIT || k < 2 ? k : 14 + k) : nullptr;
                },
                A.polls, v))
            bad = 1;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int e = t + nt * c;
            if (e < ne) raw[(e & 1) * (RAW / 2) + ST * (e / PER) + e % PER / 2] = v[c];
        }
        __syncthreads();
        // lane: an item; wavefronts: r.z and r.r of 64 items
        const int i = 64 * (w / 2) + lane;
        if (64 * (w / 2) < I.nitems) {
            const double s = wave_sum(i < I.nitems ? chain_sum<PER / 2>(raw + (w & 1) * (RAW / 2) + ST * i) : 0.0);
            if (lane == 0) P2[w & 1][w / 2] = s;
        }
        __syncthreads();
        double tz = 0.0, tr = 0.0;
        for (int k = 0; 64 * k < I.nitems; ++k) {
            tz += P2[0][k];
            tr += P2[1][k];
        }
        if (bad) {
            if (t == 0) {
                atomicOr(&T.flags, 4);
                T.done = 1;
            }
            return;
        }
        // ---- convergence, beta, p = z + beta p over the window
        const double beta = tz / rz;
        const bool notfinite = !isfinite(tr) || !isfinite(tz);
        const bool conv = tr <= thresh;
        const bool new_dir = !(notfinite || conv);
        rz = tz;
        ++iters;
        if (notfinite) {
            flags |= 2;
            done = 1;
        } else if (conv || iters >= maxit) {
            done = 1;
        }
        const bool finished = done || it + 1 >= A.max_iters;
        if (t == 0 && G.w == 0) {
            T.rr = tr;
            if (new_dir) T.rzd = tz;
        }
        auto direct = [&](int at, double z0, double z1, double z2) {
            const float4 po = pwin[at];
            pwin[at] = make_float4((float)__builtin_fma(beta, (double)po.x, z0),
                                         (float)__builtin_fma(beta, (double)po.y, z1),
                                         (float)__builtin_fma(beta, (double)po.z, z2), 0.0f);
        };
        // n rows of the halo, four rows' loads in flight per thread
        auto halo = [&](int n, auto row_of, auto place_of) {
            for (int hh = t; hh < n; hh += 4 * nt) {
                TE e[4][3];
                int row[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    row[u] = row_of(min(hh + u * nt, n - 1));
#pragma unroll
                    for (int c = 0; c < 3; ++c) e[u][c] = agent_load_f(E + (size_t)c * A.nv + row[u]);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (hh + u * nt >= n) break;
                    double z[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        z[c] = (double)e[u][c];
                        if constexpr (KIND == 0) z[c] *= (double)A.pre[3 * row[u] + c];
                    }
                    direct(place_of(hh + u * nt, row[u]), z[0], z[1], z[2]);
                }
            }
        };
        if (new_dir) {
            if (!finished) {
                halo(nh, [&](int h) { return h < h0 ? lo + h : (h < h0 + h1 ? a1 + h - h0 : hb + h - h0 - h1); },
                     [&](int, int row) { return row - lo; });
                if constexpr (FAR) halo(nfar, far_row, [&](int f, int) { return wn + f; });
            }
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                const int row = r0[j] + lane;
                if (row >= rend) continue;
                if constexpr (KIND == 0) {
                        double z[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        z[c] = (double)(RLDS ? LR[(c * NS + j) * NT + t] : rv_[RLDS ? 0 : j][c]) * (double)pre[j][c];
                    direct(row - lo, z[0], z[1], z[2]);
                } else {
                    direct(row - lo, (double)zf[j][0], (double)zf[j][1], (double)zf[j][2]);
                }
            }
        }
        if (finished) break;
        __syncthreads();
    }
    // ---- results: r, x and the own rows of p
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int row = r0[j] + lane_id();
        if (row < rend) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                R[3 * row + c] = RLDS ? LR[(c * NS + j) * NT + t0] : rv_[RLDS ? 0 : j][c];
                X[3 * row + c] = LX[(c * NS + j) * NT + t0];
            }
            const float4 po = pwin[row - lo];
            st3(A.p, row, po.x, po.y, po.z);
        }
    }
    if (t0 == 0 && G.w == 0) {
        T.rzp[par] = rz;
        T.live[0] = T.live[1] = 0;
        T.iters = iters;
        // a workgroup that gave up at the last meeting may be setting both now
        atomicOr(&T.flags, flags);
        atomicOr(&T.done, done);
    }
}

// Block-column window of every resident workgroup: the near columns (within
// `reach` rows of its own), the smallest and largest of those below and of
// those above them (contacts couple sheets whose rows lie far apart); and the
// most rows of a window of each instance.
constexpr int RES_REACH = 4096;
__global__ void __launch_bounds__(256) k_res_windows(const ResInst *inst, const int4 *wg, const int *rowptr,
                                                     const int *colidx, int reach, ResWin *win, int *inst_win) {
    __shared__ int sh[6][4];
    const int4 G = wg[blockIdx.x];
    const ResInst I = inst[G.x];
    const int rend = I.row0 + I.nrows, it0 = G.y / 16, w0 = G.y % 16;
    const int a0 = min(rend, I.row0 + 2048 * it0 + 64 * w0), a1 = min(rend, a0 + 64 * G.z);
    const int b0 = min(rend, I.row0 + 2048 * it0 + 1024 + 64 * w0), b1 = min(rend, b0 + 64 * G.z);
    const int nlo = a0 - reach, nhi = max(a1, b1) + reach;
    int v[6] = {0x7fffffff, -1, 0x7fffffff, -1, 0x7fffffff, -1};   // near, below, above: smallest, largest
    for (int run = 0; run < 2; ++run) {
        const int e0 = run ? rowptr[b0] : rowptr[a0], e1 = run ? rowptr[b1] : rowptr[a1];
        for (int k = e0 + (int)threadIdx.x; k < e1; k += blockDim.x) {
            const int c = colidx[k], q = c < nlo ? 2 : (c >= nhi ? 4 : 0);
#pragma unroll
            for (int x = 0; x < 6; x += 2)
                if (q == x) {
                    v[x] = min(v[x], c);
                    v[x + 1] = max(v[x + 1], c);
                }
        }
    }
#pragma unroll
    for (int x = 0; x < 6; ++x) {
        for (int m = 32; m >= 1; m >>= 1) {
            const int o = __shfl_xor(v[x], m, WAVE);
            v[x] = x & 1 ? max(v[x], o) : min(v[x], o);
        }
        if (lane_id() == 0) sh[x][threadIdx.x / WAVE] = v[x];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int x = 0; x < 6; ++x)
            for (int k = 1; k < (int)blockDim.x / WAVE; ++k) v[x] = x & 1 ? max(v[x], sh[x][k]) : min(v[x], sh[x][k]);
        ResWin W;
        W.lo = v[0]; W.n = v[1] - v[0] + 1;
        W.blo = v[3] < 0 ? 0 : v[2]; W.bn = v[3] < 0 ? 0 : v[3] - v[2] + 1;
        W.alo = v[5] < 0 ? 0 : v[4]; W.an = v[5] < 0 ? 0 : v[5] - v[4] + 1;
        win[blockIdx.x] = W;
        atomicMax(&inst_win[G.x], W.n + W.bn + W.an);
    }
}

// Every stored block's column as a row of its workgroup's window (where the
// window has the rows that fit; a wider one is not used).  One workgroup per
// resident workgroup, a wavefront per slice.
__global__ void __launch_bounds__(512) k_res_place(const ResInst *inst, const int4 *wg, const ResWin *win,
                                                   const int *slice_vbase, const uint8_t *slot_cnt, const int *jcol,
                                                   int16_t *place) {
    const int4 G = wg[blockIdx.x];
    const ResInst I = inst[G.x];
    const ResWin W = win[blockIdx.x];
    const int lane = lane_id();
    for (int q = threadIdx.x / WAVE; q < 2 * G.z; q += blockDim.x / WAVE) {
        const int pg = G.y + q / 2, sl = 32 * (pg / 16) + 16 * (q & 1) + pg % 16;
        if (sl >= I.nsl) continue;
        const int s = I.slice0 + sl, cnt = (int)slot_cnt[s * WAVE + lane];
        const int off = slice_vbase[s] + wave_excl_scan(slot_width(cnt));
        const int n = __popcll(__ballot(cnt > 0));
        for (int k = 0; k < n; ++k) {
            const int at = __builtin_amdgcn_readlane(off, k) + lane;
            if (lane >= __builtin_amdgcn_readlane(cnt, k)) continue;
            const int c = jcol[at];
            place[at] = (int16_t)(c < W.lo ? W.n + c - W.blo : (c < W.lo + W.n ? c - W.lo : W.n + W.bn + c - W.alo));
        }
    }
}

__global__ void k_res_clear(u64 *slots, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) slots[i] = EMPTY;
}

// ---------------------------------------------------------------- host side
// Teams.  With P = 2 or 4 pairs per workgroup (one slice per wavefront, 2 P
// wavefronts) or 8 (two slices per wavefront of 8), the smallest P whose teams
// fit the compute units at once is taken: one workgroup per unit.  P = 1 meets
// with twice the workgroups (us per iteration, P = 1 / 2, FP64 and FP32 blocks:
// 1k rows 6.1 / 6.2 and 5.8 / 5.8, 3k 8.7 / 7.6 and 8.1 / 6.9, 7k 9.4 / 8.2 and
// 8.7 / 7.5, 33k 11.7 / 9.6 and 11.1 / 9.0); with P = 4 fewer FP64 blocks stay in
// registers (3k 10.6, 33k 12.7), while FP32 gains at most 1.9 us (62k 10.9 / 9.0).  Where 8 do not fit, the instances go in
// several rounds, each to the end of the sweep.  An instance of more than
// 1,024 rows a unit does not fit any round: the three-launch iteration runs.
// (Whole items per workgroup, 2,048 rows, kept 4 of 12 blocks a row in
// registers and streamed the rest with 8 wavefronts in flight: 41.0 us against
// 43.3 us at 420k rows, but half of the chip idle just past 262k rows, and a
// batch in two such rounds 73 us against 62 us.)
pc_status resident_plan(Ctx *ctx) {
    ResPlan &P = ctx->res;
    P.planned = true;
    P.valid = false;
    P.rounds.clear();
    const int ninst = (int)ctx->inst_row0_h.size() - 1;
    int dev = 0, ncu = 0;
    PC_HIP(hipGetDevice(&dev));
    PC_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    if (ncu < 1) return PC_OK;
    ncu = std::min(ncu, 256);   // P1, P2 and RAW hold the sums of 256 workgroups
    std::vector<ResInst> inst(ninst);
    int slice0 = 0;
    for (int i = 0; i < ninst; ++i) {
        ResInst &I = inst[i];
        I.row0 = ctx->inst_row0_h[i];
        I.nrows = ctx->inst_row0_h[i + 1] - I.row0;
        I.slice0 = slice0;
        I.nsl = (I.nrows + WAVE - 1) / WAVE;
        slice0 += I.nsl;
        I.ngroups = (I.nsl + 7) / 8;
        I.nitems = (I.nsl + 31) / 32;
    }
    auto pairs_of = [](const ResInst &I) { return 16 * (I.nitems - 1) + std::min(16, I.nsl - 32 * (I.nitems - 1)); };
    auto team_of = [&](const ResInst &I, int per) { return (pairs_of(I) + per - 1) / per; };
    int per = 8;
    for (int cand : {2, 4, 8}) {
        int64_t sum = 0;
        for (const ResInst &I : inst) sum += team_of(I, cand);
        if (sum <= ncu) {
            per = cand;
            break;
        }
    }
    P.ns = per <= 4 ? 1 : 2;
    P.threads = per <= 4 ? 2 * per * WAVE : 512;
    std::vector<int4> wg;
    int npq = 0, nrz = 0, first = 0;
    for (int i = 0; i < ninst; ++i) {
        ResInst &I = inst[i];
        I.k = per;
        I.team = team_of(I, per);
        if (I.team > ncu) return PC_OK;
        if ((int)wg.size() - first + I.team > ncu) {
            P.rounds.push_back({first, (int)wg.size() - first});
            first = (int)wg.size();
        }
        const int pairs = pairs_of(I);
        for (int g = 0; g < I.team; ++g) wg.push_back(int4{i, g * per, std::min(per, pairs - g * per), g});
        I.pq_off = npq;
        I.rz_off = nrz;
        npq += per <= 4 ? 32 * I.nitems : (4 * I.nitems + 15) / 16 * 16;   // whole cache lines
        nrz += 32 * I.nitems;
    }
    P.rounds.push_back({first, (int)wg.size() - first});
    P.slot_rz = npq;
    P.slot_n = npq + nrz;
    P.slot_rep = 2 * P.slot_n + 32;
    P.coop = false;
    for (const ResInst &I : inst) P.coop = P.coop || I.team > 1;
    // one block: the instances and workgroups, in one copy, then windows and slots
    const size_t inst_bytes = (sizeof(ResInst) * ninst + 15) / 16 * 16, wg_bytes = sizeof(int4) * wg.size();
    const size_t win_at = inst_bytes + wg_bytes, slots_at = (win_at + sizeof(ResWin) * wg.size() + 127) / 128 * 128;
    const size_t bytes = slots_at + sizeof(u64) * (size_t)REPLICAS * P.slot_rep;
    if (bytes > P.mem_bytes) {
        dev_free(ctx, P.mem);
        P.mem = nullptr;
        P.mem_bytes = 0;
        if (dev_alloc(ctx, (void **)&P.mem, bytes)) return PC_OK;   // the three launches need none of it
        P.mem_bytes = bytes;
    }
    std::vector<char> up(win_at);
    std::copy_n((const char *)inst.data(), sizeof(ResInst) * ninst, up.data());
    std::copy_n((const char *)wg.data(), wg_bytes, up.data() + inst_bytes);
    PC_HIP(hipMemcpy(P.mem, up.data(), win_at, hipMemcpyHostToDevice));
    P.inst = (ResInst *)P.mem;
    P.wg = (int4 *)(P.mem + inst_bytes);
    P.win = (ResWin *)(P.mem + win_at);
    P.slots = (u64 *)(P.mem + slots_at);
    P.nwg = (int)wg.size();
    P.valid = true;
    return PC_OK;
}

void resident_free(Ctx *ctx) {
    ResPlan &P = ctx->res;
    dev_free(ctx, P.mem);
    dev_free(ctx, P.place);
    P = ResPlan{};
}

// Without contacts one near range is the whole window and the 16-bit offsets
// serve; with contacts the columns are placed per assembly (16 bits a block),
// and where there is no memory for that the solve does without.
pc_status resident_windows(Ctx *ctx, int *inst_win, bool *fits, hipStream_t s) {
    ResPlan &P = ctx->res;
    *fits = true;
    P.placed = ctx->nc > 0;
    hipLaunchKernelGGL(k_res_windows, dim3(P.nwg), dim3(256), 0, s, P.inst, P.wg, ctx->rowptr, ctx->colidx,
                       P.placed ? RES_REACH : 1 << 30, P.win, inst_win);
    if (P.placed) {
        const size_t bytes = sizeof(int16_t) * (size_t)ctx->vcap;
        if (bytes > P.place_bytes) {
            dev_free(ctx, P.place);
            P.place = nullptr;
            P.place_bytes = 0;
            if (dev_alloc(ctx, (void **)&P.place, bytes)) {
                *fits = false;
                return PC_OK;
            }
            P.place_bytes = bytes;
        }
        hipLaunchKernelGGL(k_res_place, dim3(P.nwg), dim3(512), 0, s, P.inst, P.wg, P.win, ctx->slice_vbase,
                           ctx->slot_cnt, ctx->jcol, P.place);
    }
    return PC_OK;
}

template <typename TB, typename TV, int NS, int NT, int KIND, bool FAR>
static pc_status launch_kind(Ctx *ctx, ResArgs &A, bool *taken, hipStream_t s) {
    const ResPlan &P = ctx->res;
    const size_t lds = sizeof(float4) * (size_t)P.win_rows + sizeof(TV) * (size_t)(3 * NS * NT * res_vectors(NS)) +
                       sizeof(double) * RAW;
    const void *fn = (const void *)k_pcg_resident<TB, TV, NS, NT, KIND, FAR>;
    // the function's attribute is the process's: every context and thread sets the same
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, RES_LDS);
    const size_t nslots = (size_t)REPLICAS * P.slot_rep;
    if (e == hipSuccess)
        hipLaunchKernelGGL(k_res_clear, dim3((nslots + 255) / 256), dim3(256), 0, s, A.slots, nslots);
    for (size_t k = 0; k < P.rounds.size() && e == hipSuccess; ++k) {
        A.wg0 = P.rounds[k].first;
        const dim3 grid(P.rounds[k].second), block(P.threads);
        if (P.coop) {
            void *args[] = {&A};
            e = hipLaunchCooperativeKernel(fn, grid, block, args, (unsigned)lds, s);
        } else {
            hipLaunchKernelGGL((k_pcg_resident<TB, TV, NS, NT, KIND, FAR>), grid, block, lds, s, A);
            e = hipGetLastError();
        }
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *taken = false;
    }
    return PC_OK;
}

template <typename TB, typename TV, int NS, int NT>
static pc_status launch_ns(Ctx *ctx, ResArgs &A, bool *taken, hipStream_t s) {
    if (ctx->res.placed)
        return ctx->precond == 0 ? launch_kind<TB, TV, NS, NT, 0, true>(ctx, A, taken, s)
                                 : launch_kind<TB, TV, NS, NT, 1, true>(ctx, A, taken, s);
    return ctx->precond == 0 ? launch_kind<TB, TV, NS, NT, 0, false>(ctx, A, taken, s)
                             : launch_kind<TB, TV, NS, NT, 1, false>(ctx, A, taken, s);
}

int resident_win_max(const Ctx *ctx) {
    const ResPlan &P = ctx->res;
    const int bytes = ctx->inner32 ? 4 : 8;
    const int kept = 3 * P.ns * 512 * res_vectors(P.ns) * bytes + (int)sizeof(double) * RAW;
    return (RES_LDS - kept) / (int)sizeof(float4);
}

// Storage and vector types the resident kernel is built for: FP16 and BF16
// blocks with FP32 inner vectors (their refinement sweeps), FP32 and FP64
// blocks with FP64 vectors, and FP64 blocks with FP32 inner vectors (a sweep
// after a fallback).  Wider types keep at most four slices per wavefront in
// registers.
bool resident_fits(const Ctx *ctx) {
    const bool low = ctx->dtype == PC_BF16 || ctx->dtype == PC_F16;
    return ctx->res.valid && ctx->res.win_rows > 0 && (!low || ctx->inner32);
}

template <typename TB>
pc_status resident_launch(Ctx *ctx, const SpmvArgs &M, int max_iters, bool *taken, hipStream_t s) {
    *taken = true;
    const ResPlan &P = ctx->res;
    ResArgs A{};
    A.slice_vbase = M.slice_vbase;
    A.lane_row = M.lane_row;
    A.row_lane = ctx->row_lane;
    A.slot_cnt = M.slot_cnt;
    A.jdel = P.placed ? P.place : ctx->jdel;   // within a window of at most 9,728 rows both fit 16 bits
    A.jval = M.jval;
    A.mass = M.mass;
    A.vscale_inv = ctx->f16_scale ? ctx->f16_scale + 1 : nullptr;
    A.nv = ctx->nv;
    A.inst = P.inst;
    A.wg = P.wg;
    A.win = P.win;
    A.inst_win = P.inst_win;
    A.win_rows = A.win_cap = P.win_rows;
    A.st = ctx->st;
    A.p = ctx->p;
    A.pre = ctx->precond == 0 ? ctx->dinv : ctx->binv;
    A.exch = ctx->precond == 0 && !ctx->inner32 ? (void *)ctx->q : (void *)ctx->zb;
    A.slots = P.slots;
    A.slot_n = P.slot_n;
    A.slot_rep = P.slot_rep;
    A.slot_rz = P.slot_rz;
    A.par = ctx->cg_par;
    A.max_iters = max_iters;
    A.polls = ctx->res_polls;
    A.x = ctx->inner32 ? (void *)ctx->e32 : (void *)ctx->x;
    A.r = ctx->inner32 ? (void *)ctx->r32 : (void *)ctx->r;
    constexpr bool low = std::is_same<TB, f16_t>::value || std::is_same<TB, bf16_t>::value;
    constexpr bool f64 = std::is_same<TB, double>::value;
    if constexpr (low || f64) {
        if (ctx->inner32) {
            if constexpr (f64) {   // 512 registers where 256 threads do
                if (P.threads <= 256) return launch_ns<TB, float, 1, 256>(ctx, A, taken, s);
            }
            if (P.ns == 1) return launch_ns<TB, float, 1, 512>(ctx, A, taken, s);
            if (P.ns == 2) return launch_ns<TB, float, 2, 512>(ctx, A, taken, s);
        }
    }
    if constexpr (!low) {
        if (!ctx->inner32) {
            if constexpr (f64) {
                if (P.threads <= 256) return launch_ns<TB, double, 1, 256>(ctx, A, taken, s);
            }
            if (P.ns == 1) return launch_ns<TB, double, 1, 512>(ctx, A, taken, s);
            if (P.ns == 2) return launch_ns<TB, double, 2, 512>(ctx, A, taken, s);
        }
    }
    ctx->err = "internal: resident CG variant";
    return PC_ERR_ARG;
}

template pc_status resident_launch<double>(Ctx *, const SpmvArgs &, int, bool *, hipStream_t);
template pc_status resident_launch<float>(Ctx *, const SpmvArgs &, int, bool *, hipStream_t);
template pc_status resident_launch<bf16_t>(Ctx *, const SpmvArgs &, int, bool *, hipStream_t);
template pc_status resident_launch<f16_t>(Ctx *, const SpmvArgs &, int, bool *, hipStream_t);

}  // namespace pc
