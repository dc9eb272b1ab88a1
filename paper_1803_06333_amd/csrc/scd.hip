// The SCD epoch kernels (Section 3.1): per coordinate a gather-dot of its nonzeros with the shared
// vector v, a scalar step (closed form for ridge and for the clipped hinge dual, one Newton step
// for logistic regression), and an atomic scatter of delta * a_j into v.  Many coordinates are in
// flight at once and see each other's partial updates, as in the paper's asynchronous solver.
//
// The paper's solver gives every coordinate one thread block.  On a 256-CU part with click-log
// data (a few columns holding a fifth of all rows each, a million columns of a few hundred) that
// leaves the epoch waiting for a handful of blocks, so coordinates are handled in two classes:
//   small  (<= small_max = 4096 nonzeros): one 64-wide wavefront per coordinate, four per workgroup;
//   large  (longer): split into segments of seg = 16384 nonzeros.  Every segment is two
//          work items, "dot" and "scatter".  Workgroups draw items from one atomic ticket counter
//          in epoch order; the dot items of a coordinate add their partial sums into its state and
//          the last one to arrive takes the step and publishes delta; a scatter item waits for
//          that flag.  A waiting workgroup only ever waits for workgroups that drew an earlier
//          ticket and are therefore already running, so the wait always ends; it is bounded by
//          SPIN_LIMIT all the same and raises the handle's status word instead of hanging.
#include "scd_device.h"
#include <algorithm>

namespace snap {

// ---- small coordinates: one wavefront each ----------------------------------------------------
// A wavefront walks its share of the epoch order, and what a coordinate needs is a chain of dependent
// loads: its place in the order, its two ptr entries, its indices and values, the entries of v they
// name, its own x / norm / label.  With few coordinates in flight (the cap that keeps the asynchronous
// solver convergent: some hundred rows for the hinge dual on data with popular features) that chain,
// not bandwidth, sets the pace.  So the chain is taken apart over three visits: while the gather of
// coordinate i is under way, the nonzeros and scalars of i+1, the ptr entries of i+2 and the order
// entry of i+3 are requested too, all independent of each other; only the reads of v, which must be
// as late as possible, stay in the visit they belong to.  (x[c], the norms and the labels are not
// written by other coordinates' updates.)  The part of the step that does not need v is taken while the
// gather is under way.  What was requested for later visits is waited for ahead of the scatter: memory
// operations are waited for in the order of their issue, so that waiting for it at the top of the next
// visit would also wait for the atomics of this one (3700 of the 6700 cycles of a visit with 200
// nonzeros) before the next gather has even been asked for.
//
// Up to ROUNDS nonzeros per lane travel in registers and are scattered from there; longer coordinates
// take the rest in loops of TAIL_ROUNDS independent loads.  ROUNDS is the smallest of 1, 4 and 16 that holds
// the longest coordinate (16 from 257 nonzeros on; columns of 465 nonzeros that took every fifth and
// later round through dependent loads cost 28000 cycles a visit).
//
// One wavefront per workgroup: a compute unit issues about one scattered atomic per six cycles, so
// the four wavefronts of a workgroup queued on one unit while most of the 256 units had none.
constexpr int SMALL_TPB = WAVE;
constexpr int TAIL_ROUNDS = 8;

template <int ROUNDS>
struct SmallCoord {
    int64_t c, s0, s1;            // coordinate, its range in the chunk's arrays
    uint32_t raw[ROUNDS];         // index words of this lane: nonzeros s0 + j * 64 + lane
    float a[ROUNDS];
    float xc, nc, yc;
};

template <int KIND, int ROUNDS>
__global__ void __launch_bounds__(SMALL_TPB)
k_scd_small(ChunkView cv, const uint32_t* __restrict__ order, int64_t n_small, const float* __restrict__ y,
            float* __restrict__ x, float* v, const float* __restrict__ norms, StepParams sp, int64_t n_waves) {
    const int lane = threadIdx.x;
    const int64_t wave0 = blockIdx.x;
    constexpr uint32_t IDX_MASK = KIND == K_PRIMAL_LOGISTIC ? ~LABEL_BIT : 0xFFFFFFFFu;
    // n_waves wavefronts walk the epoch order round-robin: at most n_waves coordinates in flight.
    auto order_entry = [&](int64_t wid) -> uint32_t { return wid < n_small ? order[wid] : 0u; };
    auto ptr_pair = [&](int64_t c, int64_t& p0, int64_t& p1) {
        p0 = p1 = 0;
        if (c >= 0) {
            p0 = cv.ptr[c];
            p1 = cv.ptr[c + 1];
        }
    };
    auto fetch = [&](int64_t c, int64_t s0, int64_t s1) -> SmallCoord<ROUNDS> {
        SmallCoord<ROUNDS> q;
        q.c = c, q.s0 = s0, q.s1 = s1;
        q.xc = q.nc = q.yc = 0.0f;
#pragma unroll
        for (int j = 0; j < ROUNDS; ++j) {
            const int64_t k = s0 + j * WAVE + lane;
            q.raw[j] = 0u;
            q.a[j] = 0.0f;
            if (k < s1) {
                q.raw[j] = cv.idx[k];
                q.a[j] = cv.val[k];
            }
        }
        if (c >= 0) {   // the same address in every lane: one request
            q.xc = x[c];
            q.nc = norms[c];
            if (KIND == K_DUAL) q.yc = y[c];
        }
        return q;
    };
    // fill the pipeline: three coordinates' order entries, two ptr pairs, one record
    auto coord_at = [&](int64_t wid, uint32_t entry) -> int64_t { return wid < n_small ? cv.c0 + (int64_t)entry : -1; };
    int64_t cB = coord_at(wave0 + n_waves, order_entry(wave0 + n_waves));   // its nonzeros are requested next
    uint32_t entryA = order_entry(wave0 + 2 * n_waves);                     // its ptr pair is read next
    int64_t p0B, p1B;
    SmallCoord<ROUNDS> cur;
    {
        const int64_t c = coord_at(wave0, order_entry(wave0));
        int64_t p0, p1;
        ptr_pair(c, p0, p1);
        ptr_pair(cB, p0B, p1B);
        cur = fetch(c, p0 - cv.nnz_base, p1 - cv.nnz_base);
    }
    for (int64_t wid = wave0; wid < n_small; wid += n_waves) {
        // this visit's requests
        const int64_t c = cur.c, s0 = cur.s0, s1 = cur.s1;
        uint32_t r[ROUNDS];
        float vv[ROUNDS], yy[ROUNDS];
        bool have[ROUNDS];
#pragma unroll
        for (int j = 0; j < ROUNDS; ++j) {
            have[j] = s0 + j * WAVE + lane < s1;
            r[j] = cur.raw[j] & IDX_MASK;
            vv[j] = yy[j] = 0.0f;
            if (have[j]) {
                vv[j] = load_shared(v, r[j]);
                if (KIND == K_PRIMAL_RIDGE) yy[j] = y[r[j]];
                if (KIND == K_PRIMAL_LOGISTIC) yy[j] = (cur.raw[j] & LABEL_BIT) ? -1.0f : 1.0f;
            }
        }
        SmallCoord<ROUNDS> nxt = fetch(cB, p0B - cv.nnz_base, p1B - cv.nnz_base);
        const int64_t cA = coord_at(wid + 2 * n_waves, entryA);
        int64_t p0A, p1A;
        ptr_pair(cA, p0A, p1A);
        uint32_t entry3 = order_entry(wid + 3 * n_waves);
        // nothing moves across: the requests first, then what can be computed while they are under way
        __builtin_amdgcn_sched_barrier(0);
        StepPrep prep = prepare_step<KIND>(cur.xc, cur.nc, cur.yc, sp);
        asm volatile("" : "+v"(prep.a), "+v"(prep.b), "+v"(prep.c));
        __builtin_amdgcn_sched_barrier(0);

        float g = 0.0f, h = 0.0f;
        // (these nonzeros stay in registers for the scatter pass)
#pragma unroll
        for (int j = 0; j < ROUNDS; ++j)
            if (have[j]) accumulate<KIND>(cur.a[j], vv[j], yy[j], g, h);
        for (int64_t k0 = s0 + ROUNDS * WAVE + lane; k0 < s1; k0 += TAIL_ROUNDS * WAVE) {
            uint32_t rr[TAIL_ROUNDS];
            float at[TAIL_ROUNDS], yt[TAIL_ROUNDS], vt[TAIL_ROUNDS];
#pragma unroll
            for (int j = 0; j < TAIL_ROUNDS; ++j) {        // (past the end: the lane's first nonzero with value 0)
                const int64_t k = k0 + j * WAVE;
                const bool on = k < s1;
                rr[j] = cv.idx[on ? k : k0];
                at[j] = on ? cv.val[k] : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < TAIL_ROUNDS; ++j) {
                decode<KIND>(rr[j], rr[j], yt[j], y);
                vt[j] = load_shared(v, rr[j]);
            }
#pragma unroll
            for (int j = 0; j < TAIL_ROUNDS; ++j) accumulate<KIND>(at[j], vt[j], yt[j], g, h);
        }
        g = wave_sum(g);
        if (KIND == K_PRIMAL_LOGISTIC) h = wave_sum(h);
        // every lane takes the same step
        float mult;
        const float xn = finish_step<KIND>((double)g, (double)h, cur.xc, cur.nc, cur.yc, prep, sp, mult);
        if (lane == 0) x[c] = xn;
        // the requests of this visit for later ones have arrived by now: take them over ahead of the atomics
#pragma unroll
        for (int j = 0; j < ROUNDS; ++j) asm volatile("" : "+v"(nxt.raw[j]), "+v"(nxt.a[j]));
        asm volatile("" : "+v"(nxt.xc), "+v"(nxt.nc), "+v"(nxt.yc), "+v"(p0A), "+v"(p1A), "+v"(entry3));
        __builtin_amdgcn_sched_barrier(0);
        if (mult != 0.0f) {
#pragma unroll
            for (int j = 0; j < ROUNDS; ++j)
                if (have[j]) unsafeAtomicAdd(v + r[j], mult * cur.a[j]);
            for (int64_t k0 = s0 + ROUNDS * WAVE + lane; k0 < s1; k0 += TAIL_ROUNDS * WAVE) {
                uint32_t rr[TAIL_ROUNDS];
                float at[TAIL_ROUNDS];
#pragma unroll
                for (int j = 0; j < TAIL_ROUNDS; ++j) {
                    const int64_t k = k0 + j * WAVE;
                    const bool on = k < s1;
                    rr[j] = cv.idx[on ? k : k0] & IDX_MASK;
                    at[j] = on ? cv.val[k] : 0.0f;
                }
#pragma unroll
                for (int j = 0; j < TAIL_ROUNDS; ++j)
                    if (k0 + j * WAVE < s1) unsafeAtomicAdd(v + rr[j], mult * at[j]);
            }
        }
        cur = nxt;
        cB = cA;
        p0B = p0A;
        p1B = p1A;
        entryA = entry3;
    }
}

// ---- short rows with popular features (dual forms): several rows per wavefront -----------------
// The memory side performs the atomics on one 128-byte line one request after the other, 12.7 ns each, two
// neighbouring lines 24, however many lanes a request carries.  Rows of a text-like corpus all hold the same
// few features: while every row moves (the first epochs of the hinge form) an epoch waits 48 ms per
// million rows for the two hottest lines.  So a wavefront takes R consecutive rows of the epoch
// order at once and adds their updates to the popular features in LDS; they go out, one request per line, when
// R / 2 rows have moved since the last time (most visits move no row in later epochs) and at the end.  The
// wavefront's own gathers see what is pending.  The rows in flight stay as many: fewer wavefronts.  (At R
// rows instead of R / 2 the epochs take 10 % less and the gap after the first one is five times as large.)
//
// A row has S places (32, 64 or 256 lanes of one or four registers), longer rows take the rest in plain loops.  The
// sums of all rows are taken together: each exchange step halves the registers instead of repeating the whole
// reduction per row, and lane l ends up with the sum of row row_of(l).  The steps of the rows are then taken
// side by side, each lane that of its row.
//
// Popular features: one tag per slot of a direct-mapped table, the most frequent feature of a sample of the
// rows (hot_setup).  LDS sums are fp64, rounded once: ds_add_f64 takes 39 cycles per wavefront, ds_add_f32 193.
//
// 1 M hinge rows of 50 nonzeros over 100 000 Zipf(1.1) features, 500 rows in flight, epochs from zero: 52.5, 12.0,
// 7.1, 5.6, 4.6 ms with single rows, 9.2, 7.6, 5.7, 4.9, 4.5 ms this way.  Also measured, on easier labels (48.0, 11.5,
// 4.4 ms with single rows): the popular entries of v read once per visit into LDS 10.5, 7.2, 5.4 ms (the loads
// queue at the same lines), returned by the additions 11.9, 8.7, 6.5 ms, sent out at every visit 7.3, 8.4, 5.9 ms.
constexpr int HOT_SLOTS = 512;
constexpr uint32_t HOT_NONE = 0xFFFFFFFFu;
constexpr int HOT_SAMPLE = 4096;
__device__ __forceinline__ uint32_t hot_slot(uint32_t r) { return (r ^ (r >> 9)) & (HOT_SLOTS - 1); }

template <int S, int R>
struct MergeShape {
    static constexpr int ROWS = R;                           // rows of a visit
    static constexpr int REGS = ROWS * S / WAVE;
    static constexpr int PER_ROW = S > WAVE ? S / WAVE : 1;  // registers of a row
    __device__ static __forceinline__ int row_of(int lane) { return S == 32 ? 2 * (lane & (ROWS / 2 - 1)) + (lane >> 5) : lane & (ROWS - 1); }
    __device__ static __forceinline__ int lane_of(int row) { return S == 32 ? (row >> 1) + 32 * (row & 1) : row; }
    // value of the row that register j of this lane belongs to, from the lanes that hold the rows' values
    __device__ static __forceinline__ int spread(int x, int j, bool upper) {
        if (S == 32) {
            const int a = __builtin_amdgcn_readlane(x, j), b = __builtin_amdgcn_readlane(x, 32 + j);
            return upper ? b : a;
        }
        return __builtin_amdgcn_readlane(x, j / PER_ROW);
    }
};

template <int DPP>
__device__ __forceinline__ float dpp_move(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), DPP, 0xF, 0xF, false));
}
// lanes with `bit` keep b and hand a over, the others the other way round: one register for two sums
template <int DPP>
__device__ __forceinline__ float fold_pair(float a, float b, bool bit) {
    return (bit ? b : a) + dpp_move<DPP>(bit ? a : b);
}

// p[j] = this lane's part of register j's row(s); returns the whole sum of row row_of(lane)
template <int S, int R>
__device__ __forceinline__ float sum_rows(const float (&p)[MergeShape<S, R>::REGS], int lane) {
    constexpr int QUAD_SWAP_1 = 0xB1, QUAD_SWAP_2 = 0x4E, ROW_ROR_4 = 0x124, ROW_ROR_8 = 0x128;
    constexpr int NP = MergeShape<S, R>::REGS / MergeShape<S, R>::PER_ROW;
    float q[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        q[i] = p[i * MergeShape<S, R>::PER_ROW];
#pragma unroll
        for (int k = 1; k < MergeShape<S, R>::PER_ROW; ++k) q[i] += p[i * MergeShape<S, R>::PER_ROW + k];
    }
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
    float x;
    if constexpr (NP == 8) {
        const float t0 = fold_pair<QUAD_SWAP_1>(q[0], q[1], b0), t1 = fold_pair<QUAD_SWAP_1>(q[2], q[3], b0);
        const float t2 = fold_pair<QUAD_SWAP_1>(q[4], q[5], b0), t3 = fold_pair<QUAD_SWAP_1>(q[6], q[7], b0);
        const float u0 = fold_pair<QUAD_SWAP_2>(t0, t1, b1), u1 = fold_pair<QUAD_SWAP_2>(t2, t3, b1);
        x = fold_pair<ROW_ROR_4>(u0, u1, b2);              // (each part travels to one lane of the other kind)
    } else if constexpr (NP == 1) {
        return wave_sum(q[0]);
    } else if constexpr (NP == 2) {
        x = fold_pair<QUAD_SWAP_1>(q[0], q[1], b0);
        x += dpp_move<QUAD_SWAP_2>(x);
        x += dpp_move<ROW_ROR_4>(x);
    } else {
        static_assert(NP == 4, "one, two, four or eight sums");
        const float t0 = fold_pair<QUAD_SWAP_1>(q[0], q[1], b0), t1 = fold_pair<QUAD_SWAP_1>(q[2], q[3], b0);
        x = fold_pair<QUAD_SWAP_2>(t0, t1, b1);
        x += dpp_move<ROW_ROR_4>(x);
    }
    x += dpp_move<ROW_ROR_8>(x);
    auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);
    if (S != 32) {
        auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = __uint_as_float(r32[0]) + __uint_as_float(r32[1]);
    }
    return x;
}

// moved: [0] rows whose coordinate moved, [1] wavefronts that are done; the last one writes the count
// to host memory and clears both for the next epoch.
template <int S, int R>
__global__ void __launch_bounds__(WAVE)
k_scd_merge(ChunkView cv, const uint32_t* __restrict__ order, int64_t n_small, const float* __restrict__ y,
            float* __restrict__ x, float* v, const float* __restrict__ norms, StepParams sp, int64_t n_waves,
            const uint32_t* __restrict__ hot_tag, uint32_t* moved, uint32_t* moved_out) {
    using Shape = MergeShape<S, R>;
    constexpr int ROWS = Shape::ROWS, REGS = Shape::REGS, PER_ROW = Shape::PER_ROW;
    __shared__ uint32_t s_tag[HOT_SLOTS];
    __shared__ double s_acc[HOT_SLOTS];
    const int lane = threadIdx.x;
    const bool upper = lane >= 32;
    const int row = Shape::row_of(lane);
    const bool owner = lane == Shape::lane_of(row);
    uint32_t tag[HOT_SLOTS / WAVE];
#pragma unroll
    for (int i = 0; i < HOT_SLOTS / WAVE; ++i) {
        tag[i] = hot_tag[i * WAVE + lane];
        s_tag[i * WAVE + lane] = tag[i];
        s_acc[i * WAVE + lane] = 0.0;
    }
    __syncthreads();

    struct Rows {
        int64_t c, s0;                // this lane's row: coordinate, first nonzero in the chunk's arrays
        int len;
        uint32_t raw[REGS];
        float a[REGS];
        float xc, nc, yc;
    };
    auto order_entry = [&](int64_t g) -> uint32_t { return g * ROWS + row < n_small ? order[g * ROWS + row] : 0u; };
    auto coord_at = [&](int64_t g, uint32_t entry) -> int64_t { return g * ROWS + row < n_small ? cv.c0 + (int64_t)entry : -1; };
    auto ptr_pair = [&](int64_t c, int64_t& p0, int64_t& p1) {
        p0 = p1 = 0;
        if (c >= 0) {
            p0 = cv.ptr[c];
            p1 = cv.ptr[c + 1];
        }
    };
    auto place = [&](int j) -> int { return S == 32 ? (lane & 31) : (j % PER_ROW) * WAVE + lane; };
    auto first_of = [&](int64_t s0, int j) -> int64_t {
        const uint32_t lo = (uint32_t)Shape::spread((int)(uint32_t)s0, j, upper);
        const int hi = Shape::spread((int)(s0 >> 32), j, upper);
        return (int64_t)(((uint64_t)(uint32_t)hi << 32) | lo);
    };
    auto fetch = [&](int64_t c, int64_t p0, int64_t p1) -> Rows {
        Rows q;
        q.c = c, q.s0 = c >= 0 ? p0 - cv.nnz_base : 0, q.len = (int)(p1 - p0);
        q.xc = q.nc = q.yc = 0.0f;
#pragma unroll
        for (int j = 0; j < REGS; ++j) {
            const int64_t k = first_of(q.s0, j) + place(j);
            const int len = Shape::spread(q.len, j, upper);
            q.raw[j] = 0u;
            q.a[j] = 0.0f;
            if (place(j) < len) {
                q.raw[j] = cv.idx[k];
                q.a[j] = cv.val[k];
            }
        }
        if (c >= 0) {
            q.xc = x[c];
            q.nc = norms[c];
            q.yc = y[c];
        }
        return q;
    };
    const int64_t wave0 = blockIdx.x;
    const int64_t n_visits = (n_small + ROWS - 1) / ROWS;
    uint32_t n_moved = 0;
    int64_t cB = coord_at(wave0 + n_waves, order_entry(wave0 + n_waves));
    uint32_t entryA = order_entry(wave0 + 2 * n_waves);
    int64_t p0B, p1B;
    Rows cur;
    {
        const int64_t c = coord_at(wave0, order_entry(wave0));
        int64_t p0, p1;
        ptr_pair(c, p0, p1);
        ptr_pair(cB, p0B, p1B);
        cur = fetch(c, p0, p1);
    }
    uint32_t pending = 0;                                  // rows whose updates of popular features still sit in LDS
    auto flush = [&]() {
        // (one wavefront: its LDS operations are performed in the order of their issue)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        double t[HOT_SLOTS / WAVE];
#pragma unroll
        for (int i = 0; i < HOT_SLOTS / WAVE; ++i) t[i] = s_acc[i * WAVE + lane];
#pragma unroll
        for (int i = 0; i < HOT_SLOTS / WAVE; ++i)
            if (t[i] != 0.0) {
                s_acc[i * WAVE + lane] = 0.0;
                unsafeAtomicAdd(v + tag[i], (float)t[i]);
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        pending = 0;
    };
    for (int64_t g = wave0; g < n_visits; g += n_waves) {
        float vv[REGS];
        bool have[REGS], hot[REGS];
#pragma unroll
        for (int j = 0; j < REGS; ++j) {
            have[j] = place(j) < Shape::spread(cur.len, j, upper);
            hot[j] = have[j] && s_tag[hot_slot(cur.raw[j])] == cur.raw[j];
        }
#pragma unroll
        for (int j = 0; j < REGS; ++j) vv[j] = have[j] ? load_shared(v, cur.raw[j]) : 0.0f;
        Rows nxt = fetch(cB, p0B, p1B);
        const int64_t cA = coord_at(g + 2 * n_waves, entryA);
        int64_t p0A, p1A;
        ptr_pair(cA, p0A, p1A);
        uint32_t entry3 = order_entry(g + 3 * n_waves);
        // nothing moves across: the requests first, then what can be computed while they are under way
        __builtin_amdgcn_sched_barrier(0);
        StepPrep prep = prepare_step<K_DUAL>(cur.xc, cur.nc, cur.yc, sp);
        asm volatile("" : "+v"(prep.a), "+v"(prep.b), "+v"(prep.c));
        __builtin_amdgcn_sched_barrier(0);

        float part[REGS];
#pragma unroll
        for (int j = 0; j < REGS; ++j) part[j] = cur.a[j] * (hot[j] ? vv[j] + (float)s_acc[hot_slot(cur.raw[j])] : vv[j]);
        float sum = sum_rows<S, R>(part, lane);
        const bool longer = __ballot(cur.len > S) != 0;
        if (longer) {
            for (int q = 0; q < ROWS; ++q) {
                const int l = Shape::lane_of(q), len = __builtin_amdgcn_readlane(cur.len, l);
                if (len <= S) continue;
                const int64_t s0 = ((int64_t)__builtin_amdgcn_readlane((int)(cur.s0 >> 32), l) << 32) |
                                   (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)cur.s0, l);
                float t = 0.0f;
                for (int k = S + lane; k < len; k += WAVE) t += cv.val[s0 + k] * load_shared(v, cv.idx[s0 + k]);
                t = wave_sum(t);
                if (row == q) sum += t;
            }
        }
        float mult;
        const float xn = finish_step<K_DUAL>((double)sum, 0.0, cur.xc, cur.nc, cur.yc, prep, sp, mult);
        if (cur.c < 0) mult = 0.0f;
        if (owner && cur.c >= 0) x[cur.c] = xn;
        const uint64_t movers = __ballot(owner && mult != 0.0f);
        n_moved += (uint32_t)__popcll(movers);
        // what was requested for later visits has arrived by now: take it over ahead of the atomics
#pragma unroll
        for (int j = 0; j < REGS; ++j) asm volatile("" : "+v"(nxt.raw[j]), "+v"(nxt.a[j]));
        asm volatile("" : "+v"(nxt.xc), "+v"(nxt.nc), "+v"(nxt.yc), "+v"(p0A), "+v"(p1A), "+v"(entry3));
        __builtin_amdgcn_sched_barrier(0);
        if (movers != 0) {
#pragma unroll
            for (int j = 0; j < REGS; ++j) {
                const float mj = __int_as_float(Shape::spread(__float_as_int(mult), j, upper));
                if (have[j] && mj != 0.0f) {
                    if (hot[j]) unsafeAtomicAdd(&s_acc[hot_slot(cur.raw[j])], (double)(mj * cur.a[j]));
                    else unsafeAtomicAdd(v + cur.raw[j], mj * cur.a[j]);
                }
            }
            if (longer) {
                for (int q = 0; q < ROWS; ++q) {
                    const int l = Shape::lane_of(q), len = __builtin_amdgcn_readlane(cur.len, l);
                    const float mq = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mult), l));
                    if (len <= S || mq == 0.0f) continue;
                    const int64_t s0 = ((int64_t)__builtin_amdgcn_readlane((int)(cur.s0 >> 32), l) << 32) |
                                       (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)cur.s0, l);
                    for (int k = S + lane; k < len; k += WAVE) unsafeAtomicAdd(v + cv.idx[s0 + k], mq * cv.val[s0 + k]);
                }
            }
            pending += (uint32_t)__popcll(movers);
            if (pending >= ROWS / 2) flush();
        }
        cur = nxt;
        cB = cA;
        p0B = p0A;
        p1B = p1A;
        entryA = entry3;
    }
    if (pending != 0) flush();
    if (lane == 0) {
        // the addition has been performed before the arrival is counted (it returns the old value)
        const uint32_t before = atomicAdd(&moved[0], n_moved);
        uint32_t one = 1u;
        asm volatile("" : "+v"(one) : "v"(before));
        if (atomicAdd(&moved[1], one) == (uint32_t)n_waves - 1u) {
            const uint32_t total = atomicExch(&moved[0], 0u);
            __hip_atomic_store(&moved[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(moved_out, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Features of a sample of the rows: counts, then the most frequent feature of every slot.
__global__ void __launch_bounds__(WAVE)
k_hot_count(const int64_t* __restrict__ ptr, const uint32_t* __restrict__ idx, int64_t m, int64_t small_max, int samples,
            uint32_t* __restrict__ freq) {
    const int64_t c = (int64_t)blockIdx.x * m / samples;
    const int64_t s0 = ptr[c], s1 = ptr[c + 1];
    if (s1 - s0 > small_max) return;
    for (int64_t k = s0 + threadIdx.x; k < s1; k += WAVE) atomicAdd(freq + idx[k], 1u);
}

// best[slot] = count << 32 | ~feature; best[HOT_SLOTS] = the largest count.  A feature is taken if the sampled rows hold
// line_least entries on its 128-byte line of v: a line in the table costs one request per R rows that moved.
__global__ void k_hot_pick(const uint32_t* __restrict__ freq, int64_t len, uint32_t line_least, unsigned long long* __restrict__ best) {
    constexpr int LINE = 128 / sizeof(float);
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < len; r += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t n = freq[r];
        if (n == 0) continue;
        const int64_t l0 = r & ~(int64_t)(LINE - 1), l1 = min(len, l0 + LINE);
        uint32_t on_line = 0;
        for (int64_t q = l0; q < l1; ++q) on_line += freq[q];
        if (on_line < line_least) continue;
        atomicMax(best + hot_slot((uint32_t)r), ((unsigned long long)n << 32) | (0xFFFFFFFFu - (uint32_t)r));
        atomicMax(best + HOT_SLOTS, (unsigned long long)n);
    }
}

__global__ void k_hot_tags(const unsigned long long* __restrict__ best, uint32_t* __restrict__ tag) {
    for (int s = threadIdx.x; s < HOT_SLOTS; s += blockDim.x)
        tag[s] = best[s] ? 0xFFFFFFFFu - (uint32_t)(best[s] & 0xFFFFFFFFu) : HOT_NONE;
}

// Creation, dual forms on resident sparse data: find the popular features.  Where no feature is in an eighth of
// the rows the lines of v are not contended and every row goes alone.
int hot_setup(snap_handle* h) {
    if (h->kind != K_DUAL || h->dense || h->streaming || h->m < HOT_SAMPLE || h->vlen < 1 || h->nnz_small < 1) return SNAP_OK;
    uint32_t* freq = nullptr;
    unsigned long long *best = nullptr, top = 0;
    auto find = [&]() -> int {
        SNAP_HIP(hipMalloc(&freq, (size_t)h->vlen * sizeof(uint32_t)));
        SNAP_HIP(hipMalloc(&best, (HOT_SLOTS + 1) * sizeof(*best)));
        SNAP_HIP(hipMalloc(&h->hot_tag, HOT_SLOTS * sizeof(uint32_t)));
        SNAP_HIP(hipMalloc(&h->moved, 2 * sizeof(uint32_t)));
        SNAP_TRY(fill_zero(freq, (size_t)h->vlen * sizeof(uint32_t), h->compute));
        SNAP_TRY(fill_zero(best, (HOT_SLOTS + 1) * sizeof(*best), h->compute));
        SNAP_TRY(fill_zero(h->moved, 2 * sizeof(uint32_t), h->compute));
        hipLaunchKernelGGL(k_hot_count, dim3(HOT_SAMPLE), dim3(WAVE), 0, h->compute, h->ptr, h->idx, h->m, h->small_max, HOT_SAMPLE, freq);
        hipLaunchKernelGGL(k_hot_pick, dim3((unsigned)std::min<int64_t>(1024, (h->vlen + 255) / 256)), dim3(256), 0, h->compute, freq,
                           h->vlen, (uint32_t)(HOT_SAMPLE / 8), best);
        hipLaunchKernelGGL(k_hot_tags, dim3(1), dim3(256), 0, h->compute, best, h->hot_tag);
        SNAP_HIP(hipGetLastError());
        SNAP_HIP(hipMemcpyAsync(&top, best + HOT_SLOTS, sizeof(top), hipMemcpyDeviceToHost, h->compute));
        SNAP_HIP(hipStreamSynchronize(h->compute));
        return SNAP_OK;
    };
    const int rc = find();
    (void)hipStreamSynchronize(h->compute);
    (void)hipFree(freq);
    (void)hipFree(best);
    SNAP_TRY(rc);
    if (top * 8 < (unsigned long long)HOT_SAMPLE) hot_free(h);
    hot_reset(h);
    return SNAP_OK;
}

// Creation: scratch of the epoch with v in LDS, where that may be used.
int lds_epoch_setup(snap_handle* h) {
    int lds_max = 0;
    SNAP_HIP(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, h->device));
    if (h->dense || h->nnz_small < 1 || h->grouped || h->vlen < 1 || h->vlen * (int64_t)sizeof(double) > lds_max) return SNAP_OK;
    SNAP_HIP(hipMalloc(&h->step_prep, (size_t)h->m * 2 * sizeof(double)));
    return SNAP_OK;
}

void hot_reset(snap_handle* h) { reinterpret_cast<volatile uint32_t*>(h->red.host + MOVED_WORD)[0] = 0xFFFFFFFFu; }

void hot_free(snap_handle* h) {
    (void)hipFree(h->hot_tag);
    (void)hipFree(h->moved);
    h->hot_tag = h->moved = nullptr;
}

// ---- short coordinates, short shared vector: v in the LDS of one compute unit ----------------------
// With few coordinates in flight (the cap is a quarter of v's length) an epoch is a chain of visits, and a visit waits for
// its gather and its atomics: 1.4 us for a column of 200 nonzeros (7.7 ns per scattered atomic of a compute unit), more
// where the lines are contended.  A v of up to 20 000 entries fits the LDS of one compute unit as fp64, where 64
// scattered additions take 20 cycles and 64 reads 6 (eight wavefronts; ds_add_f32 takes 192).  So one workgroup
// runs the epoch: the other 255 compute units could not have shortened the chain.  v is rounded to fp32 once, at the end.
//
// What limits it is the issue rate of four SIMDs, then the wait for the nonzeros: R coordinates per visit share the
// reduction and the step (as in k_scd_merge), the part of the step that does not need v is computed by a launch of its own
// for all coordinates (k_prepare_steps: no coordinate is visited twice in an epoch), and nonzeros are requested two visits
// ahead, in three slots that change roles by name (a register move would wait for the load).  No coordinate is longer than
// its S places.  60 013 logistic rows of up to 23 nonzeros over 5 003 features, 88 in flight: 1.85 -> 0.95 ms per epoch (1.06 with
// R = 4); 1 000 logistic columns of 200 nonzeros over 10 000 rows, 12 in flight: 118 -> 103 us, issue-bound: 180 vector
// instructions per column.
template <int KIND>
__global__ void __launch_bounds__(256)
k_prepare_steps(int64_t c0, int64_t c1, const float* __restrict__ x, const float* __restrict__ norms, const float* __restrict__ y,
                StepParams sp, double2* __restrict__ prep) {
    for (int64_t c = c0 + (int64_t)blockIdx.x * 256 + threadIdx.x; c < c1; c += (int64_t)gridDim.x * 256) {
        const StepPrep p = prepare_step<KIND>(x[c], norms[c], KIND == K_DUAL ? y[c] : 0.0f, sp);
        prep[c] = make_double2(p.a, p.b);
    }
}

// most wavefronts of the workgroup (three slots of 16 registers of nonzeros leave room for eight)
constexpr int lds_waves(int S) { return S == 1024 ? 8 : 16; }

template <int KIND, int S, int R>
__global__ void __launch_bounds__(WAVE * lds_waves(S))
k_scd_lds(ChunkView cv, const uint32_t* __restrict__ order, int64_t n_small, const float* __restrict__ y, float* __restrict__ x,
          float* __restrict__ v, int64_t vlen, const float* __restrict__ norms, const double2* __restrict__ prep, StepParams sp) {
    using Shape = MergeShape<S, R>;
    constexpr int ROWS = R, REGS = Shape::REGS, PER_ROW = Shape::PER_ROW;
    constexpr uint32_t IDX_MASK = KIND == K_PRIMAL_LOGISTIC ? ~LABEL_BIT : 0xFFFFFFFFu;
    extern __shared__ double s_shared[];
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t n_waves = blockDim.x / WAVE, wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const bool upper = lane >= 32;
    const int row = Shape::row_of(lane);
    const bool owner = lane == Shape::lane_of(row);
    // (ridge: v - y, all that the steps need of the two)
    for (int64_t i = threadIdx.x; i < vlen; i += blockDim.x) s_shared[i] = (double)v[i] - (KIND == K_PRIMAL_RIDGE ? (double)y[i] : 0.0);
    __syncthreads();

    // Every lane loads, from a valid place: what does not belong to it is masked where it is used, and no branch keeps a
    // load and its wait together.  The empty asm statements hold the arithmetic on a loaded value back to the visit
    // that uses it (the compiler would convert it right behind the load, and wait there).
    struct Rows {
        int64_t c, s0;                // this lane's coordinate, its first nonzero in the chunk's arrays
        int len;
        uint32_t raw[REGS];
        float a[REGS];
        float xc, nc, yc;
        double2 pr;
    };
    struct Range { int64_t c, p0, p1; };
    auto load_entry = [&](int64_t g) -> uint32_t { return order[min(g * ROWS + row, n_small - 1)]; };
    auto load_range = [&](int64_t g, uint32_t entry) -> Range {
        const int64_t c = cv.c0 + (int64_t)entry;
        return Range{g * ROWS + row < n_small ? c : -1, cv.ptr[c], cv.ptr[c + 1]};
    };
    auto place = [&](int j) -> int { return S == 32 ? (lane & 31) : (j % PER_ROW) * WAVE + lane; };
    auto fetch = [&](Rows& q, const Range& r) {
        const int64_t c = r.c >= 0 ? r.c : cv.c0;
        q.c = r.c, q.s0 = r.p0 - cv.nnz_base, q.len = r.c >= 0 ? (int)(r.p1 - r.p0) : 0;
        q.xc = x[c];
        q.nc = q.yc = 0.0f;
        q.pr = make_double2(0.0, 0.0);
        if (KIND != K_PRIMAL_LOGISTIC) q.pr = prep[c];
        if (KIND == K_DUAL) {
            q.nc = norms[c];
            q.yc = y[c];
        }
#pragma unroll
        for (int j = 0; j < REGS; ++j) {
            const uint32_t lo = (uint32_t)Shape::spread((int)(uint32_t)q.s0, j, upper);
            const int hi = Shape::spread((int)(q.s0 >> 32), j, upper);
            const int64_t k = (int64_t)(((uint64_t)(uint32_t)hi << 32) | lo) + place(j);
            const int64_t at = place(j) < Shape::spread(q.len, j, upper) ? k : 0;
            q.raw[j] = cv.idx[at];
            q.a[j] = cv.val[at];
        }
    };
    const int64_t n_visits = (n_small + ROWS - 1) / ROWS;
    // visit g: the order entry of visit g + 4, the range of visit g + 3 and the nonzeros of visit g + 2 are requested, in
    // this order, so that a wait for one of the first two is no wait for the nonzeros behind it
    auto visit = [&](int64_t g, Rows& cur, Rows& nxt2, Range& range3, Range& range2, uint32_t& entry4, uint32_t& entry3) {
        asm volatile("" : "+v"(entry3), "+v"(range2.p0), "+v"(range2.p1), "+v"(cur.xc), "+v"(cur.nc), "+v"(cur.yc), "+v"(cur.pr.x), "+v"(cur.pr.y));
#pragma unroll
        for (int j = 0; j < REGS; ++j) asm volatile("" : "+v"(cur.raw[j]), "+v"(cur.a[j]));
        __builtin_amdgcn_sched_barrier(0);
        // (one long coordinate must not make all others pay for its registers: four at a time are passed over)
        const int len0 = R == 1 && REGS > 4 ? __builtin_amdgcn_readlane(cur.len, 0) : 0;
        auto used = [&](int j) { return !(R == 1 && REGS > 4) || j < 4 || (j & ~3) * WAVE < len0; };
        float yy[REGS];
        bool have[REGS];
        double vv[REGS];
#pragma unroll
        for (int j = 0; j < REGS; ++j) {
            have[j] = place(j) < Shape::spread(cur.len, j, upper);
            yy[j] = 0.0f;
            if (KIND == K_PRIMAL_LOGISTIC) yy[j] = (cur.raw[j] & LABEL_BIT) ? -1.0f : 1.0f;
            vv[j] = 0.0;
            if (used(j)) vv[j] = s_shared[cur.raw[j] & IDX_MASK];
        }
        entry4 = load_entry(g + 4 * n_waves);
        range3 = load_range(g + 3 * n_waves, entry3);
        fetch(nxt2, range2);
        __builtin_amdgcn_sched_barrier(0);
        float pg[REGS], ph[REGS];
#pragma unroll
        for (int j = 0; j < REGS; ++j) {
            pg[j] = ph[j] = 0.0f;
            if (used(j) && have[j]) accumulate<KIND>(cur.a[j], (float)vv[j], yy[j], pg[j], ph[j]);
        }
        float gs = sum_rows<S, R>(pg, lane), hs = 0.0f;
        if (KIND == K_PRIMAL_LOGISTIC) hs = sum_rows<S, R>(ph, lane);
        StepPrep p{cur.pr.x, cur.pr.y, 0.0};
        if (KIND == K_DUAL) p.c = (double)cur.yc * sp.inv_lam_n;
        float mult;
        const float xn = finish_step<KIND>((double)gs, (double)hs, cur.xc, cur.nc, cur.yc, p, sp, mult);
        if (cur.c < 0) mult = 0.0f;
        if (owner && cur.c >= 0) x[cur.c] = xn;
        if (__ballot(mult != 0.0f) != 0) {
#pragma unroll
            for (int j = 0; j < REGS; ++j) {
                if (!used(j)) continue;
                const float mj = __int_as_float(Shape::spread(__float_as_int(mult), j, upper));
                if (have[j] && mj != 0.0f) unsafeAtomicAdd(&s_shared[cur.raw[j] & IDX_MASK], (double)(mj * cur.a[j]));
            }
        }
    };
    Rows q0, q1, q2;
    Range r0, r1, r2;
    uint32_t e0, e1, e2;
    e0 = load_entry(wave0);
    e1 = load_entry(wave0 + n_waves);
    e2 = load_entry(wave0 + 2 * n_waves);
    r0 = load_range(wave0, e0);
    r1 = load_range(wave0 + n_waves, e1);
    r2 = load_range(wave0 + 2 * n_waves, e2);
    e0 = load_entry(wave0 + 3 * n_waves);
    fetch(q0, r0);
    fetch(q1, r1);
    for (int64_t g = wave0; g < n_visits;) {
        visit(g, q0, q2, r0, r2, e1, e0);
        if ((g += n_waves) >= n_visits) break;
        visit(g, q1, q0, r1, r0, e2, e1);
        if ((g += n_waves) >= n_visits) break;
        visit(g, q2, q1, r2, r1, e0, e2);
        g += n_waves;
    }
    __syncthreads();
    for (int64_t i = threadIdx.x; i < vlen; i += blockDim.x)
        v[i] = (float)(s_shared[i] + (KIND == K_PRIMAL_RIDGE ? (double)y[i] : 0.0));
}

// ---- large coordinates: segments, two phases, ticket order -------------------------------------
// Everything the workgroups of one coordinate exchange (partial sums, arrival count, the published
// step) goes through device-scope atomic operations, which are performed at the level of the
// memory system that all compute dies share.  Ordering between them therefore only needs the
// earlier operations to have completed, which a data dependence on their returned values gives; a
// device-scope fence would also write back and invalidate the L2 of the die on every work item,
// which costs far more than the item itself.
static_assert(sizeof(LargeState) == 32, "one coordinate's state is one 32-byte block (hipMalloc aligns the array)");

// One workgroup: prefix sums of the items of the large coordinates in epoch order, zeroed state,
// ticket counter back to zero.
__global__ void __launch_bounds__(1024)
k_large_prepare(const int64_t* __restrict__ ptr, int64_t c0, const uint32_t* __restrict__ order_large,
                int64_t n_large, int64_t dense_len, int64_t seg_len, int64_t* __restrict__ item_start,
                LargeState* __restrict__ st, uint32_t* __restrict__ ticket) {
    __shared__ int64_t part[1024];
    const int64_t per = (n_large + 1023) / 1024;
    const int64_t lo = min(n_large, (int64_t)threadIdx.x * per), hi = min(n_large, lo + per);
    int64_t s = 0;
    for (int64_t k = lo; k < hi; ++k) {
        const int64_t c = c0 + (int64_t)order_large[k];
        const int64_t len = dense_len > 0 ? dense_len : ptr[c + 1] - ptr[c];
        s += 2 * ((len + seg_len - 1) / seg_len);
        st[k] = LargeState{0.0, 0.0, 0ull, 0u, 0u};
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        int64_t t = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += t;
        __syncthreads();
    }
    int64_t run = part[threadIdx.x] - s;
    for (int64_t k = lo; k < hi; ++k) {
        const int64_t c = c0 + (int64_t)order_large[k];
        const int64_t len = dense_len > 0 ? dense_len : ptr[c + 1] - ptr[c];
        item_start[k] = run;
        run += 2 * ((len + seg_len - 1) / seg_len);
    }
    if (threadIdx.x == 1023) item_start[n_large] = part[1023];
    if (threadIdx.x == 0) *ticket = 0u;
}

#ifndef SNAP_UNROLL
#define SNAP_UNROLL 4
#endif
constexpr int UNROLL = SNAP_UNROLL;

// index / value streams are read once per pass: load them with the non-temporal hint so that they
// do not push the lines of v out of the caches
template <typename T>
__device__ __forceinline__ T stream_load(const T* p) {
#ifdef SNAP_NO_NT
    return *p;
#else
    return __builtin_nontemporal_load(p);
#endif
}

template <int KIND, bool DENSE>
__global__ void __launch_bounds__(TPB)
k_scd_large(ChunkView cv, const uint32_t* __restrict__ order_large, int64_t n_large,
            const int64_t* __restrict__ item_start, int64_t n_items, LargeState* st, uint32_t* ticket,
            uint32_t* status, const float* __restrict__ y, float* __restrict__ x, float* v,
            const float* __restrict__ norms, StepParams sp, int64_t dense_len, int64_t seg_len) {
    __shared__ uint32_t s_ticket;
    __shared__ float s_mult;
    __shared__ float s_part[2 * WAVES_PER_WG];
    // a fixed number of workgroups (the cap on work in flight) keeps drawing tickets
    for (;;) {
        __syncthreads();                                   // s_ticket / s_mult / s_part are reused
        if (threadIdx.x == 0) s_ticket = atomicAdd(ticket, 1u);
        __syncthreads();
        const int64_t t = (int64_t)s_ticket;
        if (t >= n_items) return;
        int64_t lo = 0, hi = n_large;                      // largest k with item_start[k] <= t
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) >> 1;
            if (item_start[mid] <= t) lo = mid; else hi = mid;
        }
        const int64_t k = lo;
        const int64_t c = cv.c0 + (int64_t)order_large[k];
        int64_t b0, len;
        if (DENSE) {
            b0 = c * dense_len;
            len = dense_len;
        } else {
            b0 = cv.ptr[c] - cv.nnz_base;
            len = cv.ptr[c + 1] - cv.ptr[c];
        }
        const int64_t nseg = (len + seg_len - 1) / seg_len;
        const int64_t item = t - item_start[k];
        const bool dot_phase = item < nseg;
        const int64_t seg = dot_phase ? item : item - nseg;
        const int64_t e0 = seg * seg_len, e1 = min(len, e0 + seg_len);   // element range of the item
        const uint32_t* __restrict__ idxp = cv.idx + b0;
        const float* __restrict__ valp = cv.val + b0;

        if (dot_phase) {
            float g = 0.0f, h = 0.0f;
            int64_t e = e0 + threadIdx.x;
            // UNROLL independent index/value loads, then their gathers, then the arithmetic
            for (; e + (UNROLL - 1) * TPB < e1; e += UNROLL * TPB) {
                uint32_t r[UNROLL];
                float a[UNROLL], yy[UNROLL], vv[UNROLL];
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) {
                    const int64_t eu = e + u * TPB;
                    a[u] = stream_load(valp + eu);
                    if (DENSE) {
                        r[u] = (uint32_t)eu;
                        yy[u] = KIND == K_DUAL ? 0.0f : y[r[u]];
                    } else {
                        decode<KIND>(stream_load(idxp + eu), r[u], yy[u], y);
                    }
                }
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) vv[u] = load_shared(v, r[u]);
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) accumulate<KIND>(a[u], vv[u], yy[u], g, h);
            }
            for (; e < e1; e += TPB) {
                uint32_t r;
                float yy;
                if (DENSE) {
                    r = (uint32_t)e;
                    yy = KIND == K_DUAL ? 0.0f : y[r];
                } else {
                    decode<KIND>(idxp[e], r, yy, y);
                }
                accumulate<KIND>(valp[e], load_shared(v, r), yy, g, h);
            }
            g = wave_sum(g);
            h = wave_sum(h);
            const int w = threadIdx.x / WAVE;
            if ((threadIdx.x & (WAVE - 1)) == 0) {
                s_part[2 * w] = g;
                s_part[2 * w + 1] = h;
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                double G = 0.0, H = 0.0;
#pragma unroll
                for (int ww = 0; ww < WAVES_PER_WG; ++ww) {
                    G += (double)s_part[2 * ww];
                    H += (double)s_part[2 * ww + 1];
                }
                // Both sums must have been performed before the count goes up.  The two additions return
                // the old values, and the increment is made to depend on them: a returning atomic
                // answers only once it has been performed where all compute dies see it, so no
                // fence (and no assumption about how one is lowered) is needed.
                const double g_seen = atomicAdd(&st[k].g, G);
                const double h_seen = atomicAdd(&st[k].h, H);
                uint32_t one = 1u;
                asm volatile("" : "+v"(one) : "v"(g_seen), "v"(h_seen));
                const uint32_t arrived = atomicAdd(&st[k].done, one);
                if (arrived == (uint32_t)nseg - 1u) {              // last dot item of this coordinate
                    const double Gt = atomicAdd(&st[k].g, 0.0);
                    const double Ht = atomicAdd(&st[k].h, 0.0);
                    const float xc = x[c];
                    const float yc = KIND == K_DUAL ? y[c] : 0.0f;
                    float mult;
                    x[c] = take_step<KIND>(Gt, Ht, xc, norms[c], yc, sp, mult);
                    const uint64_t word = (1ull << 32) | (uint64_t)__float_as_uint(mult);
                    __hip_atomic_store(&st[k].published, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            continue;
        }

        // scatter phase: wait (bounded) for the step of this coordinate
        if (threadIdx.x == 0) {
            uint32_t spins = 0;
            uint64_t word;
            while (((word = __hip_atomic_load(&st[k].published, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 32) == 0) {
                __builtin_amdgcn_s_sleep(16);
                if (++spins > SPIN_LIMIT) break;
            }
            if ((word >> 32) != 0) {
                s_mult = __uint_as_float((uint32_t)word);
            } else {
                s_mult = 0.0f;
                atomicOr(status, 1u);
            }
        }
        __syncthreads();
        const float mult = s_mult;
        if (mult == 0.0f) continue;
        int64_t e = e0 + threadIdx.x;
        for (; e + (UNROLL - 1) * TPB < e1; e += UNROLL * TPB) {
            uint32_t r[UNROLL];
            float a[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int64_t eu = e + u * TPB;
                a[u] = stream_load(valp + eu);
                r[u] = DENSE ? (uint32_t)eu
                             : (stream_load(idxp + eu) & (KIND == K_PRIMAL_LOGISTIC ? ~LABEL_BIT : 0xFFFFFFFFu));
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) unsafeAtomicAdd(v + r[u], mult * a[u]);
        }
        for (; e < e1; e += TPB) {
            const uint32_t r = DENSE ? (uint32_t)e : (idxp[e] & (KIND == K_PRIMAL_LOGISTIC ? ~LABEL_BIT : 0xFFFFFFFFu));
            unsafeAtomicAdd(v + r, mult * valp[e]);
        }
    }
}

template <int KIND>
static int launch_kind(snap_handle* h, const ChunkView& cv, const snap_handle::Chunk& ck, const uint32_t* order,
                       const StepParams& sp) {
    const int64_t dense_len = h->dense ? h->ld : 0;
    if (ck.n_large > 0) {
        const uint32_t* order_large = order + ck.n_small;
        hipLaunchKernelGGL(k_large_prepare, dim3(1), dim3(1024), 0, h->compute, cv.ptr, cv.c0, order_large, ck.n_large,
                           dense_len, h->seg, h->item_start, h->lstate, h->ticket);
        int64_t wgs = ck.n_items;
        if (h->inflight_nnz > 0) wgs = std::min<int64_t>(wgs, std::max<int64_t>(1, h->inflight_nnz / h->seg));
        wgs = std::min<int64_t>(wgs, 256 * 8);          // no more than the device holds at once
        const dim3 grid((unsigned)wgs);
        if (h->dense)
            hipLaunchKernelGGL((k_scd_large<KIND, true>), grid, dim3(TPB), 0, h->compute, cv, order_large, ck.n_large,
                               h->item_start, ck.n_items, h->lstate, h->ticket, h->status, h->y, h->x, h->v, h->norms,
                               sp, dense_len, h->seg);
        else
            hipLaunchKernelGGL((k_scd_large<KIND, false>), grid, dim3(TPB), 0, h->compute, cv, order_large, ck.n_large,
                               h->item_start, ck.n_items, h->lstate, h->ticket, h->status, h->y, h->x, h->v, h->norms,
                               sp, dense_len, h->seg);
    }
    if (h->opt.profile && !h->streaming) SNAP_HIP(hipEventRecord(h->ev[3], h->compute));
    if (ck.n_small > 0) {
        int64_t waves = std::min<int64_t>(ck.n_small, 256 * 32);
        if (h->inflight_nnz > 0)
            waves = std::min<int64_t>(waves, std::max<int64_t>(1, (int64_t)((double)h->inflight_nnz / h->avg_small_len)));
        // v in LDS where it fits and the chain of visits, not the work, takes the time.  Dual forms: below the 96 rows in
        // flight from which several rows per wavefront pay (15.8 ns per row of up to 32 nonzeros against 31 ns with single rows, of
        // which the contended lines are the larger part).  Primal forms, whose lines are not contended: a column of 200
        // nonzeros takes 0.10 us of the one compute unit and 1.4 us / (columns in flight) otherwise: equal at 14.  Longer
        // columns (up to 1 024) shift both sides alike.
        const int64_t few = KIND == K_DUAL ? 95 : 14;
        if (h->step_prep && waves <= few && h->max_small_len <= 1024 && ck.nnz1 > ck.nnz0) {     // (idle lanes load the chunk's first nonzero)
            if (KIND != K_PRIMAL_LOGISTIC)
                hipLaunchKernelGGL((k_prepare_steps<KIND>), dim3((unsigned)std::min<int64_t>((cv.c1 - cv.c0 + 255) / 256, 1024)), dim3(256), 0,
                                   h->compute, cv.c0, cv.c1, h->x, h->norms, h->y, sp, (double2*)h->step_prep);
            auto launch = [&](auto kernel, int most, int rows) {
                const int64_t w = std::max<int64_t>(1, std::min<int64_t>(most, waves / rows));
                hipLaunchKernelGGL(kernel, dim3(1), dim3((unsigned)(WAVE * w)), (size_t)h->vlen * sizeof(double), h->compute, cv, order,
                                   ck.n_small, h->y, h->x, h->v, h->vlen, h->norms, (const double2*)h->step_prep, sp);
            };
            if (h->max_small_len <= 32 && waves >= 8) launch(k_scd_lds<KIND, 32, 8>, lds_waves(32), 8);
            else if (h->max_small_len <= 64 && waves >= 4) launch(k_scd_lds<KIND, 64, 4>, lds_waves(64), 4);
            else if (h->max_small_len <= 256) launch(k_scd_lds<KIND, 256, 1>, lds_waves(256), 1);
            else if (h->max_small_len <= 512) launch(k_scd_lds<KIND, 512, 1>, lds_waves(512), 1);
            else launch(k_scd_lds<KIND, 1024, 1>, lds_waves(1024), 1);
            SNAP_HIP(hipGetLastError());
            return SNAP_OK;
        }
        if constexpr (KIND == K_DUAL) {
            // Several rows per wavefront where popular features are contended for: eight while at least half of the
            // rows move (by the count of the last epoch that kept one; 0xFFFFFFFF: none yet), four down to one row in 32,
            // then single rows, whose visits are shorter (figures at k_scd_merge).  With fewer than 32 (24) wavefronts
            // left the atomics of a compute unit, 7.7 ns per scattered lane, take longer than the contended lines
            // (60 013 logistic rows of 23 nonzeros, 54 in flight: 1.9 ms single, 2.2 ms with R = 4, 2.9 with R = 8).
            const uint32_t last = reinterpret_cast<volatile uint32_t*>(h->red.host + MOVED_WORD)[0];
            const int64_t moving = last == 0xFFFFFFFFu ? ck.n_small : (int64_t)last;
            const int rows = moving * 2 >= ck.n_small && waves >= 256 && h->avg_small_len <= WAVE ? 8 : 4;
            if (h->hot_tag && moving * 32 >= ck.n_small && waves >= 96) {
                const dim3 grid((unsigned)(waves / rows));
                auto launch = [&](auto kernel) {
                    hipLaunchKernelGGL(kernel, grid, dim3(WAVE), 0, h->compute, cv, order, ck.n_small, h->y, h->x, h->v, h->norms, sp,
                                       (int64_t)grid.x, h->hot_tag, h->moved, reinterpret_cast<uint32_t*>(h->red.host_mapped + MOVED_WORD));
                };
                if (h->avg_small_len > WAVE) launch(k_scd_merge<256, 4>);
                else if (h->max_small_len <= 32) rows == 8 ? launch(k_scd_merge<32, 8>) : launch(k_scd_merge<32, 4>);
                else rows == 8 ? launch(k_scd_merge<64, 8>) : launch(k_scd_merge<64, 4>);
                SNAP_HIP(hipGetLastError());
                return SNAP_OK;
            }
        }
        const dim3 grid((unsigned)waves);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(SMALL_TPB), 0, h->compute, cv, order, ck.n_small, h->y, h->x, h->v, h->norms,
                               sp, waves);
        };
        if (h->max_small_len <= WAVE) launch(k_scd_small<KIND, 1>);
        else if (h->max_small_len <= 4 * WAVE) launch(k_scd_small<KIND, 4>);
        else launch(k_scd_small<KIND, 16>);
    }
    SNAP_HIP(hipGetLastError());
    return SNAP_OK;
}

int scd_run_chunk(snap_handle* h, const ChunkView& cv, const snap_handle::Chunk& ck, const uint32_t* order) {
    const StepParams sp = make_step_params(h);
    if (ck.n_items > 0x7FFFFFFFll || ck.n_small / WAVES_PER_WG > 0x7FFFFFFFll) {
        set_error("chunk too large for one launch");
        return SNAP_EINVAL;
    }
    switch (h->kind) {
    case K_PRIMAL_RIDGE: return launch_kind<K_PRIMAL_RIDGE>(h, cv, ck, order, sp);
    case K_PRIMAL_LOGISTIC: return launch_kind<K_PRIMAL_LOGISTIC>(h, cv, ck, order, sp);
    case K_DUAL: return launch_kind<K_DUAL>(h, cv, ck, order, sp);
    }
    set_error("unknown solver kind");
    return SNAP_EINVAL;
}

}  // namespace snap
