// Batched circuit-fitness kernels (Eq. 11 of Sec. IV-E) and unitary builders.
#include "../../include/qe.h"
#include "qe_eval_core.hpp"
#include "qe_internal.hpp"
#include "qe_reg_core.hpp"

namespace qe {

constexpr int WPB = 4;   // wavefronts (circuits) per workgroup

__device__ __forceinline__ Item resolve(const BatchArgs& a, int b, bool need_target = true) {
    return resolve_item(a, b, need_target);
}

// Gate p of a circuit as its gate source returns it: the descriptor, or
// with ANG the descriptor and its angle (0 beyond the circuit).
template <bool ANG>
__device__ __forceinline__ auto batch_gate(const Item& it, int p) {
    if constexpr (ANG)
        return p < it.L ? make_uint2((uint32_t)it.g[p], it.ang[p]) : make_uint2(0u, 0u);
    else
        return p < it.L ? (uint32_t)it.g[p] : 0u;
}

// ------------------------------------------------------------ n <= 3
// One-element-per-lane path, WPB circuits per workgroup.  FILTER: a
// mixed-width batch is served by one launch per width, each skipping the
// circuits of other widths.  ANG: the batch carries angles.
template <typename Real, int NQ, bool FILTER, bool ANG>
__global__ __launch_bounds__(64 * WPB) void wave_kernel(BatchArgs a, Real* __restrict__ f,
                                                        Real* __restrict__ g,
                                                        Real* __restrict__ delta) {
    const int b = __builtin_amdgcn_readfirstlane(blockIdx.x * WPB + (threadIdx.x >> 6));
    if (b >= a.B) return;
    const int lane = (int)lane_id();
    Item it = resolve(a, b);
    if (FILTER && it.n != NQ) return;
    if (it.err == 0 && it.n != NQ) it.err = QE_DEVERR_WIDTH;
    const Real nan = (Real)__builtin_nan("");
    FitOut<Real> o{nan, nan, nan};
    if (it.err == 0) {
        auto src = [&](int ch) { return batch_gate<ANG>(it, ch * 64 + lane); };
        const Real* T = reinterpret_cast<const Real*>(a.targets) + 2 * it.toff;
        const bool ok = run_small_path<NQ, false>(T, it.L, src, (Real*)nullptr, &o, a.mode);
        if (!ok) {
            it.err = QE_DEVERR_DESC;
            o = FitOut<Real>{nan, nan, nan};
        } else if (!(o.f == o.f)) {
            it.err = QE_DEVERR_NUMERIC;
        }
    }
    if (lane == 0) {
        f[b] = o.f;
        if (g) g[b] = o.g;
        if (delta) delta[b] = o.delta;
        if (it.err) atomicOr(a.err, it.err);
    }
}

// ------------------------------------------- register-resident, n = 4..6
// One circuit on its W wavefronts (W = 4 at n = 6, else 1; `wave` the circuit's
// wavefront): the fitness of circuit b (n = 6: every wavefront of the workgroup
// calls it, red is LDS).
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <typename Real, int NQ, bool ANG, int COLS = reg_columns<NQ>()>
__device__ __forceinline__ void reg_item(const BatchArgs& a, int b, Item it, int wave, Real (*red)[3],
                                         Real* __restrict__ f, Real* __restrict__ g,
                                         Real* __restrict__ delta) {
    const int lane = (int)lane_id();
    if (it.err == 0 && it.n != NQ) it.err = QE_DEVERR_WIDTH;
    // (wave-uniform, and in scalar registers from here on)
    it.err = (uint32_t)__builtin_amdgcn_readfirstlane((int)it.err);
    it.toff = uniform64(it.toff);
    Real fv, gv, dv;
    fv = gv = dv = (Real)__builtin_nan("");
    if (it.err == 0) {
        RegMatrix<Real, NQ, COLS> M;
        M.place(wave);
        auto src = [&](int ch) { return batch_gate<ANG>(it, ch * 64 + lane); };
        const auto dv0 = src(0);
        M.load(reinterpret_cast<const Real*>(a.targets) + 2 * it.toff);
        if (!M.template run<true>(it.L, src, dv0)) {
            it.err = QE_DEVERR_DESC;
        } else {
            fv = M.fitness(a.mode, &gv, &dv, wave, red);
            if (!(fv == fv)) it.err = QE_DEVERR_NUMERIC;
        }
    }
    if (wave == 0 && lane == 0) {
        f[b] = fv;
        if (g) g[b] = gv;
        if (delta) delta[b] = dv;
        if (it.err) atomicOr(a.err, it.err);
    }
}

// Four circuits per workgroup, one per wavefront, or (n = 6 with 16 columns per
// wavefront) one per workgroup.
template <typename Real, int NQ, bool FILTER, bool ANG, int COLS = reg_columns<NQ>()>
__global__ __launch_bounds__(256) void reg_kernel(BatchArgs a, Real* __restrict__ f, Real* __restrict__ g,
                                                  Real* __restrict__ delta) {
    __shared__ Real red[4][3];
    const int wave = (int)(threadIdx.x >> 6);
    constexpr bool WHOLE = RegGeom<NQ, COLS>::W == 4;
    const int b = __builtin_amdgcn_readfirstlane(WHOLE ? (int)blockIdx.x : (int)blockIdx.x * WPB + wave);
    if (b >= a.B) return;
    const Item it = resolve(a, b);
    if (FILTER && it.n != NQ) return;
    reg_item<Real, NQ, ANG, COLS>(a, b, it, WHOLE ? wave : 0, red, f, g, delta);
}

// Unitaries of a uniform-width batch: the product started from the identity.
template <typename Real, int NQ, bool ANG>
__global__ __launch_bounds__(256) void unitary_kernel(BatchArgs a, Real* __restrict__ out) {
    constexpr bool WHOLE = NQ == 6;
    const int wave = (int)(threadIdx.x >> 6), lane = (int)lane_id();
    const int b = __builtin_amdgcn_readfirstlane(WHOLE ? (int)blockIdx.x : (int)blockIdx.x * WPB + wave);
    if (b >= a.B) return;
    Item it = resolve(a, b, false);
    it.err = (uint32_t)__builtin_amdgcn_readfirstlane((int)it.err);
    auto src = [&](int ch) { return batch_gate<ANG>(it, ch * 64 + lane); };
    Real* U = out + ((size_t)2 << (2 * NQ)) * b;
    bool ok = it.err == 0;
    if (!ok) it.L = 0;                          // (a malformed range: NaN, no gate read)
    if constexpr (NQ <= 3) {
        ok = run_small_path<NQ, true>((const Real*)nullptr, it.L, src, U, (FitOut<Real>*)nullptr) && ok;
        if (it.err) {
            const Real nan = (Real)__builtin_nan("");
            for (int e = lane; e < (2 << (2 * NQ)); e += 64) U[e] = nan;
        }
    } else {
        RegMatrix<Real, NQ> M;
        M.place(WHOLE ? wave : 0);
        const auto dv0 = src(0);
        M.identity();
        ok = M.template run<false>(it.L, src, dv0) && ok;
        M.store(reinterpret_cast<complex_of<Real>*>(U), ok);
    }
    if (!ok && it.err == 0) it.err = QE_DEVERR_DESC;
    if (lane == 0 && (!WHOLE || wave == 0) && it.err) atomicOr(a.err, it.err);
}

// Marks circuits whose width is outside 1..6 (mixed-width batches only).
__global__ void width_check_kernel(BatchArgs a, float* f, float* g, float* delta) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= a.B) return;
    const int n = a.nq[b];
    if (n >= 1 && n <= MAX_QUBITS) return;
    f[b] = __builtin_nanf("");
    if (g) g[b] = __builtin_nanf("");
    if (delta) delta[b] = __builtin_nanf("");
    atomicOr(a.err, (uint32_t)QE_DEVERR_WIDTH);
}

// LDS-staged path, W wavefronts per circuit (see run_lds_path).
template <int NQ, int W, bool FILTER, bool ANG>
__global__ __launch_bounds__(64 * W) void lds32_kernel(BatchArgs a, float* __restrict__ f,
                                                       float* __restrict__ g,
                                                       float* __restrict__ delta) {
    constexpr int N = 1 << NQ;
    __shared__ float2 M[N * N];
    __shared__ uint4 GT[W][ANG ? GATE_TABLE_ANGLED : GATE_TABLE];
    const int b = blockIdx.x;
    const int lane = (int)lane_id(), wave = (int)(threadIdx.x >> 6);
    Item it = resolve(a, b);
    if (FILTER && it.n != NQ) return;
    if (it.err == 0 && it.n != NQ) it.err = QE_DEVERR_WIDTH;
    bool ok = it.err == 0;
    RowMap map{};
    if (ok) {
        const int L = it.L;
        auto src = [&](int ch) { return batch_gate<ANG>(it, ch * 64 + lane); };
        const float* T = reinterpret_cast<const float*>(a.targets) + 2 * it.toff;
        ok = run_lds_path<NQ, W>(M, GT[wave], T, L, src, &map);
        if (!ok) it.err = QE_DEVERR_DESC;
    }
    // fitness, in the width's fixed order
    constexpr int WR = reduction_waves<NQ>();
    static_assert(WR == 1 || WR == W, "the reduction's wavefronts are the circuit's");
    __shared__ float red[4][3];
    if constexpr (W > 1) __syncthreads();      // every wavefront's columns are in place
    if (WR == 1 && wave != 0) return;
    float gv, dlt;
    const float fv = canonical_fitness<NQ, WR>(M, map, a.mode, &gv, &dlt, WR == 1 ? 0 : wave, red);
    if (wave == 0 && lane == 0) {
        const float nan = __builtin_nanf("");
        if (ok && !(fv == fv)) it.err = QE_DEVERR_NUMERIC;
        f[b] = ok ? fv : nan;
        if (g) g[b] = ok ? gv : nan;
        if (delta) delta[b] = ok ? dlt : nan;
        if (it.err) atomicOr(a.err, it.err);
    }
}

// ----------------------------------------------- mixed widths, one launch
// Circuits of a mixed-width batch are ordered by cost, widest first and,
// within a width, longest first (classes of 8 gates), by a one-workgroup
// counting sort; one launch then gives every workgroup one work item.  In large
// batches that is one circuit for one wavefront (register-resident for widths 4 to
// 6, one entry per lane below; four circuits per workgroup held a finished one's
// registers until the others ended: 16384 circuits 90.0 -> 86.5 us, 256 GA
// populations of 64 73.9 -> 71.4); in small ones a circuit of width 6 for four
// wavefronts or four of the other widths, of similar lengths.  Workgroups are
// dispatched in index order, so the heaviest items start first
// (longest-processing-time order).
constexpr int MIX_BUCKETS = 7;          // widths 6..1, then malformed widths
// Fewest circuits of a mixed batch that run one per workgroup, those of width 6 with
// one column per lane.  The line is that of widths 3 to 6 in equal parts (8 to 64
// gates, sort included, us: 3072 circuits 34.2 against 33.6 the other way, 4095 37.5
// against 38.8, 8192 50.5 against 56.7).  Other mixes cross elsewhere (width 6 alone
// at 1300: 2048 36 against 41; widths 2 to 5 lose: 8192 35.8 against 33.3), but only
// the device knows the widths, and the launch needs its shape before.
constexpr int MIX_COLUMNS_MIN = 4096;
constexpr int MIX_LCLASSES = 16;        // lengths >= 120, 112..119, ..., 8..15, < 8

__device__ __forceinline__ int mix_bucket(int n) { return (n >= 1 && n <= MAX_QUBITS) ? 6 - n : 6; }

// Sort key of circuit b: width bucket, then length class (longest first; a
// malformed range only lands in some class, the item reports it).
__device__ __forceinline__ int mix_key(const BatchArgs& a, int b) {
    const int64_t len = a.uniform_L > 0 ? (int64_t)a.uniform_L : (int64_t)a.goff[b + 1] - a.goff[b];
    const int lc = len >= 120 ? 0 : (len < 8 ? MIX_LCLASSES - 1 : MIX_LCLASSES - 1 - (int)(len >> 3));
    return mix_bucket(a.nq[b]) * MIX_LCLASSES + lc;
}
// circuits per work item
__host__ __device__ __forceinline__ bool mix_columns(int B) { return B >= MIX_COLUMNS_MIN; }
__device__ __forceinline__ int mix_per_item(int k, bool columns) { return k == 0 || columns ? 1 : 4; }

// meta: [0..7) first order position, [8..15) first item (8 entries, the last
// the total), [16..23) count per bucket.
// One workgroup.  The LDS atomics bound it (the circuits of a wavefront mostly
// share a width, so that their counts collide): each key counts in MIX_REP
// places, by lane, and when one tile of MIX_PER circuits per thread holds the
// batch, the first pass's counts are the ranks of the second (16384 circuits:
// 14.4 -> 12.0 us) and the order goes through LDS to coalesced stores (11.8 ->
// 9.7 us: one compute unit's scattered stores take about a cycle per lane).
constexpr int MIX_SORT = 1024, MIX_PER = 16, MIX_REP = 4;
__global__ __launch_bounds__(MIX_SORT) void mix_bucket_kernel(BatchArgs a, int32_t* order, int32_t* meta) {
    constexpr int K = MIX_BUCKETS * MIX_LCLASSES * MIX_REP;
    __shared__ int cnt[K], cursor[K];
    __shared__ uint16_t sorted[MIX_PER * MIX_SORT];
    static_assert(MIX_PER * MIX_SORT <= 1 << 16, "a tile's circuits in 16 bits");
    const int tid = threadIdx.x;
    for (int k = tid; k < K; k += MIX_SORT) cnt[k] = 0;
    int key[MIX_PER], rank[MIX_PER];
    auto read_tile = [&](int b0) {
#pragma unroll
        for (int c = 0; c < MIX_PER; ++c) {
            const int b = b0 + c * MIX_SORT + tid;
            key[c] = b < a.B ? mix_key(a, b) * MIX_REP + tid % MIX_REP : -1;
        }
    };
    const bool one_tile = a.B <= MIX_PER * MIX_SORT;
    read_tile(0);
    __syncthreads();
    for (int b0 = 0; b0 < a.B; b0 += MIX_PER * MIX_SORT) {
        if (b0 > 0) read_tile(b0);
#pragma unroll
        for (int c = 0; c < MIX_PER; ++c)
            if (key[c] >= 0) rank[c] = atomicAdd(&cnt[key[c]], 1);
    }
    __syncthreads();
    static_assert(K % 64 == 0, "whole runs of counts per lane");
    if (tid < 64) {
        // exclusive prefix sum of the counts over one wavefront, a run per lane
        constexpr int RUN = K / 64;
        int c[RUN], sum = 0;
#pragma unroll
        for (int u = 0; u < RUN; ++u) {
            c[u] = cnt[tid * RUN + u];
            sum += c[u];
        }
        int incl = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(incl, d, 64);
            if (tid >= d) incl += o;
        }
        int at = incl - sum;
#pragma unroll
        for (int u = 0; u < RUN; ++u) {
            cursor[tid * RUN + u] = at;
            at += c[u];
        }
    }
    __syncthreads();
    if (tid == 0) {
        // per width: first order position, first item, count (every circuit
        // has a key, so the last width ends at B)
        int item = 0;
        for (int k = 0; k < MIX_BUCKETS; ++k) {
            const int pos = cursor[k * MIX_LCLASSES * MIX_REP];
            const int end = k + 1 < MIX_BUCKETS ? cursor[(k + 1) * MIX_LCLASSES * MIX_REP] : a.B;
            meta[k] = pos;
            meta[8 + k] = item;
            meta[16 + k] = end - pos;
            const int per = mix_per_item(k, mix_columns(a.B));
            item += (end - pos + per - 1) / per;
        }
        meta[8 + MIX_BUCKETS] = item;
    }
    __syncthreads();
    if (one_tile) {
#pragma unroll
        for (int c = 0; c < MIX_PER; ++c)
            if (key[c] >= 0) sorted[cursor[key[c]] + rank[c]] = (uint16_t)(c * MIX_SORT + tid);
        __syncthreads();
        for (int p = tid; p < a.B; p += MIX_SORT) order[p] = sorted[p];
        return;
    }
    for (int b0 = 0; b0 < a.B; b0 += MIX_PER * MIX_SORT) {
        read_tile(b0);
#pragma unroll
        for (int c = 0; c < MIX_PER; ++c)
            if (key[c] >= 0) order[atomicAdd(&cursor[key[c]], 1)] = b0 + c * MIX_SORT + tid;
    }
}

template <int NQ>
__device__ __forceinline__ void mix_wave_item(const BatchArgs& a, int b, float* f, float* g,
                                              float* delta) {
    const int lane = (int)lane_id();
    Item it = resolve(a, b);
    FitOut<float> o{__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf("")};
    if (it.err == 0) {
        const uint16_t* gp = it.g;
        const int L = it.L;
        auto src = [&](int ch) -> uint32_t {
            const int p = ch * 64 + lane;
            return p < L ? (uint32_t)gp[p] : 0u;
        };
        const float* T = reinterpret_cast<const float*>(a.targets) + 2 * it.toff;
        if (!run_small_path<NQ, false>(T, L, src, (float*)nullptr, &o, a.mode)) {
            it.err = QE_DEVERR_DESC;
            o = FitOut<float>{__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf("")};
        } else if (!(o.f == o.f)) {
            it.err = QE_DEVERR_NUMERIC;
        }
    }
    if (lane == 0) {
        f[b] = o.f;
        if (g) g[b] = o.g;
        if (delta) delta[b] = o.delta;
        if (it.err) atomicOr(a.err, it.err);
    }
}

// COLUMNS: circuits of width 6 with one column per lane (large batches).  (They
// and the other widths in two launches, so that the small widths keep the
// occupancy of 52 VGPRs: no gain at 16384 circuits, and 55
// against 37 us at 4096, where each launch ends in a nearly empty round.)
template <bool COLUMNS>
__global__ __launch_bounds__(256) void mix_kernel(BatchArgs a, const int32_t* __restrict__ order,
                                                  const int32_t* __restrict__ meta,
                                                  float* __restrict__ f, float* __restrict__ g,
                                                  float* __restrict__ delta) {
    __shared__ float red[4][3];
    if (a.gates_odd && (((a.gen_ptr ? *a.gen_ptr : 0ull) + a.gen) & 1ull)) a.gates = a.gates_odd;
    const int item = blockIdx.x;
    if (item >= meta[8 + MIX_BUCKETS]) return;
    int k = 0;
    while (k + 1 < MIX_BUCKETS && item >= meta[8 + k + 1]) ++k;
    const int wave = (int)(threadIdx.x >> 6);
    const int per = mix_per_item(k, COLUMNS);
    const int local = (item - meta[8 + k]) * per;
    const int sub = per == 1 ? 0 : wave;       // (COLUMNS: one wavefront)
    int b = local + sub < meta[16 + k] ? order[meta[k] + local + sub] : -1;
    if (b >= a.B) b = -1;        // an order written for another batch never indexes past this one
    b = __builtin_amdgcn_readfirstlane(b);
    if (b < 0) return;           // (four wavefronts per circuit: the whole workgroup)
    switch (k) {
        case 0:
            if constexpr (COLUMNS) reg_item<float, 6, false, 64>(a, b, resolve(a, b), 0, red, f, g, delta);
            else reg_item<float, 6, false>(a, b, resolve(a, b), wave, red, f, g, delta);
            break;
        case 1: reg_item<float, 5, false>(a, b, resolve(a, b), 0, red, f, g, delta); break;
        case 2: reg_item<float, 4, false>(a, b, resolve(a, b), 0, red, f, g, delta); break;
        case 3: mix_wave_item<3>(a, b, f, g, delta); break;
        case 4: mix_wave_item<2>(a, b, f, g, delta); break;
        case 5: mix_wave_item<1>(a, b, f, g, delta); break;
        default:
            if (lane_id() == 0) {
                const float nan = __builtin_nanf("");
                f[b] = nan;
                if (g) g[b] = nan;
                if (delta) delta[b] = nan;
                atomicOr(a.err, (uint32_t)QE_DEVERR_WIDTH);
            }
            break;
    }
}

// ------------------------------------------- FP64, mixed widths in one launch
__global__ __launch_bounds__(256) void lds_kernel(BatchArgs a, double* __restrict__ f, double* __restrict__ g,
                                                  double* __restrict__ delta) {
    const int b = blockIdx.x;
    Item it = resolve(a, b);
    const double* T = it.err ? nullptr : reinterpret_cast<const double*>(a.targets) + 2 * it.toff;
    // dynamic LDS: two planes of 4^n reals for the largest width
    double* Mr = generic_lds<double>();
    double* Mi = Mr + ((size_t)1 << (2 * MAX_QUBITS));
    lds_generic_body<double>(it.n, it.L, it.g, it.ang, T, it.err, f + b, g ? g + b : nullptr,
                             delta ? delta + b : nullptr, a.err, a.mode, Mr, Mi);
}

// ------------------------------------------------------------------ launchers
// Per-width schedule: which kernel evaluates a circuit of width n on the
// FP32 path.  path: QE_PATH_FP32 (default schedule), QE_PATH_FP32_REG,
// QE_PATH_FP32_LDS.
static bool use_lds(int n, int path, int L, int lib_class) {
    if (n <= 3) return false;
    if (path == QE_PATH_FP32_REG) return false;
    if (path == QE_PATH_FP32_LDS) return true;
    return schedule_for(n, L, lib_class).lds != 0;
}

// length of the batch's circuits for the schedule (uneven batches: the long class)
static int sched_len(const BatchArgs& a) { return a.uniform_L > 0 ? a.uniform_L : 32; }

// One launch over the batch's circuits of width n.  n <= 3: the
// one-element-per-lane kernel; above, the register-resident or the LDS-staged
// one.
template <bool FILTER, bool ANG>
static void launch_width(const BatchArgs& a, int n, int path, float* f, float* g, float* delta,
                         hipStream_t s) {
    const dim3 wgrid((a.B + WPB - 1) / WPB), wblock(64 * WPB);
    constexpr int LIB = ANG ? SCHED_ISING : SCHED_DISCRETE;
    const bool lds = use_lds(n, path, sched_len(a), LIB);
    switch (n) {
        case 1: wave_kernel<float, 1, FILTER, ANG><<<wgrid, wblock, 0, s>>>(a, f, g, delta); break;
        case 2: wave_kernel<float, 2, FILTER, ANG><<<wgrid, wblock, 0, s>>>(a, f, g, delta); break;
        case 3: wave_kernel<float, 3, FILTER, ANG><<<wgrid, wblock, 0, s>>>(a, f, g, delta); break;
        case 4:
            if (lds) lds32_kernel<4, 1, FILTER, ANG><<<a.B, 64, 0, s>>>(a, f, g, delta);
            else reg_kernel<float, 4, FILTER, ANG><<<wgrid, wblock, 0, s>>>(a, f, g, delta);
            break;
        case 5:
            if (!lds) reg_kernel<float, 5, FILTER, ANG><<<wgrid, wblock, 0, s>>>(a, f, g, delta);
            else if (schedule_for(5, sched_len(a), LIB).waves == 2)
                lds32_kernel<5, 2, FILTER, ANG><<<a.B, 128, 0, s>>>(a, f, g, delta);
            else
                lds32_kernel<5, 1, FILTER, ANG><<<a.B, 64, 0, s>>>(a, f, g, delta);
            break;
        default:
            if (lds) lds32_kernel<6, 4, FILTER, ANG><<<a.B, 256, 0, s>>>(a, f, g, delta);
            else if ((uint32_t)a.B >= reg6_columns_min(ANG))
                reg_kernel<float, 6, FILTER, ANG, 64><<<wgrid, wblock, 0, s>>>(a, f, g, delta);
            else reg_kernel<float, 6, FILTER, ANG><<<a.B, 256, 0, s>>>(a, f, g, delta);
            break;
    }
}

hipError_t launch_eval_fp32(const BatchArgs& a, int path, float* f, float* g, float* delta,
                            int32_t* work, hipStream_t s) {
    if (a.B == 0) return hipSuccess;
    if (a.angles) {
        if (a.uniform_n > 0) {
            launch_width<false, true>(a, a.uniform_n, path, f, g, delta, s);
        } else {
            width_check_kernel<<<(a.B + 255) / 256, 256, 0, s>>>(a, f, g, delta);
            for (int n = 1; n <= MAX_QUBITS; ++n) launch_width<true, true>(a, n, path, f, g, delta, s);
        }
    } else if (a.uniform_n > 0) {
        launch_width<false, false>(a, a.uniform_n, path, f, g, delta, s);
    } else if (path == QE_PATH_FP32 && work) {
        // one launch over width-sorted work items (register-resident for n >= 4,
        // whatever the schedule says)
        mix_bucket_kernel<<<1, MIX_SORT, 0, s>>>(a, work + MIX_WORK_META, work);
        return launch_mix_eval(a, work, f, g, delta, s);
    } else {
        width_check_kernel<<<(a.B + 255) / 256, 256, 0, s>>>(a, f, g, delta);
        for (int n = 1; n <= MAX_QUBITS; ++n) launch_width<true, false>(a, n, path, f, g, delta, s);
    }
    return hipGetLastError();
}

// The phase-insensitive fitness is sum |U_ij|^2 |T_ij|^2 / 2^n; the kernels
// evaluate it as the diagonal overlap of U T^dagger, which equals it exactly
// when every entry of T has modulus 0 or 1.  One wavefront per circuit (one in
// all for a shared target) checks the target; a circuit whose target has an
// entry of modulus strictly between gets NaN and QE_DEVERR_TARGET.  Runs
// after the evaluation, whose outputs it overwrites.
template <typename Real>
__global__ void target_check_kernel(BatchArgs a, Real* f, Real* g, Real* delta) {
    const int lane = (int)lane_id();
    const bool shared = a.tstride == 0 && a.uniform_n > 0;
    const int b = shared ? 0 : (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (b >= a.B || (shared && (blockIdx.x > 0 || threadIdx.x >= 64))) return;
    const Item it = resolve(a, b, true);
    if (it.err) return;                    // malformed circuits report already
    const int NN = 1 << (2 * it.n);
    const Real* T = reinterpret_cast<const Real*>(a.targets) + 2 * it.toff;
    const Real tol = sizeof(Real) == 8 ? (Real)1e-9 : (Real)1e-5;
    bool bad = false;
    for (int e = lane; e < NN; e += 64) {
        const Real x = T[2 * e], y = T[2 * e + 1];
        const Real m = x * x + y * y;
        if (!(m <= tol || (m - (Real)1 <= tol && (Real)1 - m <= tol))) bad = true;
    }
    if (__ballot(bad) == 0ull) return;
    const Real nan = (Real)__builtin_nan("");
    auto mark = [&](int c) {
        f[c] = nan;
        if (g) g[c] = nan;
        if (delta) delta[c] = nan;
    };
    if (shared) {
        for (int c = lane; c < a.B; c += 64) mark(c);
    } else if (lane == 0) {
        mark(b);
    }
    if (lane == 0) atomicOr(a.err, (uint32_t)QE_DEVERR_TARGET);
}

hipError_t launch_target_check(const BatchArgs& a, bool fp64, void* f, void* g, void* delta,
                               hipStream_t s) {
    if (a.B == 0 || a.mode != QE_FIT_PHASE_INSENSITIVE) return hipSuccess;
    const unsigned grid = (a.tstride == 0 && a.uniform_n > 0) ? 1u : (unsigned)((a.B + 3) / 4);
    if (fp64) target_check_kernel<double><<<grid, 256, 0, s>>>(a, (double*)f, (double*)g, (double*)delta);
    else target_check_kernel<float><<<grid, 256, 0, s>>>(a, (float*)f, (float*)g, (float*)delta);
    return hipGetLastError();
}

hipError_t launch_mix_sort(const BatchArgs& a, int32_t* work, hipStream_t s) {
    if (a.B > 0) mix_bucket_kernel<<<1, MIX_SORT, 0, s>>>(a, work + MIX_WORK_META, work);
    return hipGetLastError();
}

hipError_t launch_mix_eval(const BatchArgs& a, const int32_t* work, float* f, float* g, float* delta,
                           hipStream_t s) {
    if (a.B == 0) return hipSuccess;
    // (the workgroups past the items leave: how many there are of each width is
    // known on the device only)
    const int32_t* order = work + MIX_WORK_META;
    if (mix_columns(a.B)) mix_kernel<true><<<a.B, 64, 0, s>>>(a, order, work, f, g, delta);
    else mix_kernel<false><<<a.B, 256, 0, s>>>(a, order, work, f, g, delta);
    return hipGetLastError();
}

template <bool ANG>
static void launch_fp64_width(const BatchArgs& a, double* f, double* g, double* delta, hipStream_t s) {
    const unsigned wgs = (unsigned)((a.B + WPB - 1) / WPB);
    switch (a.uniform_n) {
        case 1: wave_kernel<double, 1, false, ANG><<<wgs, 64 * WPB, 0, s>>>(a, f, g, delta); break;
        case 2: wave_kernel<double, 2, false, ANG><<<wgs, 64 * WPB, 0, s>>>(a, f, g, delta); break;
        case 3: wave_kernel<double, 3, false, ANG><<<wgs, 64 * WPB, 0, s>>>(a, f, g, delta); break;
        case 4: reg_kernel<double, 4, false, ANG><<<wgs, 64 * WPB, 0, s>>>(a, f, g, delta); break;
        case 5: reg_kernel<double, 5, false, ANG><<<wgs, 64 * WPB, 0, s>>>(a, f, g, delta); break;
        default: reg_kernel<double, 6, false, ANG><<<a.B, 256, 0, s>>>(a, f, g, delta); break;
    }
}

hipError_t launch_eval_fp64(const BatchArgs& a, double* f, double* g, double* delta, hipStream_t s) {
    if (a.B == 0) return hipSuccess;
    if (a.uniform_n == 0)
        lds_kernel<<<a.B, 256, generic_lds_bytes(MAX_QUBITS, 8), s>>>(a, f, g, delta);
    else if (a.angles) launch_fp64_width<true>(a, f, g, delta, s);
    else launch_fp64_width<false>(a, f, g, delta, s);
    return hipGetLastError();
}

template <typename Real, bool ANG>
static void launch_unitary_width(const BatchArgs& a, Real* out, hipStream_t s) {
    const unsigned wgs = (unsigned)((a.B + WPB - 1) / WPB);
    switch (a.uniform_n) {
        case 1: unitary_kernel<Real, 1, ANG><<<wgs, 64 * WPB, 0, s>>>(a, out); break;
        case 2: unitary_kernel<Real, 2, ANG><<<wgs, 64 * WPB, 0, s>>>(a, out); break;
        case 3: unitary_kernel<Real, 3, ANG><<<wgs, 64 * WPB, 0, s>>>(a, out); break;
        case 4: unitary_kernel<Real, 4, ANG><<<wgs, 64 * WPB, 0, s>>>(a, out); break;
        case 5: unitary_kernel<Real, 5, ANG><<<wgs, 64 * WPB, 0, s>>>(a, out); break;
        default: unitary_kernel<Real, 6, ANG><<<a.B, 256, 0, s>>>(a, out); break;
    }
}

hipError_t launch_unitary(const BatchArgs& a, bool fp64, void* out, hipStream_t s) {
    if (a.B == 0) return hipSuccess;
    if (fp64) {
        if (a.angles) launch_unitary_width<double, true>(a, (double*)out, s);
        else launch_unitary_width<double, false>(a, (double*)out, s);
    } else {
        if (a.angles) launch_unitary_width<float, true>(a, (float*)out, s);
        else launch_unitary_width<float, false>(a, (float*)out, s);
    }
    return hipGetLastError();
}

}  // namespace qe
