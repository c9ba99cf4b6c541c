// Register-resident evaluation core of widths 4, 5 and 6 (FP32 and FP64).
//
// The circuit's N x N product M = U T^dagger (N = 2^n) never leaves the
// registers: a wavefront holds CW columns (16; 32 at n = 5), lane l owns
// column j = l mod CW (plus the wavefront's first column) and, with
// q = l div CW, the rows whose lane-slot bits equal q, in E = N * CW / 64
// complex registers.  n = 6 takes four wavefronts, the others one (and n = 6
// with enough circuits to fill the GPU one, COLS = 64: a lane holds its whole
// column in 128 VGPRs, so that no wire is ever in a lane slot).  Row bits
// sit in slots: the lane bits above the column (LB = 2; 1 at n = 5) and the
// bits of the register index.  The gates run in reg_gates (qe_reg_asm.hpp): at
// n = 5, 6 a wire that a gate needs and that sits in a lane slot is exchanged
// with a register slot (v_permlane16/32_swap, one instruction per pair of
// registers) and stays there (per two-wire gate of random circuits 0.29 exchanges
// at n = 5, 0.51 at n = 6; 6.5 for the 24 gates that act in a sampled circuit of 40
// at n = 5).
//
// What bounds it: the VALU instructions of the gate bodies (8 or 10 per row pair of
// a CV) and the scalar instructions of their dispatch.  Against the same gates on
// M in LDS (run_lds_path) there is no LDS traffic, no address arithmetic, no gate
// table and no LDS round trip per gate, and the occupancy is set by about 70 VGPRs
// instead of 8 to 32 KB of LDS per circuit.  Measured: 8192 circuits of 48 gates
// (n = 6) 175 -> 84 us; the fused kernel of 65536 circuits of 40 gates (n = 5) 225 ->
// 170 us, its VALU busy 98 % of the time; FP64, 2048 circuits of 40 gates (n = 5),
// against the generic body 76 -> 19 us.
//
// The arithmetic of each element (one rounding per operation, the same
// operations in the same gate order) and the order of the reduction are those
// of run_lds_path and canonical_fitness, so the results are the same bits.
#pragma once
#include "qe_eval_core.hpp"
#include "qe_reg_asm.hpp"

namespace qe {

// COLS: columns per wavefront
template <int NQ>
constexpr int reg_columns() { return NQ == 5 ? 32 : 16; }
template <int NQ, int COLS>
struct RegGeom {
    static_assert(NQ >= 4 && NQ <= 6, "widths 4 to 6");
    static constexpr int N = 1 << NQ, CW = COLS, W = N / CW;
    static constexpr int Q = 64 / CW, LB = Q == 4 ? 2 : (Q == 2 ? 1 : 0), EB = NQ - LB, E = 1 << EB;
    // a lane's rows never move between slots (width 4, and one column per lane)
    static constexpr bool STATIC = NQ == 4 || LB == 0;
};

// Two complex numbers (one 16-byte load from memory aligned for one float2).
struct __attribute__((aligned(8))) float2x2 {
    float ax, ay, bx, by;
};

template <typename Real, int E>
struct RegVec;
template <> struct RegVec<float, 16> { using type = f32x32; };
template <> struct RegVec<float, 4> { using type = f32x8; };
template <> struct RegVec<float, 64> { using type = f32x128; };
template <> struct RegVec<double, 16> { using type = f64x32; };
template <> struct RegVec<double, 4> { using type = f64x8; };

template <typename Real, int NQ, int COLS = reg_columns<NQ>()>
struct RegMatrix {
    using G = RegGeom<NQ, COLS>;
    static constexpr int N = G::N, E = G::E, EB = G::EB, LB = G::LB, Q = G::Q;
    typename RegVec<Real, E>::type x;     // the lane's E elements
    SlotMap map;
    int j;                 // the lane's column
    uint32_t q;            // its lane-slot bits (lane slot s: bit s)

    __device__ __forceinline__ Real re(int m) const { return reg_get(x, 2 * m); }
    __device__ __forceinline__ Real im(int m) const { return reg_get(x, 2 * m + 1); }
    __device__ __forceinline__ void put(int m, Real r, Real i) {
        reg_set(x, 2 * m, r);
        reg_set(x, 2 * m + 1, i);
    }

    __device__ __forceinline__ void place(int wave) {
        const int lane = (int)lane_id();
        j = wave * G::CW + lane % G::CW;
        q = (uint32_t)lane / G::CW;
        // n = 5, 6: register slots hold the low row bits, lane slots the high
        // ones, so that a lane's E elements of M_0 = T^dagger are contiguous
        // in T; wire w is row bit NQ-1-w
        map.w2s = map.s2w = 0u;
        if constexpr (!G::STATIC) {
#pragma unroll
            for (int p = 0; p < NQ; ++p) {
                const uint32_t w = NQ - 1 - p;
                map.w2s |= (uint32_t)p << (4 * w);
                map.s2w |= 4u * w << (5 * p);
            }
        }
    }
    // M_0 = T^dagger: M[r][j] = conj(T[j][r])
    __device__ __forceinline__ void load(const float* __restrict__ T) {
        if constexpr (NQ == 4) {
            const float2* t = reinterpret_cast<const float2*>(T) + ((size_t)j * N + q);
#pragma unroll
            for (int m = 0; m < E; ++m) {
                const float2 v = t[Q * m];
                put(m, v.x, -v.y);
            }
        } else {
            const float2x2* t = reinterpret_cast<const float2x2*>(T + 2 * ((size_t)j * N + q * E));
#pragma unroll
            for (int m = 0; m < E; m += 2) {
                const float2x2 v = t[m / 2];
                put(m, v.ax, -v.ay);
                put(m + 1, v.bx, -v.by);
            }
        }
    }
    __device__ __forceinline__ void load(const double* __restrict__ T) {
        const complex128* t = reinterpret_cast<const complex128*>(T) + ((size_t)j * N + q * (NQ == 4 ? 1 : E));
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const complex128 v = t[(NQ == 4 ? Q : 1) * m];
            put(m, v.x, -v.y);
        }
    }
    __device__ __forceinline__ void identity() {
#pragma unroll
        for (int m = 0; m < E; ++m)
            put(m, (int)(NQ == 4 ? q + Q * m : q * E + m) == j ? (Real)1 : (Real)0, (Real)0);
    }

    // The word of a gate (its descriptor checked) for reg_gates: table, target and
    // control (the target again for a single-wire gate).
    // (exact: the bodies for exact values of a sampled circuit)
    static __device__ __forceinline__ uint32_t gate_word(uint32_t d, bool exact) {
        const uint32_t kind = d & 15u, t = (d >> 4) & 15u;
        const uint32_t c = kind_two_wire((int)kind) ? (d >> 8) & 15u : t;
        if constexpr (LB == 0) {
            // tables by kind: NOT 2, CNOT 1, CV, CV+ 0, H 0, T 1, R_x 3, R_y 4, R_z 5, J 2
            const uint32_t table = (uint32_t)((exact ? 0x33120ull : 0x25431000120ull) >> (4u * kind)) & 15u;
            const uint32_t ts = NQ - 1 - t, cs = NQ - 1 - c;
            const bool flip = kind == KIND_ZZ && ts > cs;            // (symmetric: one order)
            return 256u * table + 32u * (flip ? cs : ts) + 4u * (flip ? ts : cs);
        }
        // tables by kind: NOT, CNOT 2, CV 0, CV+ 1, H 0, T 1, R_x 3, R_y 4, R_z 5, J 3
        const uint32_t table = (uint32_t)((exact ? 0x43220ull : 0x35431010220ull) >> (4u * kind)) & 15u;
        if constexpr (NQ == 4) {
            // entries 0, 1: row bits 2, 3 (register bits); 2, 3: row bits 0, 1 (lane
            // slots); wire w is row bit 3 - w
            const uint32_t ts = (5u - t) & 3u, cs = (5u - c) & 3u;
            return 256u * table + 32u * ts + 4u * cs;
        } else {
            return 0x04040000u | (4u * c << 8) | (table << 5) | (4u * t);
        }
    }

    // ------------------------------------------------------------ circuits
    // Applies the circuit; false if a descriptor was invalid (M is then
    // garbage).  RESTORE: and leaves the slots in canonical order.  dv0: the
    // source's first chunk, fetched by the caller.
    // NCV: the source only yields what the QEQEA sampler decodes; units: the target
    // holds only 0, +-1 and +-i.
    template <bool RESTORE, bool NCV = false, typename GateSrc, typename SrcT>
    __device__ __forceinline__ bool run(int L, GateSrc&& src, const SrcT dv0, bool units = false) {
        constexpr bool ANG = src_angled<GateSrc>();
        static_assert(!NCV || !ANG, "sampled discrete circuits hold no angles");
        constexpr int GATES = ANG ? GATES_ANGLED : (NCV ? GATES_SAMPLED : GATES_DISCRETE);
        uint32_t cvs = 0u;                     // CV and CV+ gates so far
        const int lane = (int)lane_id();
        L = __builtin_amdgcn_readfirstlane(L);
        const int chunks = (L + 63) >> 6;
        // (an empty circuit still restores the slots; the next chunk is fetched
        // at the end of the body, so that there is one copy of the gate loop)
        SrcT dvv = dv0;
        int ch = 0;
        do {
            const uint32_t dv = desc_of(dvv);
            const bool in = lane < min(64, L - ch * 64);
            if (__ballot(in && !desc_valid<ANG>(dv, NQ))) return false;
            const int kind = (int)(dv & 15u);
            const bool live = in && kind != KIND_I;
            // the gates in order into the lanes up to 62, the others behind them
            const uint64_t todo = __ballot(live);
            const uint32_t cnt = (uint32_t)__popcll(todo);
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(todo >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)todo, 0u));
            const int to = 4 * (int)(((live ? rank - cnt : (uint32_t)lane - rank) - 1u) & 63u);
            bool exact = false;
            if constexpr (NCV) {
                cvs += (uint32_t)__popcll(__ballot(live && kind >= KIND_CV));
                exact = units && cvs <= EXACT_CV_MAX;
            }
            const uint32_t word = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(live ? gate_word(dv, exact) : 0u));
            Real gc = (Real)0.70710678118654752440084436210485, gs = (Real)0;
            if constexpr (LB == 0) {           // (CV and CV+ come with their signs)
                if (kind == KIND_CV) gc = exact ? (Real)1 : (Real)0.5;
                if (kind == KIND_CVDG) gc = exact ? (Real)-1 : (Real)-0.5;
                gs = -gc;
            }
            if constexpr (ANG)
                if (in && kind_ising(kind)) half_angle(angle_of(dvv), &gc, &gs);
            if constexpr (ANG || LB == 0) {
                gc = push_lane(to, gc);
                gs = push_lane(to, gs);
            }
            reg_gates<NQ, GATES>(x, word, cnt, gc, gs, map, RESTORE && ch + 1 >= chunks);
            if (++ch < chunks) dvv = src(ch);
        } while (ch < chunks);
        return true;
    }

    // Row-major store of M (the slots in any order).
    template <typename C2>
    __device__ __forceinline__ void store(C2* U, bool ok) const {
        auto bit = [&](int slot) -> uint32_t { return NQ - 1 - ((map.s2w >> (5 * slot + 2)) & 7u); };
        uint32_t row = q;                       // the lane slots' part
        if constexpr (!G::STATIC) {
            row = 0u;
#pragma unroll
            for (int s = 0; s < LB; ++s) row |= ((q >> s) & 1u) << bit(4 + s);
        }
#pragma unroll
        for (int m = 0; m < E; ++m) {
            uint32_t r = row;
#pragma unroll
            for (int k = 0; k < EB; ++k)
                if ((m >> k) & 1) r |= G::STATIC ? (uint32_t)Q << k : 1u << bit(k);
            const Real nan = (Real)__builtin_nan("");
            C2 v;
            v.x = ok ? re(m) : nan;
            v.y = ok ? im(m) : nan;
            U[(size_t)r * N + j] = v;
        }
    }

    // Eq. 11 (or, by `mode`, the phase-insensitive form) in the order of
    // canonical_fitness, of a matrix whose slots were restored.  Four wavefronts
    // per circuit (n = 6): all of them call it, red 4 x 3 values of LDS, w the
    // wavefront.  Returns f on every lane.
    __device__ __forceinline__ Real fitness(int mode, Real* g_out, Real* delta_out, int w, Real (*red)[3]) {
        if constexpr (LB == 0) return fitness_columns(mode, g_out, delta_out);
        else return fitness_groups(mode, g_out, delta_out, w, red);
    }

    // One column per lane (n = 6): the sums that canonical_fitness's wavefront
    // v makes of columns 16 v.. and row groups q (rows q, q + 4, ...) are formed
    // from the lane's four partial sums in the same order: over the 16 columns
    // of each q, over the groups, then over the wavefronts.
    __device__ __forceinline__ float fitness_columns(int mode, float* g_out, float* delta_out) const {
        float off[4] = {0.0f, 0.0f, 0.0f, 0.0f}, dr = 0.0f, di = 0.0f;
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const bool dg = m == j;
            const float xr = re(m), xi = im(m), m2 = xr * xr + xi * xi;
            off[m & 3] += dg ? 0.0f : m2;
            dr = dg ? xr : dr;
            di = dg ? xi : di;
        }
        // the four wavefronts' sums, in lanes 0, 16, 32, 48, added in order
        auto over_waves = [](float v) -> float {
            float t = 0.0f;
#pragma unroll
            for (int k = 0; k < 4; ++k) t += read_lane(v, 16 * k);
            return t;
        };
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            off[g] += dpp_mov<0xB1>(off[g]);
            off[g] += dpp_mov<0x4E>(off[g]);
            off[g] += dpp_mov<0x141>(off[g]);
            off[g] += dpp_mov<0x140>(off[g]);
        }
        const float offs = over_waves((off[0] + off[1]) + (off[2] + off[3]));
        if (mode == QE_FIT_PHASE_INSENSITIVE) {
            float fv;
            fitness_pi(offs, N, &fv, g_out, delta_out);
            return fv;
        }
        // a diagonal entry belongs to row group j mod 4: the columns of a group
        // (lanes 4 and 8 apart), then the groups
        auto total = [&](float v) -> float {
            v += dpp_mov<0x1B>(dpp_mov<0x141>(v));     // lane ^ 4: l ^ 7, then l ^ 3
            v += dpp_mov<0x128>(v);                    // lane ^ 8
            v += dpp_mov<0xB1>(v);
            v += dpp_mov<0x4E>(v);
            return over_waves(v);
        };
        const float tr = total(dr), ti = total(di);
        const float am = sqrtf(tr * tr + ti * ti);
        float er = 1.0f, ei = 0.0f;
        if (am > 0.0f) { er = tr / am; ei = ti / am; }
        const float xr = dr - er, xi = di - ei;
        const float dlt = 0.5f * (offs + total(xr * xr + xi * xi));
        *g_out = am / (float)N;
        *delta_out = dlt;
        return 1.0f - sqrtf(clamp01(dlt / (float)N));
    }

    __device__ __forceinline__ Real fitness_groups(int mode, Real* g_out, Real* delta_out, int w, Real (*red)[3]) {
        const int lane = (int)lane_id();
        const int key = (j % Q) == (int)q ? j / Q : -1;       // register of the diagonal entry
        // (one chain of E terms in FP64 too.  Four partial sums per lane are nearer on
        // dense columns, 0.65 against 0.86 units of 2^-53, but further off on circuits
        // near a target, whose products have few and like entries: n = 5, f of 10
        // gates 7.0e-17 against 6.5e-17, delta 3.7e-15 against 3.2e-15.)
        Real off = (Real)0, dr = (Real)0, di = (Real)0;
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const bool dg = m == key;
            const Real xr = re(m), xi = im(m), m2 = xr * xr + xi * xi;
            off += dg ? (Real)0 : m2;
            dr = dg ? xr : dr;
            di = dg ? xi : di;
        }
        // sums over the circuit's wavefronts, added in order
        auto total = [&](Real x) -> Real {
            const Real s = wave_sum(x);
            if constexpr (G::W == 1) {
                return s;
            } else {
                __syncthreads();
                if (lane == 0) red[w][0] = s;
                __syncthreads();
                Real t = (Real)0;
#pragma unroll
                for (int k = 0; k < G::W; ++k) t += red[k][0];
                return t;
            }
        };
        const Real offs = total(off);
        if (mode == QE_FIT_PHASE_INSENSITIVE) {
            Real fv;
            fitness_pi(offs, N, &fv, g_out, delta_out);
            return fv;
        }
        Real tr, ti;
        if constexpr (G::W == 1) {
            tr = wave_sum(dr);
            ti = wave_sum(di);
        } else {
            // (one pair of barriers for both components)
            const Real sr = wave_sum(dr), si = wave_sum(di);
            __syncthreads();
            if (lane == 0) { red[w][1] = sr; red[w][2] = si; }
            __syncthreads();
            tr = (Real)0;
            ti = (Real)0;
#pragma unroll
            for (int k = 0; k < G::W; ++k) { tr += red[k][1]; ti += red[k][2]; }
        }
        const Real am = real_sqrt(tr * tr + ti * ti);
        Real er = (Real)1, ei = (Real)0;
        if (am > (Real)0) { er = tr / am; ei = ti / am; }
        Real dl = (Real)0;
        if (key >= 0) { const Real xr = dr - er, xi = di - ei; dl = xr * xr + xi * xi; }
        const Real dlt = (Real)0.5 * (offs + total(dl));
        const Real qq = clamp01(dlt / (Real)N);
        *g_out = am / (Real)N;
        *delta_out = dlt;
        return (Real)1 - real_sqrt(qq);
    }
};

}  // namespace qe
