// Gate loop of the register-resident core (qe_reg_core.hpp), in assembly.
//
// One block runs a chunk of gates on a matrix held in a fixed run of VGPRs
// (element k: real part, then imaginary part).  A gate's word gives its table
// and its wires; the wires' slots pick the table's entry, which leads to a
// body that updates the registers in place and returns to the loop.  Written
// in C++ the same bodies under a dispatch cost 16 to 50 register moves per gate
// (the compiler turns the dispatch into a chain of merges and copies what a
// body swapped at each) and a tree of compares; here a gate costs its
// arithmetic, a dozen scalar instructions and two branches.
//
// What bounds it: the VALU's and the scalar unit's issue slots together (a SIMD
// issues one of each per four cycles and a wavefront one at a time): ten more
// instructions per gate of n = 5 circuits cost the fused generation of 65536 of
// them (180 us) 17 us as scalar and 9 us as vector instructions.  Hence the words
// that are s_bfe operands, the maps that are shift amounts, the gate count that
// carries out, and the loop's head at the end of every body (against a plain loop of
// about 20 scalar instructions a gate and 54 an exchange: 185 -> 176 us there).
//
// Tables of 64 entries (target 8 t, control c; t = c: a single-wire gate):
//   0 CV, H   1 CV+, T   2 CNOT, NOT   3 interaction, R_x   4 R_y   5 R_z
// (sampled circuits, which hold no other kinds: 0 CV  1 CV+  2 CNOT, NOT and 3 CV
// 4 CV+ of exact values); with 16 registers per lane also the exchanges of register
// bits 0..3 and lane slots 4, 5 (4 times the higher, plus the lower, always a
// register bit).  Entries that nothing has lead to the block's end.
//
// 16 registers (widths 5, 6): a wire is in any slot (maps W: wire to slot, S:
// slot to wire).  A gate whose wire is in a lane slot first
// exchanges that slot with a register bit, by choice one that the next gate
// does not use.  4 registers (width 4): every wire keeps its slot (entries 0,
// 1: register bits, 2, 3: lane slots) and the bodies deal with the lane slots
// themselves: with 4 registers every other gate would need an exchange, and
// keeping the maps would cost more scalar instructions than that saves.
//
// 64 registers (width 6, one column per lane): every wire is a register bit, so
// a gate's word is its entry, in the tables
//   0 CV and CV+, H   1 CNOT, T   2 interaction (t < c), NOT   3 R_x   4 R_y   5 R_z
// (sampled circuits: 2 NOT and 3 CV and CV+ of exact values)
//
// Multiplies and adds stay separate (one rounding each) except in CV, whose
// last step is a fused multiply-add of exact halves.
//
// Exact values: from a target whose entries are 0, +-1 and +-i, k gates CV or CV+
// (CNOT and NOT only move values) leave entries that are multiples of
// 2^-ceil(k/2) no larger than 8 (a column's norm does not grow).  With k <= 36
// (EXACT_CV_MAX) every sum of the bodies fits 24 bits, nothing is ever rounded,
// and a body of 8 operations per row pair instead of 10 gives the same bits (n = 6:
// a generation of 4096 circuits of 48 gates 65.2 -> 60.9 us; n = 5, 65536 circuits
// of 40 gates: 9 % fewer vector instructions, the fused kernel 187 -> 185 us).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qe {

// The lane's registers: element k is values 2k and 2k + 1.  (An asm operand
// holds at most 32 VGPRs, so 32 doubles are two.)
typedef float f32x32 __attribute__((ext_vector_type(32)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef double f64x16 __attribute__((ext_vector_type(16)));
typedef double f64x8 __attribute__((ext_vector_type(8)));
struct f64x32 {
    f64x16 lo, hi;
};
struct f32x128 {
    f32x32 a, b, c, d;
};
template <typename V>
__device__ __forceinline__ auto reg_get(const V& x, int i) { return x[i]; }
__device__ __forceinline__ double reg_get(const f64x32& x, int i) { return i < 16 ? x.lo[i] : x.hi[i - 16]; }
__device__ __forceinline__ float reg_get(const f32x128& x, int i) {
    return i < 32 ? x.a[i] : i < 64 ? x.b[i - 32] : i < 96 ? x.c[i - 64] : x.d[i - 96];
}
template <typename V, typename R>
__device__ __forceinline__ void reg_set(V& x, int i, R v) { x[i] = v; }
__device__ __forceinline__ void reg_set(f32x128& x, int i, float v) {
    if (i < 32) x.a[i] = v;
    else if (i < 64) x.b[i - 32] = v;
    else if (i < 96) x.c[i - 64] = v;
    else x.d[i - 96] = v;
}
__device__ __forceinline__ void reg_set(f64x32& x, int i, double v) {
    if (i < 16) x.lo[i] = v;
    else x.hi[i - 16] = v;
}

// Wave-uniform maps: wire w's slot in bits 4 w.. of w2s, slot s's wire times 4 in bits
// 5 s.. of s2w; register bit k is slot k, lane slot s slot 4 + s.
struct SlotMap {
    uint32_t w2s, s2w;
};

// What a circuit may hold: the discrete libraries, angled gates as well, or only
// what the QEQEA sampler decodes ({I, NOT, CNOT, CV, CV+}).
enum : int { GATES_DISCRETE = 0, GATES_ANGLED = 1, GATES_SAMPLED = 2 };
constexpr uint32_t EXACT_CV_MAX = 36;

// ------------------------------------------------------------ assembler text
// Registers of element k (x real, y imaginary part), the temporaries and the
// gate's scalars, then the arithmetic, per precision.
#define QR_X32(k) "v[QRB+2*(" k ")]"
#define QR_Y32(k) "v[QRB+2*(" k ")+1]"
#define QR_T32(i) "v[QRT+" #i "]"
#define QR_A32 "s60"
#define QR_B32 "s62"
#define QR_ADD32(d, a, b) "v_add_f32 " d "," a "," b "\n"
#define QR_SUB32(d, a, b) "v_sub_f32 " d "," a "," b "\n"
#define QR_MUL32(d, a, b) "v_mul_f32 " d "," a "," b "\n"
#define QR_FMA32(d, a, b, c) "v_fma_f32 " d "," a "," b "," c "\n"
#define QR_FMAC32(d, a, b) "v_fmac_f32 " d "," a "," b "\n"
#define QR_XCH32(ins, k, l)                                                                          \
    ins " v[QRB+2*(" k ")],v[QRB+2*(" l ")]\n" ins " v[QRB+2*(" k ")+1],v[QRB+2*(" l ")+1]\n"
// 1 / sqrt 2, for H and T
#define QR_CONST32 "s_mov_b32 s60,0x3f3504f3\n"
#define QR_ANGLE32 "v_readlane_b32 s60,%[gc],s42\nv_readlane_b32 s62,%[gs],s42\n"

#define QR_X64(k) "v[QRB+4*(" k "):QRB+4*(" k ")+1]"
#define QR_Y64(k) "v[QRB+4*(" k ")+2:QRB+4*(" k ")+3]"
#define QR_T64(i) "v[QRT+2*" #i ":QRT+2*" #i "+1]"
#define QR_A64 "s[60:61]"
#define QR_B64 "s[62:63]"
#define QR_ADD64(d, a, b) "v_add_f64 " d "," a "," b "\n"
#define QR_SUB64(d, a, b) "v_add_f64 " d "," a ",-" b "\n"
#define QR_MUL64(d, a, b) "v_mul_f64 " d "," a "," b "\n"
#define QR_FMA64(d, a, b, c) "v_fma_f64 " d "," a "," b "," c "\n"
#define QR_FMAC64(d, a, b) "v_fmac_f64 " d "," a "," b "\n"
#define QR_XCH64(ins, k, l)                                                                          \
    ins " v[QRB+4*(" k ")],v[QRB+4*(" l ")]\n" ins " v[QRB+4*(" k ")+1],v[QRB+4*(" l ")+1]\n"        \
    ins " v[QRB+4*(" k ")+2],v[QRB+4*(" l ")+2]\n" ins " v[QRB+4*(" k ")+3],v[QRB+4*(" l ")+3]\n"
#define QR_CONST64 "s_mov_b32 s60,0x667f3bcd\ns_mov_b32 s61,0x3fe6a09e\n"
#define QR_ANGLE64                                                                                   \
    "v_readlane_b32 s60,%[gcl],s42\nv_readlane_b32 s61,%[gch],s42\n"                                 \
    "v_readlane_b32 s62,%[gsl],s42\nv_readlane_b32 s63,%[gsh],s42\n"

#define QR_ELEMS16 "0,1,2,3,4,5,6,7,8,9,10,11,12,13,14,15"
#define QR_ELEMS4 "0,1,2,3"
#define QR_ELEMS64                                                                                   \
    "0,1,2,3,4,5,6,7,8,9,10,11,12,13,14,15,16,17,18,19,20,21,22,23,24,25,26,27,28,29,30,31,"         \
    "32,33,34,35,36,37,38,39,40,41,42,43,44,45,46,47,48,49,50,51,52,53,54,55,56,57,58,59,60,61,62,63"

// The rows a of a gate whose target and control are register bits QT, QC, and
// their partners.
#define QR_A "\\a"
#define QR_P "\\a+(1<<QT)"
#define QR_ROWS(E, cond, text) ".irp a," QR_ELEMS##E "\n.if " cond "\n" text ".endif\n.endr\n"
#define QR_ROWS1(E, text) QR_ROWS(E, "((\\a>>QT)&1)==0", text)
#define QR_ROWS2(E, text) QR_ROWS(E, "(((\\a>>QT)&1)==0)&(((\\a>>QC)&1)==1)", text)

// u + iv = a - b, p + iq = (a + b) / 2: a' = p - hs v + i (q + hs u), b' = p + hs v
// + i (q - hs u); HP = hs, HM = -hs
#define QR_CVROW(P, HP, HM)                                                                          \
                QR_SUB##P(QR_T##P(0), QR_X##P(QR_A), QR_X##P(QR_P))                                  \
                QR_SUB##P(QR_T##P(1), QR_Y##P(QR_A), QR_Y##P(QR_P))                                  \
                QR_ADD##P(QR_X##P(QR_A), QR_X##P(QR_A), QR_X##P(QR_P))                               \
                QR_ADD##P(QR_Y##P(QR_A), QR_Y##P(QR_A), QR_Y##P(QR_P))                               \
                QR_MUL##P(QR_X##P(QR_P), "0.5", QR_X##P(QR_A))                                       \
                QR_MUL##P(QR_Y##P(QR_P), "0.5", QR_Y##P(QR_A))                                       \
                QR_FMA##P(QR_X##P(QR_A), HM, QR_T##P(1), QR_X##P(QR_P))                              \
                QR_FMA##P(QR_Y##P(QR_A), HP, QR_T##P(0), QR_Y##P(QR_P))                              \
                QR_FMAC##P(QR_X##P(QR_P), HP, QR_T##P(1))                                            \
                QR_FMAC##P(QR_Y##P(QR_P), HM, QR_T##P(0))
#define QR_CV(P, E, HP, HM) QR_ROWS2(E, QR_CVROW(P, HP, HM))
// The same in 8 operations, for exact values (as above; the same bits there): with
// g + ih = (1 -+ i) (u + iv) / 2 a' = a - (g + ih), b' = b + (g + ih)
#define QR_CVROW8(P, ADDG, SUBH)                                                                     \
                QR_SUB##P(QR_T##P(0), QR_X##P(QR_A), QR_X##P(QR_P))                                  \
                QR_SUB##P(QR_T##P(1), QR_Y##P(QR_A), QR_Y##P(QR_P))                                  \
                ADDG##P(QR_T##P(2), QR_T##P(0), QR_T##P(1))                                          \
                SUBH##P(QR_T##P(3), QR_T##P(1), QR_T##P(0))                                          \
                QR_FMAC##P(QR_X##P(QR_A), "-0.5", QR_T##P(2))                                        \
                QR_FMAC##P(QR_Y##P(QR_A), "-0.5", QR_T##P(3))                                        \
                QR_FMAC##P(QR_X##P(QR_P), "0.5", QR_T##P(2))                                         \
                QR_FMAC##P(QR_Y##P(QR_P), "0.5", QR_T##P(3))
#define QR_CXROW(P) QR_XCH##P("v_swap_b32", QR_A, QR_P)
#define QR_CNOT(P, E) QR_ROWS2(E, QR_CXROW(P))
#define QR_NOT(P, E) QR_ROWS1(E, QR_XCH##P("v_swap_b32", QR_A, QR_P))
#define QR_H(P, E)                                                                                   \
    QR_ROWS1(E, QR_SUB##P(QR_T##P(0), QR_X##P(QR_A), QR_X##P(QR_P))                                  \
                QR_SUB##P(QR_T##P(1), QR_Y##P(QR_A), QR_Y##P(QR_P))                                  \
                QR_ADD##P(QR_X##P(QR_A), QR_X##P(QR_A), QR_X##P(QR_P))                               \
                QR_ADD##P(QR_Y##P(QR_A), QR_Y##P(QR_A), QR_Y##P(QR_P))                               \
                QR_MUL##P(QR_X##P(QR_A), QR_A##P, QR_X##P(QR_A))                                     \
                QR_MUL##P(QR_Y##P(QR_A), QR_A##P, QR_Y##P(QR_A))                                     \
                QR_MUL##P(QR_X##P(QR_P), QR_A##P, QR_T##P(0))                                        \
                QR_MUL##P(QR_Y##P(QR_P), QR_A##P, QR_T##P(1)))
#define QR_TG(P, E)                                                                                  \
    QR_ROWS1(E, QR_SUB##P(QR_T##P(0), QR_X##P(QR_P), QR_Y##P(QR_P))                                  \
                QR_ADD##P(QR_Y##P(QR_P), QR_X##P(QR_P), QR_Y##P(QR_P))                               \
                QR_MUL##P(QR_X##P(QR_P), QR_A##P, QR_T##P(0))                                        \
                QR_MUL##P(QR_Y##P(QR_P), QR_A##P, QR_Y##P(QR_P)))
// rotations, A + iB = e^{i theta/2}: temporaries B times the four parts, then
// the parts scaled by A
#define QR_ROT(P, E, t0, t1, t2, t3, rest)                                                           \
    QR_ROWS1(E, QR_MUL##P(QR_T##P(0), QR_B##P, t0) QR_MUL##P(QR_T##P(1), QR_B##P, t1)                \
                QR_MUL##P(QR_T##P(2), QR_B##P, t2) QR_MUL##P(QR_T##P(3), QR_B##P, t3)                \
                QR_MUL##P(QR_X##P(QR_A), QR_A##P, QR_X##P(QR_A))                                     \
                QR_MUL##P(QR_Y##P(QR_A), QR_A##P, QR_Y##P(QR_A))                                     \
                QR_MUL##P(QR_X##P(QR_P), QR_A##P, QR_X##P(QR_P))                                     \
                QR_MUL##P(QR_Y##P(QR_P), QR_A##P, QR_Y##P(QR_P)) rest)
// a' = c a - i s b, b' = c b - i s a
#define QR_RX(P, E)                                                                                  \
    QR_ROT(P, E, QR_Y##P(QR_P), QR_X##P(QR_P), QR_Y##P(QR_A), QR_X##P(QR_A),                         \
           QR_ADD##P(QR_X##P(QR_A), QR_X##P(QR_A), QR_T##P(0))                                       \
           QR_SUB##P(QR_Y##P(QR_A), QR_Y##P(QR_A), QR_T##P(1))                                       \
           QR_ADD##P(QR_X##P(QR_P), QR_X##P(QR_P), QR_T##P(2))                                       \
           QR_SUB##P(QR_Y##P(QR_P), QR_Y##P(QR_P), QR_T##P(3)))
// a' = c a - s b, b' = s a + c b
#define QR_RY(P, E)                                                                                  \
    QR_ROT(P, E, QR_X##P(QR_P), QR_Y##P(QR_P), QR_X##P(QR_A), QR_Y##P(QR_A),                         \
           QR_SUB##P(QR_X##P(QR_A), QR_X##P(QR_A), QR_T##P(0))                                       \
           QR_SUB##P(QR_Y##P(QR_A), QR_Y##P(QR_A), QR_T##P(1))                                       \
           QR_ADD##P(QR_X##P(QR_P), QR_T##P(2), QR_X##P(QR_P))                                       \
           QR_ADD##P(QR_Y##P(QR_P), QR_T##P(3), QR_Y##P(QR_P)))
// a' = (c - i s) a, b' = (c + i s) b
#define QR_RZ(P, E)                                                                                  \
    QR_ROT(P, E, QR_Y##P(QR_A), QR_X##P(QR_A), QR_Y##P(QR_P), QR_X##P(QR_P),                         \
           QR_ADD##P(QR_X##P(QR_A), QR_X##P(QR_A), QR_T##P(0))                                       \
           QR_SUB##P(QR_Y##P(QR_A), QR_Y##P(QR_A), QR_T##P(1))                                       \
           QR_SUB##P(QR_X##P(QR_P), QR_X##P(QR_P), QR_T##P(2))                                       \
           QR_ADD##P(QR_Y##P(QR_P), QR_Y##P(QR_P), QR_T##P(3)))
// e^{-i theta/2} where the two wires' bits agree, e^{i theta/2} where they differ
#define QR_ZZ(P, E)                                                                                  \
    ".irp a," QR_ELEMS##E "\n"                                                                       \
    QR_MUL##P(QR_T##P(0), QR_B##P, QR_Y##P(QR_A)) QR_MUL##P(QR_T##P(1), QR_B##P, QR_X##P(QR_A))      \
    QR_MUL##P(QR_X##P(QR_A), QR_A##P, QR_X##P(QR_A)) QR_MUL##P(QR_Y##P(QR_A), QR_A##P, QR_Y##P(QR_A)) \
    ".if ((\\a>>QT)&1)==((\\a>>QC)&1)\n"                                                             \
    QR_ADD##P(QR_X##P(QR_A), QR_X##P(QR_A), QR_T##P(0))                                              \
    QR_SUB##P(QR_Y##P(QR_A), QR_Y##P(QR_A), QR_T##P(1))                                              \
    ".else\n"                                                                                        \
    QR_SUB##P(QR_X##P(QR_A), QR_X##P(QR_A), QR_T##P(0))                                              \
    QR_ADD##P(QR_Y##P(QR_A), QR_Y##P(QR_A), QR_T##P(1))                                              \
    ".endif\n.endr\n"

// Lane slot S with register bit K.  v_permlane*_swap reads a register two wait
// states or more after the VALU wrote it, hence the s_nop.
#define QR_SWAPS(P, E, SW, K) QR_ROWS(E, "((\\a>>(" K "))&1)==0", QR_XCH##P(SW, QR_A, "\\a+(1<<(" K "))"))
#define QR_LANE2(P, E, S, K)                                                                         \
    "s_nop 1\n.if (" S ")==0\n" QR_SWAPS(P, E, "v_permlane16_swap_b32", K) ".else\n"                 \
    QR_SWAPS(P, E, "v_permlane32_swap_b32", K) ".endif\n"
#define QR_LANE1(P, E, S, K) "s_nop 1\n" QR_SWAPS(P, E, "v_permlane32_swap_b32", K)

#define QR_BODY(name, list, text) ".irp n," list "\n.Lqr%=" name "\\n:\n" text "qrnext%=\n.endr\n"
#define QR_TWO16 "1,2,3,8,10,11,16,17,19,24,25,26"
#define QR_ONE16 "0,9,18,27"
#define QR_SETTC ".set QT,\\n>>3\n.set QC,\\n&7\n"
// widths 5, 6: target and control are register bits
#define QR_TWO_16(name, text) QR_BODY(name, QR_TWO16, QR_SETTC text)
#define QR_ONE_16(name, text) QR_BODY(name, QR_ONE16, QR_SETTC text)
// width 4: slots 2, 3 are lane slots (S = 0, 1).  A lane slot's target is
// exchanged with a register bit around the body (of a controlled gate with a
// register control: only the rows it changes); a lane slot's control, and the
// one row that T changes, are masked lanes; the diagonal rotations take the
// sign of B from the lane.
#define QR_MASK(slot)      /* the lanes whose lane slot (2 or 3) is 1 */                              \
    ".if (" slot ")==2\n.set QML,0xffff0000\n.set QMH,0xffff0000\n.else\n.set QML,0\n.set QMH,0xffffffff\n.endif\n"
#define QR_EXEC "s_mov_b32 exec_lo,QML\ns_mov_b32 exec_hi,QMH\n"
#define QR_EXEC_ALL "s_mov_b64 exec,-1\n"
#define QR_LANEROWS(P, S)                                                                            \
    "s_nop 1\n.if (" S ")==0\n" QR_ROWS2(4, QR_XCH##P("v_permlane16_swap_b32", QR_A, QR_P))          \
    ".else\n" QR_ROWS2(4, QR_XCH##P("v_permlane32_swap_b32", QR_A, QR_P)) ".endif\n"
#define QR_CTL4(P, name, row)                                                                        \
    QR_BODY(name, QR_TWO16, QR_SETTC                                                                  \
        ".if (QT<2)&(QC<2)\n" QR_ROWS2(4, row)                                                       \
        ".elseif QT<2\n" QR_MASK("QC") QR_EXEC QR_ROWS1(4, row) QR_EXEC_ALL                          \
        ".elseif QC<2\n.set QS0,QT-2\n.set QT,1-QC\n"                                                \
        QR_LANEROWS(P, "QS0") QR_ROWS2(4, row) QR_LANEROWS(P, "QS0")                                 \
        ".else\n.set QS0,QT-2\n.set QT,0\n" QR_LANE2(P, 4, "QS0", "0")                               \
        QR_MASK("QC") QR_EXEC QR_ROWS1(4, row) QR_EXEC_ALL QR_LANE2(P, 4, "QS0", "0") ".endif\n")
#define QR_ONE4(P, name, text)                                                                       \
    QR_BODY(name, QR_ONE16, QR_SETTC                                                                  \
        ".if QT<2\n" text ".else\n.set QS0,QT-2\n.set QT,0\n"                                        \
        QR_LANE2(P, 4, "QS0", "0") text QR_LANE2(P, 4, "QS0", "0") ".endif\n")
#define QR_TROW(P)                                                                                   \
    QR_SUB##P(QR_T##P(0), QR_X##P(QR_A), QR_Y##P(QR_A)) QR_ADD##P(QR_Y##P(QR_A), QR_X##P(QR_A), QR_Y##P(QR_A)) \
    QR_MUL##P(QR_X##P(QR_A), QR_A##P, QR_T##P(0)) QR_MUL##P(QR_Y##P(QR_A), QR_A##P, QR_Y##P(QR_A))
#define QR_T4(P)                                                                                     \
    QR_BODY("t", QR_ONE16, QR_SETTC                                                                   \
        ".if QT<2\n" QR_ROWS(4, "((\\a>>QT)&1)==1", QR_TROW(P))                                      \
        ".else\n" QR_MASK("QT") QR_EXEC QR_ROWS(4, "1", QR_TROW(P)) QR_EXEC_ALL ".endif\n")
// temporary 3: B, negated in the lanes of the mask; then row a times A - i B3, or
// (odd rows) A + i B3
#define QR_SIGN32                                                                                    \
    "v_mov_b32 v[QRT+3]," QR_B32 "\ns_mov_b32 s50,QML\ns_mov_b32 s51,QMH\n"                          \
    "v_cndmask_b32_e64 v[QRT+3],v[QRT+3],-v[QRT+3],s[50:51]\n"
#define QR_SIGN64                                                                                    \
    "v_mov_b32 v[QRT+6],s62\nv_mov_b32 v[QRT+7],s63\ns_mov_b32 s50,QML\ns_mov_b32 s51,QMH\n"         \
    "v_cndmask_b32_e64 v[QRT+7],v[QRT+7],-v[QRT+7],s[50:51]\n"
#define QR_PHASE(P, odd)                                                                             \
    ".irp a," QR_ELEMS4 "\n"                                                                         \
    QR_MUL##P(QR_T##P(0), QR_T##P(3), QR_Y##P(QR_A)) QR_MUL##P(QR_T##P(1), QR_T##P(3), QR_X##P(QR_A)) \
    QR_MUL##P(QR_X##P(QR_A), QR_A##P, QR_X##P(QR_A)) QR_MUL##P(QR_Y##P(QR_A), QR_A##P, QR_Y##P(QR_A)) \
    ".if " odd "\n"                                                                                  \
    QR_SUB##P(QR_X##P(QR_A), QR_X##P(QR_A), QR_T##P(0)) QR_ADD##P(QR_Y##P(QR_A), QR_Y##P(QR_A), QR_T##P(1)) \
    ".else\n"                                                                                        \
    QR_ADD##P(QR_X##P(QR_A), QR_X##P(QR_A), QR_T##P(0)) QR_SUB##P(QR_Y##P(QR_A), QR_Y##P(QR_A), QR_T##P(1)) \
    ".endif\n.endr\n"
#define QR_RZ4(P)                                                                                    \
    QR_BODY("rz", QR_ONE16, QR_SETTC                                                                  \
        ".if QT<2\n" QR_RZ(P, 4) ".else\n" QR_MASK("QT") QR_SIGN##P QR_PHASE(P, "0") ".endif\n")
#define QR_ZZ4(P)                                                                                    \
    QR_BODY("zz", QR_TWO16, QR_SETTC                                                                  \
        ".if (QT<2)&(QC<2)\n" QR_ZZ(P, 4)                                                            \
        ".elseif QT<2\n" QR_MASK("QC") QR_SIGN##P QR_PHASE(P, "((\\a>>QT)&1)==1")                    \
        ".elseif QC<2\n" QR_MASK("QT") QR_SIGN##P QR_PHASE(P, "((\\a>>QC)&1)==1")                    \
        ".else\n.set QML,0xffff0000\n.set QMH,0x0000ffff\n" QR_SIGN##P QR_PHASE(P, "0") ".endif\n")

// a table: bodies of two wires and of one, by name (QRN slots, those from QRL on
// lead to the exchange)
#define QR_TABLE(test, two, one)                                                                     \
    ".irp n," QR_ELEMS64 "\n.if ((\\n>>3)>=QRN)|((\\n&7)>=QRN)|(" test ")\ns_branch .Lqr%=e\n"       \
    ".elseif ((\\n>>3)>=QRL)|((\\n&7)>=QRL)\ns_branch .Lqr%=s\n"                                     \
    ".elseif (\\n>>3)==(\\n&7)\ns_branch .Lqr%=" one "\n.else\ns_branch .Lqr%=" two "\n.endif\n.endr\n"
#define QR_TAB(two, one) QR_TABLE("0", two "\\n", one "\\n")
#define QR_TAB1(one) QR_TABLE("(\\n>>3)!=(\\n&7)", "e", one "\\n")
#define QR_TAB2(two) QR_TABLE("(\\n>>3)==(\\n&7)", two "\\n", "e")
#define QR_TABLES0 QR_TAB("cv", "h") QR_TAB("cd", "t") QR_TAB("cx", "x")
#define QR_TABLES1 QR_TABLES0 QR_TAB("zz", "rx") QR_TAB1("ry") QR_TAB1("rz")
#define QR_TABLES2 QR_TAB2("cv") QR_TAB2("cd") QR_TAB("cx", "x") QR_TAB2("cw") QR_TAB2("ce")
#define QR_BODIES16_0(P)                                                                             \
    QR_TWO_16("cv", QR_CV(P, 16, "0.5", "-0.5")) QR_TWO_16("cd", QR_CV(P, 16, "-0.5", "0.5"))        \
    QR_TWO_16("cx", QR_CNOT(P, 16)) QR_ONE_16("h", QR_H(P, 16)) QR_ONE_16("t", QR_TG(P, 16))         \
    QR_ONE_16("x", QR_NOT(P, 16))
#define QR_BODIES16_1(P)                                                                             \
    QR_BODIES16_0(P) QR_TWO_16("zz", QR_ZZ(P, 16)) QR_ONE_16("rx", QR_RX(P, 16))                     \
    QR_ONE_16("ry", QR_RY(P, 16)) QR_ONE_16("rz", QR_RZ(P, 16))
#define QR_BODIES16_2(P)                                                                             \
    QR_TWO_16("cv", QR_CV(P, 16, "0.5", "-0.5")) QR_TWO_16("cd", QR_CV(P, 16, "-0.5", "0.5"))        \
    QR_TWO_16("cw", QR_ROWS2(16, QR_CVROW8(P, QR_ADD, QR_SUB)))                                      \
    QR_TWO_16("ce", QR_ROWS2(16, QR_CVROW8(P, QR_SUB, QR_ADD)))                                      \
    QR_TWO_16("cx", QR_CNOT(P, 16)) QR_ONE_16("x", QR_NOT(P, 16))
#define QR_BODIES4_0(P)                                                                              \
    QR_CTL4(P, "cv", QR_CVROW(P, "0.5", "-0.5")) QR_CTL4(P, "cd", QR_CVROW(P, "-0.5", "0.5"))        \
    QR_CTL4(P, "cx", QR_CXROW(P)) QR_ONE4(P, "h", QR_H(P, 4)) QR_T4(P) QR_ONE4(P, "x", QR_NOT(P, 4))
#define QR_BODIES4_2(P)                                                                              \
    QR_CTL4(P, "cv", QR_CVROW(P, "0.5", "-0.5")) QR_CTL4(P, "cd", QR_CVROW(P, "-0.5", "0.5"))        \
    QR_CTL4(P, "cw", QR_CVROW8(P, QR_ADD, QR_SUB)) QR_CTL4(P, "ce", QR_CVROW8(P, QR_SUB, QR_ADD))    \
    QR_CTL4(P, "cx", QR_CXROW(P)) QR_ONE4(P, "x", QR_NOT(P, 4))
#define QR_BODIES4_1(P)                                                                              \
    QR_BODIES4_0(P) QR_ZZ4(P) QR_ONE4(P, "rx", QR_RX(P, 4)) QR_ONE4(P, "ry", QR_RY(P, 4)) QR_RZ4(P)
#define QR_SCALARS0(P)
#define QR_SCALARS2(P)
#define QR_START2(P)
#define QR_SCALARS1(P) QR_ANGLE##P
#define QR_START0(P) QR_CONST##P
#define QR_START1(P)

// s[40:41] the tables' address, s43 the next gate's word, s42 its lane (mod 64): the
// gates lie in the lanes up to 62 (the first in lane 63 - cnt), so that counting
// s42 up carries out behind the last.  qrnext: goes to the next gate's body, or
// leaves (the end of every body has its own copy: one branch fewer per gate).
#define QR_HEAD(BASE, TMP, N, L) ".set QRB," BASE "\n.set QRT," TMP "\n.set QRN," N "\n.set QRL," L "\n"
#define QR_PC(rest)                                                                                  \
    "s_getpc_b64 s[40:41]\n.Lqr%=p:\n" rest "s_sub_u32 s42,-1,%[cnt]\nv_readlane_b32 s43,%[p],s42\n"
#define QR_COUNT(end) "s_add_u32 s42,s42,1\ns_cbranch_scc1 .Lqr%=" end "\n"

// Width 4, and 64 registers: the word is the gate's entry (bytes).
#define QR_ENTRY                                                                                     \
    QR_COUNT("e") "s_add_u32 s48,s40,s43\ns_addc_u32 s49,s41,0\nv_readlane_b32 s43,%[p],s42\n"       \
    "s_setpc_b64 s[48:49]\n"
#define QR_TEXT4(P, BASE, TMP, ANG)                                                                  \
    QR_HEAD(BASE, TMP, "4", "8") QR_START##ANG(P)                                                    \
    QR_PC("s_add_u32 s40,s40,.Lqr%=tab-.Lqr%=p\ns_addc_u32 s41,s41,0\n")                             \
    ".macro qrnext%=\n" QR_SCALARS##ANG(P) QR_ENTRY ".endm\nqrnext%=\n"                              \
    ".Lqr%=tab:\n" QR_TABLES##ANG QR_BODIES4_##ANG(P) ".Lqr%=e:\n"

// Widths 5, 6: the word holds 4 * target wire (bits 0..4), the table (bits 5..7), 4 *
// control wire (target again for a single-wire gate; bits 8..12), and 4 in bits
// 16.. and 24.., so that it and its half from bit 8 on are s_bfe's offset and width
// of the wires' slots in W.  A gate is in s45, s46 (its slots) and s50 (its table).
#define QR_GO16                                                                                      \
    "s_lshl3_add_u32 s47,s45,s46\ns_lshl1_add_u32 s47,s50,s47\ns_lshl2_add_u32 s48,s47,s40\n"         \
    "s_addc_u32 s49,s41,0\ns_setpc_b64 s[48:49]\n"
#define QR_WANT(slot, wire, label)                                                                   \
    "s_bfe_u32 s47,%[W],0x40000+4*" wire "\ns_cmp_eq_u32 s47," slot "\ns_cbranch_scc1 " label "\n"
#define QR_CALL(label)                                                                               \
    "s_getpc_b64 s[58:59]\n.Lqr%=p" label ":\ns_add_u32 s58,s58,.Lqr%=" label "-.Lqr%=p" label "\n"  \
    "s_addc_u32 s59,s59,0\ns_branch .Lqr%=x\n.Lqr%=" label ":\n"
// canonical order: the lane slots, then register bits 0..2; L0, L1: the wires of
// lane slots 4, 5, R0..R2: those of register bits 0..2
#define QR_LANE_BACK2(L0, L1)                                                                        \
    QR_WANT("4", L0, ".Lqr%=r1")                                                                     \
    /* (from the other lane slot by way of register bit 0) */                                        \
    "s_mov_b32 s54,s47\ns_cmp_lt_u32 s47,4\ns_cbranch_scc1 .Lqr%=r0\n"                               \
    "s_mov_b32 s54,0\n" QR_CALL("c0") "s_mov_b32 s54,0\n"                                            \
    ".Lqr%=r0:\ns_mov_b32 s47,4\n" QR_CALL("c1") ".Lqr%=r1:\n"                                       \
    QR_WANT("5", L1, ".Lqr%=r2") "s_mov_b32 s54,s47\ns_mov_b32 s47,5\n" QR_CALL("c2") ".Lqr%=r2:\n"
#define QR_LANE_BACK1(L0, L1)                                                                        \
    QR_WANT("4", L0, ".Lqr%=r2") "s_mov_b32 s54,s47\ns_mov_b32 s47,4\n" QR_CALL("c2") ".Lqr%=r2:\n"
// exchanges slots s47 and s54 in the maps and in the registers; then to s[58:59]
#define QR_EXCHANGE                                                                                  \
    "s_lshl2_add_u32 s51,s54,s54\ns_lshl2_add_u32 s52,s47,s47\n"                                     \
    "s_lshr_b32 s53,%[S],s51\ns_lshr_b32 s55,%[S],s52\n"                                             \
    "s_xor_b32 s48,s53,s55\ns_and_b32 s48,s48,31\ns_lshl_b32 s51,s48,s51\ns_lshl_b32 s52,s48,s52\n"   \
    "s_xor_b32 %[S],%[S],s51\ns_xor_b32 %[S],%[S],s52\n"                                             \
    "s_xor_b32 s48,s54,s47\ns_lshl_b32 s53,s48,s53\ns_lshl_b32 s55,s48,s55\n"                        \
    "s_xor_b32 %[W],%[W],s53\ns_xor_b32 %[W],%[W],s55\n"                                             \
    "s_lshl2_add_u32 s51,s47,s54\ns_lshl2_add_u32 s48,s51,s56\ns_addc_u32 s49,s57,0\ns_setpc_b64 s[48:49]\n"
#define QR_WHICH1 "s_mov_b32 s47,4\n"
#define QR_WHICH2 "s_cmp_gt_u32 s45,3\ns_cselect_b32 s47,s45,s46\n"
#define QR_TEXT16(P, BASE, TMP, LS, ANG, L0, L1, R0, R1, R2)                                         \
    QR_HEAD(BASE, TMP, "4+" #LS, "4") QR_START##ANG(P)                                               \
    QR_PC("s_add_u32 s56,s40,.Lqr%=xt-.Lqr%=p\ns_addc_u32 s57,s41,0\n"                                \
          "s_add_u32 s58,s40,.Lqr%=g-.Lqr%=p\ns_addc_u32 s59,s41,0\n"                                 \
          "s_add_u32 s40,s40,.Lqr%=tab-.Lqr%=p\ns_addc_u32 s41,s41,0\n")                              \
    ".macro qrnext%=\n" QR_SCALARS##ANG(P) QR_COUNT("b")                                             \
    "s_lshr_b32 s47,s43,8\ns_bfe_u32 s45,%[W],s43\ns_bfe_u32 s46,%[W],s47\ns_and_b32 s50,s43,0xe0\n"  \
    "v_readlane_b32 s43,%[p],s42\n" /* (past the last gate it only steers a choice) */               \
    QR_GO16 ".endm\nqrnext%=\n"                                                                      \
    /* a wire of the gate in lane slot s47: the register bit s54 it goes to is not the gate's */     \
    /* other wire's nor, if it can be, the next gate's */                                            \
    ".Lqr%=s:\n"                                                                                     \
    "s_lshr_b32 s52,s43,8\ns_bfe_u32 s51,%[W],s43\ns_bfe_u32 s52,%[W],s52\n"                         \
    "s_mov_b32 s53,15\ns_bitset0_b32 s53,s45\ns_bitset0_b32 s53,s46\n"                               \
    "s_mov_b32 s54,s53\ns_bitset0_b32 s54,s51\ns_bitset0_b32 s54,s52\n"                              \
    "s_cmp_lg_u32 s54,0\ns_cselect_b32 s54,s54,s53\ns_ff1_i32_b32 s54,s54\n" QR_WHICH##LS            \
    "s_cmp_eq_u32 s45,s47\ns_cselect_b32 s45,s54,s45\ns_cmp_eq_u32 s46,s47\ns_cselect_b32 s46,s54,s46\n" \
    ".Lqr%=x:\n" QR_EXCHANGE                                                                         \
    ".Lqr%=g:\n" QR_GO16                                                                             \
    ".Lqr%=tab:\n" QR_TABLES##ANG                                                                    \
    ".Lqr%=xt:\n.irp n,0,1,2,3,4,5,6,7,8,9,10,11,12,13,14,15,16,17,18,19,20,21,22,23\n"              \
    ".if ((\\n>>2)>(\\n&3))&((\\n>>2)<4+" #LS ")\ns_branch .Lqr%=v\\n\n.else\ns_branch .Lqr%=e\n.endif\n.endr\n" \
    QR_BODIES16_##ANG(P)                                                                             \
    ".irp n,4,8,9,12,13,14\n.Lqr%=v\\n:\n"                                                           \
    QR_ROWS(16, "(((\\a>>(\\n>>2))&1)==0)&(((\\a>>(\\n&3))&1)==1)",                                  \
            QR_XCH##P("v_swap_b32", QR_A, "\\a+(1<<(\\n>>2))-(1<<(\\n&3))"))                         \
    "s_setpc_b64 s[58:59]\n.endr\n"                                                                  \
    ".irp n,16,17,18,19,20,21,22,23\n.if (\\n>>2)<4+" #LS "\n.Lqr%=v\\n:\n"                          \
    QR_LANE##LS(P, 16, "(\\n>>2)-4", "\\n&3") "s_setpc_b64 s[58:59]\n.endif\n.endr\n"                \
    /* after the last gate */                                                                        \
    ".Lqr%=b:\ns_cmp_eq_u32 %[restore],0\ns_cbranch_scc1 .Lqr%=e\n" QR_LANE_BACK##LS(L0, L1)         \
    QR_WANT("0", R0, ".Lqr%=r3") "s_mov_b32 s54,0\n" QR_CALL("c3") ".Lqr%=r3:\n"                     \
    QR_WANT("1", R1, ".Lqr%=r4") "s_mov_b32 s54,1\n" QR_CALL("c4") ".Lqr%=r4:\n"                     \
    QR_WANT("2", R2, ".Lqr%=e") "s_mov_b32 s54,2\n" QR_CALL("c5")                                    \
    ".Lqr%=e:\n"

// Width 6, 64 registers: the gate's scalars always come with it (CV and CV+
// share a body: A, B = +-1/2, which keeps the bodies within 40 KB of
// instruction cache).
#define QR_TWO64 "1,2,3,4,5,8,10,11,12,13,16,17,19,20,21,24,25,26,28,29,32,33,34,35,37,40,41,42,43,44"
#define QR_ONE64 "0,9,18,27,36,45"
#define QR_UP64 "1,2,3,4,5,10,11,12,13,19,20,21,28,29,37"      /* t < c */
#define QR_B2_64(name, text) QR_BODY(name, QR_TWO64, QR_SETTC text)
#define QR_B1_64(name, text) QR_BODY(name, QR_ONE64, QR_SETTC text)
#define QR_TABU(up, one) QR_TABLE("(\\n>>3)>(\\n&7)", up "\\n", one "\\n")
#define QR_TABLES64_0 QR_TAB("cv", "h") QR_TAB("cx", "t") QR_TAB1("x")
#define QR_TABLES64_1                                                                                \
    QR_TAB("cv", "h") QR_TAB("cx", "t") QR_TABU("zz", "x") QR_TAB1("rx") QR_TAB1("ry") QR_TAB1("rz")
#define QR_TABLES64_2 QR_TAB2("cv") QR_TAB2("cx") QR_TAB1("x") QR_TAB2("cw")
// (the signs of CV and CV+ as factors +-1: A, B)
#define QR_CVROW8S(P)                                                                                \
                QR_SUB##P(QR_T##P(0), QR_X##P(QR_A), QR_X##P(QR_P))                                  \
                QR_SUB##P(QR_T##P(1), QR_Y##P(QR_A), QR_Y##P(QR_P))                                  \
                QR_FMA##P(QR_T##P(2), QR_A##P, QR_T##P(1), QR_T##P(0))                               \
                QR_FMA##P(QR_T##P(3), QR_B##P, QR_T##P(0), QR_T##P(1))                               \
                QR_FMAC##P(QR_X##P(QR_A), "-0.5", QR_T##P(2))                                        \
                QR_FMAC##P(QR_Y##P(QR_A), "-0.5", QR_T##P(3))                                        \
                QR_FMAC##P(QR_X##P(QR_P), "0.5", QR_T##P(2))                                         \
                QR_FMAC##P(QR_Y##P(QR_P), "0.5", QR_T##P(3))
#define QR_BODIES64_2                                                                                \
    QR_B2_64("cv", QR_CV(32, 64, QR_A32, QR_B32)) QR_B2_64("cx", QR_CNOT(32, 64))                    \
    QR_B2_64("cw", QR_ROWS2(64, QR_CVROW8S(32))) QR_B1_64("x", QR_NOT(32, 64))
#define QR_BODIES64_0                                                                                \
    QR_B2_64("cv", QR_CV(32, 64, QR_A32, QR_B32)) QR_B2_64("cx", QR_CNOT(32, 64))                    \
    QR_B1_64("h", QR_H(32, 64)) QR_B1_64("t", QR_TG(32, 64)) QR_B1_64("x", QR_NOT(32, 64))
#define QR_BODIES64_1                                                                                \
    QR_BODIES64_0 QR_BODY("zz", QR_UP64, QR_SETTC QR_ZZ(32, 64)) QR_B1_64("rx", QR_RX(32, 64))                        \
    QR_B1_64("ry", QR_RY(32, 64)) QR_B1_64("rz", QR_RZ(32, 64))
#define QR_TEXT64(ANG)                                                                               \
    QR_HEAD("16", "144", "6", "8") QR_PC("s_add_u32 s40,s40,.Lqr%=tab-.Lqr%=p\ns_addc_u32 s41,s41,0\n") \
    ".macro qrnext%=\n" QR_ANGLE32 QR_ENTRY ".endm\nqrnext%=\n"                                      \
    ".Lqr%=tab:\n" QR_TABLES64_##ANG QR_BODIES64_##ANG ".Lqr%=e:\n"

#define QR_CLOBBER                                                                                   \
    "scc", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", "s48", "s49", "s50", "s51", "s52", \
        "s53", "s54", "s55", "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63"

// A wave-uniform value, into a scalar register.
__device__ __forceinline__ uint32_t scalar(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

// A chunk's cnt gates: words in p (gate i in lane (i - 1 - cnt) mod 64), with angles the
// gates' scalars (cos, sin of theta / 2; 1 / sqrt 2 for H and T) in gc, gs.
// restore: leaves the slots in canonical order (slot: row bit; lane slot s:
// row bit s, register bit k: row bit LS + k).  Every lane is active.
template <int NQ, int GATES>
__device__ __forceinline__ void reg_gates(f32x8& x, uint32_t p, uint32_t cnt, float gc, float gs, SlotMap&, bool) {
    static_assert(NQ == 4, "4 registers: width 4");
    cnt = scalar(cnt);
    if constexpr (GATES == GATES_ANGLED)
        asm volatile(QR_TEXT4(32, "16", "24", 1)
                     : "+{v[16:23]}"(x) : [p] "v"(p), [cnt] "s"(cnt), [gc] "v"(gc), [gs] "v"(gs)
                     : QR_CLOBBER, "v24", "v25", "v26", "v27");
    else if constexpr (GATES == GATES_SAMPLED)
        asm volatile(QR_TEXT4(32, "16", "24", 2)
                     : "+{v[16:23]}"(x) : [p] "v"(p), [cnt] "s"(cnt)
                     : QR_CLOBBER, "v24", "v25", "v26", "v27");
    else
        asm volatile(QR_TEXT4(32, "16", "24", 0)
                     : "+{v[16:23]}"(x) : [p] "v"(p), [cnt] "s"(cnt)
                     : QR_CLOBBER, "v24", "v25", "v26", "v27");
}
template <int NQ, int GATES>
__device__ __forceinline__ void reg_gates(f32x128& x, uint32_t p, uint32_t cnt, float gc, float gs, SlotMap&, bool) {
    static_assert(NQ == 6, "64 registers: width 6");
    cnt = scalar(cnt);
#define QR_ASM64C(ANG_)                                                                              \
    asm volatile(QR_TEXT64(ANG_)                                                                     \
                 : "+{v[16:47]}"(x.a), "+{v[48:79]}"(x.b), "+{v[80:111]}"(x.c), "+{v[112:143]}"(x.d) \
                 : [p] "v"(p), [cnt] "s"(cnt), [gc] "v"(gc), [gs] "v"(gs)                            \
                 : QR_CLOBBER, "v144", "v145", "v146", "v147")
    if constexpr (GATES == GATES_ANGLED) QR_ASM64C(1);
    else if constexpr (GATES == GATES_SAMPLED) QR_ASM64C(2);
    else QR_ASM64C(0);
#undef QR_ASM64C
}
template <int NQ, int GATES>
__device__ __forceinline__ void reg_gates(f64x8& x, uint32_t p, uint32_t cnt, double gc, double gs, SlotMap&, bool) {
    static_assert(NQ == 4, "4 registers: width 4");
    cnt = scalar(cnt);
    if constexpr (GATES == GATES_ANGLED)
        asm volatile(QR_TEXT4(64, "16", "32", 1)
                     : "+{v[16:31]}"(x)
                     : [p] "v"(p), [cnt] "s"(cnt), [gcl] "v"(__double2loint(gc)), [gch] "v"(__double2hiint(gc)),
                       [gsl] "v"(__double2loint(gs)), [gsh] "v"(__double2hiint(gs))
                     : QR_CLOBBER, "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39");
    else
        asm volatile(QR_TEXT4(64, "16", "32", 0)
                     : "+{v[16:31]}"(x) : [p] "v"(p), [cnt] "s"(cnt)
                     : QR_CLOBBER, "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39");
}
// (row bit b is wire NQ - 1 - b)
#define QR_W5(P, TMP, ANG) QR_TEXT16(P, "16", TMP, 1, ANG, "4", "", "3", "2", "1")
#define QR_W6(P, TMP, ANG) QR_TEXT16(P, "16", TMP, 2, ANG, "5", "4", "3", "2", "1")
template <int NQ, int GATES>
__device__ __forceinline__ void reg_gates(f32x32& x, uint32_t p, uint32_t cnt, float gc, float gs, SlotMap& map,
                                          bool restore) {
    const uint32_t rs = scalar(restore ? 1u : 0u);
    uint32_t w2s = scalar(map.w2s), s2w = scalar(map.s2w);
    cnt = scalar(cnt);
#define QR_ASM32(TEXT, ANG)                                                                          \
    asm volatile(TEXT(32, "48", ANG)                                                                 \
                 : "+{v[16:47]}"(x), [W] "+s"(w2s), [S] "+s"(s2w)                            \
                 : [p] "v"(p), [cnt] "s"(cnt), [restore] "s"(rs), [gc] "v"(gc), [gs] "v"(gs) \
                 : QR_CLOBBER, "v48", "v49", "v50", "v51")
    if constexpr (NQ == 5) {
        if constexpr (GATES == GATES_ANGLED) QR_ASM32(QR_W5, 1);
        else if constexpr (GATES == GATES_SAMPLED) QR_ASM32(QR_W5, 2);
        else QR_ASM32(QR_W5, 0);
    } else {
        if constexpr (GATES == GATES_ANGLED) QR_ASM32(QR_W6, 1);
        else if constexpr (GATES == GATES_SAMPLED) QR_ASM32(QR_W6, 2);
        else QR_ASM32(QR_W6, 0);
    }
#undef QR_ASM32
    map.w2s = w2s;
    map.s2w = s2w;
}
template <int NQ, int GATES>
__device__ __forceinline__ void reg_gates(f64x32& x, uint32_t p, uint32_t cnt, double gc, double gs, SlotMap& map,
                                          bool restore) {
    const uint32_t rs = scalar(restore ? 1u : 0u);
    uint32_t w2s = scalar(map.w2s), s2w = scalar(map.s2w);
    cnt = scalar(cnt);
#define QR_ASM64(TEXT, ANG)                                                                          \
    asm volatile(TEXT(64, "80", ANG)                                                                 \
                 : "+{v[16:47]}"(x.lo), "+{v[48:79]}"(x.hi), [W] "+s"(w2s), [S] "+s"(s2w)    \
                 : [p] "v"(p), [cnt] "s"(cnt), [restore] "s"(rs),                        \
                   [gcl] "v"(__double2loint(gc)), [gch] "v"(__double2hiint(gc)),                     \
                   [gsl] "v"(__double2loint(gs)), [gsh] "v"(__double2hiint(gs))                      \
                 : QR_CLOBBER, "v80", "v81", "v82", "v83", "v84", "v85", "v86", "v87")
    if constexpr (NQ == 5) {
        if constexpr (GATES == GATES_ANGLED) QR_ASM64(QR_W5, 1); else QR_ASM64(QR_W5, 0);
    } else {
        if constexpr (GATES == GATES_ANGLED) QR_ASM64(QR_W6, 1); else QR_ASM64(QR_W6, 0);
    }
#undef QR_ASM64
    map.w2s = w2s;
    map.s2w = s2w;
}

}  // namespace qe
