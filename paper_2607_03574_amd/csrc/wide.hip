// Wide replay kernel: forward replay and reverse sweep of a program, one
// thread per lane, with matrices four (Section 3.5: one structural walk, numeric payloads
// widened over the batch axis).  The program format and its reasons are in
// wide.h.
//
// The interpreter is one inline-asm block: the compiler cannot express the
// VGPR index mode over a file of this size, nor keep the double-buffered
// program words in fixed scalar registers.  Library functions are compiled as
// ordinary device functions, which the interpreter calls by the platform's
// calling convention (arguments in v[0:1], v[2:3], ..., result in v[0:1],
// return address in s[30:31]; they may change v0-v38, matrix functions v0-v94, s0-s25 and vcc).  The
// compiled parts are held below the interpreter's registers by
// amdgpu_num_vgpr (counted in pairs of architectural and accumulation
// registers: 20 is 40 vector registers).
#include <hip/hip_runtime.h>

#include <mutex>

#include "../../include/ndvm.h"
#include "slot.h"
#include "wide.h"
#include "wide_exec.h"

namespace ndvm {
namespace {

#define AS_GLOBAL __attribute__((address_space(1)))
#define AS_CONST __attribute__((address_space(4)))

// Scalar registers: bytes of a checkpoint row s26, code base s[28:29], program
// s[34:35], the halves of the program buffer s[36:67] and s[68:99], jump
// target s[100:101]; vcc is scratch.
// Vector registers: temporaries v0 - v39 (matrices: v95); addresses of this
// lane's checkpoint column PCK, observations POB, loss PLO and gradient PGR;
// the file from F on.  The two kernels define these names (below).
#define T "v[0:1]"
#define U "v[2:3]"
// a class's code in one half: a region of kRegion bytes (too long a text does not assemble)
#define REGION(text) "77:\n" text ".skip 1024-(.-77b)\n"
// operand access: M0 from the low or high half of word k of the micro-op
#define LO(k) "s_mov_b32 m0, s[wq+" #k "]\n"
#define HI(k) "s_lshr_b32 m0, s[wq+" #k "], 16\n"
#define MOV(d, s) "v_mov_b64 " d ", " s "\n"
// End of a block in one half: block b + 1's words have landed in the other
// half; this half receives block b + 2's.
#define DISPATCH_A \
    "s_waitcnt lgkmcnt(0)\ns_add_u32 s100, s28, s66\ns_addc_u32 s101, s29, 0\n" \
    "s_load_dwordx16 s[36:51], s[34:35], s67\ns_load_dwordx16 s[52:67], s[34:35], s67 offset:0x40\n" \
    "s_setpc_b64 s[100:101]\n"
#define DISPATCH_B \
    "s_waitcnt lgkmcnt(0)\ns_add_u32 s100, s28, s98\ns_addc_u32 s101, s29, 0\n" \
    "s_load_dwordx16 s[68:83], s[34:35], s99\ns_load_dwordx16 s[84:99], s[34:35], s99 offset:0x40\n" \
    "s_setpc_b64 s[100:101]\n"
// n micro-ops of w words, the last ending at the word before the headers
#define BODY(end, n, w, text) ".set wq, " #end "-" #n "*" #w "\n.rept " #n "\n" text ".set wq, wq+" #w "\n.endr\n"
#define CLASS(first, n, w, text) \
    REGION(first BODY(66, n, w, text) DISPATCH_A) REGION(first BODY(98, n, w, text) DISPATCH_B)

#define FMA_TEXT LO(0) MOV(T, F) HI(0) "v_mul_f64 " T ", " F ", " T "\n" \
    LO(1) "v_add_f64 " T ", " F ", " T "\n" HI(1) MOV(F, T)
#define DUAL_TEXT \
    LO(0) MOV(T, F) HI(0) MOV(F, "0") "v_cmpx_neq_f64_e32 vcc, 0, " T "\n" \
    LO(1) "v_mul_f64 " U ", " F ", " T "\n" HI(1) "v_add_f64 " F ", " F ", " U "\n" \
    LO(2) "v_mul_f64 " U ", " F ", " T "\n" HI(2) "v_add_f64 " F ", " F ", " U "\n" \
    "s_mov_b64 exec, -1\n"
#define SEL_TEXT \
    LO(0) MOV(T, F) HI(0) "v_cmp_gt_f64_e32 vcc, " F ", " T "\n" LO(1) MOV(U, F) \
    HI(1) "v_cndmask_b32_e32 v0, " FLO ", v2, vcc\nv_cndmask_b32_e32 v1, " FHI ", v3, vcc\n" LO(2) MOV(F, T)
#define SELADJ_TEXT \
    LO(0) MOV(T, F) HI(0) MOV(F, "0") LO(1) MOV(U, F) HI(1) "v_cmpx_gt_f64_e32 vcc, " F ", " U "\n" \
    LO(2) "v_add_f64 " F ", " F ", " T "\n" "s_not_b64 exec, exec\n" \
    HI(2) "v_add_f64 " F ", " F ", " T "\n" "s_mov_b64 exec, -1\n"
// q = n / d by the division instructions (scaled reciprocal, two Newton
// steps, one correction, unscaling and fix-up); v[10:17] are scratch.  M0 must
// apply to no operand.
#define DIVIDE(q, n, d) \
    "v_div_scale_f64 v[10:11], vcc, " d ", " d ", " n "\nv_rcp_f64_e32 v[12:13], v[10:11]\n" \
    "v_div_scale_f64 v[14:15], vcc, " n ", " d ", " n "\nv_fma_f64 v[16:17], -v[10:11], v[12:13], 1.0\n" \
    "v_fma_f64 v[12:13], v[12:13], v[16:17], v[12:13]\nv_fma_f64 v[16:17], -v[10:11], v[12:13], 1.0\n" \
    "v_fma_f64 v[12:13], v[12:13], v[16:17], v[12:13]\nv_mul_f64 v[16:17], v[14:15], v[12:13]\n" \
    "v_fma_f64 v[10:11], -v[10:11], v[16:17], v[14:15]\n" \
    "v_div_fmas_f64 v[10:11], v[10:11], v[12:13], v[16:17]\nv_div_fixup_f64 " q ", v[10:11], " d ", " n "\n"
#define DIV_TEXT LO(0) MOV(T, F) HI(0) MOV(U, F) "s_mov_b32 m0, 0\n" DIVIDE("v[0:1]", "v[0:1]", "v[2:3]") LO(1) MOV(F, T)
#define DIVADJ_TEXT \
    LO(0) MOV(T, F) HI(0) MOV(F, "0") LO(1) MOV(U, F) LO(2) "v_mul_f64 v[4:5], " F ", " T "\n" "s_mov_b32 m0, 0\n" \
    DIVIDE("v[6:7]", "v[0:1]", "v[2:3]") DIVIDE("v[4:5]", "v[4:5]", "v[2:3]") \
    "v_cmpx_neq_f64_e32 vcc, 0, " T "\n" HI(1) "v_add_f64 " F ", " F ", v[6:7]\n" \
    HI(2) "v_add_f64 " F ", " F ", -v[4:5]\n" "s_mov_b64 exec, -1\n"
#define ACCD_TEXT \
    LO(0) MOV(T, F) HI(0) MOV(F, "0") LO(1) MOV(U, F) LO(2) MOV("v[4:5]", F) "s_mov_b32 m0, 0\n" \
    DIVIDE("v[4:5]", "v[4:5]", "v[2:3]") "v_cmpx_neq_f64_e32 vcc, 0, " T "\n" \
    HI(1) "v_add_f64 " F ", " F ", v[4:5]\n" "s_mov_b64 exec, -1\n"
// v[2:3] = address of a checkpoint row in this lane's column
#define ROWADDR(k) "s_mul_i32 vcc_lo, s[wq+" #k "], s26\ns_mul_hi_u32 vcc_hi, s[wq+" #k "], s26\nv_lshl_add_u64 " U ", vcc, 0, " PCK "\n"
#define CKST_TEXT LO(0) MOV(T, F) ROWADDR(1) "global_store_dwordx2 " U ", " T ", off\n"
// (M0 still holds the roles of the operand accessed last, which would apply
// to the address: no role here)
#define LDK_TEXT "s_mov_b32 m0, 0\n" ROWADDR(0) "global_load_dwordx2 v[vq:vq+1], " U ", off\n.set vq, vq+2\n"
#define LDO_TEXT "s_mov_b32 m0, 0\ns_mov_b32 vcc_lo, s[wq]\ns_mov_b32 vcc_hi, 0\nv_lshl_add_u64 " U ", vcc, 0, " POB "\n" \
    "global_load_dwordx2 v[vq:vq+1], " U ", off\n.set vq, vq+2\n"
// a line of the program per thread (into PDUMP, the temporary that no function
// uses: a load may land at any time)
#define PF_TEXT "s_mov_b32 m0, 0\nv_mbcnt_lo_u32_b32 v2, -1, 0\nv_mbcnt_hi_u32_b32 v2, -1, v2\nv_lshlrev_b32 v2, 6, v2\n" \
    "v_add_u32 v2, s[wq], v2\nglobal_load_dword " PDUMP ", v2, s[34:35]\n"
#define LOADS(reg, n, text) \
    REGION(".set vq, " FBASE "+" #reg "\n" BODY(66, n, 1, text) DISPATCH_A) \
    REGION(".set vq, " FBASE "+" #reg "\n" BODY(98, n, 1, text) DISPATCH_B)
#define STLOSS_TEXT LO(0) MOV(T, F) "global_store_dwordx2 " PLO ", " T ", off\n"
#define STGRAD_TEXT LO(0) MOV(T, F) "s_mov_b32 vcc_lo, s[wq+1]\ns_mov_b32 vcc_hi, 0\nv_lshl_add_u64 " U ", vcc, 0, " PGR "\n" \
    "global_store_dwordx2 " U ", " T ", off\n"
// Call of a library function, past its first instruction: a function begins
// with a wait for every outstanding load (4 bytes), which its arguments, all
// computed here, do not need and which would end the loads issued ahead.
#define CALL(f) "s_set_gpr_idx_off\n" CALL_ONLY(f)
#define CALL_ONLY(f) \
    "s_getpc_b64 s[100:101]\ns_add_u32 s100, s100, " f "@rel32@lo+8\n" \
    "s_addc_u32 s101, s101, " f "@rel32@hi+16\ns_swappc_b64 s[30:31], s[100:101]\n"
#define RESULT_LO(k) "s_set_gpr_idx_on s[wq+" #k "], 0x8\n" MOV(F, T)
#define RESULT_HI(k) "s_lshr_b32 vcc_lo, s[wq+" #k "], 16\ns_set_gpr_idx_on vcc_lo, 0x8\n" MOV(F, T)
#define CALL1(f) CLASS("", 10, 1, LO(0) MOV("v[0:1]", F) CALL(f) RESULT_HI(0))
#define CALL2(f) CLASS("", 10, 2, LO(0) MOV("v[0:1]", F) HI(0) MOV("v[2:3]", F) CALL(f) RESULT_LO(1))
#define CALL3(f) \
    CLASS("", 10, 2, LO(0) MOV("v[0:1]", F) HI(0) MOV("v[2:3]", F) LO(1) MOV("v[4:5]", F) CALL(f) RESULT_HI(1))
#define CALL4(f) \
    CLASS("", 10, 3, LO(0) MOV("v[0:1]", F) HI(0) MOV("v[2:3]", F) LO(1) MOV("v[4:5]", F) HI(1) MOV("v[6:7]", F) \
          CALL(f) RESULT_LO(2))

// ---- matrices: LDS address of a matrix (a word of the micro-op) for this
// lane, and for this lane's thread's element of a quad
#define ADDR(v, k) "v_add_u32 v" #v ", s[wq+" #k "], v104\n"
#define ADDR4(v, k) "v_add_u32 v" #v ", s[wq+" #k "], v105\n"
#define STE_TEXT LO(0) MOV(T, F) ADDR(2, 1) "ds_write_b64 v2, " T "\n"
#define STE4_TEXT LO(0) MOV(T, F) ADDR4(2, 1) "ds_write_b64 v2, " T "\n"
#define LDE_TEXT "s_mov_b32 m0, 0\n" ADDR(2, 0) "ds_read_b64 " T ", v2\ns_waitcnt lgkmcnt(0)\n" LO(1) MOV(F, T)
#define CKSTM_TEXT "s_mov_b32 m0, 0\n" ADDR4(2, 0) "ds_read_b64 " T ", v2\n" ROWADDR(1) "s_waitcnt lgkmcnt(0)\n" \
    "global_store_dwordx2 " U ", " T ", off\n"
// calls with three matrices, and with two, a scalar and a scalar result; the
// immediate in s27
#define CALLM(f) \
    CLASS("", 7, 4, "s_set_gpr_idx_off\n" ADDR(0, 0) ADDR(1, 1) ADDR(2, 2) "s_mov_b32 s27, s[wq+3]\n" CALL_ONLY(f) \
          "s_set_gpr_idx_on s26, 0x0\n")
#define CALLS(f) \
    CLASS("", 7, 4, LO(3) MOV("v[2:3]", F) "s_set_gpr_idx_off\n" ADDR(0, 0) ADDR(1, 1) "s_mov_b32 s27, s[wq+2]\n" \
          CALL_ONLY(f) RESULT_HI(3))

}  // namespace

// Library functions (C linkage: the interpreter names them).  None uses
// scratch memory: the interpreter sets up no stack.
#define NDVM_WIDE_FN \
    extern "C" __device__ __attribute__((used, noinline, visibility("hidden"))) double
NDVM_WIDE_FN ndvm_wide_exp(double x) { return exp(x); }
NDVM_WIDE_FN ndvm_wide_sin(double x) { return sin(x); }
NDVM_WIDE_FN ndvm_wide_cos(double x) { return cos(x); }
NDVM_WIDE_FN ndvm_wide_logc(double x) { return wide::f_logc(x); }
NDVM_WIDE_FN ndvm_wide_sqrtc(double x) { return wide::f_sqrtc(x); }
NDVM_WIDE_FN ndvm_wide_pow(double x, double y) { return pow(x, y); }
NDVM_WIDE_FN ndvm_wide_accsin(double x, double y, double w) { return wide::f_accsin(x, y, w); }
NDVM_WIDE_FN ndvm_wide_acccos(double x, double y, double w) { return wide::f_acccos(x, y, w); }
NDVM_WIDE_FN ndvm_wide_acclog(double x, double y, double w) { return wide::f_acclog(x, y, w); }
NDVM_WIDE_FN ndvm_wide_accabs(double x, double y, double w) { return wide::f_accabs(x, y, w); }
NDVM_WIDE_FN ndvm_wide_accpow(double x, double y, double z, double w) { return wide::f_accpow(x, y, z, w); }
NDVM_WIDE_FN ndvm_wide_accsqrt(double x, double y, double z, double w) { return wide::f_accsqrt(x, y, z, w); }
NDVM_WIDE_FN ndvm_wide_abs(double x) { return fabs(x); }

// ---- matrix functions: a lane's four threads (t / 16) take a row each, or
// every fourth element; a thread past the last row repeats it (the same values
// to the same places).  Past the first instruction of a function only its own
// LDS operations and scalar loads of the program are in flight; a wait for all
// but the n newest of both covers the function's older ones.
namespace {
struct LdsMem {
    __device__ __forceinline__ double ld(uint32_t p, uint32_t e) const {
        return *(__attribute__((address_space(3))) double *)(size_t)(p + e * wide::kLdsRow);
    }
    __device__ __forceinline__ void st(uint32_t p, uint32_t e, double v) const {
        *(__attribute__((address_space(3))) double *)(size_t)(p + e * wide::kLdsRow) = v;
    }
};
__device__ __forceinline__ uint32_t lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }
__device__ __forceinline__ uint32_t quarter() { return lane_id() >> 4; }
__device__ __forceinline__ uint32_t immediate() {
    uint32_t v;
    asm volatile("s_mov_b32 %0, s27" : "=s"(v));
    return v;
}
// whether any of a lane's four threads has `b`
__device__ __forceinline__ bool any_of_lane(bool b) {
    const uint64_t m = __ballot(b);
    uint32_t f = uint32_t(m) | uint32_t(m >> 32);
    f |= f >> 16;
    return (f >> (lane_id() & 15u)) & 1u;
}
}  // namespace
#define NDVM_WIDE_MATRIX extern "C" __device__ __attribute__((used, noinline, visibility("hidden")))
NDVM_WIDE_MATRIX void ndvm_wide_mm(uint32_t a, uint32_t b, uint32_t d) {
    const uint32_t im = immediate(), m = im & 7u, k = (im >> 3) & 7u, n = (im >> 6) & 7u, r = min(quarter(), m - 1);
#define ROW(K, N) wide::mm_row<K, N>(LdsMem{}, a, b, d, r)
    NDVM_WIDE_SIDES(k, n, ROW)
#undef ROW
}
NDVM_WIDE_MATRIX void ndvm_wide_mma(uint32_t g, uint32_t b, uint32_t t) {
    const uint32_t im = immediate(), m = im & 7u, k = (im >> 3) & 7u, n = (im >> 6) & 7u, r = min(quarter(), m - 1);
    const bool first = im & wide::kFirstBit;
#define ROW(K, N) wide::mma_row<K, N>(LdsMem{}, g, b, t, r, first, any_of_lane)
    NDVM_WIDE_SIDES(k, n, ROW)
#undef ROW
}
NDVM_WIDE_MATRIX void ndvm_wide_mmb(uint32_t a, uint32_t g, uint32_t t) {
    const uint32_t im = immediate(), m = im & 7u, k = (im >> 3) & 7u, n = (im >> 6) & 7u, p = min(quarter(), k - 1);
    const bool first = im & wide::kFirstBit;
#define ROW(M, N) wide::mmb_row<M, N>(LdsMem{}, a, g, t, p, k, first)
    NDVM_WIDE_SIDES(m, n, ROW)
#undef ROW
}
NDVM_WIDE_MATRIX void ndvm_wide_vadd(uint32_t a, uint32_t b, uint32_t d) {
    wide::vadd(LdsMem{}, a, b, d, quarter(), immediate());
}
NDVM_WIDE_MATRIX void ndvm_wide_vacc(uint32_t g, uint32_t, uint32_t t) {
    wide::vacc(LdsMem{}, g, t, quarter(), immediate());
}
NDVM_WIDE_MATRIX void ndvm_wide_trans(uint32_t a, uint32_t, uint32_t d) {
    wide::transpose(LdsMem{}, a, d, quarter(), immediate());
}
NDVM_WIDE_MATRIX void ndvm_wide_transacc(uint32_t g, uint32_t, uint32_t t) {
    wide::transpose_acc(LdsMem{}, g, t, quarter(), immediate());
}
NDVM_WIDE_MATRIX void ndvm_wide_inv2(uint32_t a, uint32_t, uint32_t d) { wide::inv2(LdsMem{}, a, d); }
NDVM_WIDE_MATRIX void ndvm_wide_inv2acc(uint32_t z, uint32_t g, uint32_t t) {
    wide::inv2_acc(LdsMem{}, z, g, t, immediate());
}
NDVM_WIDE_MATRIX double ndvm_wide_vscale(uint32_t a, uint32_t d, double s) {
    wide::vscale(LdsMem{}, a, d, s, quarter(), immediate());
    return 0.0;
}
NDVM_WIDE_MATRIX double ndvm_wide_vaccs(uint32_t g, uint32_t t, double s) {
    const uint32_t im = immediate(), n = im & 511u;
    wide::vaccs(LdsMem{}, g, t, s, quarter(), n, im & wide::kFirstBit, wide::any_of(LdsMem{}, g, n));
    return 0.0;
}
NDVM_WIDE_MATRIX double ndvm_wide_sdot(uint32_t g, uint32_t a, double) { return wide::sdot(LdsMem{}, g, a, immediate()); }
NDVM_WIDE_MATRIX double ndvm_wide_det2(uint32_t a, uint32_t, double) {
    double v[4];
    wide::load4(LdsMem{}, a, v);
    return wide::det2(v);
}
NDVM_WIDE_MATRIX double ndvm_wide_logdetacc(uint32_t a, uint32_t t, double g) {
    wide::logdet2_acc(LdsMem{}, a, t, g, immediate());
    return 0.0;
}

// The interpreter's start and its classes' code (order of wide::Class).
#define START \
    "s_load_dwordx16 s[36:51], s[34:35], s100\ns_load_dwordx16 s[52:67], s[34:35], s100 offset:0x40\n" \
    "s_getpc_b64 s[28:29]\n.Lpc%=:\ns_add_u32 s28, s28, .Lbase%=-.Lpc%=\ns_addc_u32 s29, s29, 0\n" \
    "s_set_gpr_idx_on s26, 0x0\n" DISPATCH_B ".p2align 8\n.Lbase%=:\n"
#define SCALAR_CLASSES \
    CLASS("", 15, 2, FMA_TEXT) \
    CLASS("", 10, 3, DUAL_TEXT) \
    CLASS("", 10, 3, SEL_TEXT) \
    CLASS("", 10, 3, SELADJ_TEXT) \
    CLASS("", 8, 2, DIV_TEXT) \
    CLASS("", 4, 3, DIVADJ_TEXT) \
    CLASS("", 6, 3, ACCD_TEXT) \
    CLASS("", 15, 2, CKST_TEXT) \
    LOADS(16, 12, LDK_TEXT) \
    LOADS(40, 12, LDK_TEXT) \
    LOADS(0, 4, LDO_TEXT) \
    LOADS(8, 4, LDO_TEXT) \
    REGION("s_waitcnt vmcnt(0)\n" DISPATCH_A) REGION("s_waitcnt vmcnt(0)\n" DISPATCH_B) \
    CLASS("s_waitcnt vmcnt(0)\n", 1, 1, PF_TEXT) \
    CLASS("", 2, 1, PF_TEXT) \
    CLASS("", 1, 1, STLOSS_TEXT) \
    CLASS("", 8, 2, STGRAD_TEXT) \
    CALL1("ndvm_wide_exp") \
    CALL1("ndvm_wide_sin") \
    CALL1("ndvm_wide_cos") \
    CALL1("ndvm_wide_logc") \
    CALL1("ndvm_wide_sqrtc") \
    CALL2("ndvm_wide_pow") \
    CALL3("ndvm_wide_accsin") \
    CALL3("ndvm_wide_acccos") \
    CALL3("ndvm_wide_acclog") \
    CALL3("ndvm_wide_accabs") \
    CALL4("ndvm_wide_accpow") \
    CALL4("ndvm_wide_accsqrt") \
    CALL1("ndvm_wide_abs") \
    REGION("s_branch .Lend%=\n") REGION("s_branch .Lend%=\n")
#define MATRIX_CLASSES \
    CLASS("", 15, 2, STE_TEXT) \
    CLASS("", 15, 2, STE4_TEXT) \
    CLASS("", 15, 2, LDE_TEXT) \
    CLASS("", 15, 2, CKSTM_TEXT) \
    CALLM("ndvm_wide_mm") \
    CALLM("ndvm_wide_mma") \
    CALLM("ndvm_wide_mmb") \
    CALLM("ndvm_wide_vadd") \
    CALLM("ndvm_wide_vacc") \
    CALLM("ndvm_wide_trans") \
    CALLM("ndvm_wide_transacc") \
    CALLM("ndvm_wide_inv2") \
    CALLM("ndvm_wide_inv2acc") \
    CALLS("ndvm_wide_vscale") \
    CALLS("ndvm_wide_vaccs") \
    CALLS("ndvm_wide_sdot") \
    CALLS("ndvm_wide_det2") \
    CALLS("ndvm_wide_logdetacc")
#define FINISH ".Lend%=:\ns_set_gpr_idx_off\ns_waitcnt vmcnt(0) lgkmcnt(0)\n"
#define CLOBBERS \
    "s0", "s1", "s2", "s3", "s4", "s5", "s6", "s7", "s8", "s9", "s10", "s11", "s12", "s13", "s14", "s15", "s16", \
    "s17", "s18", "s19", "s20", "s21", "s22", "s23", "s24", "s25", "s26", "s28", "s29", "s30", "s31", "s34", \
    "s101", "m0", "vcc", "scc", "memory", "v0", "v39", "v255"

// Prologue of a workgroup: its program, the scalar registers of the
// interpreter; false: no work.
struct Item {
    wide::Prog D;
    uint32_t q, bx;
};
__device__ __forceinline__ bool item_of(const LaunchArgs &A, const wide::Prog *table, const wide::Prog &single, Item &w) {
    w.q = blockIdx.y;
    w.bx = blockIdx.x;
    if (A.wg_items) {
        const uint64_t it = A.wg_items[blockIdx.x];
        if (it == ~uint64_t(0)) return false;
        w.q = uint32_t(it >> 32);
        w.bx = uint32_t(it);
    }
    w.D = table ? table[w.q] : single;
    return true;
}
__device__ __forceinline__ void set_scalars(const LaunchArgs &A, const wide::Prog &D, uint32_t pitch) {
    asm volatile("s_mov_b32 s26, %[pitch]\ns_mov_b64 s[34:35], %[code]\n"
                 "s_mov_b32 s100, %[f0]\ns_mov_b32 s98, %[f1]\ns_mov_b32 s99, %[f2]\n" ::[pitch] "s"(pitch),
                 [code] "s"(uint64_t(size_t(D.code))), [f0] "s"(D.first[0]), [f1] "s"(D.first[1]), [f2] "s"(D.first[2])
                 : "s26", "s34", "s35", "s98", "s99", "s100", "scc");
}
// static registers through set(register, value): parameters, their adjoints
// (+0), the sink, constants
template <class S>
__device__ __forceinline__ void set_statics(const LaunchArgs &A, const Item &w, int64_t lc, S set) {
    const AS_GLOBAL double *prow =
        (const AS_GLOBAL double *)(A.params + int64_t(w.q) * A.prog_stride_p) + lc * A.ld_p;
    const uint32_t P = w.D.n_params;
    uint32_t r = wide::kSlots;
    for (uint32_t p = 0; p < P; p += 4) {
        double v[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) v[i] = prow[p + i < P ? p + i : P - 1];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i)
            if (p + i < P) set(r + p + i, v[i]);
    }
    r += P;
    const uint32_t zeros = (w.D.adjoints ? P : 0) + 1;
    for (uint32_t i = 0; i < zeros; ++i) set(r + i, 0.0);
    r += zeros;
    const AS_CONST double *cs = (const AS_CONST double *)w.D.consts;
    for (uint32_t i = 0; i < w.D.n_consts; ++i) set(r + i, cs[i]);
}
#define SET_REG(r, v) \
    asm volatile("s_set_gpr_idx_on %[i], 0x8\n" MOV(F, "%[x]") "s_set_gpr_idx_off\n" ::[i] "s"(2 * (r)), [x] "v"(v) \
                 : "m0", "v255")
#define SET_ADDRESS(reg, p) asm volatile(MOV(reg, "%[x]")::[x] "v"(p) : "v255")

#define FBASE "48"
#define F "v[48:49]"
#define FLO "v48"
#define FHI "v49"
#define PCK "v[40:41]"
#define PDUMP "v39"
#define POB "v[42:43]"
#define PLO "v[44:45]"
#define PGR "v[46:47]"
// One wave per workgroup.  Bound by instruction issue: a lone wave issues an
// instruction every 4.5 cycles, so an FMA micro-op takes 32 cycles and a DUAL
// 72 (24 of them for the two changes of EXEC), a block's dispatch 61, a division
// 84, a library call 110 and the function; two waves on a SIMD (256 vector
// registers each) take 1.3 to 1.5 times as long together as one alone.
__global__ void __launch_bounds__(64) __attribute__((amdgpu_num_vgpr(20)))
ndvm_wide(LaunchArgs A, const wide::Prog *__restrict__ table, wide::Prog single) {
    static_assert(wide::kFileBase == 48, "registers named here");
    Item w;
    if (!item_of(A, table, single, w)) return;
    const int64_t lane = int64_t(w.bx) * 64 + threadIdx.x;
    const bool active = lane < A.L;
    int64_t lc = active ? lane : A.L - 1;
    const double *obs = A.obs;
    if (A.n_points > 0) {   // flattened data axis: parameter row and data point of the lane
        obs += (lc % A.n_points) * A.obs_stride;
        lc = lc / A.n_points;
    }
    set_statics(A, w, lc, [](uint32_t r, double v) { SET_REG(r, v); });
    // addresses; the lanes past the last one write to the trash rows
    double *trash = A.ws + int64_t(w.D.trash_row) * A.Lpad + lane;
    SET_ADDRESS(PCK, A.ws + int64_t(w.D.ckpt_row0) * A.Lpad + lane);
    SET_ADDRESS(POB, obs);
    SET_ADDRESS(PLO, active ? A.loss + int64_t(w.q) * A.L + lane : trash);
    SET_ADDRESS(PGR, active && w.D.adjoints ? A.grad + int64_t(w.q) * A.prog_stride_g + lane * A.ld_g : trash);
    set_scalars(A, w.D, uint32_t(A.Lpad * 8));
    // nothing of the compiled part is live from here on
    asm volatile(START SCALAR_CLASSES FINISH ::: CLOBBERS, "v39");
}

#undef FBASE
#undef F
#undef FLO
#undef FHI
#undef PCK
#undef PDUMP
#undef POB
#undef PLO
#undef PGR
#define FBASE "106"
#define F "v[106:107]"
#define FLO "v106"
#define FHI "v107"
#define PCK "v[96:97]"
#define PDUMP "v95"
#define POB "v[98:99]"
#define PLO "v[100:101]"
#define PGR "v[102:103]"
// Programs with matrices: 16 lanes a wave, four threads a lane, matrices in
// LDS (v104: this lane's LDS offset, v105: with its thread's element of a quad).
// Bound by the chain of matrix calls: each waits for LDS (some 130 cycles for
// its first operands) and for fused multiply-adds in a fixed order; a wave has
// the launch's parallelism only through its four rows, and 16,384 lanes are one
// wave per SIMD.  Kalman filter of four states, 200 steps, 16,384 lanes: 6.93 ms
// in the slot kernel, whose slots shared a row's operands through four issues of
// every LDS access, 4.20 here.
__global__ void __launch_bounds__(64) __attribute__((amdgpu_num_vgpr(48)))
ndvm_wide_matrix(LaunchArgs A, const wide::Prog *__restrict__ table, wide::Prog single) {
    static_assert(wide::kMatFileBase == 106, "registers named here");
    Item w;
    if (!item_of(A, table, single, w)) return;
    const uint32_t t = threadIdx.x, quarter = t / wide::kMatLanes;
    const int64_t lane = int64_t(w.bx) * wide::kMatLanes + t % wide::kMatLanes;
    const bool active = lane < A.L;
    int64_t lc = active ? lane : A.L - 1;
    const double *obs = A.obs;
    if (A.n_points > 0) {
        obs += (lc % A.n_points) * A.obs_stride;
        lc = lc / A.n_points;
    }
    set_statics(A, w, lc, [](uint32_t r, double v) { SET_REG(r, v); });
    double *trash = A.ws + int64_t(w.D.trash_row) * A.Lpad + lane;
    SET_ADDRESS(PCK, A.ws + int64_t(w.D.ckpt_row0 + quarter) * A.Lpad + lane);
    SET_ADDRESS(POB, obs);
    SET_ADDRESS(PLO, active ? A.loss + int64_t(w.q) * A.L + lane : trash);
    SET_ADDRESS(PGR, active && w.D.adjoints ? A.grad + int64_t(w.q) * A.prog_stride_g + lane * A.ld_g : trash);
    asm volatile("v_mov_b32 v104, %[a]\nv_mov_b32 v105, %[b]\n" ::[a] "v"(t % wide::kMatLanes * 8), [b] "v"(t * 8)
                 : "v255");
    set_scalars(A, w.D, uint32_t(A.Lpad * 32));
    asm volatile(START SCALAR_CLASSES MATRIX_CLASSES FINISH ::: CLOBBERS, "v95");
}

hipError_t launch_wide(const LaunchArgs &A, const wide::Prog *d_table, const wide::Prog &single, uint32_t n_prog,
                       uint32_t lds_bytes, hipStream_t stream) {
    const uint32_t lanes = lds_bytes ? wide::kMatLanes : 64;
    const dim3 grid = A.wg_items ? dim3(A.n_wg) : dim3(uint32_t((A.L + lanes - 1) / lanes), n_prog);
    if (lds_bytes) {
        static std::once_flag once[64];
        int dev = 0;
        (void)hipGetDevice(&dev);
        std::call_once(once[dev & 63], [dev]() {
            int most = 0;
            (void)hipDeviceGetAttribute(&most, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
            (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&ndvm_wide_matrix),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, most);
        });
        hipLaunchKernelGGL(ndvm_wide_matrix, grid, dim3(64), lds_bytes, stream, A, d_table, single);
    } else {
        hipLaunchKernelGGL(ndvm_wide, grid, dim3(64), 0, stream, A, d_table, single);
    }
    return hipGetLastError();
}

}  // namespace ndvm
