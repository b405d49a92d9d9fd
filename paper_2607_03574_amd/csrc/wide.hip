// Wide replay kernel: forward replay and reverse sweep of a scalar program,
// one thread per lane (Section 3.5: one structural walk, numeric payloads
// widened over the batch axis).  The program format and its reasons are in
// wide.h.
//
// The interpreter is one inline-asm block: the compiler cannot express the
// VGPR index mode over a file of this size, nor keep the double-buffered
// program words in fixed scalar registers.  Library functions are compiled as
// ordinary device functions, which the interpreter calls by the platform's
// calling convention (arguments in v[0:1], v[2:3], ..., result in v[0:1],
// return address in s[30:31]; they may change v0-v39, s0-s29 and vcc).  The
// compiled parts are held below the interpreter's registers by
// amdgpu_num_vgpr (counted in pairs of architectural and accumulation
// registers: 20 is 40 vector registers).
#include <hip/hip_runtime.h>

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
// Vector registers: temporaries v0 - v39; addresses of this lane's checkpoint
// column v[40:41], observations v[42:43], loss v[44:45] and gradient v[46:47];
// the file from v48 on.
#define T "v[0:1]"
#define U "v[2:3]"
#define F "v[48:49]"
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
    HI(1) "v_cndmask_b32_e32 v0, v48, v2, vcc\nv_cndmask_b32_e32 v1, v49, v3, vcc\n" LO(2) MOV(F, T)
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
#define ROW(k) "s_mul_i32 vcc_lo, s[wq+" #k "], s26\ns_mul_hi_u32 vcc_hi, s[wq+" #k "], s26\nv_lshl_add_u64 " U ", vcc, 0, v[40:41]\n"
#define CKST_TEXT LO(0) MOV(T, F) ROW(1) "global_store_dwordx2 " U ", " T ", off\n"
// (M0 still holds the roles of the operand accessed last, which would apply
// to the address: no role here)
#define LDK_TEXT "s_mov_b32 m0, 0\n" ROW(0) "global_load_dwordx2 v[vq:vq+1], " U ", off\n.set vq, vq+2\n"
#define LDO_TEXT "s_mov_b32 m0, 0\ns_mov_b32 vcc_lo, s[wq]\ns_mov_b32 vcc_hi, 0\nv_lshl_add_u64 " U ", vcc, 0, v[42:43]\n" \
    "global_load_dwordx2 v[vq:vq+1], " U ", off\n.set vq, vq+2\n"
// a line of the program per thread (nothing reads v39)
#define PF_TEXT "s_mov_b32 m0, 0\nv_mbcnt_lo_u32_b32 v2, -1, 0\nv_mbcnt_hi_u32_b32 v2, -1, v2\nv_lshlrev_b32 v2, 6, v2\n" \
    "v_add_u32 v2, s[wq], v2\nglobal_load_dword v39, v2, s[34:35]\n"
#define LOADS(reg, n, text) \
    REGION(".set vq, " #reg "\n" BODY(66, n, 1, text) DISPATCH_A) REGION(".set vq, " #reg "\n" BODY(98, n, 1, text) DISPATCH_B)
#define STLOSS_TEXT LO(0) MOV(T, F) "global_store_dwordx2 v[44:45], " T ", off\n"
#define STGRAD_TEXT LO(0) MOV(T, F) "s_mov_b32 vcc_lo, s[wq+1]\ns_mov_b32 vcc_hi, 0\nv_lshl_add_u64 " U ", vcc, 0, v[46:47]\n" \
    "global_store_dwordx2 " U ", " T ", off\n"
// Call of a library function, past its first instruction: a function begins
// with a wait for every outstanding load (4 bytes), which its arguments, all
// computed here, do not need and which would end the loads issued ahead.
#define CALL(f) \
    "s_set_gpr_idx_off\ns_getpc_b64 s[100:101]\ns_add_u32 s100, s100, " f "@rel32@lo+8\n" \
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

// The file register `r` = v (prologue).
__device__ __forceinline__ void set_reg(uint32_t r, double v) {
    asm volatile("s_set_gpr_idx_on %[i], 0x8\n" MOV(F, "%[v]") "s_set_gpr_idx_off\n" ::[i] "s"(2 * r), [v] "v"(v)
                 : "m0", "v255");
}

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

// One wave per workgroup.  Bound by instruction issue: a lone wave issues an
// instruction every 4.5 cycles, so an FMA micro-op takes 32 cycles and a DUAL
// 72 (24 of them for the two changes of EXEC), a block's dispatch 61, a division
// 84, a library call 110 and the function; two waves on a SIMD (256 vector
// registers each) take 1.3 to 1.5 times as long together as one alone.
__global__ void __launch_bounds__(64) __attribute__((amdgpu_num_vgpr(20)))
ndvm_wide(LaunchArgs A, const wide::Prog *__restrict__ table, wide::Prog single) {
    uint32_t q = blockIdx.y, bx = blockIdx.x;
    if (A.wg_items) {
        const uint64_t it = A.wg_items[blockIdx.x];
        if (it == ~uint64_t(0)) return;
        q = uint32_t(it >> 32);
        bx = uint32_t(it);
    }
    const wide::Prog D = table ? table[q] : single;
    const int64_t lane = int64_t(bx) * 64 + threadIdx.x;
    const bool active = lane < A.L;
    int64_t lc = active ? lane : A.L - 1;
    const double *obs = A.obs;
    if (A.n_points > 0) {   // flattened data axis: parameter row and data point of the lane
        obs += (lc % A.n_points) * A.obs_stride;
        lc = lc / A.n_points;
    }
    const AS_GLOBAL double *prow = (const AS_GLOBAL double *)(A.params + int64_t(q) * A.prog_stride_p) + lc * A.ld_p;
    const uint32_t P = D.n_params;
    // static registers: parameters, their adjoints (+0), the sink, constants
    {
        uint32_t r = wide::kSlots;
        for (uint32_t p = 0; p < P; p += 4) {
            double v[4];
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i) v[i] = prow[p + i < P ? p + i : P - 1];
#pragma unroll
            for (uint32_t i = 0; i < 4; ++i)
                if (p + i < P) set_reg(r + p + i, v[i]);
        }
        r += P;
        const uint32_t zeros = (D.adjoints ? P : 0) + 1;
        for (uint32_t i = 0; i < zeros; ++i) set_reg(r + i, 0.0);
        r += zeros;
        const AS_CONST double *cs = (const AS_CONST double *)D.consts;
        for (uint32_t i = 0; i < D.n_consts; ++i) set_reg(r + i, cs[i]);
    }
    // addresses; the lanes past the last one write to the trash rows
    double *col = A.ws + int64_t(D.ckpt_row0) * A.Lpad + lane;
    double *trash = A.ws + int64_t(D.trash_row) * A.Lpad + lane;
    double *loss = active ? A.loss + int64_t(q) * A.L + lane : trash;
    double *grad = active && D.adjoints ? A.grad + int64_t(q) * A.prog_stride_g + lane * A.ld_g : trash;
    asm volatile(MOV("v[40:41]", "%[a]") MOV("v[42:43]", "%[b]") MOV("v[44:45]", "%[c]") MOV("v[46:47]", "%[d]")
                 ::[a] "v"(col), [b] "v"(obs), [c] "v"(loss), [d] "v"(grad)
                 : "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47");
    asm volatile("s_mov_b32 s26, %[pitch]\ns_mov_b64 s[34:35], %[code]\n"
                 "s_mov_b32 s100, %[f0]\ns_mov_b32 s98, %[f1]\ns_mov_b32 s99, %[f2]\n" ::[pitch] "s"(uint32_t(A.Lpad * 8)),
                 [code] "s"(uint64_t(size_t(D.code))), [f0] "s"(D.first[0]), [f1] "s"(D.first[1]), [f2] "s"(D.first[2])
                 : "s26", "s34", "s35", "s98", "s99", "s100", "scc");
    // nothing of the compiled part is live from here on
    asm volatile(
        "s_load_dwordx16 s[36:51], s[34:35], s100\ns_load_dwordx16 s[52:67], s[34:35], s100 offset:0x40\n"
        "s_getpc_b64 s[28:29]\n.Lpc%=:\ns_add_u32 s28, s28, .Lbase%=-.Lpc%=\ns_addc_u32 s29, s29, 0\n"
        "s_set_gpr_idx_on s26, 0x0\n"
        DISPATCH_B
        ".p2align 8\n.Lbase%=:\n"
        CLASS("", 15, 2, FMA_TEXT)
        CLASS("", 10, 3, DUAL_TEXT)
        CLASS("", 10, 3, SEL_TEXT)
        CLASS("", 10, 3, SELADJ_TEXT)
        CLASS("", 8, 2, DIV_TEXT)
        CLASS("", 4, 3, DIVADJ_TEXT)
        CLASS("", 6, 3, ACCD_TEXT)
        CLASS("", 15, 2, CKST_TEXT)
        LOADS(64, 12, LDK_TEXT)
        LOADS(88, 12, LDK_TEXT)
        LOADS(48, 4, LDO_TEXT)
        LOADS(56, 4, LDO_TEXT)
        REGION("s_waitcnt vmcnt(0)\n" DISPATCH_A) REGION("s_waitcnt vmcnt(0)\n" DISPATCH_B)
        CLASS("s_waitcnt vmcnt(0)\n", 1, 1, PF_TEXT)
        CLASS("", 2, 1, PF_TEXT)
        CLASS("", 1, 1, STLOSS_TEXT)
        CLASS("", 8, 2, STGRAD_TEXT)
        CALL1("ndvm_wide_exp")
        CALL1("ndvm_wide_sin")
        CALL1("ndvm_wide_cos")
        CALL1("ndvm_wide_logc")
        CALL1("ndvm_wide_sqrtc")
        CALL2("ndvm_wide_pow")
        CALL3("ndvm_wide_accsin")
        CALL3("ndvm_wide_acccos")
        CALL3("ndvm_wide_acclog")
        CALL3("ndvm_wide_accabs")
        CALL4("ndvm_wide_accpow")
        CALL4("ndvm_wide_accsqrt")
        CALL1("ndvm_wide_abs")
        REGION("s_branch .Lend%=\n") REGION("s_branch .Lend%=\n")
        ".Lend%=:\ns_set_gpr_idx_off\ns_waitcnt vmcnt(0) lgkmcnt(0)\n"
        ::: "s0", "s1", "s2", "s3", "s4", "s5", "s6", "s7", "s8", "s9", "s10", "s11", "s12", "s13", "s14", "s15", "s16",
          "s17", "s18", "s19", "s20", "s21", "s22", "s23", "s24", "s25", "s26", "s28", "s29", "s30", "s31", "s34",
          "s101", "m0", "vcc", "scc", "memory", "v0", "v39", "v255");
}

hipError_t launch_wide(const LaunchArgs &A, const wide::Prog *d_table, const wide::Prog &single, uint32_t n_prog,
                       hipStream_t stream) {
    const dim3 grid = A.wg_items ? dim3(A.n_wg) : dim3(uint32_t((A.L + 63) / 64), n_prog);
    hipLaunchKernelGGL(ndvm_wide, grid, dim3(64), 0, stream, A, d_table, single);
    return hipGetLastError();
}

}  // namespace ndvm
