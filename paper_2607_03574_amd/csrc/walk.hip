// Device walker kernel: the structural walk of a stack-bytecode program on
// the GPU, one wave per 64 lanes of one program (definitions and layout in
// walk.h).
//
// Control is the same for every lane of a wave.  The operand stack's and the
// locals' node numbers and the loop counters live in vector registers, entry i
// in lane i, read and written as wave-uniform values by a lane index; the next
// instruction word is read ahead.  Numbers are per lane.  The forward
// walk keeps the operand stack's top in a register and its values and the
// locals' in LDS rows (one double per lane); every node it records is also
// stored, as a coalesced row of 64 doubles, to the wave's slot in HBM for the
// reverse sweep.  A numeric IFLT takes one ballot: each arm runs under the mask
// of the lanes that take it, an arm no lane takes is not walked at all, and when
// both arms ran their differing stack positions and locals become MERGE nodes
// (Section 6, lane masking).  The reverse sweep visits the recorded operations
// from last to first and applies the adjoint rules of Appendix C, table
// tab:adjoints, per lane, gated on a nonzero incoming adjoint; a node no rule
// reached is skipped.  Records are read 64 at a time and the values a rule needs
// one node ahead.  Adjoints live in a few LDS rows, each tagged with its node:
// most are formed and used within a few nodes, so they take no memory traffic and
// no wait for stores; when all rows are taken, one moves to the wave's slot.
// The parameters' values and adjoints stay in LDS.
//
// What bounds it is the chain of one wave: a word costs its dispatch and an LDS
// read, a node its dispatch, two LDS reads and what is left of a memory read.
// 128 random programs of 128 points on 1,000 lanes each: 11.4 ms with structure
// in LDS, adjoints in HBM and structured control flow (some 1,700 cycles a word
// forward, 2,100 an operation in reverse), 6.5 now (880 and 1,250); 1,024
// programs of 16 points on 1,024 lanes 7.8 against 3.9 ms, one program of 64
// points on one lane 1.67 against 1.08.  Measured on the way: unstructured
// control flow 11.0 -> 7.6 ms, adjoints in LDS and one visit ahead 7.3, three
// visits ahead 6.4.  Instruction words in vector registers, 128 at a time, in
// place of the scalar read one word ahead: 6.3 -> 6.5, not kept.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>

#include "common.h"
#include "walk.h"

namespace ndvm {
namespace {

using walk::Args;
using walk::ProgDesc;

constexpr uint32_t kUnset = 0xFFFFFFFFu;

// Read-only inputs (the program buffer, the observations) are read through
// the constant address space, so wave-uniform reads become scalar loads that
// wait for nothing else (a vector load would wait for every store the walk
// has in flight before it).
#define AS_CONST __attribute__((address_space(4)))
// The wave's rows and words are named by their address space, so that no
// access goes through a generic address.
#define AS_LDS __attribute__((address_space(3)))
#define AS_HBM __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ const AS_CONST T *cst(const T *p) {
    return (const AS_CONST T *)(p);
}

__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
    return uint64_t(uni(uint32_t(v))) | uint64_t(uni(uint32_t(v >> 32))) << 32;
}

__device__ __forceinline__ double clampv(double x) { return x < 1e-8 ? 1e-8 : x; }

__device__ __forceinline__ bool is_binary(uint32_t op) {
    return op == bc::ADD || op == bc::SUB || op == bc::MUL || op == bc::DIV || op == bc::POW;
}

// Library functions whose code branches per lane, out of line: the interpreter's
// own control flow stays free of such branches, and so free of the flow blocks
// they would put around every handler.  A call by the platform's convention,
// past the function's first instruction, a wait for every load and store in
// flight (4 bytes), which its arguments do not need.  None uses scratch memory
// or registers past those named as changed.
#define NDVM_WALK_FN extern "C" __device__ __attribute__((used, noinline, visibility("hidden"))) double
NDVM_WALK_FN ndvm_walk_sin(double x) { return sin(x); }
NDVM_WALK_FN ndvm_walk_cos(double x) { return cos(x); }
NDVM_WALK_FN ndvm_walk_pow(double x, double y) { return pow(x, y); }
#define CALL_TEXT(f) \
    "s_getpc_b64 s[28:29]\ns_add_u32 s28, s28, " f "@rel32@lo+8\ns_addc_u32 s29, s29, " f "@rel32@hi+16\n" \
    "s_swappc_b64 s[30:31], s[28:29]\n"
#define CALL_CHANGES \
    "s0", "s1", "s2", "s3", "s4", "s5", "s6", "s7", "s8", "s9", "s10", "s11", "s12", "s13", "s14", "s15", "s16", "s17", \
    "s18", "s19", "s20", "s21", "s22", "s23", "s24", "s25", "s26", "s27", "s28", "s29", "s30", "s31", "vcc", "scc", \
    "v4", "v5", "v6", "v7", "v8", "v9", "v10", "v11", "v12", "v13", "v14", "v15", "v16", "v17", "v18", "v19", "v20", \
    "v21", "v22", "v23", "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35", "v36", \
    "v37", "v38", "v39"
__device__ __forceinline__ double call_sin(double x) {
    double r;
    asm volatile(CALL_TEXT("ndvm_walk_sin") : "={v[0:1]}"(r) : "0"(x) : "v2", "v3", CALL_CHANGES);
    return r;
}
__device__ __forceinline__ double call_cos(double x) {
    double r;
    asm volatile(CALL_TEXT("ndvm_walk_cos") : "={v[0:1]}"(r) : "0"(x) : "v2", "v3", CALL_CHANGES);
    return r;
}
__device__ __forceinline__ double call_pow(double x, double y) {
    double r, gone;
    asm volatile(CALL_TEXT("ndvm_walk_pow") : "={v[0:1]}"(r), "={v[2:3]}"(gone) : "0"(x), "1"(y) : CALL_CHANGES);
    return r;
}

// forward value of a scalar word
__device__ __forceinline__ double forward(uint32_t op, double x, double y) {
    switch (op) {
    case bc::ADD: return x + y;
    case bc::SUB: return x - y;
    case bc::MUL: return x * y;
    case bc::DIV: return x / y;
    case bc::NEG: return -x;
    case bc::SQRT: return sqrt(clampv(x));
    case bc::ABS: return fabs(x);
    case bc::EXP: return exp(x);
    case bc::LOG: return log(clampv(x));
    case bc::SIN: return call_sin(x);
    case bc::COS: return call_cos(x);
    default: return call_pow(x, y);
    }
}

// a recorded operation as one 16-byte access: kind, operands, number
typedef uint32_t Node4 __attribute__((ext_vector_type(4), aligned(8)));

struct Wave {
    uint32_t lane;
    // LDS: value rows (64 doubles each)
    AS_LDS double *VP;   // parameters' values
    AS_LDS double *VS;   // operand stack values (forward)
    AS_LDS double *VL;   // locals' values (forward)
    AS_LDS double *GP;   // parameters' adjoints (reverse; the rows of VS and VL on)
    AS_LDS double *GC;   // adjoint rows of other nodes (reverse)
    // LDS: IFLT frames, words that nothing reads (one per lane), one flag bit
    // per node (its adjoint row is in HBM)
    AS_LDS uint32_t *frm, *dump, *flg;
    uint32_t snap, fsz, depth;
    // HBM slot of the wave
    AS_HBM double *V, *G;
    AS_HBM Node4 *E;
    AS_HBM uint64_t *M;   // ballot words of MERGE nodes

    __device__ __forceinline__ AS_LDS double &s(uint32_t i) const { return VS[i * 64 + lane]; }
    __device__ __forceinline__ AS_LDS double &l(uint32_t j) const { return VL[j * 64 + lane]; }
};

__device__ __forceinline__ uint32_t get(uint32_t v, uint32_t i) { return __builtin_amdgcn_readlane(v, i); }
__device__ __forceinline__ void put(uint32_t &v, uint32_t i, uint32_t x) { v = threadIdx.x == i ? x : v; }

// A value whose load is waited for here, in the rare path that needs one, and
// not where paths meet: there the wait would be for the values read ahead too.
template <class T>
__device__ __forceinline__ T landed(T v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Walk one work item (64 lanes of one program); returns false when a bound
// the host validation guarantees was not met (the lanes then hold NaN).
__device__ bool walk_item(const Args &A, const Wave &W, const ProgDesc &D, uint32_t q, int64_t l0) {
    const uint32_t lane = W.lane;
    const int64_t lg = l0 + lane;
    const bool active = lg < A.L;
    const int64_t lc = active ? lg : A.L - 1;
    const AS_CONST uint32_t *code = cst(A.buf + D.code_off);
    const AS_CONST int32_t *match = cst(reinterpret_cast<const int32_t *>(A.buf + D.match_off));
    const AS_CONST double *K = cst(reinterpret_cast<const double *>(A.buf + D.const_off));
    const AS_CONST double *obs = cst(A.obs);
    const double *prm = A.params + int64_t(q) * A.prog_stride_p + lc * A.ld_p;
    const uint32_t n_nodes = D.n_nodes, P = D.n_params;
    if (n_nodes > A.n_nodes_max || D.depth > A.depth || D.n_locals > A.n_locals || D.n_loops > A.n_loops ||
        D.n_frames > A.n_frames || P > A.n_params || D.n_instr == 0)
        return false;

    for (uint32_t i = lane; i < (n_nodes + 31) / 32; i += 64) W.flg[i] = 0;
    for (uint32_t p = 0; p < P; ++p) W.VP[p * 64 + lane] = prm[p];

    // value of node k in the forward walk (parameters in LDS, the others in
    // HBM; a leaf's number carries kLeafBit)
    auto value = [&](uint32_t k) -> double {
        k &= ~walk::kLeafBit;
        return k < P ? W.VP[k * 64 + lane] : W.V[k * 64u + lane];
    };
    // entry i of the stack, the locals and the loops in lane i
    uint32_t stk = 0, loc = kUnset, loop_pc = 0, loop_trips = 0, loop_at = 0;
    uint64_t mask = uni64(__ballot(active));
    uint32_t n = P, sp = 0, lp = 0, fp = 0, pc = 0, steps = 0;
    double top = 0.0;   // value of stack position sp - 1 (its LDS row holds it too)
    // operation records, 64 at a time: record m in lane m % 64
    uint32_t m = 0, r_op = 0, r_a = 0, r_b = 0, r_k = 0;
    auto record = [&](uint32_t op, uint32_t a, uint32_t b, double val) {
        W.V[n * 64u + lane] = val;
        const uint32_t i = m % 64;
        put(r_op, i, op);
        put(r_a, i, a);
        put(r_b, i, b);
        put(r_k, i, n);
        if (++m % 64 == 0) W.E[m - 64 + lane] = Node4{r_op, r_a, r_b, r_k};
        return n++;
    };
    auto leaf = [&](double x) {
        W.V[n * 64u + lane] = x;
        W.s(sp) = top = x;
        put(stk, sp++, n++ | walk::kLeafBit);
    };
    auto reload_top = [&]() { top = W.s(sp ? sp - 1 : 0); };
    // node numbers of the stack and the locals (a snapshot of an IFLT's frame)
    auto save = [&](AS_LDS uint32_t *to) {
        *(lane < sp ? to + lane : W.dump + lane) = stk;
        *(lane < D.n_locals ? to + W.depth + lane : W.dump + lane) = loc;
    };

    const uint32_t last = D.n_instr - 1;
    uint32_t w0 = code[0], imm = code[1];   // the word at pc
    for (;;) {
        if (pc > last || ++steps > D.n_steps) return false;   // the walk always ends within both
        // the next word, and the value below the top, are read ahead
        const uint32_t at = pc < last ? pc + 1 : last;
        const uint32_t next0 = code[2 * at], next_imm = code[2 * at + 1];
        const double below = W.s(sp < 2 ? 0 : sp - 2);
        const uint32_t op = w0 & 0xFFu, wa = (w0 >> 8) & 0xFFu;
        // bounds the host validation guarantees (kept so that a broken
        // guarantee can only give NaN lanes, never an access out of bounds);
        // the host packs each word's stack effect into it
        const uint32_t pops = (w0 >> 16) & 3u, pushes = (w0 >> 18) & 3u;
        if (sp < pops || sp - pops + pushes > W.depth) return false;   // the other bounds: in their words
        switch (op) {
        case bc::HALT:
            goto reverse;
        case bc::PUSH:
            if (n >= n_nodes) return false;
            leaf(K[imm]);
            break;
        case bc::OBS: {
            if (n >= n_nodes || wa > lp || wa > last - pc) return false;
            int64_t idx = imm;
            // The first stride is in the word read ahead, and the word behind the
            // strides is read together with the observation: one scalar read after
            // another otherwise (one program on one lane 1.08 -> 1.05 ms, 1,024
            // programs on 1,024 lanes 3.93 -> 3.85).
            if (wa) idx += int64_t(int32_t(next_imm)) * int64_t(get(loop_at, lp - 1));
            for (uint32_t d = 1; d < wa; ++d)
                idx += int64_t(int32_t(code[2 * (pc + 1 + d) + 1])) * int64_t(get(loop_at, lp - 1 - d));
            const uint32_t behind = wa < last - pc ? pc + wa + 1 : last;
            w0 = code[2 * behind];
            imm = code[2 * behind + 1];
            double x = obs[idx];
            asm volatile("" : "+s"(w0), "+s"(imm), "+s"(x));   // one wait for the three
            leaf(x);
            pc += wa + 1;
            continue;
        }
        case bc::PARAM:
            if (imm >= P) return false;
            W.s(sp) = top = W.VP[imm * 64 + lane];
            put(stk, sp++, imm);
            break;
        case bc::LOADL: {
            if (imm >= D.n_locals) return false;
            const uint32_t id = get(loc, imm);
            if (id == kUnset) return false;
            W.s(sp) = top = W.l(imm);
            put(stk, sp++, id);
            break;
        }
        case bc::STOREL:
            if (imm >= D.n_locals) return false;
            --sp;
            W.l(imm) = top;
            put(loc, imm, get(stk, sp));
            top = below;
            break;
        case bc::DUP:
            W.s(sp) = top;
            put(stk, sp, get(stk, sp - 1));
            ++sp;
            break;
        case bc::OVER:
            W.s(sp) = top = below;
            put(stk, sp, get(stk, sp - 2));
            ++sp;
            break;
        case bc::SWAP: {
            const uint32_t t = get(stk, sp - 1), u = get(stk, sp - 2);
            W.s(sp - 1) = below;
            W.s(sp - 2) = top;
            top = below;
            put(stk, sp - 1, u);
            put(stk, sp - 2, t);
            break;
        }
        case bc::DROP:
            --sp;
            top = below;
            break;
        case bc::LOOP:
            if (lp >= A.n_loops) return false;
            if (imm == 0) {
                pc = uni(uint32_t(match[pc])) + 1;
                goto jumped;
            }
            put(loop_pc, lp, pc + 1);
            put(loop_trips, lp, imm);
            put(loop_at, lp, 0);
            ++lp;
            break;
        case bc::ENDLOOP: {
            if (lp == 0) return false;
            const uint32_t k = get(loop_at, lp - 1) + 1;
            if (k < get(loop_trips, lp - 1)) {
                put(loop_at, lp - 1, k);
                pc = get(loop_pc, lp - 1);
                goto jumped;
            }
            --lp;
            break;
        }
        case bc::IFLT: {
            if (fp >= A.n_frames) return false;
            sp -= 2;
            const uint64_t tm = uni64(__ballot(below < top)) & mask, em = mask & ~tm;
            reload_top();
            // frame: outer mask, first-arm mask, second-arm mask, phase, entry
            // depth, then the entry snapshot and the first arm's exit snapshot
            // (node numbers of stack positions and locals)
            AS_LDS uint32_t *f = W.frm + fp * W.fsz;
            ++fp;
            f[0] = uint32_t(mask);
            f[1] = uint32_t(mask >> 32);
            f[2] = uint32_t(tm);
            f[3] = uint32_t(tm >> 32);
            f[4] = uint32_t(em);
            f[5] = uint32_t(em >> 32);
            f[6] = 0;
            f[7] = sp;
            save(f + walk::kFrameFixed);
            if (tm) {
                mask = tm;
                break;
            }
            mask = em;   // no lane takes the first arm: it is not walked
            pc = uni(uint32_t(match[pc])) + 1;
            goto jumped;
        }
        case bc::ELSE: {   // end of a walked first arm
            if (fp == 0) return false;
            AS_LDS uint32_t *f = W.frm + (fp - 1) * W.fsz;
            const uint64_t em = uint64_t(uni(f[4])) | uint64_t(uni(f[5])) << 32;
            f[6] = 1u | sp << 1;
            save(f + walk::kFrameFixed + W.snap);
            if (em) {
                // the second arm starts from the entry state: restore the
                // stack and locals values that differ from it
                const uint32_t sp0 = uni(f[7]);
                if (sp0 > W.depth) return false;
                const uint32_t s0 = f[walk::kFrameFixed + (lane < sp0 ? lane : 0u)];
                const uint32_t j0 = f[walk::kFrameFixed + W.depth + (lane < D.n_locals ? lane : 0u)];
                for (uint64_t d = uni64(__ballot(lane < sp0 && (lane >= sp || s0 != stk))); d; d &= d - 1) {
                    const uint32_t i = uint32_t(__builtin_ctzll(d));
                    W.s(i) = value(get(s0, i));
                }
                for (uint64_t d = uni64(__ballot(lane < D.n_locals && j0 != loc && j0 != kUnset)); d; d &= d - 1) {
                    const uint32_t i = uint32_t(__builtin_ctzll(d));
                    W.l(i) = value(get(j0, i));
                }
                stk = s0;
                loc = j0;
                sp = sp0;
                reload_top();
                mask = em;
                break;
            }
            pc = uni(uint32_t(match[pc]));   // to the ENDIF
            goto jumped;
        }
        case bc::ENDIF: {
            if (fp == 0) return false;
            const AS_LDS uint32_t *f = W.frm + (fp - 1) * W.fsz;
            const uint32_t ph = uni(f[6]);
            const uint64_t tm = uint64_t(uni(f[2])) | uint64_t(uni(f[3])) << 32;
            const uint64_t em = uint64_t(uni(f[4])) | uint64_t(uni(f[5])) << 32;
            if ((ph & 1u) && em) {   // both arms walked: merge what they left different
                if ((ph >> 1) != sp) return false;
                const bool first = (tm >> lane) & 1u;
                const uint32_t s1 = f[walk::kFrameFixed + W.snap + (lane < sp ? lane : 0u)];
                const uint32_t j1 = f[walk::kFrameFixed + W.snap + W.depth + (lane < D.n_locals ? lane : 0u)];
                for (uint64_t d = uni64(__ballot(lane < sp && s1 != stk)); d; d &= d - 1) {
                    const uint32_t i = uint32_t(__builtin_ctzll(d)), x = get(s1, i);
                    if (n >= n_nodes) return false;
                    const double then = value(x), other = W.s(i), val = first ? then : other;
                    W.s(i) = val;
                    W.M[n] = tm;
                    put(stk, i, record(walk::kMerge, x, get(stk, i), val));
                }
                for (uint64_t d = uni64(__ballot(lane < D.n_locals && j1 != loc)); d; d &= d - 1) {
                    const uint32_t i = uint32_t(__builtin_ctzll(d)), x = get(j1, i), y = get(loc, i);
                    if (x == kUnset || y == kUnset || n >= n_nodes) return false;
                    const double then = value(x), other = W.l(i), val = first ? then : other;
                    W.l(i) = val;
                    W.M[n] = tm;
                    put(loc, i, record(walk::kMerge, x, y, val));
                }
                reload_top();
            }
            mask = uint64_t(uni(f[0])) | uint64_t(uni(f[1])) << 32;
            --fp;
            break;
        }
        default: {   // a scalar numeric word
            if (n >= n_nodes) return false;
            const bool bin = is_binary(op);
            const uint32_t hi = get(stk, sp - 1);
            const uint32_t bi = bin ? hi : 0u, ai = bin ? get(stk, sp - 2) : hi;
            sp -= bin ? 2 : 1;
            top = forward(op, bin ? below : top, top);
            W.s(sp) = top;
            put(stk, sp++, record(op, ai, bi, top));
        }
        }
        ++pc;
        w0 = next0;
        imm = next_imm;
        continue;
    jumped:
        if (pc > last) return false;
        w0 = code[2 * pc];
        imm = code[2 * pc + 1];
    }

reverse: {
    const uint32_t loss_id = get(stk, 0);
    const double loss = W.s(0);
    if (lane < m % 64) W.E[m / 64 * 64 + lane] = Node4{r_op, r_a, r_b, r_k};
    for (uint32_t p = 0; p < P; ++p) W.GP[p * 64 + lane] = 0.0;
    // Adjoint rows: row r of GC belongs to node tag[r] (lane r).  A row whose
    // node the sweep has passed (or kUnset) is free; lanes past the rows match
    // no node.  in_hbm counts the nodes whose adjoint was moved out.
    constexpr uint64_t kRows = (1ull << walk::kAdjointRows) - 1;
    uint32_t tag = lane < walk::kAdjointRows ? kUnset : kUnset >> 1, in_hbm = 0, turn = 0;
    auto flagged = [&](uint32_t j) { return in_hbm && ((uni(W.flg[j >> 5]) >> (j & 31)) & 1u); };
    auto flip = [&](uint32_t j) { W.flg[j >> 5] = uni(W.flg[j >> 5]) ^ 1u << (j & 31); };
    auto row_of = [&](uint32_t j) { return uni64(__ballot(tag == j)); };
    // Row of target j while node k is visited (never row `keep`), and its
    // adjoint so far: 0 before the first contribution.
    auto target = [&](uint32_t j, uint32_t k, uint32_t keep, double *base) -> uint32_t {
        const uint64_t hit = row_of(j);
        if (hit) {
            const uint32_t r = uint32_t(__builtin_ctzll(hit));
            *base = W.GC[r * 64 + lane];
            return r;
        }
        *base = 0.0;
        if (flagged(j)) {
            *base = landed(W.G[j * 64u + lane]);
            flip(j);
            --in_hbm;
        }
        const uint64_t open = uni64(__ballot(tag >= k)) & kRows & ~(1ull << keep);
        uint32_t r;
        if (open) {
            r = uint32_t(__builtin_ctzll(open));
        } else {
            if (turn == keep) turn = (turn + 1) % walk::kAdjointRows;
            r = turn;
            turn = (turn + 1) % walk::kAdjointRows;
            const uint32_t old = get(tag, r);
            W.G[old * 64u + lane] = W.GC[r * 64 + lane];
            flip(old);
            ++in_hbm;
        }
        put(tag, r, j);
        return r;
    };
    if (!(loss_id & walk::kLeafBit)) {   // seed: 0 + 1
        if (loss_id < P) {
            W.GP[loss_id * 64 + lane] = 1.0;
        } else {
            put(tag, 0, loss_id);
            W.GC[lane] = 1.0;
        }
    }
    // Records of the chunk of 64 operations visited and of the one below it.
    // The values an operation's rules read are loaded kAhead visits ahead, all
    // three whatever the rule (a load in some paths only would be waited for in
    // all; a parameter's row in the slot is read and not used).
    uint32_t chunk = m ? (m - 1) / 64 : 0;
    Node4 cur{}, low{};
    if (m && lane <= (m - 1) % 64) cur = W.E[chunk * 64 + lane];
    if (chunk) low = W.E[(chunk - 1) * 64 + lane];
    struct Values {
        double x, y, z;
    };
    auto load = [&](uint32_t e) __attribute__((always_inline)) {
        const uint32_t i = e % 64;
        const bool here = e / 64 == chunk;
        const uint32_t a = get(here ? cur.y : low.y, i), b = get(here ? cur.z : low.z, i),
                       k = get(here ? cur.w : low.w, i);
        return Values{W.V[(a & ~walk::kLeafBit) * 64u + lane], W.V[(b & ~walk::kLeafBit) * 64u + lane],
                      W.V[k * 64u + lane]};
    };
    auto visit = [&](uint32_t e, const Values &v) __attribute__((always_inline)) {
        if (e / 64 != chunk) {
            cur = low;
            --chunk;
            if (chunk) low = landed(W.E[(chunk - 1) * 64 + lane]);
        }
        const uint32_t i = e % 64;
        const uint32_t op = get(cur.x, i), a = get(cur.y, i), b = get(cur.z, i), k = get(cur.w, i);
        const uint64_t mine = row_of(k);
        double g;
        if (mine) {
            g = W.GC[uint32_t(__builtin_ctzll(mine)) * 64 + lane];
        } else {
            if (!flagged(k)) return;   // no adjoint reached it
            g = landed(W.G[k * 64u + lane]);
            flip(k);
            --in_hbm;
        }
        const bool two = is_binary(op) || op == walk::kMerge;
        const bool has_a = !(a & walk::kLeafBit), has_b = two && !(b & walk::kLeafBit);
        // the targets' rows (constants and observations take no adjoint); one
        // named twice (x * x) takes its second contribution on top of the first
        double ga = 0.0, gb = 0.0;
        uint32_t row_a = 0, row_b = 0, keep = 63;   // rows from GP on
        if (has_a) {
            if (a < P) {
                row_a = a;
                ga = W.GP[a * 64 + lane];
            } else {
                keep = target(a, k, 63, &ga);
                row_a = A.n_params + keep;
            }
        }
        if (has_b && b != a) {
            if (b < P) {
                row_b = b;
                gb = W.GP[b * 64 + lane];
            } else {
                row_b = A.n_params + target(b, k, keep, &gb);
            }
        }
        const double x = a < P ? W.VP[a * 64 + lane] : v.x, y = b < P ? W.VP[b * 64 + lane] : v.y, z = v.z;
        const bool on = g != 0.0;
        // contributions: value, where it applies, subtracted
        double ca = 0.0, cb = 0.0;
        bool pa = on, pb = on, na = false, nb = false;
        switch (op) {
        case walk::kMerge: {
            const bool first = (uni64(W.M[k]) >> lane) & 1u;
            ca = cb = g;
            pa = on && first;
            pb = on && !first;
            break;
        }
        case bc::ADD:
            ca = cb = g;
            break;
        case bc::SUB:
            ca = cb = g;
            nb = true;
            break;
        case bc::MUL:
            ca = g * y;
            cb = g * x;
            break;
        case bc::DIV:
            ca = g / y;
            cb = (g * z) / y;
            nb = true;
            break;
        case bc::NEG:
            ca = g;
            na = true;
            break;
        case bc::EXP:
            ca = g * z;
            break;
        case bc::LOG:
            pa = on && x > 1e-8;
            ca = g / x;
            break;
        case bc::SQRT:
            pa = on && x > 1e-8;
            ca = g / (2.0 * z);
            break;
        case bc::SIN:
            ca = g * call_cos(x);
            break;
        case bc::COS:
            ca = g * call_sin(x);
            na = true;
            break;
        case bc::ABS:
            ca = x > 0.0 ? g : (x < 0.0 ? -g : 0.0);
            break;
        default:   // POW
            ca = ((g * y) * z) / x;
            cb = (g * z) * log(x);
        }
        if (has_a) {
            const double nv = na ? ga - ca : ga + ca;
            ga = pa ? nv : ga;
            W.GP[row_a * 64 + lane] = ga;
        }
        if (has_b) {
            if (b == a) {
                gb = ga;
                row_b = row_a;
            }
            const double nv = nb ? gb - cb : gb + cb;
            W.GP[row_b * 64 + lane] = pb ? nv : gb;
        }
    };
    if (m) {
        constexpr uint32_t kAhead = 3;
        auto before = [&](uint32_t e, uint32_t d) { return e > d ? e - d : 0; };
        Values v0 = load(m - 1), v1 = load(before(m - 1, 1)), v2 = load(before(m - 1, 2));
        for (uint32_t e = m - 1;; --e) {
            visit(e, v0);
            v0 = load(before(e, kAhead));
            if (e-- == 0) break;
            visit(e, v1);
            v1 = load(before(e, kAhead));
            if (e-- == 0) break;
            visit(e, v2);
            v2 = load(before(e, kAhead));
            if (e == 0) break;
        }
    }
    if (active) {
        A.loss[int64_t(q) * A.L + lg] = loss;
        double *gr = A.grad + int64_t(q) * A.prog_stride_g + lg * A.ld_g;
        for (uint32_t p = 0; p < P; ++p) gr[p] = W.GP[p * 64 + lane];
    }
}
    return true;
}

__global__ void __launch_bounds__(64) ndvm_walk(Args A) {
    extern __shared__ double sh[];
    Wave W;
    W.lane = threadIdx.x;
    W.depth = A.depth;
    W.snap = A.depth + A.n_locals;
    W.fsz = walk::kFrameFixed + 2 * W.snap;
    W.VP = (AS_LDS double *)sh;
    W.VS = W.VP + A.n_params * 64;
    W.VL = W.VS + A.depth * 64;
    W.GP = W.VS;
    W.GC = W.GP + A.n_params * 64;
    W.frm = (AS_LDS uint32_t *)(W.VP + walk::launch_rows(A.depth, A.n_locals, A.n_params) * 64);
    W.dump = W.frm + A.n_frames * W.fsz;
    W.flg = W.dump + walk::kDumpWords;
    uint8_t *slot = A.ws + uint64_t(blockIdx.x) * A.n_nodes_max * walk::ws_bytes_per_node();
    W.V = (AS_HBM double *)slot;
    W.G = W.V + uint64_t(A.n_nodes_max) * 64;
    W.E = (AS_HBM Node4 *)(W.G + uint64_t(A.n_nodes_max) * 64);
    W.M = (AS_HBM uint64_t *)(W.E + A.n_nodes_max);
    const uint64_t per_prog = uint64_t((A.L + 63) / 64);
    const AS_CONST uint32_t *descs = cst(A.buf);   // ProgDesc records, word by word
    for (uint64_t item = blockIdx.x; item < A.n_items; item += gridDim.x) {
        const uint32_t q = uint32_t(item / per_prog);
        const int64_t l0 = int64_t(item % per_prog) * 64;
        ProgDesc D;
        uint32_t *dw = reinterpret_cast<uint32_t *>(&D);
        for (uint32_t i = 0; i < sizeof(ProgDesc) / 4; ++i) dw[i] = descs[uint64_t(q) * (sizeof(ProgDesc) / 4) + i];
        if (!walk_item(A, W, D, q, l0)) {
            // a bound the validation guarantees was not met: report it and
            // leave this item's lanes NaN
            if (W.lane == 0) atomicOr(A.status, 1);
            const int64_t lg = l0 + W.lane;
            if (lg < A.L) {
                A.loss[int64_t(q) * A.L + lg] = NAN;
                double *gr = A.grad + int64_t(q) * A.prog_stride_g + lg * A.ld_g;
                for (uint32_t p = 0; p < D.n_params; ++p) gr[p] = NAN;
            }
        }
    }
}

// Clears the status word (a kernel: a memset node of a captured graph may not
// take effect on its later replays).
__global__ void ndvm_walk_clear(int *status) { *status = 0; }

}  // namespace

hipError_t launch_walk(const walk::Args &A, uint32_t grid, hipStream_t stream) {
    hipLaunchKernelGGL(ndvm_walk_clear, dim3(1), dim3(1), 0, stream, A.status);
    if (grid == 0) return hipGetLastError();
    static std::once_flag once[64];
    static hipError_t raised[64];   // the LDS limit, per device
    int dev = 0;
    (void)hipGetDevice(&dev);
    hipError_t &st = raised[dev & 63];
    std::call_once(once[dev & 63], [&st]() {
        st = hipFuncSetAttribute(reinterpret_cast<const void *>(&ndvm_walk), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 int(walk::kMaxLaunchLdsBytes));
    });
    if (st != hipSuccess) return st;
    hipLaunchKernelGGL(ndvm_walk, dim3(grid), dim3(64), size_t(A.lds_bytes), stream, A);
    return hipGetLastError();
}

}  // namespace ndvm
