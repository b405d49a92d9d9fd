// Scheduler of the wide replay kernel: a scalar tape becomes one sequence of
// micro-ops per lane (forward sweep, then per checkpoint segment restore,
// recompute, adjoint rules), over virtual registers that a linear scan places
// in the lane's register file, then cut into blocks of one class.
//
// Which values are computed, stored and recomputed, and the order of the
// contributions to every adjoint, are those of the slot scheduler (Info,
// Builder), so both kernels give the same bits.
#include "wide.h"

#include <algorithm>
#include <stdexcept>
#include <unordered_map>

#include "plan.h"
#include "slot.h"
#include "wide_exec.h"

namespace ndvm {

namespace {

using namespace wide;

struct WOp {
    uint8_t cls = 0, n = 0;
    bool late = false;     // a load of a row the loss is formed from
    uint32_t imm = 0;      // row, observation index or output index
    uint32_t r[6] = {};    // registers in the order of the class's half words
    uint8_t n_mem = 0;
    uint32_t m[3] = {}, e[3] = {};   // matrices and elements in the order of the class's offset words
};

// Half words of a class and their roles: 'u' read, 'd' written after the
// reads, 'e' written before the last read, 'm' read and written, '-' unused;
// the immediate's word ('i') stands for two halves.  Whole words: 'R' offset of
// a matrix read, 'W' written, 'M' read and written, 'z' nothing.
const char *roles(uint32_t cls) {
    switch (cls) {
    case FMA: return "uuud";
    case DUAL: return "ueumum";
    case SEL: return "uuuud-";
    case SELADJ: return "ueuumm";
    case DIV: case POW: return "uud-";
    case DIVADJ: return "ueumum";
    case ACCD: return "ueumu-";
    case CKST: case STGRAD: return "u-i";
    case LDK0: case LDK1: case LDO0: case LDO1: case WAITPF: case PF: return "i";
    case STLOSS: return "u-";
    case EXP: case SIN: case COS: case LOGC: case SQRTC: case ABS: return "ud";
    case ACCSIN: case ACCCOS: case ACCLOG: case ACCABS: return "uuud";
    case ACCPOW: case ACCSQRT: return "uuuud-";
    case STE: case STE4: return "u-W";
    case LDE: return "Rd-";
    case CKSTM: return "Ri";
    case MM: case VADD: return "RRWi";
    case MMA: case MMB: case INV2ACC: return "RRMi";
    case VACC: case TRANSACC: return "RzMi";
    case TRANS: case INV2: return "RzWi";
    case VSCALE: return "RWiud";
    case VACCS: case LOGDETACC: return "RMiud";
    case SDOT: return "RRiud";
    case DET2: return "Rziud";
    default: return "";
    }
}

constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr uint32_t kUnsetTime = 0xFFFFFFFFu;
constexpr uint32_t kVirtual = 1u << 20;   // register numbers from here on are virtual
// micro-ops a value may wait in its load slot before its last reader; beyond
// that it is copied to a register so that the slot's next load can start
constexpr uint32_t kSlotHold = 24;
// micro-ops to look back for one that can clear a second first-contribution target
constexpr uint32_t kLookBack = 48;

// Estimated cycles of a lone wave per micro-op and per block (an instruction
// issues about every 4.5 cycles; a change of EXEC by a compare costs 20 more).
uint32_t class_cost(uint32_t cls) {
    switch (cls) {
    case FMA: return 32;
    case DUAL: return 72;
    case SEL: return 46;
    case SELADJ: return 80;
    case DIV: return 90;
    case DIVADJ: return 200;
    case ACCD: return 130;
    case CKST: return 35;
    case LDK0: case LDK1: case LDO0: case LDO1: return 25;
    case EXP: return 330;
    case SIN: case COS: case ACCSIN: case ACCCOS: return 450;
    case LOGC: case ACCPOW: return 450;
    case POW: return 1100;
    case ACCLOG: case ACCSQRT: case SQRTC: return 280;
    case PF: case WAITPF: return 30;
    case STE: case STE4: return 30;
    case LDE: case CKSTM: return 110;
    case MM: case MMA: case MMB: return 430;
    case VADD: case VACC: case TRANS: case TRANSACC: case VSCALE: case VACCS: return 300;
    case INV2: case INV2ACC: case LOGDETACC: case SDOT: case DET2: return 450;
    default: return 150;
    }
}
constexpr uint32_t kDispatchCost = 62;

// Measured cycles of a lone wave per micro-op and per block: least squares over
// the launches named at the slot kernel's lone_cycles, times within 13%
// (gradients 10%, programs with matrices 20%); class_cost stays what the choice
// between programs was tuned on.
uint32_t lone_cycles(uint32_t cls) {
    switch (cls) {
    case FMA: return 27;
    case DUAL: return 70;
    case SEL: return 84;
    case SELADJ: return 122;
    case DIV: return 86;
    case DIVADJ: return 189;
    case ACCD: return 151;
    case CKST: return 10;
    case LDK0: case LDK1: return 70;
    case LDO0: case LDO1: case STGRAD: return 5;
    case WAIT: case WAITPF: return 172;
    case PF: return 40;
    case EXP: return 331;
    case SIN: return 530;
    case COS: return 482;
    case LOGC: return 554;
    case SQRTC: return 239;
    case POW: return 1289;
    case ACCSIN: return 621;
    case ACCCOS: return 681;
    case ACCLOG: return 269;
    case ACCABS: return 199;
    case ACCPOW: return 679;
    case ACCSQRT: return 307;
    case ABS: return 101;
    case STE: return 46;
    case STE4: return 76;
    case LDE: case CKSTM: return 155;
    case MM: return 420;
    case MMA: case MMB: return 830;
    case VADD: case VACC: return 460;
    case TRANS: case TRANSACC: return 620;
    case INV2: case VSCALE: return 560;
    case INV2ACC: case LOGDETACC: return 700;
    case VACCS: return 1000;
    case SDOT: return 1200;
    case DET2: return 400;
    default: return 0;
    }
}
bool is_call(uint32_t cls) { return cls >= EXP && cls <= ACCSQRT; }
// what else a program with matrices does four times, once a thread of a lane, or
// waits for alone
bool is_element(uint32_t cls) { return cls == STE || cls == LDE || cls == DIV || cls == DIVADJ || cls == ACCD; }
constexpr uint32_t kLoneDispatch = 43;

struct Lower {
    const Info &I;
    Builder &B;
    const Tape &t;
    const bool with_grad;
    const uint32_t N, P;
    std::vector<double> consts;
    std::unordered_map<uint64_t, uint32_t> const_of;   // bits -> constant number
    uint32_t kSink = 0, kConst0 = 0, n_static = 0;
    std::vector<WOp> ops;
    uint32_t n_virtual = 0;                            // virtual registers so far (ids from kSlots + n_static)
    std::unordered_map<uint32_t, uint32_t> neg_param;  // parameter -> register holding its negation
    std::vector<uint32_t> fval, adj;
    // of the segment being reversed: the register of each value, and the
    // checkpoint row of each live-in value (valid where the mark is segment + 1)
    std::vector<uint32_t> rval, rval_of, row, row_of;
    std::vector<uint32_t> first_row;                   // of each segment's live-in values
    // loads, in the order their values are first needed: position in ops of
    // the placeholder that takes the value (an FMA move whose r[0] becomes the slot)
    struct Load {
        uint32_t at, reg;
        bool ckpt;
        uint32_t imm;
        uint32_t after;   // op that stores the row (0 for an observation)
        bool late;        // read when the loss is formed last
    };
    std::vector<Load> loads;
    std::vector<uint32_t> stored_at;   // op that stores each checkpoint row

    const bool mats;                                   // a program with matrices
    std::vector<uint32_t> mem_size;                    // elements of each matrix (padded to quads)

    Lower(const Info &info, Builder &b, bool grad, bool matrices)
        : I(info), B(b), t(info.t), with_grad(grad), N(info.N), P(info.P), mats(matrices) {}

    // ---- matrices: values and adjoints of more than one element are named by
    // matrix numbers where scalars are named by registers
    uint32_t mem(uint32_t nel) {
        mem_size.push_back((nel + 3) / 4 * 4);
        return uint32_t(mem_size.size() - 1);
    }
    uint32_t place_of(uint32_t s) { return I.nel[s] == 1 ? vreg() : mem(I.nel[s]); }
    void put_m(uint32_t cls, std::initializer_list<uint32_t> m, uint32_t imm = 0, std::initializer_list<uint32_t> r = {},
               uint32_t element = 0) {
        put(cls, r, imm);
        WOp &u = ops.back();
        for (uint32_t x : m) u.m[u.n_mem++] = x;
        u.e[0] = element;
    }
    // the matrix operand s (a scalar put into a matrix of its own)
    uint32_t as_matrix(uint32_t nel, uint32_t where) {
        if (nel > 1) return where;
        const uint32_t m = mem(1);
        put_m(STE, {m}, 0, {where});
        return m;
    }
    uint32_t element(uint32_t m, uint32_t e) {
        const uint32_t v = vreg();
        put_m(LDE, {m}, 0, {v}, e);
        return v;
    }
    uint32_t quads(uint32_t nel) const { return (nel + 3) / 4; }
    uint32_t rows_of(uint32_t s) const { return mats ? quads(I.nel[s]) : 1; }

    uint32_t konst(double v) {
        uint64_t bits;
        std::memcpy(&bits, &v, 8);
        auto it = const_of.emplace(bits, uint32_t(consts.size()));
        if (it.second) consts.push_back(v);
        return kConst0 + it.first->second;
    }
    uint32_t vreg() { return kVirtual + n_virtual++; }
    void put(uint32_t cls, std::initializer_list<uint32_t> r, uint32_t imm = 0) {
        WOp u;
        u.cls = uint8_t(cls);
        u.imm = imm;
        for (uint32_t x : r) u.r[u.n++] = x;
        ops.push_back(u);
    }
    void fma(uint32_t a, uint32_t x, uint32_t y, uint32_t z) { put(FMA, {x, y, z, a}); }
    // (used by most micro-ops: found once)
    uint32_t common[4] = {kNone, kNone, kNone, kNone};
    uint32_t konst(uint32_t i, double v) { return common[i] != kNone ? common[i] : common[i] = konst(v); }
    uint32_t one() { return konst(0, 1.0); }
    uint32_t minus_one() { return konst(1, -1.0); }
    uint32_t neg_zero() { return konst(2, -0.0); }
    uint32_t zero() { return konst(3, 0.0); }
    uint32_t param(uint32_t p) const { return kSlots + p; }
    uint32_t param_adj(uint32_t p) const { return kSlots + P + p; }

    // a value loaded from memory: taken from its slot by the placeholder
    uint32_t load(bool ckpt, uint32_t imm, bool late_row = false) {
        const uint32_t v = vreg();
        loads.push_back({uint32_t(ops.size()), v, ckpt, imm, ckpt ? stored_at.at(imm) : 0, late_row});
        fma(v, 0, one(), neg_zero());
        return v;
    }
    void store(uint32_t s, uint32_t where, uint32_t row) {
        for (uint32_t q = 0; q < rows_of(s); ++q, ++row) {
            if (stored_at.size() <= row) stored_at.resize(row + 1, 0);
            stored_at[row] = uint32_t(ops.size());
            if (I.nel[s] == 1) put(CKST, {where}, row);
            else put_m(CKSTM, {where}, row, {}, 4 * q);
        }
    }

    // register of a static slot negated
    uint32_t negated(uint32_t s) {
        s = I.rep[s];
        if (I.kind[s] == K_CONST) return konst(-t.consts[t.ops[s].imm]);
        const uint32_t p = t.ops[s].imm;
        auto it = neg_param.find(p);
        return it != neg_param.end() ? it->second : kNone;
    }

    // whether forward_matrix and reverse_matrix are asked about an op: those of a
    // program with matrices, and matrix words on scalars (moves) in any program
    bool has_matrix_form(const TapeOp &o) const {
        return mats || o.code == tp::TRANSPOSE || o.code == tp::PACK || o.code == tp::INDEX;
    }
    // a value with a matrix among its operands or as its result; false: none
    template <class F>
    bool forward_matrix(uint32_t k, F operand, uint32_t dst) {
        const TapeOp &o = t.ops[k];
        const uint32_t n = I.nel[k];
        switch (o.code) {
        case tp::MATMUL: {
            const uint32_t a = as_matrix(I.nel[o.a], operand(o.a)), b = as_matrix(I.nel[o.b], operand(o.b));
            const uint32_t d = n == 1 ? mem(1) : dst;
            put_m(MM, {a, b, d}, mat_imm(t.ops[o.a].rows, t.ops[o.a].cols, t.ops[o.b].cols));
            if (n == 1) put_m(LDE, {d}, 0, {dst});
            return true;
        }
        case tp::ADD: case tp::SUB:
            if (n == 1) return false;
            put_m(VADD, {operand(o.a), operand(o.b), dst}, quads(n) | (o.code == tp::SUB ? kNegBit : 0u));
            return true;
        case tp::MUL: {
            if (n == 1) return false;
            const bool as = I.nel[o.a] == 1;
            const uint32_t x = operand(as ? o.a : o.b);
            put_m(VSCALE, {operand(as ? o.b : o.a), dst}, quads(n), {x, kSink});
            return true;
        }
        case tp::TRANSPOSE:
            if (n == 1) fma(dst, operand(o.a), one(), neg_zero());
            else put_m(TRANS, {operand(o.a), dst}, mat_imm(t.ops[o.a].rows, t.ops[o.a].cols, 0));
            return true;
        case tp::PACK:
            for (uint32_t i = 0; i < o.b; ++i) {
                const uint32_t x = operand(t.aux[o.a + i]);
                if (n == 1) fma(dst, x, one(), neg_zero());
                else put_m(STE, {dst}, 0, {x}, i);
            }
            return true;
        case tp::INDEX:
            if (I.nel[o.a] == 1) fma(dst, operand(o.a), one(), neg_zero());
            else put_m(LDE, {operand(o.a)}, 0, {dst}, o.imm);
            return true;
        case tp::INV:
            put_m(INV2, {operand(o.a), dst});
            return true;
        case tp::LOGDET: {
            const uint32_t d = vreg();
            put_m(DET2, {operand(o.a)}, 0, {one(), d});
            put(LOGC, {d, dst});
            return true;
        }
        default: return false;
        }
    }

    template <class F>
    void forward_op(uint32_t k, F operand, uint32_t dst) {
        const TapeOp &o = t.ops[k];
        if (has_matrix_form(o) && forward_matrix(k, operand, dst)) return;
        switch (o.code) {
        case tp::ADD: case tp::SUB: case tp::MUL: {
            if (I.fmul[k]) {
                const uint32_t m = I.fmul[k] - 1;
                const bool first = I.rep[o.a] == m;
                const uint32_t z = operand(first ? o.b : o.a);
                uint32_t x = operand(t.ops[m].a), y = operand(t.ops[m].b);
                if (o.code == tp::SUB) {   // z - x*y, one factor static
                    if (I.is_static(t.ops[m].a))
                        x = negated(t.ops[m].a);
                    else
                        y = negated(t.ops[m].b);
                }
                fma(dst, x, y, z);
                return;
            }
            const uint32_t a = operand(o.a), b = operand(o.b);
            if (o.code == tp::ADD) fma(dst, a, one(), b);
            else if (o.code == tp::SUB) fma(dst, b, minus_one(), a);
            else fma(dst, a, b, neg_zero());
            return;
        }
        case tp::NEG: fma(dst, operand(o.a), minus_one(), neg_zero()); return;
        case tp::SELECT:
            put(SEL, {operand(o.a), operand(o.b), operand(o.c), operand(o.d), dst});
            return;
        default: break;
        }
        switch (o.code) {
        case tp::DIV: put(DIV, {operand(o.a), operand(o.b), dst}); return;
        case tp::POW: put(POW, {operand(o.a), operand(o.b), dst}); return;
        case tp::EXP: put(EXP, {operand(o.a), dst}); return;
        case tp::LOG: put(LOGC, {operand(o.a), dst}); return;
        case tp::SQRT: put(SQRTC, {operand(o.a), dst}); return;
        case tp::SIN: put(SIN, {operand(o.a), dst}); return;
        case tp::COS: put(COS, {operand(o.a), dst}); return;
        case tp::ABS: put(ABS, {operand(o.a), dst}); return;
        default: throw std::logic_error("unknown tape op in the wide scheduler");
        }
    }

    uint32_t fwd_operand(uint32_t s) {
        s = I.rep[s];
        switch (I.kind[s]) {
        case K_CONST: return konst(t.consts[t.ops[s].imm]);
        case K_PARAM: return param(t.ops[s].imm);
        case K_OBS:
            if (fval[s] == kNone) fval[s] = load(false, 8 * t.ops[s].imm);
            return fval[s];
        default: return fval[s];
        }
    }

    uint32_t rev_operand(uint32_t s, uint32_t j) {
        s = I.rep[s];
        if (I.kind[s] == K_CONST || I.kind[s] == K_PARAM) return fwd_operand(s);
        if (I.kind[s] == K_COMP && B.resident[s]) return fval[s];
        if (rval_of[s] == j + 1) return rval[s];
        if (I.kind[s] != K_OBS && row_of[s] != j + 1) throw std::logic_error("value read outside its segment");
        if (I.nel[s] == 1) {
            set_rval(s, j, I.kind[s] == K_OBS ? load(false, 8 * t.ops[s].imm) : load(true, row[s]));
        } else {
            const uint32_t m = mem(I.nel[s]);
            for (uint32_t q = 0; q < rows_of(s); ++q) put_m(STE4, {m}, 0, {load(true, row[s] + q)}, 4 * q);
            set_rval(s, j, m);
        }
        return rval[s];
    }
    void set_rval(uint32_t s, uint32_t j, uint32_t v) {
        rval[s] = v;
        rval_of[s] = j + 1;
    }

    // register of a target's adjoint; *first: its first contribution
    uint32_t target(uint32_t s, bool *first) {
        *first = false;
        if (I.kind[s] == K_PARAM) return param_adj(t.ops[s].imm);
        if (I.kind[s] != K_COMP || !I.active[s]) return kNone;
        if (adj[s] == kNone) {
            adj[s] = place_of(s);
            *first = true;
        }
        return adj[s];
    }

    // +0 in register r: an earlier micro-op near by that clears none does it,
    // else one of its own (a zero adjoint contributes nothing)
    void clear(uint32_t r) {
        for (size_t i = ops.size(), n = 0; i-- > rev_begin && n < kLookBack; ++n)
            if ((ops[i].cls == DUAL || ops[i].cls == SELADJ || ops[i].cls == DIVADJ || ops[i].cls == ACCD) &&
                ops[i].r[1] == kSink) {
                ops[i].r[1] = r;
                return;
            }
        put(DUAL, {zero(), r, one(), kSink, one(), kSink});
    }
    size_t rev_begin = 0;

    // a1 += g * y1, a2 += g * y2 where g != 0
    void dual(uint32_t g, uint32_t a1, bool f1, uint32_t y1, uint32_t a2, bool f2, uint32_t y2) {
        if (a1 == kNone && a2 == kNone) return;
        uint32_t zr = kSink;
        if (a1 == kNone) a1 = kSink, y1 = one();
        if (a2 == kNone) a2 = kSink, y2 = one();
        if (f1) zr = a1;
        if (f2) {
            if (zr != kSink) clear(a2);
            else zr = a2;
        }
        put(DUAL, {g, zr, y1, a1, y2, a2});
    }
    // a, or +0 for a first contribution
    uint32_t base(uint32_t a, bool first) { return first ? zero() : a; }

    // The adjoint rule of an op with matrices; false: it has none.  Where the
    // contribution is the adjoint itself no gate is needed: a zero changes no
    // sum, which is never -0 (it starts at +0).
    bool reverse_matrix(uint32_t k, uint32_t j, uint32_t g) {
        const TapeOp &o = t.ops[k];
        const uint32_t n = I.nel[k];
        auto v = [&](uint32_t s) { return rev_operand(s, j); };
        bool f1 = false, f2 = false;
        auto first = [](bool f) { return f ? kFirstBit : 0u; };
        // a += c for a scalar target
        auto add = [&](uint32_t a, bool f, uint32_t c) { fma(a, c, one(), base(a, f)); };
        switch (o.code) {
        case tp::ADD: case tp::SUB: {
            if (n == 1) return false;
            const uint32_t a1 = target(o.a, &f1);
            if (a1 != kNone) put_m(VACC, {g, a1}, quads(n) | first(f1));
            const uint32_t a2 = target(o.b, &f2);
            if (a2 != kNone) put_m(VACC, {g, a2}, quads(n) | first(f2) | (o.code == tp::SUB ? kNegBit : 0u));
            return true;
        }
        case tp::MUL: {
            if (n == 1) return false;
            const bool as = I.nel[o.a] == 1;
            const uint32_t sc = as ? o.a : o.b, ma = as ? o.b : o.a;
            auto scalar = [&]() {
                const uint32_t M = I.takes_adjoint(sc) ? v(ma) : 0, a = target(sc, &f1);
                if (a == kNone) return;
                const uint32_t c = vreg();
                put_m(SDOT, {g, M}, n, {one(), c});
                add(a, f1, c);
            };
            auto matrix = [&]() {
                const uint32_t S = I.takes_adjoint(ma) ? v(sc) : 0, a = target(ma, &f2);
                if (a != kNone) put_m(VACCS, {g, a}, n | first(f2), {S, kSink});
            };
            if (as) scalar(), matrix();
            else matrix(), scalar();
            return true;
        }
        case tp::MATMUL: {
            const uint32_t imm = mat_imm(t.ops[o.a].rows, t.ops[o.a].cols, t.ops[o.b].cols);
            const uint32_t G = as_matrix(n, g);
            for (int side = 0; side < 2; ++side) {
                const uint32_t x = side ? o.b : o.a, y = side ? o.a : o.b;
                const uint32_t other = I.takes_adjoint(x) ? as_matrix(I.nel[y], v(y)) : 0;
                const uint32_t a = target(x, &f1);
                if (a == kNone) continue;
                const bool sc = I.nel[x] == 1;
                const uint32_t T = sc ? mem(1) : a, im = imm | first(sc || f1);
                if (side) put_m(MMB, {other, G, T}, im);
                else put_m(MMA, {G, other, T}, im);
                if (sc) add(a, f1, element(T, 0));
            }
            return true;
        }
        case tp::TRANSPOSE: {
            const uint32_t a = target(o.a, &f1);
            if (a == kNone) return true;
            if (n == 1) add(a, f1, g);
            else put_m(TRANSACC, {g, a}, mat_imm(t.ops[o.a].rows, t.ops[o.a].cols, 0) | first(f1));
            return true;
        }
        case tp::PACK:
            for (uint32_t i = 0; i < o.b; ++i) {
                const uint32_t a = target(t.aux[o.a + i], &f1);
                if (a != kNone) add(a, f1, n == 1 ? g : element(g, i));
            }
            return true;
        case tp::INDEX: {
            const uint32_t a = target(o.a, &f1), ne = I.nel[o.a];
            if (a == kNone) return true;
            if (ne == 1) {
                add(a, f1, g);
                return true;
            }
            for (uint32_t i = 0; f1 && i < ne; ++i)
                if (i != o.imm) put_m(STE, {a}, 0, {zero()}, i);
            const uint32_t c = vreg();
            fma(c, g, one(), f1 ? zero() : element(a, o.imm));
            put_m(STE, {a}, 0, {c}, o.imm);
            return true;
        }
        case tp::INV: {
            const uint32_t Z = v(k), a = target(o.a, &f1);
            if (a != kNone) put_m(INV2ACC, {Z, g, a}, first(f1));
            return true;
        }
        case tp::LOGDET: {
            const uint32_t A = v(o.a), a = target(o.a, &f1);
            if (a != kNone) put_m(LOGDETACC, {A, a}, first(f1), {g, kSink});
            return true;
        }
        default: return false;
        }
    }

    void reverse_op(uint32_t k, uint32_t j) {
        const TapeOp &o = t.ops[k];
        const uint32_t g = adj[k];
        if (g == kNone) throw std::logic_error("adjoint rule laid out before any contribution to it");
        auto v = [&](uint32_t s) { return rev_operand(s, j); };
        if (has_matrix_form(o) && reverse_matrix(k, j, g)) return;
        bool f1 = false, f2 = false;
        switch (o.code) {
        case tp::ADD: case tp::SUB: {
            const uint32_t a1 = target(o.a, &f1), a2 = target(o.b, &f2);
            dual(g, a1, f1, one(), a2, f2, o.code == tp::ADD ? one() : minus_one());
            return;
        }
        case tp::MUL: {
            const uint32_t A = I.takes_adjoint(o.b) ? v(o.a) : 0, Bv = I.takes_adjoint(o.a) ? v(o.b) : 0;
            const uint32_t a1 = target(o.a, &f1), a2 = target(o.b, &f2);
            dual(g, a1, f1, Bv, a2, f2, A);
            return;
        }
        case tp::NEG: {
            const uint32_t a1 = target(o.a, &f1);
            dual(g, a1, f1, minus_one(), kNone, false, 0);
            return;
        }
        case tp::EXP: {
            const uint32_t Z = v(k), a1 = target(o.a, &f1);
            dual(g, a1, f1, Z, kNone, false, 0);
            return;
        }
        case tp::DIV: {
            const uint32_t Bv = v(o.b), Z = I.takes_adjoint(o.b) ? v(k) : 0;
            uint32_t a1 = target(o.a, &f1), a2 = target(o.b, &f2);
            if (a2 == kNone) {
                if (a1 != kNone) put(ACCD, {g, f1 ? a1 : kSink, Bv, a1, g});
                return;
            }
            if (a1 == kNone) a1 = kSink;
            uint32_t zr = f1 ? a1 : kSink;
            if (f2) {
                if (zr != kSink) clear(a2);
                else zr = a2;
            }
            put(DIVADJ, {g, zr, Bv, a1, Z, a2});
            return;
        }
        case tp::POW: {
            const uint32_t A = v(o.a), Bv = I.takes_adjoint(o.a) ? v(o.b) : 0, Z = v(k);
            const uint32_t a1 = target(o.a, &f1);
            if (a1 != kNone) {   // ((g * b) * z) / a
                const uint32_t t1 = vreg(), t2 = vreg();
                fma(t1, g, Bv, neg_zero());
                fma(t2, t1, Z, neg_zero());
                put(ACCD, {g, f1 ? a1 : kSink, A, a1, t2});
            }
            const uint32_t a2 = target(o.b, &f2);
            if (a2 != kNone) {   // (g * z) * ln a
                const uint32_t t3 = vreg();
                fma(t3, g, Z, neg_zero());
                put(ACCPOW, {g, A, t3, base(a2, f2), a2});
            }
            return;
        }
        case tp::LOG: case tp::SIN: case tp::COS: case tp::ABS: {
            const uint32_t A = v(o.a), a1 = target(o.a, &f1);
            if (a1 == kNone) return;
            const uint32_t cls = o.code == tp::LOG ? ACCLOG : o.code == tp::SIN ? ACCSIN : o.code == tp::COS ? ACCCOS : ACCABS;
            put(cls, {g, A, base(a1, f1), a1});
            return;
        }
        case tp::SQRT: {
            const uint32_t A = v(o.a), Z = v(k), a1 = target(o.a, &f1);
            if (a1 != kNone) put(ACCSQRT, {g, A, Z, base(a1, f1), a1});
            return;
        }
        case tp::SELECT: {
            const uint32_t A = v(o.a), Bv = v(o.b);
            uint32_t a1 = target(o.c, &f1), a2 = target(o.d, &f2);
            if (a1 == kNone && a2 == kNone) return;
            if (a1 == kNone) a1 = kSink;
            if (a2 == kNone) a2 = kSink;
            uint32_t zr = f1 ? a1 : kSink;
            if (f2) {
                if (zr != kSink) clear(a2);
                else zr = a2;
            }
            put(SELADJ, {g, zr, A, Bv, a1, a2});
            return;
        }
        default:
            throw std::logic_error("unknown tape op in the wide reverse scheduler");
        }
    }

    // ---- values that only the loss needs
    // The recompute policy forms a value twice: in the forward sweep and in its
    // segment's reverse sweep.  Where nothing the reverse sweep starts from
    // depends on it (terms of a sum: only the loss reads them), the forward
    // sweep leaves it out, the reverse sweep stores the last such values that
    // it recomputes, and the loss is formed from them at the end, by the same
    // operations in the same order.  Done where the operations left out cost
    // more than the rows' stores and loads (kRowCost each).
    static constexpr uint32_t kRowCost = 110;
    std::vector<uint8_t> in_forward;                    // computed by the forward sweep
    std::vector<uint8_t> late;                          // computed after the reverse sweep
    std::unordered_map<uint32_t, uint32_t> late_row;    // value -> row it is stored to for the end
    void plan_late() {
        in_forward.assign(N, 1);
        late.assign(N, 0);
        if (!with_grad || mats || B.save_reads || I.kind[t.loss] != K_COMP) return;
        std::vector<uint8_t> need(N, 0), recomputed(N, 0);
        for (const auto &v : B.livein)
            for (uint32_t s : v) need[s] = 1;
        for (uint32_t s = 0; s < N; ++s) need[s] = need[s] || (B.resident[s] && B.comp_live(s));
        for (uint32_t k = N; k-- > 0;)
            if (need[k] && I.kind[k] == K_COMP) I.for_operands(k, [&](uint32_t s) { need[s] = 1; });
        for (const auto &v : B.recomp)
            for (uint32_t s : v) recomputed[s] = 1;
        // from the loss back: what is formed at the end, what is loaded
        std::vector<uint8_t> end(N, 0);
        std::vector<uint32_t> rows;
        end[I.rep[t.loss]] = 1;
        for (uint32_t k = N; k-- > 0;) {
            if (!end[k] || I.kind[k] != K_COMP) continue;
            if (B.resident[k]) continue;
            if (recomputed[k] || need[k]) {
                rows.push_back(k);
                continue;
            }
            late[k] = 1;
            I.for_operands(k, [&](uint32_t s) { end[s] = 1; });
        }
        uint64_t saved = 0;
        for (uint32_t k = 0; k < N; ++k)
            if (B.comp_live(k) && I.rep[k] == k && !need[k] && !late[k]) saved += class_cost(class_of(k));
        if (saved <= uint64_t(kRowCost) * rows.size()) {
            late.assign(N, 0);
            return;
        }
        for (uint32_t k = 0; k < N; ++k) in_forward[k] = need[k];
        for (uint32_t k : rows) late_row[k] = n_rows++;
    }
    // class of a value's operation
    uint32_t class_of(uint32_t k) const {
        switch (t.ops[k].code) {
        case tp::DIV: return DIV;
        case tp::POW: return POW;
        case tp::EXP: return EXP;
        case tp::LOG: return LOGC;
        case tp::SQRT: return SQRTC;
        case tp::SIN: return SIN;
        case tp::COS: return COS;
        case tp::ABS: return ABS;
        case tp::SELECT: return SEL;
        default: return FMA;
        }
    }

    void run() {
        const uint32_t m = uint32_t(B.cuts.size());
        // static registers: parameters, their adjoints, the sink, constants
        kSink = kSlots + P + (with_grad ? P : 0);
        kConst0 = kSink + 1;
        fval.assign(N, kNone);
        adj.assign(N, kNone);
        rval.assign(N, 0);
        rval_of.assign(N, 0);
        row.assign(N, 0);
        row_of.assign(N, 0);
        n_rows = 0;
        for (uint32_t j = 0; with_grad && j < m; ++j) {
            first_row.push_back(n_rows);
            for (uint32_t s : B.livein[j]) n_rows += rows_of(s);
        }
        plan_late();
        const bool late_loss = !late_row.empty();
        // negated parameters that folded differences multiply by
        for (uint32_t k = 0; k < N; ++k) {
            if (!I.fmul[k] || t.ops[k].code != tp::SUB) continue;
            const TapeOp &mo = t.ops[I.fmul[k] - 1];
            const uint32_t s = I.rep[I.is_static(mo.a) ? mo.a : mo.b];
            if (I.kind[s] != K_PARAM || neg_param.count(t.ops[s].imm)) continue;
            const uint32_t r = vreg();
            neg_param[t.ops[s].imm] = r;
            fma(r, param(t.ops[s].imm), minus_one(), neg_zero());
        }
        std::unordered_map<uint32_t, std::vector<uint32_t>> saves_of;   // save policy: rows of each stored value
        if (with_grad && B.save_reads)
            for (uint32_t j = 0; j < m; ++j)
                for (uint32_t i = 0, r = first_row[j]; i < B.livein[j].size(); r += rows_of(B.livein[j][i]), ++i)
                    saves_of[B.livein[j][i]].push_back(r);
        uint32_t next_cut = 1;
        auto fwd = [&](uint32_t s) { return fwd_operand(s); };
        for (uint32_t k = 0; k < N; ++k) {
            if (with_grad && !B.save_reads)
                while (next_cut < m && B.cuts[next_cut] == k) {
                    uint32_t r = first_row[next_cut];
                    for (uint32_t s : B.livein[next_cut]) {
                        store(s, fval[s], r);
                        r += rows_of(s);
                    }
                    ++next_cut;
                }
            if (!B.comp_live(k) || I.rep[k] != k || !in_forward[k]) continue;
            const uint32_t dst = place_of(k);
            forward_op(k, fwd, dst);
            fval[k] = dst;
            auto lr = late_row.find(k);
            if (lr != late_row.end()) store(k, dst, lr->second);
            if (with_grad && B.save_reads) {
                auto it = saves_of.find(k);
                if (it != saves_of.end())
                    for (uint32_t r : it->second) store(k, dst, r);
            }
        }
        if (!late_loss) put(STLOSS, {fwd_operand(t.loss)});
        if (with_grad) {
            rev_begin = ops.size();
            bool f;
            const uint32_t seed = target(t.loss, &f);
            if (seed != kNone) {
                if (f) fma(seed, one(), one(), neg_zero());
                else fma(seed, one(), one(), seed);   // the loss is a parameter
            }
            for (uint32_t j = m; j-- > 0;) {
                uint32_t r = first_row[j];
                for (uint32_t s : B.livein[j]) {
                    row[s] = r;
                    row_of[s] = j + 1;
                    r += rows_of(s);
                }
                for (uint32_t s : B.recomp[j]) {
                    if (I.kind[s] == K_OBS) continue;   // loaded where first read
                    auto opnd = [&](uint32_t x) { return rev_operand(x, j); };
                    const uint32_t dst = place_of(s);
                    forward_op(s, opnd, dst);
                    set_rval(s, j, dst);
                    auto lr = late_row.find(s);
                    if (lr != late_row.end() && !in_forward[s] && !(lr->second < stored_at.size() && stored_at[lr->second]))
                        store(s, dst, lr->second);
                }
                for (uint32_t k : B.revops[j]) reverse_op(k, j);
            }
            for (uint32_t p = 0; p < P; ++p) put(STGRAD, {param_adj(p)}, 8 * p);
            if (late_loss) {
                // the observations read at the end are loaded anew, the values
                // of the forward sweep (residents apart) are gone
                for (uint32_t k = 0; k < N; ++k)
                    if (!(I.kind[k] == K_COMP && B.resident[k])) fval[k] = kNone;
                auto opnd = [&](uint32_t s) {
                    s = I.rep[s];
                    if (I.kind[s] == K_COMP && fval[s] == kNone) fval[s] = load(true, late_row.at(s), true);
                    return fwd_operand(s);
                };
                for (uint32_t k = 0; k < N; ++k) {
                    if (!late[k]) continue;
                    const uint32_t dst = vreg();
                    forward_op(k, opnd, dst);
                    fval[k] = dst;
                }
                put(STLOSS, {opnd(t.loss)});
            }
        }
        put(END, {});
        n_static = (with_grad ? 2 : 1) * P + 1 + uint32_t(consts.size());
    }
    uint32_t n_rows = 0;
};

// Checkpoint slots per half that a program uses: a recomputing program
// restores a few rows per segment and is short of registers; a saving one
// restores every value a rule reads and has registers to spare.  The rows the
// loss is formed from at the end come one after the other with little work
// between them, and few registers are live by then: they use all slots.
uint32_t ck_slots(bool save_reads, bool matrices) { return save_reads || matrices ? kCkSlots : 4; }

// Loads issued ahead: the loads of each kind (observations, checkpoint rows)
// go in batches of up to half its slots.  While the values of one batch are
// used the next one is in flight: it is issued when the first value of the
// batch before is taken, or when the last value of the batch before that has
// left its slot, if later.  The first value taken of a batch waits for it.  A
// value whose last reader is near is read from its slot directly (its
// placeholder goes).
// *late_at: the op from which on every checkpoint slot may be in use.
std::vector<WOp> place_loads(const Lower &W, uint32_t ck_cap, uint32_t *late_at) {
    const uint32_t n = uint32_t(W.ops.size());
    std::vector<uint32_t> last(W.n_virtual, 0);
    for (uint32_t i = 0; i < n; ++i)
        for (uint32_t q = 0; q < W.ops[i].n; ++q)
            if (W.ops[i].r[q] >= kVirtual) last[W.ops[i].r[q] - kVirtual] = i;
    struct At {
        std::vector<WOp> before, after;   // of an op
    };
    std::unordered_map<uint32_t, At> at;
    std::vector<uint8_t> drop(n, 0), marked(n, 0);     // marked: in `at`
    std::vector<uint32_t> alias(W.n_virtual, kNone);   // virtual register -> slot
    std::unordered_map<uint32_t, uint32_t> slot_at;    // placeholder -> slot
    std::vector<WOp> head;                             // issued at the program's start
    for (int kind = 0; kind < 2; ++kind) {
        const bool ckpt = kind == 1;
        const uint32_t size = ckpt ? kCkSlots : kObsSlots;
        std::vector<const Lower::Load *> q;
        for (const auto &l : W.loads)
            if (l.ckpt == ckpt) q.push_back(&l);
        uint32_t done[2] = {kUnsetTime, kUnsetTime};   // last use of the values of the batch in each half
        // batches: a row is stored before its batch's first value is taken
        std::vector<size_t> begin{0};
        for (size_t i = 0; i < q.size(); ++i) {
            const Lower::Load &f = *q[begin.back()];
            const uint32_t cap = !ckpt ? kObsSlots : f.late ? kCkSlots : ck_cap;
            if (i - begin.back() == cap || q[i]->after >= f.at || q[i]->late != f.late) begin.push_back(i);
        }
        begin.push_back(q.size());
        for (size_t nb = 0, half = 0; nb + 1 < begin.size() && !q.empty(); ++nb, half ^= 1) {
            const size_t b = begin[nb];
            const uint32_t c = uint32_t(begin[nb + 1] - b);
            const uint32_t slot0 = (ckpt ? 2 * kObsSlots : 0) + uint32_t(half) * size;
            // every value of the batch leaves its slot before the first value
            // of the half's next batch is taken
            const uint32_t limit = nb + 3 < begin.size() ? q[begin[nb + 2]]->at : n;
            std::vector<WOp> issue;
            uint32_t end_of_batch = 0, stored = 0;
            for (uint32_t i = 0; i < c; ++i) {
                const Lower::Load &l = *q[b + i];
                const uint32_t slot = slot0 + size - c + i;   // a short batch enters its block late
                WOp u;
                u.cls = uint8_t((ckpt ? LDK0 : LDO0) + half);
                u.imm = l.imm;
                u.late = l.late;
                issue.push_back(u);
                stored = std::max(stored, l.after);
                const uint32_t end = last[l.reg - kVirtual];
                if (end - l.at <= kSlotHold && end < limit) {
                    alias[l.reg - kVirtual] = slot;
                    drop[l.at] = 1;
                    end_of_batch = std::max(end_of_batch, end);
                } else {
                    slot_at[l.at] = slot;
                    at[l.at];   // (marked below)
                    end_of_batch = std::max(end_of_batch, l.at);
                }
            }
            // Issued when the first value of the batch before is taken, when the
            // half's last values have left it, and (checkpoint rows) when the
            // rows have been stored, whichever is last; the first two batches
            // of observations at the program's start.
            std::vector<WOp> *dst = &head;
            uint32_t after = nb >= 2 ? done[half] : 0;
            if (ckpt) after = std::max(after, stored);
            if (nb >= 2 || ckpt) {
                const uint32_t first_before = nb >= 1 ? q[begin[nb - 1]]->at : 0;
                dst = nb >= 1 && after < first_before ? &at[first_before].before : &at[after].after;
            }
            dst->insert(dst->end(), issue.begin(), issue.end());
            WOp w;
            w.cls = WAIT;
            auto &before = at[q[b]->at].before;
            before.insert(before.begin(), w);
            done[half] = end_of_batch;
        }
    }
    std::vector<WOp> out;
    out.reserve(n + W.loads.size() * 2);
    *late_at = UINT32_MAX;
    bool pending = false;   // loads issued since the last wait
    auto add = [&](const WOp &u) {
        if (u.cls == WAIT && !pending) return;
        if (u.cls == WAIT) pending = false;
        if (u.cls >= LDK0 && u.cls <= LDO1) pending = true;
        if (u.late && *late_at == UINT32_MAX) *late_at = uint32_t(out.size());
        out.push_back(u);
    };
    for (const WOp &u : head) add(u);
    for (const auto &a : at) marked[a.first] = 1;
    for (uint32_t i = 0; i < n; ++i) {
        const At *here = marked[i] ? &at.at(i) : nullptr;
        if (here)
            for (const WOp &u : here->before) add(u);
        if (!drop[i]) {
            WOp u = W.ops[i];
            if (here) {
                auto s = slot_at.find(i);
                if (s != slot_at.end()) u.r[0] = s->second;
            }
            for (uint32_t q = 0; q < u.n; ++q)
                if (u.r[q] >= kVirtual && alias[u.r[q] - kVirtual] != kNone) u.r[q] = alias[u.r[q] - kVirtual];
            out.push_back(u);
        }
        if (here)
            for (const WOp &u : here->after) add(u);
    }
    return out;
}

// Linear scan: every virtual register to the lowest register free over its
// whole life.  A register read for the last time by a micro-op may be the one
// it writes at its end.  `spare`: registers below the statics that are free
// (load slots the program does not use); `early`: those free for lives that
// end before op late_at, the one freed last first.  Returns the registers used,
// or `limit` + 1 where they are more than `limit` (at most 128).
uint32_t place_registers(std::vector<WOp> &ops, uint32_t n_virtual, uint32_t n_static,
                         const std::vector<uint32_t> &spare, const std::vector<uint32_t> &early, uint32_t late_at,
                         uint32_t limit) {
    // Lives, in half op steps (a write at a micro-op's end is the later half).
    std::vector<uint32_t> first(n_virtual, kUnsetTime), last(n_virtual, 0), order;
    order.reserve(n_virtual);
    for (uint32_t i = 0; i < ops.size(); ++i) {
        const WOp &u = ops[i];
        const char *role = roles(u.cls);
        const size_t seen = order.size();
        for (uint32_t q = 0; q < u.n; ++q) {
            if (u.r[q] < kVirtual) continue;
            const uint32_t v = u.r[q] - kVirtual;
            const uint32_t when = 2 * i + (role[q] == 'd' ? 1 : 0);
            if (first[v] == kUnsetTime) {
                first[v] = when;
                order.push_back(v);
            }
            last[v] = std::max(last[v], when);
        }
        if (order.size() > seen + 1)
            std::sort(order.begin() + seen, order.end(),
                      [&](uint32_t a, uint32_t b) { return first[a] != first[b] ? first[a] < first[b] : a < b; });
    }
    // free registers by number, the early ones as a stack; the lives that end
    // at each half step as a list
    uint64_t open[2] = {0, 0};
    auto release = [&](uint32_t r) { open[r / 64] |= 1ull << (r % 64); };
    for (uint32_t r : spare) release(r);
    std::vector<uint32_t> free_early(early.rbegin(), early.rend());
    std::vector<uint8_t> is_early(kSlots, 0);
    for (uint32_t r : early) is_early[r] = 1;
    std::vector<uint32_t> reg(n_virtual, 0), ends(2 * ops.size(), kNone), link(n_virtual, kNone), ended;
    uint32_t next = kSlots + n_static, now = 0;
    for (uint32_t v : order) {
        for (; now < first[v]; ++now) {
            if (ends[now] == kNone) continue;
            ended.clear();
            for (uint32_t x = ends[now]; x != kNone; x = link[x]) ended.push_back(reg[x]);
            if (ended.size() > 1) std::sort(ended.begin(), ended.end());
            for (uint32_t r : ended) {
                if (r < kSlots && is_early[r]) free_early.push_back(r);
                else release(r);
            }
        }
        uint32_t r;
        if (!free_early.empty() && last[v] / 2 < late_at) {
            r = free_early.back();
            free_early.pop_back();
        } else if (open[0] | open[1]) {
            r = open[0] ? uint32_t(__builtin_ctzll(open[0])) : 64 + uint32_t(__builtin_ctzll(open[1]));
            open[r / 64] &= open[r / 64] - 1;
        } else {
            r = next++;
            if (next > limit) return next;
        }
        reg[v] = r;
        link[v] = ends[last[v]];
        ends[last[v]] = v;
    }
    for (WOp &u : ops)
        for (uint32_t q = 0; q < u.n; ++q)
            if (u.r[q] >= kVirtual) u.r[q] = reg[u.r[q] - kVirtual];
    return next;
}

// Orders the micro-ops of a scalar program into longer runs of one class (a
// block costs kDispatchCost however few it holds).  Between loads and waits,
// where the slots' contents change, any order that keeps each register's reads
// and writes in order gives the same bits.  Of the `window` oldest micro-ops
// left, the class is taken next that the longest run can be made of (a run may
// hold micro-ops that depend on each other); the window bounds what the order
// adds to the values held at a time.  Estimated cycles of a lone wave, in program
// order against windows of 8, 16, 32 and 64 (thousands): logistic saving 776
// against 671, 647, 646, 646; Lotka-Volterra saving 1849 against 1590, 1583,
// 1559, 1559, recomputing (runs of 9 as it is) 1646 against 1649, 1648, 1647,
// 1646; twelve random programs 11.8 against 11.6, 11.2, 11.0, 11.0 million.
constexpr uint32_t kOrderWindow = 32;   // (at most 64: members are bits of a word)
void order_ops(std::vector<WOp> &ops, uint32_t n_virtual, uint32_t sink, uint32_t late_at, uint32_t window) {
    const uint32_t n_regs = kRegs + n_virtual;
    auto reg_of = [&](uint32_t r) { return r < kVirtual ? r : kRegs + (r - kVirtual); };
    // of each register, in this region: its last writer, and the readers since
    std::vector<uint32_t> writer(n_regs, 0), seen(n_regs, 0);
    std::vector<std::vector<uint32_t>> readers(n_regs);
    uint32_t region = 0;
    std::vector<uint32_t> preds, preds_of;   // of op i in the region: preds[preds_of[i] .. preds_of[i + 1]]
    std::vector<uint32_t> mark_of;           // run that last held the op (0: none; kNone: placed)
    std::vector<uint32_t> ahead, run, best, classes;   // ahead: the window's ops, in order
    uint64_t members[kClasses];
    std::vector<WOp> out;
    auto fixed = [&](uint32_t cls) { return cls >= LDK0 && cls <= WAITPF; };
    for (uint32_t b = 0; b < ops.size();) {
        uint32_t e = b;
        while (e < ops.size() && !fixed(ops[e].cls) && ops[e].cls != PF && ops[e].cls != WAIT &&
               !(e == late_at && e > b))
            ++e;
        if (e - b < 3) {
            b = std::max(e, b + 1);
            continue;
        }
        const uint32_t n = e - b;
        ++region;
        preds.clear();
        preds_of.assign(1, 0);
        for (uint32_t i = 0; i < n; ++i) {
            const WOp &u = ops[b + i];
            const char *role = roles(u.cls);
            for (uint32_t q = 0; q < u.n; ++q) {
                if (role[q] == '-' || u.r[q] == sink) continue;
                const uint32_t r = reg_of(u.r[q]);
                if (seen[r] != region) {
                    seen[r] = region;
                    writer[r] = kNone;
                    readers[r].clear();
                }
                if (writer[r] != kNone && writer[r] != i) preds.push_back(writer[r]);
                if (role[q] == 'u') {
                    readers[r].push_back(i);
                } else {
                    for (uint32_t k : readers[r])
                        if (k != i) preds.push_back(k);
                    readers[r].clear();
                    writer[r] = i;
                }
            }
            preds_of.push_back(uint32_t(preds.size()));
        }
        mark_of.assign(n, 0);
        uint32_t mark = 0, next = 0;
        out.clear();
        ahead.clear();
        for (;;) {
            while (next < n && ahead.size() < window) ahead.push_back(next++);
            if (ahead.empty()) break;
            best.clear();
            uint64_t present = 0;   // classes in the window; the ops of each, in the order of the classes' first
            classes.clear();
            for (uint32_t k = 0; k < ahead.size(); ++k) {
                const uint32_t cls = ops[b + ahead[k]].cls;
                if (!(present >> cls & 1u)) {
                    present |= 1ull << cls;
                    members[cls] = 0;
                    classes.push_back(cls);
                }
                members[cls] |= 1ull << k;
            }
            for (uint32_t cls : classes) {
                if (uint32_t(__builtin_popcountll(members[cls])) <= best.size()) continue;   // no longer run
                ++mark;
                run.clear();
                for (uint64_t left = members[cls]; left && run.size() < kInfo[cls].max; left &= left - 1) {
                    const uint32_t i = ahead[__builtin_ctzll(left)];
                    bool ready = true;
                    for (uint32_t p = preds_of[i + 1]; ready && p-- > preds_of[i];)
                        ready = mark_of[preds[p]] == kNone || mark_of[preds[p]] == mark;
                    if (!ready) continue;
                    mark_of[i] = mark;
                    run.push_back(i);
                }
                if (run.size() > best.size()) best.swap(run);
            }
            for (uint32_t i : best) {
                mark_of[i] = kNone;
                out.push_back(ops[b + i]);
            }
            ahead.erase(std::remove_if(ahead.begin(), ahead.end(), [&](uint32_t i) { return mark_of[i] == kNone; }),
                        ahead.end());
        }
        std::copy(out.begin(), out.end(), ops.begin() + b);
        b = e;
    }
}

// Places of the matrices in LDS, in elements: in the order they are first
// written, each to the lowest run of elements free over its whole life (the
// micro-op that writes a matrix may read the others throughout).  Returns the
// elements used.
uint32_t place_matrices(std::vector<WOp> &ops, const std::vector<uint32_t> &size) {
    const uint32_t n = uint32_t(size.size());
    std::vector<uint32_t> first(n, kUnsetTime), last(n, 0), order, at(n, 0);
    for (uint32_t i = 0; i < ops.size(); ++i)
        for (uint32_t q = 0; q < ops[i].n_mem; ++q) {
            const uint32_t v = ops[i].m[q];
            if (first[v] == kUnsetTime) {
                first[v] = i;
                order.push_back(v);
            }
            last[v] = i;
        }
    struct Run {
        uint32_t at, size, end;   // elements, last use
    };
    std::vector<Run> live;        // by place
    uint32_t top = 0;
    for (uint32_t v : order) {
        live.erase(std::remove_if(live.begin(), live.end(), [&](const Run &r) { return r.end < first[v]; }), live.end());
        uint32_t place = 0;
        size_t i = 0;
        for (; i < live.size() && live[i].at < place + size[v]; ++i) place = live[i].at + live[i].size;
        live.insert(live.begin() + i, {place, size[v], last[v]});
        at[v] = place;
        top = std::max(top, place + size[v]);
    }
    for (WOp &u : ops)
        for (uint32_t q = 0; q < u.n_mem; ++q) u.e[q] += at[u.m[q]];
    return top;
}

// words of one micro-op
void encode(const WOp &u, std::vector<uint32_t> *out) {
    uint32_t q = 0, word = 0, halves = 0, mem = 0;
    for (const char *c = roles(u.cls); *c; ++c) {
        if (*c == 'R' || *c == 'W' || *c == 'M') {
            out->push_back(u.e[mem++] * kLdsRow);
            continue;
        }
        if (*c == 'z') {
            out->push_back(0);
            continue;
        }
        if (*c == 'i') {
            out->push_back(u.imm);
            continue;
        }
        const uint32_t h = *c == '-' ? 0u
                                     : 2 * u.r[q++] | (*c == 'u' ? kSrc : *c == 'm' ? kSrc | kDst : kDst);
        word |= h << (16 * (halves & 1u));
        if (halves++ & 1u) {
            out->push_back(word);
            word = 0;
        }
    }
}

// The program is read once, by every wave in turn, and its blocks are short:
// a block's scalar loads are issued one block ahead, which hides an L2 hit
// but not a miss.  So the waves also fetch the program into the L2 cache some
// kPrefetch bytes ahead, where they wait for loads anyway (the fetch must not
// be in flight at the next wait), or in a block of its own.
void emit(const std::vector<WOp> &in, WideSchedule *S) {
    std::vector<WOp> ops;
    ops.reserve(in.size() + in.size() / 64 + 4);
    uint64_t total = 4 * kBlockWords;
    for (const WOp &u : in) total += 4 * kInfo[u.cls].words + 4;   // a header for every other micro-op
    // blocks of consecutive micro-ops of one class
    std::vector<std::pair<uint32_t, uint32_t>> blocks;   // (first, count)
    uint64_t at = 4 * kBlockWords, fetched = 0;          // bytes laid out, bytes fetched ahead
    auto fetch = [&](uint32_t cls) {
        WOp u;
        u.cls = uint8_t(cls);
        u.imm = uint32_t(fetched);
        fetched += kPrefetch;
        return u;
    };
    if (total > 2 * kPrefetch) {   // (a shorter program is read before a fetch of it would help)
        for (int i = 0; i < 2; ++i) ops.push_back(fetch(PF));
        blocks.push_back({0, 2});
        at += 4 * (2 * kInfo[PF].words + 2);
    } else {
        fetched = UINT64_MAX / 2;
    }
    for (uint32_t i = 0; i < in.size();) {
        uint32_t n = 1;
        while (n < kInfo[in[i].cls].max && i + n < in.size() && in[i + n].cls == in[i].cls) ++n;
        const bool wait = in[i].cls == WAIT;
        if (fetched < total && (wait ? at + 2 * kPrefetch > fetched : at + kPrefetch > fetched)) {
            const uint32_t cls = wait ? WAITPF : PF;
            blocks.push_back({uint32_t(ops.size()), 1});
            ops.push_back(fetch(cls));
            at += 4 * (kInfo[cls].words + 2);
            if (wait) {
                i += n;
                continue;
            }
        }
        blocks.push_back({uint32_t(ops.size()), n});
        for (uint32_t q = 0; q < n; ++q) ops.push_back(in[i + q]);
        at += 4 * (uint64_t(n) * kInfo[in[i].cls].words + 2);
        i += n;
    }
    const uint32_t nb = uint32_t(blocks.size());
    auto entry_of = [&](uint32_t b) {
        return b < nb ? entry(ops[blocks[b].first].cls, blocks[b].second, b & 1) : 0u;
    };
    // where the words of each block are read from: a whole half ending with
    // the block's headers
    std::vector<uint32_t> start(nb);
    uint64_t words = kBlockWords;
    for (uint32_t b = 0; b < nb; ++b) {
        words += uint64_t(blocks[b].second) * kInfo[ops[blocks[b].first].cls].words + 2;
        if (words > 0x3FFFFFFFu) throw std::length_error("wide program beyond 32-bit offsets");
        start[b] = uint32_t(4 * (words - kBlockWords));
    }
    auto start_of = [&](uint32_t b) { return start[std::min(b, nb - 1)]; };
    S->code.assign(kBlockWords, 0);
    S->code.reserve(words);
    for (uint32_t b = 0; b < nb; ++b) {
        for (uint32_t i = 0; i < blocks[b].second; ++i) encode(ops[blocks[b].first + i], &S->code);
        S->code.push_back(entry_of(b + 1));
        S->code.push_back(start_of(b + 2));
        const uint32_t cls = ops[blocks[b].first].cls, n = blocks[b].second;
        S->cost += kDispatchCost + uint64_t(n) * class_cost(cls);
        S->lone += kLoneDispatch + uint64_t(n) * lone_cycles(cls);
        if (is_call(cls) || (S->matrices && is_element(cls))) S->calls += uint64_t(n) * lone_cycles(cls);
    }
    // what the fetches read past the program's end
    S->code.resize(std::max<size_t>(S->code.size(), fetched < UINT64_MAX / 2 ? fetched / 4 : 0), 0);
    S->first[0] = start_of(0);
    S->first[1] = entry_of(0);
    S->first[2] = start_of(1);
    S->n_blocks = nb;
    S->n_uops = ops.size();
}

}  // namespace

bool wide_takes(const Tape &t, bool *matrices) {
    *matrices = false;
    for (const TapeOp &o : t.ops) *matrices = *matrices || o.rows != 1 || o.cols != 1 || o.code == tp::MATMUL;
    auto nel = [&](uint32_t s) { return t.nel(s); };
    for (const TapeOp &o : t.ops) {
        if (o.rows > 4 || o.cols > 4) return false;
        const bool scalar = o.rows == 1 && o.cols == 1;
        switch (o.code) {
        case tp::CONST: case tp::PARAM: case tp::OBS: case tp::ADD: case tp::SUB:
        case tp::MATMUL: case tp::TRANSPOSE: case tp::PACK: case tp::INDEX:
            break;
        case tp::MUL:   // scalars, or a scalar and a matrix
            if (!scalar && nel(o.a) != 1 && nel(o.b) != 1) return false;
            break;
        case tp::DIV: case tp::NEG: case tp::EXP: case tp::LOG: case tp::SQRT: case tp::SIN: case tp::COS:
        case tp::POW: case tp::ABS: case tp::SELECT:
            if (!scalar) return false;
            break;
        case tp::INV: case tp::LOGDET:
            if (nel(o.a) != 4) return false;
            break;
        default: return false;
        }
    }
    return kSlots + 2 * uint64_t(t.n_params) + 8 <= (*matrices ? kMatRegs : kRegs) && t.n_obs < 1u << 29;
}

// A matrix operation costs the wide kernel a call (some 300 cycles before its
// first product), and the scalars of a program with matrices use a quarter of
// the lanes that a wave could serve; the slot kernel costs less where the
// operations are small.  Steps of a 4x4 product and a scaling (40 products or
// elements an operation) on 16,384 lanes, 150 steps, slot against wide kernel,
// us: losses 107 against 97, gradients 753 against 669; 3x3 (18 an operation)
// 129 against 82, 871 against 470; 2x2 (6) 49 against 60, 345 against 317; a
// 4x4 matrix on a vector, scaled, and its norm (7) 188 against 137, 566 against
// 575, of 2x2 (2.5) 109 against 128, 449 against 525.
constexpr uint64_t kMatWork = 12;
bool wide_pays(const Tape &t) {
    uint64_t n = 0, work = 0;   // matrix operations, their products or elements
    for (const TapeOp &o : t.ops) {
        if (o.code != tp::MATMUL && ((o.rows == 1 && o.cols == 1) || o.code == tp::PACK)) continue;
        n += 1;
        work += o.code == tp::MATMUL ? uint64_t(t.nel(o.a)) * o.cols : uint64_t(o.rows) * o.cols;
    }
    return work >= kMatWork * n;
}

namespace {
WideSchedule schedule_in(const Tape &t, bool with_grad, bool save_reads, uint32_t lds_rows, bool order) {
    WideSchedule none;
    bool mats;
    if (!wide_takes(t, &mats)) return none;
    const uint32_t regs = mats ? kMatRegs : kRegs;
    Info I(t);
    I.fold_static_subtrahend = true;
    I.fold_scalars_only = true;
    I.exact_revreads = true;
    I.analyse();
    uint64_t total = 0;
    for (uint32_t k = 0; k < I.N; ++k)
        if (I.kind[k] == K_COMP && I.vlive[k]) total += I.nel[k];
    total = std::max<uint64_t>(total, 1);
    uint64_t read_elems = 0;
    if (with_grad) {
        std::vector<uint8_t> read(I.N, 0);
        auto count = [&](uint32_t s) {
            if (I.kind[s] == K_COMP && !read[s]) read[s] = 1, read_elems += I.nel[s];
        };
        for (uint32_t k = 0; k < I.N; ++k)
            if (I.need_rev[k]) I.for_revreads(k, count);
    }
    bool lds_fit = true;   // whether the last trial's matrices fitted, if its registers did
    // (a search over sizes needs the registers only; the chosen one is encoded)
    auto trial = [&](uint64_t size, std::vector<WOp> *out) {
        Builder B(I);
        B.save_reads = save_reads;
        B.resident.assign(I.N, 0);
        B.res_off.assign(I.N, 0);
        if (with_grad) {
            B.set_cuts(B.choose_cuts(size));
            B.plan(false);
            B.choose_residents(2);
            B.set_cuts(B.choose_cuts(size));
            B.plan(true);
        } else {
            B.set_cuts({0});
        }
        Lower W(I, B, with_grad, mats);
        W.run();
        WideSchedule S;
        lds_fit = true;
        // (what follows numbers every register below kVirtual as one of the file)
        if (kSlots + uint64_t(W.n_static) > regs) return S;
        const uint32_t ck_cap = ck_slots(save_reads, mats);
        uint32_t late_at;
        std::vector<WOp> ops = place_loads(W, ck_cap, &late_at);
        std::vector<uint32_t> spare, early;
        bool obs[2] = {false, false}, ck[2] = {false, false};
        for (const WOp &u : ops) {
            if (u.cls == LDO0 || u.cls == LDO1) obs[u.cls - LDO0] = true;
            if ((u.cls == LDK0 || u.cls == LDK1) && !u.late) ck[u.cls - LDK0] = true;
        }
        for (uint32_t half = 0; half < 2; ++half) {
            for (uint32_t i = 0; i < kObsSlots && !obs[half]; ++i) spare.push_back(half * kObsSlots + i);
            for (uint32_t i = 0; i < kCkSlots; ++i)
                if (!ck[half] || i < kCkSlots - ck_cap)
                    (late_at == UINT32_MAX ? spare : early).push_back(2 * kObsSlots + half * kCkSlots + i);
        }
        if (order && !mats) order_ops(ops, W.n_virtual, W.kSink, late_at, kOrderWindow);
        S.n_regs = place_registers(ops, W.n_virtual, W.n_static, spare, early, late_at, regs);
        if (S.n_regs > regs) return S;
        S.matrices = mats;
        S.lds_rows = place_matrices(ops, W.mem_size);
        lds_fit = S.lds_rows <= lds_rows;
        S.n_ckpt_rows = W.n_rows * (mats ? 4 : 1);
        S.n_segments = uint32_t(B.cuts.size());
        S.values = total;
        S.read_elems = read_elems;
        for (const auto &v : B.livein)
            for (uint32_t s : v) S.ckpt_elems += I.nel[s];
        S.consts = W.consts;
        S.ok = lds_fit && S.n_ckpt_rows < (1u << 31);
        *out = std::move(ops);
        return S;
    };
    std::vector<WOp> ops;
    WideSchedule best;
    auto encoded = [&](WideSchedule &&S) {
        if (S.ok) emit(ops, &S);
        return std::move(S);
    };
    if (!with_grad) return encoded(trial(0, &ops));
    // The largest segment size that fits the register file (doubled or halved
    // from a usual one, then bisection), and the size that cuts the trace
    // evenly into as many segments (which cuts every step of a loop at the
    // same point): the cheaper of the two.
    constexpr uint64_t kShortest = 4;
    std::vector<WOp> last;
    auto fits = [&](uint64_t size) {   // `best` and `ops`: of the last size that does
        WideSchedule S = trial(size, &last);
        if (!S.ok) return false;
        best = std::move(S);
        ops.swap(last);
        return true;
    };
    if (fits(total)) return encoded(std::move(best));   // the whole trace in one segment
    uint64_t lo = std::min<uint64_t>(80, total), hi = 0;   // lo fits, hi does not
    while (!fits(lo)) {
        // where the matrices of the shortest segments do not fit either, no
        // length between is tried (a longer one holds more at a time)
        if (!hi && !lds_fit && !fits(kShortest) && !lds_fit) return none;
        hi = lo;
        lo /= 2;
        if (lo < kShortest) return none;
    }
    while (!hi) {
        if (fits(2 * lo)) lo *= 2;
        else hi = 2 * lo;
    }
    while (hi - lo > std::max<uint64_t>(4, lo / 16)) {
        const uint64_t mid = lo + (hi - lo) / 2;
        (fits(mid) ? lo : hi) = mid;
    }
    best = encoded(std::move(best));
    const uint64_t even = total / best.n_segments;
    if (even > 0 && even != lo) {
        WideSchedule alt = encoded(trial(even, &ops));
        if (alt.ok && alt.cost < best.cost) best = std::move(alt);
    }
    return best;
}
}  // namespace

// (in program order where the longer runs need registers that are not there)
WideSchedule schedule_wide(const Tape &t, bool with_grad, bool save_reads, uint32_t lds_rows) {
    WideSchedule S = schedule_in(t, with_grad, save_reads, lds_rows, true);
    bool mats;
    if (!S.ok && wide_takes(t, &mats) && !mats) S = schedule_in(t, with_grad, save_reads, lds_rows, false);
    return S;
}

}  // namespace ndvm
