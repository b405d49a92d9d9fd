// Host emulator of slot programs -- a checking tool for the scheduler, built
// into its own library (libndvm_emu.so) that only the CPU tests load; the
// product binding never calls it.
//
// It schedules a tape exactly as ndvm_tape_upload / ndvm_grad do and runs the
// resulting program lane by lane through the same micro-op handlers the GPU
// kernel uses.  Every slot of an instruction reads before any slot writes
// (writes are buffered until the instruction ends, as on the GPU); every
// register access is bounds-checked, every read of a never-written register
// is reported, and so is a slot that reads or writes a register another slot
// of the same instruction writes.  That exposes register-allocation,
// checkpoint, packing and first-contribution mistakes without a GPU.
#include <cmath>
#include <algorithm>
#include <cstdio>
#include <vector>

#include "common.h"
#include "sched.h"
#include "slot_exec.h"
#include "wide.h"
#include "wide_exec.h"

using namespace ndvm;

namespace {

// Payload of one slot: register fields decoded from byte offsets into
// register numbers (the host context's handles).
struct P4 {
    uint32_t w[4], hdr, slot, reg_bytes;
    uint32_t *n_loaded;   // calls of loaded() (a hot handler makes exactly one)
    uint32_t a() const { return w[0] / reg_bytes; }
    uint32_t x() const { return w[1] / reg_bytes; }
    uint32_t y() const { return w[2] / reg_bytes; }
    uint32_t z() const { return w[3] / reg_bytes; }
    uint32_t ix() const { return w[1]; }
    uint32_t imm() const { return hdr >> slot::kImmShift; }
    bool first() const { return (hdr >> (slot::kFirstShift + slot)) & 1u; }
    void loaded() const { ++*n_loaded; }
};

struct HostCtx {
    double *regs;
    uint8_t *written;
    uint32_t n_regs, sink;
    const double *consts, *obs, *params;
    uint32_t n_consts, n_obs, n_params;
    double *loss, *grad;
    double *ckpt;
    uint32_t n_ckpt;   // rows including the trash row
    int *fault;        // first problem seen: 1 register range, 2 unwritten read, 3 pool/param/obs index,
                       // 4 ckpt row, 6 read of a register another slot writes, 7 two slots write one register,
                       // 8 form differs between slots, 9 output store or skip test inside a skipped arm,
                       // 10 a hot handler marked its operand reads other than once
    uint32_t cur_slot = 0;
    bool cur_dummy = false;   // an unused slot (result to the sink): its reads are never checked
    std::vector<std::pair<uint32_t, double>> *pending;
    std::vector<uint32_t> *pend_slot;

    static uint32_t uni(uint32_t x) { return x; }
    uint32_t slot() const { return cur_slot; }
    uint32_t *fault_reg = nullptr;   // register of the first fault (when it concerns one)
    void flag(int code, uint32_t r = 0xFFFFFFFFu) const {
        if (*fault == 0) {
            *fault = code;
            if (fault_reg) *fault_reg = r;
        }
    }
    void check_pending_read(uint32_t r) const {
        if (cur_dummy) return;
        for (size_t i = 0; i < pending->size(); ++i)
            if ((*pending)[i].first == r && (*pend_slot)[i] != cur_slot) flag(6);
    }
    static uint32_t adv(uint32_t h, uint32_t n) { return h + n; }
    double ld(uint32_t r) const {
        if (r >= n_regs) { flag(1); return NAN; }
        check_pending_read(r);
        if (!written[r] && !cur_dummy) flag(2, r);   // an unused slot may read an unwritten sink
        return regs[r];
    }
    double ld_raw(uint32_t r) const {
        if (r >= n_regs) { flag(1); return NAN; }
        if (r < sink || r >= sink + slot::kMaxBlock) check_pending_read(r);
        return regs[r];
    }
    void st(uint32_t r, double v) const {
        if (r >= n_regs) { flag(1); return; }
        if (poison) {
            if (cur_accum) return;
            v = NAN;
        }
        if (r < sink || r >= sink + slot::kMaxBlock)
            for (size_t i = 0; i < pending->size(); ++i)
                if ((*pending)[i].first == r && (*pend_slot)[i] != cur_slot) flag(7);
        pending->push_back({r, v});
        pend_slot->push_back(cur_slot);
    }
    void commit() const {
        for (const auto &pw : *pending) {
            regs[pw.first] = pw.second;
            written[pw.first] = 1;
        }
        pending->clear();
        pend_slot->clear();
    }
    double konst(uint32_t i) const {
        if (i >= n_consts) { flag(3); return NAN; }
        return consts[i];
    }
    double obsv(uint32_t i) const {
        if (i >= n_obs) { flag(3); return NAN; }
        return obs[i];
    }
    double param(uint32_t p) const {
        if (p >= n_params) { flag(3); return NAN; }
        return params[p];
    }
    void store_loss(double v, bool on) const {
        if (poison) flag(9);
        if (on) *loss = v;
    }
    void store_grad(uint32_t p, double v, bool on) const {
        if (poison) flag(9);
        if (!on) return;
        if (p >= n_params) { flag(3); return; }
        grad[p] = v;
    }
    void ckst(uint32_t row, double v) const {
        if (row >= n_ckpt) { flag(4); return; }
        ckpt[row] = poison ? NAN : v;
    }
    static void settle(double) {}
    void check_written(uint32_t r) const {
        if (r < n_regs && !written[r] && !cur_dummy) flag(2, r);
    }
    // SKIP, one lane at a time: the lane skips the arm it does not take (the
    // most skipping any wave of lanes could do)
    mutable uint32_t skip = 0;
    bool never_skip = false;
    // An instruction of an arm this lane skips.  On the GPU its registers
    // keep whatever they held; here every value it would form anew (forward
    // values, temporaries, first contributions) is set to NaN and every
    // adjoint it would add to keeps its value, so a result that depends on a
    // skipped arm comes out NaN or differs from the run without skipping.
    bool poison = false;
    bool cur_accum = false;   // the slot's writes add to their own register (not formed anew)
    void skip_arm(bool then_taken, uint32_t imm) const {
        const bool else_arm = (imm >> slot::kSkipSideShift) & 1u;
        if (poison) flag(9);
        if (!never_skip && (else_arm ? then_taken : !then_taken)) skip = imm & slot::kSkipCountMask;
    }
    double ckld(uint32_t row) const {
        if (row >= n_ckpt) { flag(4); return NAN; }
        return ckpt[row];
    }
};

// forms whose writes add to the register written (an adjoint update that is
// not the first contribution)
bool accumulates(uint32_t form, const P4 &p) {
    switch (form) {
    case slot::ACC: return p.z() == p.a();
    case slot::MACG: case slot::ACCD: case slot::ACCND: case slot::DOTACC: case slot::ACCSEL: case slot::ACCABS:
    case slot::DOTBACC:
        return !p.first();
    default:
        return false;
    }
}

// with_grad: 0 forward only, 1 gradient (recompute policy), 2 gradient (save
// policy); arm_min: smallest arm behind a skip test (0: none)
Schedule schedule(const Tape &t, int with_grad, uint32_t reg_budget, uint32_t slots, uint32_t arm_min) {
    return with_grad ? schedule_grad(t, reg_budget, slots, with_grad == 2, arm_min)
                     : schedule_forward(t, slots, reg_budget, arm_min);
}
// mode bits 8 / 16: arms as the NDVM_BRANCH_SKIP option lays them out / every
// arm however small
uint32_t arm_min_of(int mode) { return (mode & 16) ? 1 : (mode & 8) ? kArmMinElems : 0; }

}  // namespace

extern "C" {

/*
 * Schedule `tape` (forward-only when with_grad == 0, else the gradient
 * program for `reg_budget` registers) with `slots` micro-ops per instruction
 * and run it for L lanes on the host.  with_grad: 0 forward only, 1 gradient
 * (recompute policy), 2 gradient (save policy); + 4: never skip a branch arm;
 * + 8: branch arms behind skip tests (as the NDVM_BRANCH_SKIP option lays
 * them out); + 16: every branch arm behind a skip test, however small.
 * stats (optional, 11 entries): n_regs, n_ckpt_rows, n_segments, n_instr, fwd
 * ops, recompute ops, reverse ops, checkpoint elements stored, micro-ops,
 * slots used, skippable arms.
 * Returns 0, an ndvm_status from parsing, or 100 + fault code.
 */
int ndvm_emu_run(const uint8_t *tape, size_t len, int with_grad, uint32_t reg_budget, uint32_t slots,
                 const double *params, int64_t L, int64_t ld_p, const double *obs, int64_t n_obs, double *loss,
                 double *grad, int64_t ld_g, uint64_t *stats) {
    const bool never_skip = (with_grad & 4) != 0;   // run both arms of every branch
    const uint32_t arm_min = arm_min_of(with_grad);
    with_grad &= 3;
    Tape t;
    ndvm_status st = parse_tape(tape, len, &t);
    if (st != NDVM_OK) return st;
    if (n_obs != int64_t(t.n_obs)) return NDVM_E_ARG;
    if (slots != 1 && slots != 2 && slots != 4) return NDVM_E_ARG;
    Schedule S;
    try {
        S = schedule(t, with_grad, reg_budget, slots, arm_min);
    } catch (const std::exception &e) {
        set_error(e.what());
        return NDVM_E_UNSUPPORTED;
    }
    if (stats) {
        uint64_t v[11] = {S.n_regs, S.n_ckpt_rows, S.n_segments, S.n_instr, S.n_fwd_ops,
                          S.n_recompute_ops, S.n_rev_ops, S.ckpt_elems_stored, S.n_uops, S.n_slots_used,
                          S.n_skips};
        for (int i = 0; i < 11; ++i) stats[i] = v[i];
    }
    const uint32_t sink = 2 * t.n_params;
    std::vector<double> regs(S.n_regs), ck(size_t(S.n_ckpt_rows) + slot::kMaxBlock);
    std::vector<uint8_t> written(S.n_regs);
    std::vector<std::pair<uint32_t, double>> pending;
    std::vector<uint32_t> pend_slot;
    const uint32_t K = slot::kChunk;
    const uint32_t reg_bytes = 8 * (64 / slots);
    for (int64_t l = 0; l < L; ++l) {
        std::fill(written.begin(), written.end(), 0);
        int fault = 0;
        HostCtx c{regs.data(), written.data(), S.n_regs, sink, S.consts.data(), obs, params + l * ld_p,
                  uint32_t(S.consts.size()), uint32_t(n_obs), t.n_params, loss + l,
                  grad ? grad + l * ld_g : nullptr, ck.data(), S.n_ckpt_rows + slot::kMaxBlock, &fault, 0, false, &pending,
                  &pend_slot};
        uint32_t fault_reg = 0xFFFFFFFFu, fault_form = 0;
        uint64_t fault_instr = 0;
        c.fault_reg = &fault_reg;
        c.never_skip = never_skip;
        bool ended = false;
        uint32_t skipped = 0;   // instructions of a skipped arm still to come
        for (uint64_t i = 0; i < uint64_t(S.n_chunks) * K && !ended && !fault; ++i) {
            c.poison = skipped > 0;
            if (skipped) --skipped;
            const uint32_t hdr = S.code[S.hdr_off + i];
            const uint32_t form = hdr & slot::kFormMask;
            fault_instr = i;
            fault_form = form;
            if (form == slot::END) {
                ended = true;
                break;
            }
            for (uint32_t sl = 0; sl < slots; ++sl) {
                // slot sl's words sit in rows sl * 4 / S ..; take the first
                const uint32_t r = sl * slot::kRows / slots;
                const uint32_t *w = &S.code[size_t(i / K) * slot::kChunkWords + (size_t(r) * K + i % K) * 4];
                uint32_t n_loaded = 0;
                const P4 p{{w[0], w[1], w[2], w[3]}, hdr, sl, reg_bytes, &n_loaded};
                c.cur_slot = sl;
                c.cur_dummy = c.poison || (slot::writes_a(form) && p.a() == sink) ||
                              (form == slot::CKST && (p.ix() & slot::kCkRowMask) == S.n_ckpt_rows);
                c.cur_accum = accumulates(form, p);
                if (slot::is_hot(form)) {
                    slotx::exec_hot(c, form, p);
                    if (n_loaded != 1) c.flag(10);
                } else
                    slotx::exec_cold(c, form, p);
            }
            c.commit();
            if (c.skip) {   // the arm's instructions run poisoned
                skipped = c.skip;
                c.skip = 0;
            }
        }
        if (!ended && !fault) fault = 5;
        if (fault) {
            char m[160];
            std::snprintf(m, sizeof m, "emulator fault %d in lane %lld at instruction %llu (form %u), register %u",
                          fault, (long long)l, (unsigned long long)fault_instr, fault_form, fault_reg);
            set_error(m);
            return 100 + fault;
        }
    }
    return 0;
}

/*
 * Copy the device program the scheduler makes for `tape` (slot words,
 * chunk-major ([chunk][row][instr][4]), then the headers; slot.h) into `out`
 * when it holds `cap` words;
 * returns the number of words, or -1 on an error.
 */
int64_t ndvm_emu_program(const uint8_t *tape, size_t len, int with_grad, uint32_t reg_budget, uint32_t slots,
                         uint32_t *out, size_t cap, uint32_t *hdr_off) {
    Tape t;
    if (parse_tape(tape, len, &t) != NDVM_OK) return -1;
    Schedule S;
    try {
        S = schedule(t, with_grad & 3, reg_budget, slots, arm_min_of(with_grad));
    } catch (const std::exception &e) {
        set_error(e.what());
        return -1;
    }
    const size_t n = S.code.size();
    if (out && cap >= n) std::copy(S.code.begin(), S.code.end(), out);
    if (hdr_off) *hdr_off = S.hdr_off;
    return int64_t(n);
}

/*
 * Which kernel runs a launch of `lanes` lanes of `tape` (mode 0 losses, 1
 * gradients, 2 saving gradients) on a GPU of `cus` CUs of 160 KB LDS, `budget`
 * slot registers a lane: out[0] 1 slot, 0 wide; out[1], out[2] estimated cycles of
 * a lone wave of either; out[3] the wide program's cycles in library functions.
 * Result as ndvm_emu_wide.
 */
int ndvm_emu_route(const uint8_t *tape, size_t len, int mode, int64_t lanes, uint32_t budget, uint32_t cus, uint64_t *out) {
    Tape t;
    ndvm_status st = parse_tape(tape, len, &t);
    if (st != NDVM_OK) return -int(st);
    const WideSchedule S = schedule_wide(t, mode != 0, mode == 2, mode ? std::max(320u, budget) : 320u);
    if (!S.ok) return 1;
    const Schedule D = mode ? schedule_grad(t, budget, 4, mode == 2) : schedule_forward(t, 4, budget);
    const bool leads = !mode || short_segments(S) || slot_leads(schedule_forward(t, 4, 1280).lone, schedule_wide(t, false, mode == 2, 320).lone);
    out[0] = slot_may_win(S, mode != 0) && leads && D.n_regs <= budget &&
             slot_wins(D.lone, 1280 / std::max(D.n_regs, 1u), uint64_t(lanes + 15) / 16, cus, S.lone, S.matrices, mode == 0);
    out[1] = D.lone;
    out[2] = S.lone;
    out[3] = S.calls;
    return 0;
}

/*
 * How the wide kernel would serve ndvm_grad_noalloc of `tape` over `lanes` lanes
 * on an array of `bytes`: out[0] lanes at a time (0: not at all), out[1] whether
 * the slot kernel with `budget` registers may fit the array, out[2] workspace
 * rows.  Arguments and result otherwise as ndvm_emu_wide.
 */
int ndvm_emu_scratch(const uint8_t *tape, size_t len, int mode, uint32_t lds_rows, int64_t lanes, uint32_t budget,
                     uint64_t bytes, int64_t *out) {
    Tape t;
    ndvm_status st = parse_tape(tape, len, &t);
    if (st != NDVM_OK) return -int(st);
    const WideSchedule S = schedule_wide(t, true, mode == 2, lds_rows);
    if (!S.ok) return 1;
    const uint64_t rows = uint64_t(S.n_ckpt_rows) + slot::kMaxBlock;
    out[1] = slot_may_fit(S, mode == 2, budget, lanes, bytes);
    out[0] = scratch_part(rows, lanes, bytes, out[1]);
    out[2] = int64_t(rows);
    return 0;
}

/*
 * Schedule `tape` for the wide kernel (mode: 0 forward only, 1 gradient with
 * the recompute policy, 2 with the save policy) and run its blocks for L lanes
 * on the host, micro-op by micro-op as the kernel does.  Reads of registers
 * never written, of load slots whose loads have not been waited for, and
 * registers, rows and indices out of range are faults.  stats (optional, 7
 * entries): registers, checkpoint rows, segments, blocks, micro-ops, estimated
 * cycles, matrix elements.  Returns 0, 1 for a tape the wide kernel does not take, an
 * ndvm_status from parsing (negated), or 100 + fault code.  lds_rows: matrix
 * elements a wave may hold.
 */
int ndvm_emu_wide(const uint8_t *tape, size_t len, int mode, uint32_t lds_rows, const double *params, int64_t L, int64_t ld_p,
                  const double *obs, int64_t n_obs, double *loss, double *grad, int64_t ld_g, uint64_t *stats) {
    using namespace wide;
    Tape t;
    ndvm_status st = parse_tape(tape, len, &t);
    if (st != NDVM_OK) return -int(st);
    WideSchedule S;
    try {
        S = schedule_wide(t, mode != 0, mode == 2, lds_rows);
    } catch (const std::exception &e) {
        set_error(std::string("wide scheduler: ") + e.what());
        return 100;
    }
    if (!S.ok) return 1;
    if (stats) {
        const uint64_t v[8] = {S.n_regs, S.n_ckpt_rows, S.n_segments, S.n_blocks, S.n_uops, S.cost, S.lds_rows, wide_pays(t)};
        for (int i = 0; i < 8; ++i) stats[i] = v[i];
    }
    const uint32_t NS = S.matrices ? 4 : 1, n_rows = S.n_ckpt_rows / NS;   // threads per lane, checkpoint rows of one store
    struct Lds {
        std::vector<double> *v;
        int *fault;
        double ld(uint32_t p, uint32_t e) const { return at(p, e); }
        void st(uint32_t p, uint32_t e, double x) const { at(p, e) = x; }
        double &at(uint32_t p, uint32_t e) const {
            const uint32_t i = p / kLdsRow + e;
            if (p % kLdsRow || i >= v->size()) {
                *fault = *fault ? *fault : 8;
                return (*v)[0];
            }
            return (*v)[i];
        }
    };
    for (int64_t l = 0; l < L; ++l) {
        std::vector<double> reg(kRegs * NS, NAN), ck(S.n_ckpt_rows, NAN), lds(std::max(4u, S.lds_rows), NAN);
        std::vector<uint8_t> state(kRegs * NS, 0);   // 1 written, 2 load in flight
        int fault = 0;
        uint32_t sl = 0;                             // thread of the lane
        const Lds mem{&lds, &fault};
        uint32_t fault_cls = 0, cur_cls = 0;
        auto flag = [&](int c) {
            if (!fault) fault = c, fault_cls = cur_cls;
        };
        uint32_t r0 = kSlots;
        auto init = [&](double v) {
            if (r0 >= kRegs) return flag(1);
            for (uint32_t i = 0; i < NS; ++i) {
                reg[r0 * NS + i] = v;
                state[r0 * NS + i] = 1;
            }
            ++r0;
        };
        for (uint32_t p = 0; p < t.n_params; ++p) init(params[l * ld_p + p]);
        for (uint32_t p = 0; mode && p < t.n_params; ++p) init(0.0);
        const uint32_t sink = r0;
        init(0.0);
        for (double v : S.consts) init(v);
        auto idx = [&](uint32_t h, uint32_t roles) -> uint32_t {
            if ((h & 0xF000u) != roles || (h & 0x0F00u) || (h & 1u) || (h & 0xFFu) / 2 >= S.n_regs) flag(2);
            return (h & 0xFFu) / 2 < kRegs ? (h & 0xFFu) / 2 : 0;
        };
        auto get = [&](uint32_t h, uint32_t roles) {
            const uint32_t r = idx(h, roles) * NS + sl;
            if (state[r] != 1) flag(3);
            return reg[r];
        };
        auto set = [&](uint32_t h, uint32_t roles, double v) {
            const uint32_t r = idx(h, roles);
            // statics are never overwritten, parameter adjoints and the sink apart
            if (r >= kSlots && r < r0 && (r < kSlots + t.n_params || r > sink)) flag(4);
            reg[r * NS + sl] = v;
            state[r * NS + sl] = 1;
        };
        const uint32_t SD = kSrc | kDst;
        uint64_t start = S.first[0], next = S.first[2];   // where this block's and the next one's words are read
        uint32_t where = S.first[1];
        bool ended = false;
        for (uint64_t b = 0; !ended && !fault; ++b) {
            const uint32_t region = where / kRegion, cls = region / 2;
            if (cls >= kClasses || (region & 1u) != (b & 1u) || start / 4 + kBlockWords > S.code.size() || start % 4) {
                flag(5);
                break;
            }
            const ClassInfo info = kInfo[cls];
            const uint32_t skipped = info.bytes ? (where % kRegion) / info.bytes : 0, n = info.max - skipped;
            if (skipped >= info.max || entry(cls, n, b & 1u) != where) {
                flag(5);
                break;
            }
            const uint32_t *hdr = S.code.data() + start / 4 + kBlockWords - 2;
            const uint32_t *w = hdr - size_t(n) * info.words;
            for (uint32_t i = 0; i < n && !fault && !ended; ++i, w += info.words) {
                const uint32_t a = info.words > 0 ? w[0] : 0, c = info.words > 1 ? w[1] : 0,
                               d = info.words > 2 ? w[2] : 0;
                const uint32_t al = a & 0xFFFFu, ah = a >> 16, cl = c & 0xFFFFu, ch = c >> 16, dl = d & 0xFFFFu,
                               dh = d >> 16;
                auto add = [&](uint32_t h, bool on, double v) {
                    const double o = get(h, SD);
                    if (on) set(h, SD, o + v);
                };
                cur_cls = cls;
                const uint32_t w3 = info.words > 3 ? w[3] : 0, M = (w3 & 7u), K = (w3 >> 3) & 7u, N = (w3 >> 6) & 7u;
                const bool fst = w3 & kFirstBit;
                bool matrix = true;
                sl = 0;
                switch (cls) {   // one matrix for the lane's threads
                case MM:
#define ROW(k, n) mm_row<k, n>(mem, a, c, d, r)
                    for (uint32_t r = 0; r < M; ++r) NDVM_WIDE_SIDES(K, N, ROW)
#undef ROW
                    break;
                case MMA: {
                    const bool on = any_of(mem, a, M * N);
                    auto gate = [&](bool) { return on; };
#define ROW(k, n) mma_row<k, n>(mem, a, c, d, r, fst, gate)
                    for (uint32_t r = 0; r < M; ++r) NDVM_WIDE_SIDES(K, N, ROW)
#undef ROW
                    break;
                }
                case MMB:
#define ROW(m, n) mmb_row<m, n>(mem, a, c, d, r, K, fst)
                    for (uint32_t r = 0; r < K; ++r) NDVM_WIDE_SIDES(M, N, ROW)
#undef ROW
                    break;
                case VADD: for (uint32_t e = 0; e < 4; ++e) vadd(mem, a, c, d, e, w3); break;
                case VACC: for (uint32_t e = 0; e < 4; ++e) vacc(mem, a, d, e, w3); break;
                case TRANS: for (uint32_t e = 0; e < 4; ++e) transpose(mem, a, d, e, w3); break;
                case TRANSACC: for (uint32_t e = 0; e < 4; ++e) transpose_acc(mem, a, d, e, w3); break;
                case INV2: inv2(mem, a, d); break;
                case INV2ACC: inv2_acc(mem, a, c, d, w3); break;
                case VSCALE: for (uint32_t e = 0; e < 4; ++e) vscale(mem, a, c, get(w3 & 0xFFFFu, kSrc), e, d); break;
                case VACCS: {
                    const bool on = any_of(mem, a, d & 511u);
                    for (uint32_t e = 0; e < 4; ++e)
                        vaccs(mem, a, c, get(w3 & 0xFFFFu, kSrc), e, d & 511u, d & kFirstBit, on);
                    break;
                }
                case LOGDETACC: logdet2_acc(mem, a, c, get(w3 & 0xFFFFu, kSrc), d); break;
                default: matrix = false;
                }
                for (sl = 0; sl < NS && !matrix; ++sl) switch (cls) {
                case STE: mem.st(c, 0, get(al, kSrc)); break;
                case STE4: mem.st(c, sl, get(al, kSrc)); break;
                case LDE: set(cl, kDst, mem.ld(a, 0)); break;
                case CKSTM:
                    if (c >= n_rows) flag(6);
                    else ck[NS * c + sl] = mem.ld(a, sl);
                    break;
                case SDOT: set(w3 >> 16, kDst, sdot(mem, a, c, d)); break;
                case DET2: {
                    double v[4];
                    load4(mem, a, v);
                    set(w3 >> 16, kDst, det2(v));
                    break;
                }
                case FMA: {
                    const double x = get(al, kSrc), y = get(ah, kSrc), z = get(cl, kSrc), p = x * y;
                    set(ch, kDst, p + z);
                    break;
                }
                case DUAL: {
                    const double g = get(al, kSrc);
                    set(ah, kDst, 0.0);
                    const double y = get(cl, kSrc);
                    add(ch, g != 0.0, y * g);
                    const double z = get(dl, kSrc);
                    add(dh, g != 0.0, z * g);
                    break;
                }
                case SEL: {
                    const bool lt = get(al, kSrc) < get(ah, kSrc);
                    const double x = get(cl, kSrc), y = get(ch, kSrc);
                    set(dl, kDst, lt ? x : y);
                    break;
                }
                case SELADJ: {
                    const double g = get(al, kSrc);
                    set(ah, kDst, 0.0);
                    const bool lt = get(cl, kSrc) < get(ch, kSrc);
                    add(dl, lt, g);
                    add(dh, !lt, g);
                    break;
                }
                case DIV: {
                    const double x = get(al, kSrc), y = get(ah, kSrc);
                    set(cl, kDst, x / y);
                    break;
                }
                case DIVADJ: {
                    const double g = get(al, kSrc);
                    set(ah, kDst, 0.0);
                    const double y = get(cl, kSrc), gz = get(dl, kSrc) * g;
                    add(ch, g != 0.0, g / y);
                    add(dh, g != 0.0, -(gz / y));
                    break;
                }
                case ACCD: {
                    const double g = get(al, kSrc);
                    set(ah, kDst, 0.0);
                    const double y = get(cl, kSrc), z = get(dl, kSrc);
                    add(ch, g != 0.0, z / y);
                    break;
                }
                case CKST:
                    if (c >= n_rows) flag(6);
                    else ck[NS * c + sl] = get(al, kSrc);
                    break;
                case LDK0: case LDK1: case LDO0: case LDO1: {
                    const bool k = cls == LDK0 || cls == LDK1;
                    const uint32_t half = k ? cls - LDK0 : cls - LDO0;
                    const uint32_t slot = (k ? 2 * kObsSlots + half * kCkSlots : half * kObsSlots) + skipped + i;
                    if (k ? a >= n_rows : (a % 8 || a / 8 >= uint32_t(n_obs))) {
                        flag(6);
                        break;
                    }
                    reg[slot * NS + sl] = k ? ck[NS * a + sl] : obs[a / 8];
                    state[slot * NS + sl] = 2;
                    break;
                }
                case PF: case WAITPF:
                    if (a + kPrefetch > 4 * S.code.size()) flag(6);
                    if (cls == PF) break;
                    [[fallthrough]];
                case WAIT:
                    for (uint32_t s = 0; s < kSlots; ++s)
                        if (state[s * NS + sl] == 2) state[s * NS + sl] = 1;
                    break;
                case STLOSS: loss[l] = get(al, kSrc); break;
                case STGRAD:
                    if (c % 8 || c / 8 >= t.n_params || !grad) flag(6);
                    else grad[l * ld_g + c / 8] = get(al, kSrc);
                    break;
                case EXP: set(ah, kDst, exp(get(al, kSrc))); break;
                case SIN: set(ah, kDst, sin(get(al, kSrc))); break;
                case COS: set(ah, kDst, cos(get(al, kSrc))); break;
                case LOGC: set(ah, kDst, f_logc(get(al, kSrc))); break;
                case SQRTC: set(ah, kDst, f_sqrtc(get(al, kSrc))); break;
                case ABS: set(ah, kDst, fabs(get(al, kSrc))); break;
                case POW: set(cl, kDst, pow(get(al, kSrc), get(ah, kSrc))); break;
                case ACCSIN: set(ch, kDst, f_accsin(get(al, kSrc), get(ah, kSrc), get(cl, kSrc))); break;
                case ACCCOS: set(ch, kDst, f_acccos(get(al, kSrc), get(ah, kSrc), get(cl, kSrc))); break;
                case ACCLOG: set(ch, kDst, f_acclog(get(al, kSrc), get(ah, kSrc), get(cl, kSrc))); break;
                case ACCABS: set(ch, kDst, f_accabs(get(al, kSrc), get(ah, kSrc), get(cl, kSrc))); break;
                case ACCPOW: set(dl, kDst, f_accpow(get(al, kSrc), get(ah, kSrc), get(cl, kSrc), get(ch, kSrc))); break;
                case ACCSQRT: set(dl, kDst, f_accsqrt(get(al, kSrc), get(ah, kSrc), get(cl, kSrc), get(ch, kSrc))); break;
                default: ended = true;
                }
            }
            where = hdr[0];
            start = next;
            next = hdr[1];
        }
        if (fault) {
            char m[96];
            std::snprintf(m, sizeof m, "wide emulator fault %d in lane %lld, class %u", fault, (long long)l, fault_cls);
            set_error(m);
            return 100 + fault;
        }
    }
    return 0;
}

const char *ndvm_emu_error(void) { return get_error(); }

}  // extern "C"
