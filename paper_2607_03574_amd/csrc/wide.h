// Device program format of the wide replay kernel ("wide" programs).  Produced
// by the wide scheduler from a validated tape; not part of the public interface.
//
// Scalar programs run one thread per lane, 64 lanes a wave.  Programs with
// small matrices run four threads per lane, 16 lanes a wave (thread t serves
// lane t % 16): the four hold the same scalars and share the work of a matrix
// (a row each, or every fourth element).  Each thread holds its lane's whole
// register file of scalars in vector registers: file register r is v[kFileBase + 2r :
// kFileBase + 2r + 1], reached through the VGPR index mode (M0 holds the
// wave-uniform index), so an operand costs one scalar move and no memory
// access, and a result is ready for the next micro-op a few cycles later.
// Micro-ops of a thread run one after the other, so they need no packing
// and may depend on their neighbours.
//
// The program is a sequence of blocks.  A block holds 1 .. kMax micro-ops of
// one class and ends with two header words; it is read through scalar loads
// into one half of a double buffer (kBlockWords words ending with the headers,
// so a short block's words are the last of the half) while the block before
// it runs.  The class's code is straight-line for kMax micro-ops, each reading
// its words from fixed scalar registers, and a block of n micro-ops enters it
// at micro-op kMax - n, so nothing is tested inside a block.  Blocks alternate
// between the halves, which have code of their own.
//
// Headers of block b: the entry point of block b + 1 (byte offset from the
// code base), and where the kBlockWords words of block b + 2 start (byte
// offset in the program).
//
// Matrices live in LDS, row-major: element e of a matrix at byte offset o is
// at o + 128 e of the wave's LDS, 8 bytes for each of the 16 lanes; a matrix
// takes a multiple of four elements.  A checkpoint row holds one value per
// lane; of a program with matrices, four (thread t stores and loads element
// t / 16 of a quad, or the scalar).
//
// A micro-op's operands are half words: bits 0-7 twice the register number,
// bits 12-15 the operand roles the index applies to (kSrc: source 0, kDst:
// destination), the form M0 takes.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace ndvm {

struct Tape;

namespace wide {

// The vector registers below the file: 40 for temporaries and library
// functions, then four addresses.
constexpr uint32_t kFileBase = 48;
constexpr uint32_t kRegs = (256 - kFileBase) / 2;
// With matrices: 96 for temporaries and functions, four addresses, two LDS
// addresses.
constexpr uint32_t kMatFileBase = 106;
constexpr uint32_t kMatRegs = (256 - kMatFileBase) / 2;
constexpr uint32_t kMatLanes = 16;
constexpr uint32_t kLdsRow = 8 * kMatLanes;   // bytes of one matrix element of a wave
// Load slots: registers the loads of observations (two halves of kObsSlots
// from 0) and of checkpoint rows (two halves of kCkSlots behind them) write.
// The slots a program does not use are ordinary registers.
constexpr uint32_t kObsSlots = 4, kCkSlots = 12;
constexpr uint32_t kSlots = 2 * kObsSlots + 2 * kCkSlots;

constexpr uint32_t kSrc = 0x1000, kDst = 0x8000;

// Half words of each class: x (y, z, w) read, d written, a read and written,
// zr cleared before the adjoint update, "-" unused.  The adjoint forms add to
// w (a register holding +0 for a first contribution) or to a (cleared by zr).
enum Class : uint32_t {
    FMA = 0,   // d = x * y + z (product rounded, then sum rounded): x, y | z, d
    DUAL,      // the linear adjoint rule with two targets: zr = +0, then where g != 0:
               // a += g * y, b += g * z: g, zr | y, a | z, b
    SEL,       // d = x < y ? z : w (unordered takes w): x, y | z, w | d, -
    SELADJ,    // adjoint of a select: zr = +0, then a += g where x < y, b += g elsewhere:
               // g, zr | x, y | a, b
    DIV,       // d = x / y: x, y | d, -
    DIVADJ,    // adjoint of z = x / y: zr = +0, then where g != 0: a += g / y, b += -((g * z) / y):
               // g, zr | y, a | z, b
    ACCD,      // zr = +0, then where g != 0: a += z / y: g, zr | y, a | z, -
    CKST,      // checkpoint row of this lane = x: x, - | row
    LDK0, LDK1,   // load slot (by position, of a half) = checkpoint row: row
    LDO0, LDO1,   // load slot (by position, of a half) = observation: byte offset
    WAIT,      // the loads have landed
    WAITPF,    // WAIT, then PF
    PF,        // fetch kPrefetch bytes of the program into the L2 cache: byte offset
    STLOSS,    // loss[lane] = x: x, -
    STGRAD,    // grad[lane, p] = x: x, - | 8 p
    // library functions
    EXP,       // d = exp(x): x, d
    SIN,       // d = sin(x)
    COS,       // d = cos(x)
    LOGC,      // d = log(max(x, 1e-8)), NaN kept
    SQRTC,     // d = sqrt(max(x, 1e-8)), NaN kept
    POW,       // d = pow(x, y): x, y | d, -
    ACCSIN,    // d = x != 0 ? w + x * cos(y) : w: x, y | w, d
    ACCCOS,    // d = x != 0 ? w + x * -sin(y) : w
    ACCLOG,    // d = x != 0 && y > 1e-8 ? w + x / y : w
    ACCABS,    // d = x != 0 ? w + (y > 0 ? x : y < 0 ? -x : 0) : w
    ACCPOW,    // d = x != 0 ? w + z * log(y) : w: x, y | z, w | d, -
    ACCSQRT,   // d = x != 0 && y > 1e-8 ? w + x / (2 z) : w
    ABS,       // d = |x|: x, d
    END,       // the program's end
    // ---- matrices (A, B, D, G, T: LDS byte offsets; i: immediate, see
    // wide_exec.h; a one-element matrix is a scalar register)
    STE,       // D[0] = x: x, - | D
    STE4,      // D[t / 16] = x: x, - | D
    LDE,       // d = A[0]: A | d, -
    CKSTM,     // checkpoint row = A[0 .. 3]: A | row
    MM,        // D = A B: A | B | D | i
    MMA,       // T += G B^T: G | B | T | i
    MMB,       // T += A^T G: A | G | T | i
    VADD,      // D = A +/- B: A | B | D | i
    VACC,      // T += +/- G: G | - | T | i
    TRANS,     // D = A^T: A | - | D | i
    TRANSACC,  // T += G^T: G | - | T | i
    INV2,      // D = A^-1: A | - | D | i
    INV2ACC,   // T -= Z^T G Z^T: Z | G | T | i
    VSCALE,    // D = x A: A | D | i | x, sink
    VACCS,     // T += x G: G | T | i | x, sink
    SDOT,      // d = sum of G A: G | A | i | x, d
    DET2,      // d = det A: A | A | i | x, d
    LOGDETACC, // T += x A^-T where det A > 1e-8: A | T | i | x, sink
    kClasses
};
// words per micro-op, micro-ops per block, code bytes per micro-op
struct ClassInfo {
    uint8_t words, max, bytes;
};
constexpr ClassInfo kInfo[kClasses] = {
    {2, 15, 40}, {3, 10, 72}, {3, 10, 44}, {3, 10, 64}, {2, 8, 112}, {3, 4, 240}, {3, 6, 140}, {2, 15, 32},
    {1, kCkSlots, 28}, {1, kCkSlots, 28}, {1, kObsSlots, 28}, {1, kObsSlots, 28}, {0, 1, 0}, {1, 1, 40},
    {1, 2, 36}, {1, 1, 16}, {2, 8, 32},
    {1, 10, 48}, {1, 10, 48}, {1, 10, 48}, {1, 10, 48}, {1, 10, 48}, {2, 10, 52}, {2, 10, 64}, {2, 10, 64},
    {2, 10, 64}, {2, 10, 64}, {3, 10, 68}, {3, 10, 68}, {1, 10, 48}, {0, 1, 0},
    {2, 15, 20}, {2, 15, 20}, {2, 15, 28}, {2, 15, 44}, {4, 7, 48}, {4, 7, 48}, {4, 7, 48}, {4, 7, 48}, {4, 7, 48},
    {4, 7, 48}, {4, 7, 48}, {4, 7, 48}, {4, 7, 48}, {4, 7, 60}, {4, 7, 60}, {4, 7, 60}, {4, 7, 60}, {4, 7, 60}};
constexpr uint32_t kPrefetch = 4096;   // one line of 64 bytes per thread
constexpr uint32_t kRegion = 1024;   // code bytes reserved per class and half
constexpr uint32_t kBlockWords = 32;

// code offset of a block's entry point
constexpr uint32_t entry(uint32_t cls, uint32_t n, uint32_t half) {
    return (2 * cls + half) * kRegion + (kInfo[cls].max - n) * kInfo[cls].bytes;
}

// Per-program constants read by the kernel.
struct Prog {
    const uint32_t *code;    // the blocks, with kBlockWords words of padding in front
    const double *consts;    // static constants, in register order
    uint64_t ckpt_row0;      // checkpoint row r of lane l at ws[(ckpt_row0 + r) * Lpad + l]
    uint64_t trash_row;      // row that the lanes past the last one write their results to
    uint32_t first[3];       // where the words of block 0 start, entry of block 0, where those of block 1 start
    uint32_t n_params, n_consts;
    uint32_t adjoints;       // the program has parameter adjoints (n_params registers after the parameters)
    uint32_t lds_bytes;      // matrices: LDS of one wave (0: a scalar program)
};

}  // namespace wide

struct WideSchedule {
    bool ok = false;              // false: not a program this kernel takes (matrices, too many registers)
    std::vector<uint32_t> code;   // words; kBlockWords padding words in front, kPrefetch bytes behind
    std::vector<double> consts;
    uint32_t n_regs = 0, n_ckpt_rows = 0, n_segments = 1, n_blocks = 0;
    uint32_t first[3] = {0, 0, 0};
    uint64_t n_uops = 0;
    uint64_t cost = 0;            // estimated cycles of a lone wave, by which programs are chosen
    uint64_t lone = 0, calls = 0; // measured ones, and those of library functions (and elements, with matrices)
    bool matrices = false;
    uint32_t lds_rows = 0;        // matrix elements in LDS
    uint64_t values = 0;          // elements of the computed values
    uint64_t read_elems = 0;      // elements of the values that adjoint rules read (leaves apart)
    uint64_t ckpt_elems = 0;      // elements of the segments' stored inputs
};

constexpr uint64_t padded_lanes(int64_t lanes) { return uint64_t(lanes + 63) / 64 * 64; }
// Whether a launch of the slot kernel over `lanes` lanes, with `budget` registers
// each, may fit an array of `bytes` where the wide program is S: an estimate with
// a factor of two to spare, made so that the slot program need not be.  Saving,
// that kernel too stores what the adjoint rules read, save what its registers
// hold.  Recomputing, its registers hold the values read of one segment, and each
// segment but the first stores as many elements as one of S's.
constexpr bool slot_may_fit(const WideSchedule &S, bool save_reads, uint32_t budget, int64_t lanes, uint64_t bytes) {
    if (lanes == 0) return true;
    const uint64_t rows = bytes / (8 * padded_lanes(lanes));
    if (save_reads) return S.read_elems <= 2 * (rows + budget);
    const uint64_t inputs = S.n_segments > 1 ? S.ckpt_elems / (S.n_segments - 1) : 0;
    return S.read_elems / std::max(budget, 1u) * inputs <= 2 * rows;
}
// Lanes that a gradient launch of `rows` workspace rows runs at a time on the
// static scratch array of `bytes`: all of them, or a multiple of 64 where the
// launch needs no more than four arrays; where the slot kernel may have fitted
// the array (its registers hold up to twelve times as much, and no rows are
// padded to quads there: up to 87 times the rows for a recomputing recurrence on
// 8,192 lanes), 128 arrays, so that what it took is not refused.  0 beyond that
// and where not even 64 lanes fit.
constexpr uint64_t kFewArrays = 4, kManyArrays = 128;
constexpr int64_t scratch_part(uint64_t rows, int64_t lanes, uint64_t bytes, bool slot_fits) {
    const uint64_t fit = bytes / (8 * rows) / 64 * 64, need = 8 * rows * padded_lanes(lanes);
    if (need <= bytes) return lanes;
    return need <= (slot_fits ? kManyArrays : kFewArrays) * bytes ? int64_t(fit) : 0;
}

// A launch of few waves lasts as long as one wave.  A wave of the slot kernel
// (16 lanes) computes up to four independent library functions at a time, one of
// the wide kernel (64 lanes) one: of programs that spend their time there, losses
// above all, the slot kernel's is done earlier.  Sums of 64 terms on 4,096 lanes,
// us, slot against wide kernel: losses of powers of powers 40 against 82, of
// powers 27 against 48, of exponential, log and root 27 against 46, of sines of
// cosines 31 against 42, of products 21 against 14; gradients 160 against 156, 95
// against 93, 82 against 82, 94 against 95, 57 against 39 (of sines of sines of
// sines 110 against 125; of a random tree whose parameters do not reach its
// functions 228 against 285).  Whether the slot kernel wins, from the cycles
// of a lone wave of both: as many of its waves per CU as its registers leave
// room for run at a time, one per SIMD (each one more costs 4% and 0.4 us).
// Over 96 programs other than those the cycles were measured on, 64 to 16,384
// lanes, the kernel chosen takes at most 1.06 times as long as the other, losses,
// and 1.08, gradients, 1.001 on the mean (the wide kernel alone up to 2.4 and 1.13).
constexpr uint32_t kLoneWaves = 4;   // per CU: beyond that the wide kernel's lanes a wave count for more
// (With matrices a wave of either kernel has 16 lanes: no more of the one than of
// the other; and losses, whose estimates are rougher, take a lead of 10%.)
constexpr bool slot_wins(uint64_t slot_cycles, uint64_t resident, uint64_t waves, uint64_t cus, uint64_t wide_cycles,
                         bool matrices, bool losses) {
    const uint64_t per_cu = (waves + cus - 1) / cus, at_once = std::min<uint64_t>(kLoneWaves, std::max<uint64_t>(resident, 1));
    const uint64_t rounds = (per_cu + at_once - 1) / at_once, more = matrices ? 0 : std::min(at_once, per_cu) - 1;
    return per_cu > 0 && per_cu <= kLoneWaves && rounds * (slot_cycles * (100 + 4 * more + (matrices && losses ? 10 : 0)) / 100) + 1000 * more < wide_cycles;
}
// A gradient whose registers leave room for segments of a few values only
// restores and recomputes for most of its time, where the slot kernel's registers
// hold whole steps: a network of 8 hidden units (25 parameters, 8 values a
// segment) on 40 points, 4,096 lanes, 215 against 275 us; of 6 (48 values) 164
// against 146; no program of 24 values or more a segment was slower.
constexpr bool short_segments(const WideSchedule &S) { return S.n_segments > 1 && S.values < 16 * uint64_t(S.n_segments); }
// Whether the slot kernel may win, so that its program is worth making: by the
// share of the wide program's cycles in library functions.  No program with less
// than 40% there, gradients 60%, ran more than 3% faster on the slot kernel.
// Programs with matrices hold the scalars of a lane in each of its four threads:
// where they pack and take apart matrices around library functions and divisions
// (the share counts all these) the slot kernel's wave is done earlier too: an
// extended Kalman filter of four states, 24 steps, 4,096 lanes, us, losses 94
// against 134, gradients 438 against 505, saving 559 against 455; a linear one, 40
// steps, 200 against 199, 1,069 against 782.  None with less than 20%, gradients
// 43%, ran more than 9% faster on the slot kernel.
constexpr bool slot_may_win(const WideSchedule &S, bool with_grad) {
    if (with_grad && short_segments(S)) return true;
    return S.calls * 100 >= S.lone * (S.matrices ? with_grad ? 43 : 20 : with_grad ? 60 : 40);
}
// A gradient's slot program, whose schedule is dear, is worth making only where
// the forward program's wave is done in 85% of the wide one's cycles (no gradient
// was faster on the slot kernel with less of a lead there).
constexpr bool slot_leads(uint64_t slot_forward, uint64_t wide_forward) { return slot_forward * 100 <= wide_forward * 85; }

// Wide program of a tape: forward only, or forward and reverse (save_reads as
// schedule_grad).  lds_rows: matrix elements a wave may hold in LDS.
WideSchedule schedule_wide(const Tape &t, bool with_grad, bool save_reads, uint32_t lds_rows);
// Whether a tape is one of matrices and scalars that the wide kernel takes,
// and whether it has matrices.
bool wide_takes(const Tape &t, bool *matrices);
// Whether it is faster there than on the slot kernel.
bool wide_pays(const Tape &t);

}  // namespace ndvm
