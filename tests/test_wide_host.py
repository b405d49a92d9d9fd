"""Wide replay kernel, no GPU: its scheduler's programs run on the host
emulator against the oracle, and its machine code against the format (entry
points, operand roles, registers of the library functions)."""
import os
import re
import shutil
import subprocess
import time

import numpy as np
import pytest

import emu
from conftest import ROOT
from parity import compare
from wide_cases import (cases, extended_filter, long_recurrence, lookups, network, one_element_forms,
                        scalars_and_a_product, sum_of_terms)
from workloads import configs
from workloads.bytecode import Asm

nd = pytest.importorskip("paper_2607_03574_amd")
CASES = cases() + one_element_forms()


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_programs_equal_oracle(oracle_mod, mode):
    """Every case, forward only and both policies, by the strict bar."""
    for name, code, obs, p in CASES:
        got = emu.wide(nd.tape_build(code), p, obs, mode)
        assert got is not None and got[2]["pays"], name
        ol, og, _ = oracle_mod.run(code, p, obs)
        grads = (got[1], og) if mode and og.size else (None, None)
        compare(got[0], grads[0], ol, grads[1])


def test_same_bits_as_the_slot_programs():
    for name, code, obs, p in CASES:
        t = nd.tape_build(code)
        for mode in (1, 2):
            wl, wg, _ = emu.wide(t, p, obs, mode)
            sl, sg, _ = emu.run(t, p, obs, save=mode == 2)
            for a, b in ((wl, sl), (wg, sg)):
                same = (a.view(np.int64) == b.view(np.int64)) | (np.isnan(a) & np.isnan(b))
                assert same.all(), (name, mode, a, b)


def test_segments_and_the_loss_formed_last():
    """Cases that need several checkpoint segments, and sums whose terms the
    forward sweep leaves out."""
    w = configs.lotka_volterra(L=1, T=60)
    _, _, st = emu.wide(nd.tape_build(w.bytecode), w.params, w.obs)
    assert st["n_segments"] > 5 and st["n_ckpt_rows"] > 0
    w = configs.exp_decay(L=1)
    t = nd.tape_build(w.bytecode)
    _, _, st = emu.wide(t, w.params, w.obs)
    assert st["n_ckpt_rows"] >= 64     # each term's residual, for the sum at the end
    fwd = emu.wide(t, w.params, w.obs, 0)[2]
    assert fwd["n_ckpt_rows"] == 0


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_parameters_and_constants_at_the_files_end(oracle_mod, mode):
    """Programs whose parameters and constants alone fill the register file or
    pass its end: the wide scheduler refuses those it cannot place (the
    emulator's build checks every container access on the way) and both
    kernels' programs give the oracle's values."""
    for name, code, obs, p, fits in lookups():
        t = nd.tape_build(code)
        ol, og, _ = oracle_mod.run(code, p, obs)
        got = emu.wide(t, p, obs, mode)
        if mode:
            assert (got is not None) == fits, name
        for loss, grad in ([got[:2]] if got else []) + [emu.run(t, p, obs, with_grad=mode > 0, save=mode == 2)[:2]]:
            compare(loss, grad if mode else None, ol, og if mode else None)


@pytest.mark.parametrize("policy", [nd.POLICY_RECOMPUTE, nd.POLICY_SAVE])
def test_upload_takes_one_element_forms(policy):
    """A pack of one element, an element of a scalar and a transposed scalar:
    an upload, alone or among others, ends as that of a plain product does (on
    a host without a device, at the device)."""
    def status(f):
        try:
            f()
        except nd.NdvmError as e:
            return e.status
        return 0
    plain = nd.tape_build(Asm(2, 0).param(0).param(1).mul().halt().bytes())
    want = status(lambda: nd.tape_upload(plain, policy, 0))
    assert want != nd.E_INTERNAL
    for name, code, _, _ in one_element_forms():
        t = nd.tape_build(code)
        assert status(lambda: nd.tape_upload(t, policy, 0)) == want, (name, nd.last_error())
        assert status(lambda: nd.tape_upload_many([plain, t], policy, 0)) == want, (name, nd.last_error())


def test_scheduling_short_programs_costs_no_more_than_for_the_slot_kernel():
    """CPU time of a gradient schedule (no lane is run), least of several: short
    recurrences once took 1.6 to 1.9 times the slot scheduler's (now 0.9 to
    1.0; the bar leaves room for a busy machine)."""
    def spent(f):
        t0 = time.process_time()
        f()
        return time.process_time() - t0
    for T in (50, 100):
        w = configs.logistic(L=1, T=T)
        t, none = nd.tape_build(w.bytecode), w.params[:0]
        both = [(spent(lambda: emu.run(t, none, w.obs, budget=1280)), spent(lambda: emu.wide(t, none, w.obs)))
                for _ in range(12)]
        slot, wide = (min(x) for x in zip(*both))
        assert wide < 1.4 * slot, (T, wide, slot)


@pytest.mark.parametrize("mode", [1, 2])
def test_half_the_lds_a_wave(oracle_mod, mode):
    """Products of a step fit half the LDS a wave with shorter segments, at a cost
    that two waves a SIMD repay; a Kalman filter does not, however short."""
    obs, p = np.zeros(1), np.random.default_rng(2).uniform(0.2, 0.3, (2, 4))
    for side, n in ((4, 0), (3, 0), (4, 4)):
        code = scalars_and_a_product(60, side, n)
        t = nd.tape_build(code)
        full, half = (emu.wide(t, p, obs, mode, lds_rows=r) for r in (320, 160))
        assert half[2]["lds_rows"] <= 160 and half[2]["cost"] * 7 < full[2]["cost"] * 10
        if mode == 1:
            assert full[2]["lds_rows"] > 160 and half[2]["n_segments"] > full[2]["n_segments"]
        ol, og, _ = oracle_mod.run(code, p, obs)
        compare(half[0], half[1], ol, og)
    for T in (12, 50, 200):
        w = configs.kalman(L=1, T=T)
        assert emu.wide(nd.tape_build(w.bytecode), w.params[:0], w.obs, mode, lds_rows=160) is None


@pytest.mark.parametrize("ops,mode,slot,wide", [
    # lanes that the slot kernel runs, lanes that the wide kernel runs, with the
    # measured us of both (slot, wide): losses 40, 82 and 82, 85; 27, 46 and 54, 46
    ("pow pow", 0, [1, 64, 4096, 8192], [17000, 65536]), ("exp log sqrt", 0, [64, 4096], [16384, 65536]),
    # losses without a library function: 21, 14
    ("mul mul mul mul", 0, [], [64, 4096, 65536]), ("div", 0, [], [64, 4096]),
    # gradients 110, 125; 160, 156; 44, 39; saving 195, 132
    ("sin sin sin", 1, [64, 4096, 8192], [17000]), ("pow pow", 1, [], [64, 4096, 16384]),
    ("exp", 1, [], [64, 4096]), ("sin sin sin", 2, [], [64, 4096])])
def test_launches_of_few_waves(ops, mode, slot, wide):
    """Which kernel runs programs of independent library functions."""
    t = nd.tape_build(sum_of_terms(ops, 64))
    for lanes, want in [(n, True) for n in slot] + [(n, False) for n in wide]:
        assert emu.route(t, lanes, mode, _slot_budget(lanes) if mode else 1280)[0] == want, lanes


@pytest.mark.parametrize("name,mode,slot,wide", [
    # losses 94, 134 and 90, 109; 8,192 lanes 178, 134
    ("ekf4", 0, [1, 4096], [8192, 65536]), ("ekf3", 0, [64, 4096], [8192]),
    # gradients 541, 631 and 483, 403; saving 674, 568
    ("ekf4", 1, [64, 8192], [32768]), ("ekf3", 1, [], [64, 4096]), ("ekf4", 2, [], [64, 4096]),
    # a linear filter: losses 200, 199, gradients 1,069, 782; products and scalars: 46, 25, 228, 142
    ("kalman", 0, [], [1, 4096]), ("kalman", 1, [], [64, 4096]), ("products", 0, [], [64]), ("products", 1, [], [64, 4096])])
def test_launches_of_few_waves_with_matrices(name, mode, slot, wide):
    code = {"ekf4": lambda: extended_filter(24, 4, 2), "ekf3": lambda: extended_filter(24, 3, 1),
            "kalman": lambda: configs.kalman(L=1, T=40).bytecode, "products": lambda: scalars_and_a_product(20, 4, 12)}[name]()
    t = nd.tape_build(code)
    for lanes, want in [(n, True) for n in slot] + [(n, False) for n in wide]:
        assert emu.route(t, lanes, mode, _slot_budget(lanes) if mode else 1280)[0] == want, lanes


@pytest.mark.parametrize("units,slot", [(6, False), (8, True), (10, True)])
def test_launches_of_few_waves_with_short_segments(units, slot):
    """Gradients, 40 points, 4,096 lanes, us: 164, 146; 215, 275; 271, 355."""
    t = nd.tape_build(network(units, 40))
    for lanes in (1, 4096, 16384):
        assert emu.route(t, lanes, 1, _slot_budget(lanes))[0] == slot
    assert not emu.route(t, 16385, 1, _slot_budget(16385))[0] and not emu.route(t, 4096, 2)[0]


def test_timed_models_stay_on_the_wide_kernel():
    for w in (configs.lotka_volterra(L=1, T=60), configs.logistic(L=1, T=60)):
        t = nd.tape_build(w.bytecode)
        assert not any(emu.route(t, lanes, mode)[0] for lanes in (1, 4096) for mode in (0, 1, 2))
    t = nd.tape_build(configs.exp_decay(L=1).bytecode)
    assert not emu.route(t, 256, 1)[0] and emu.route(t, 256, 0)[0]      # losses of 64 exponentials: 16, 18 us


def _slot_budget(lanes):
    """Registers a lane of the slot kernel at `lanes` lanes (16 lanes a wave, 256
    CUs of 160 KB LDS, at most 16 waves each)."""
    waves = -(-lanes // 16)
    return 160 * 1024 // min(16, -(-waves // 256)) // 128


def _slot_rows(t, p, obs, lanes, save):
    """Workspace rows of the slot kernel's launch: checkpoints, trash, spills (a
    program that does not fit takes the budget of fewer waves a CU)."""
    b = _slot_budget(lanes)
    st = emu.run(t, p, obs, budget=b, save=save)[2]
    if st["n_regs"] > b:
        b2 = 160 * 1024 // max(1, 160 * 1024 // (st["n_regs"] * 128)) // 128
        if b2 > b:
            b, st = b2, emu.run(t, p, obs, budget=b2, save=save)[2]
    return st["n_ckpt_rows"] + 4 + max(0, st["n_regs"] - b)


SCRATCH = 64 << 20


@pytest.mark.parametrize("name", ["lotka", "logistic", "kalman", "mixed", "products"])
def test_slot_launches_that_fit_the_scratch_array_are_expected_to(name):
    """The estimate of the slot kernel's rows, by which a launch that exceeds the
    scratch array on the wide kernel is served or refused, excludes no launch
    whose slot program fits."""
    if name in ("lotka", "logistic", "kalman"):
        w = {"lotka": lambda: configs.lotka_volterra(L=1, T=300), "logistic": lambda: configs.logistic(L=1, T=1000),
             "kalman": lambda: configs.kalman(L=1, T=60)}[name]()
        t, p, obs = nd.tape_build(w.bytecode), w.params, w.obs
    else:
        code = scalars_and_a_product(100, 4, 30) if name == "mixed" else scalars_and_a_product(150, 3, 0)
        t, p, obs = nd.tape_build(code), np.full((1, 4), 0.25), np.zeros(1)
    seen = set()
    assert emu.scratch(t, 0)[:2] == (0, True)
    for lanes in (64, 1000, 4096, 8192, 16384, 32768):
        for mode in (1, 2):
            b = _slot_budget(lanes)
            part, may, rows = emu.scratch(t, lanes, mode, max(320, b), b)
            padded = -(-lanes // 64) * 64
            need = 8 * rows * padded
            whole = min(lanes, SCRATCH // (8 * rows) // 64 * 64)
            assert part == (lanes if need <= SCRATCH else whole if need <= (128 if may else 4) * SCRATCH else 0)
            fits = _slot_rows(t, p, obs, lanes, mode == 2) * padded * 8 <= SCRATCH
            assert may or not fits, (lanes, mode)
            seen.add((fits, may))
    assert (True, True) in seen and (False, False) in seen


@pytest.mark.parametrize("name,lanes,mode,served", [
    # what the slot kernel took stays served: 13 rows there, 9 arrays here; 583 and 6 arrays, a program with matrices
    ("logistic2000", 32768, 1, True), ("mixed200", 8192, 1, True),
    # what it refused is refused again beyond four arrays, however few the lanes of a part
    ("kalman200", 16384, 1, False), ("lotka1000", 4096, 2, False), ("long43000", 4096, 2, False), ("lotka300", 9999, 2, False),
    # up to four arrays in parts
    ("lotka1000", 13007, 1, True), ("kalman60", 4096, 2, True)])
def test_scratch_launches_in_parts(name, lanes, mode, served):
    kind, n = name.rstrip("0123456789"), int(name.lstrip("abcdefghijklmnopqrstuvwxyz"))
    code = {"lotka": lambda: configs.lotka_volterra(L=1, T=n).bytecode, "kalman": lambda: configs.kalman(L=1, T=n).bytecode,
            "logistic": lambda: configs.logistic(L=1, T=n).bytecode, "long": lambda: long_recurrence(n),
            "mixed": lambda: scalars_and_a_product(n, 4, 30)}[kind]()
    b = _slot_budget(lanes)
    part, _, rows = emu.scratch(nd.tape_build(code), lanes, mode, max(320, b), b)
    assert 8 * rows * lanes > SCRATCH
    assert (part >= 64 and part % 64 == 0 and 8 * rows * part <= SCRATCH) if served else part == 0


def test_rows_beyond_the_scratch_array():
    """A wave's rows on both sides of the array's size: the wide program is made
    either way, and the array serves the smaller one."""
    for steps, fits in ((43000, True), (44500, False)):
        t = nd.tape_build(long_recurrence(steps))
        part, may, rows = emu.scratch(t, 64, 2)
        assert (rows * 64 * 8 <= SCRATCH) == fits and part == (64 if fits else 0) and may
    part, may, rows = emu.scratch(nd.tape_build(long_recurrence(90000)), 64, 2)
    assert part == 0 and not may


def test_programs_left_to_the_slot_kernel():
    A = Asm(50, 0)
    A.param(0)
    for i in range(1, 50):
        A.param(i).mul()
    assert emu.wide(nd.tape_build(A.halt().bytes()), np.ones((1, 50)), np.zeros(0)) is None   # parameters
    A = Asm(4, 0)
    for i in range(4):
        A.param(i)
    A.pack(2, 2).exp().trace()
    assert emu.wide(nd.tape_build(A.halt().bytes()), np.ones((1, 4)), np.zeros(0)) is None    # a form without a class
    w = configs.kalman(L=1, T=4)
    t = nd.tape_build(w.bytecode)
    assert emu.wide(t, w.params, w.obs, 1, lds_rows=100) is None                               # LDS
    assert emu.wide(t, w.params, w.obs, 1, lds_rows=260)[2]["n_segments"] > 1
    assert emu.wide(t, w.params, w.obs, 1, lds_rows=1280)[2]["n_segments"] == 1


# ------------------------------------------------------------ machine code
CSRC = os.path.join(ROOT, "paper_2607_03574_amd", "csrc")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
ROLE = {"u": {"S"}, "d": {"D"}, "e": {"D"}, "m": {"S", "D"}, "-": set()}


def _format():
    hdr = open(os.path.join(CSRC, "wide.h")).read()
    body = re.sub(r"//.*", "", re.search(r"enum Class : uint32_t \{(.*?)kClasses", hdr, re.S).group(1))
    names = [x.split("=")[0].strip() for x in body.split(",") if x.strip()]
    assert names.index("END") + 1 == names.index("STE")
    num = dict(kCkSlots="12", kObsSlots="4")
    assert "kObsSlots = 4, kCkSlots = 12" in hdr and "kRegion = 1024" in hdr and "kFileBase = 48" in hdr and "kMatFileBase = 106" in hdr
    info = re.search(r"kInfo\[kClasses\] = \{(.*?)\};", hdr, re.S).group(1)
    info = [tuple(int(num.get(x.strip(), x)) for x in t.split(",")) for t in re.findall(r"\{([^{}]*)\}", info)]
    sch = open(os.path.join(CSRC, "wide_sched.cpp")).read()
    roles = {}
    for line in re.search(r"const char \*roles\(uint32_t cls\) \{(.*?)\n\}", sch, re.S).group(1).split(";"):
        m = re.search(r'return "(.*?)"', line)
        if m:
            roles.update({n: m.group(1) for n in re.findall(r"case (\w+):", line)})
    assert len(names) == len(info)
    return list(zip(names, info)), roles


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """Disassembly of the wide kernels: {address: text}, the functions' address
    ranges by name, and of each kernel (scalar, matrices) the code base, the
    file's first vector register and its classes."""
    import importlib.util
    spec = importlib.util.spec_from_file_location("_b", os.path.join(ROOT, "paper_2607_03574_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    if not os.path.exists(b.HIPCC) or not os.path.exists(OBJDUMP):
        pytest.skip("no device compiler")
    obj = str(tmp_path_factory.mktemp("wide") / "wide.o")
    subprocess.run([b.HIPCC] + b.COMMON + b.DEVICE + b.WIDE + ["--cuda-device-only", "--no-gpu-bundle-output", "-c",
                    os.path.join(CSRC, "wide.hip"), "-o", obj], check=True, capture_output=True)
    text = subprocess.run([OBJDUMP, "-d", obj], check=True, capture_output=True, text=True).stdout
    ins, fn, cur = {}, {}, None
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(.*)>:", line)
        if m:
            cur = m.group(1)
            fn[cur] = []
        m = re.match(r"\s+(.*?)\s+// ([0-9A-F]+): ", line)
        if m:
            a = int(m.group(2), 16)
            ins[a] = m.group(1)
            fn[cur].append(a)
    addrs = sorted(ins)
    fmt, _ = _format()
    scalar = 1 + [n for n, _ in fmt].index("END")
    kernels = []
    for name, first, n in (("ndvm_wideE", 48, scalar), ("ndvm_wide_matrixE", 106, len(fmt))):
        at = next(fn[f] for f in fn if name in f)
        i = next(a for a in at if ins[a].startswith("s_getpc_b64 s[28:29]"))
        j = addrs[addrs.index(i) + 1]
        kernels.append((j + int(ins[j].split(",")[-1], 16), first, fmt[:n]))
    return ins, fn, kernels


def test_entry_points_start_micro_ops(code):
    """Each class's code starts its micro-ops where the format says, reads the
    words of the half it serves, and ends in that half's dispatch."""
    ins, _, kernels = code
    addrs = sorted(ins)
    for base, c, name, (words, most, size) in [(b, c, *f) for b, _, fmt in kernels for c, f in enumerate(fmt)]:
        for half in range(2):
            region = base + (2 * c + half) * 1024
            end = 66 + 32 * half
            for k in range(most):
                at = region + k * size
                assert at in ins, (name, half, k)
                text = [ins[a] for a in addrs if at <= a < at + size]
                used = {int(x) for t in text for x in re.findall(r"\bs(\d+)\b", t)} & set(range(36, 100))
                first = end - (most - k) * words
                assert used <= set(range(first, first + words)), (name, half, k, used)
            after = [ins[a] for a in addrs if region + most * size <= a][:3]
            if name == "END":
                assert after[0].startswith("s_branch")
            elif name == "WAIT":
                assert after[0] == "s_waitcnt vmcnt(0)" and after[2] == f"s_add_u32 s100, s28, s{end}"
            else:
                assert after[0].startswith("s_waitcnt lgkmcnt(0)") and after[1] == f"s_add_u32 s100, s28, s{end}", name


def test_operand_roles(code):
    """The VGPR index applies to exactly the operands that name the file's base
    register, with the role the micro-op's half word carries."""
    ins, _, kernels = code
    addrs = sorted(ins)
    roles = _format()[1]
    for base, file, c, name, (words, most, size) in [(b, f, c, *x) for b, f, fmt in kernels for c, x in enumerate(fmt)]:
        if name in ("WAIT", "END"):
            continue
        halves = []
        for r in roles[name]:
            halves += [r, r] if r in "iRWMz" else [r]      # a whole word
        for half in range(2):
            for k in range(most):
                at = base + (2 * c + half) * 1024 + k * size
                first = 66 + 32 * half - (most - k) * words
                m0, on = None, True

                def role(operand, high):
                    return halves[2 * (int(operand[1:]) - first) + high]

                for a in addrs:
                    if not at <= a < at + size:
                        continue
                    op, _, rest = ins[a].partition(" ")
                    o = [x.strip() for x in rest.split(",")]
                    if op == "s_mov_b32" and o[0] == "m0":
                        m0 = set() if o[1] == "0" else ROLE[role(o[1], 0)]
                    elif op == "s_lshr_b32" and o[0] == "m0":
                        m0 = ROLE[role(o[1], 1)]
                    elif op == "s_lshr_b32" and o[0] == "vcc_lo":
                        assert role(o[1], 1) == "d"
                    elif op == "s_set_gpr_idx_off":
                        on = False
                    elif op == "s_set_gpr_idx_on":
                        on, m0 = True, {"D"} if "DST" in o[1] else set()
                        assert "SRC" not in o[1] and (not m0 or o[0] == "vcc_lo" or role(o[0], 0) == "d")
                    elif op.startswith("v_") and on:
                        dst = [] if op.startswith("v_cmp") else o[:1]
                        src = o[2:] if op.startswith("v_div_scale") else o[1:]
                        for i, x in [(-1, x) for x in dst] + list(enumerate(src)):
                            m = re.match(r"-?v\[?(\d+)", x)
                            if m:
                                assert m0 is not None, (name, ins[a])
                                indexed = "D" in m0 if i < 0 else i == 0 and "S" in m0
                                assert (int(m.group(1)) in (file, file + 1)) == indexed, (name, ins[a], m0)


def test_library_functions_keep_to_their_registers(code):
    """The functions the interpreter calls use no scratch memory, stay below the
    registers it holds across a call, and begin with the wait that the calls
    skip (each call's target is a function's second instruction)."""
    ins, fn, _ = code
    names = [f for f in fn if f.startswith("ndvm_wide_")]
    assert len(names) == 27
    scalar = {"ndvm_wide_" + x for x in ("exp", "sin", "cos", "logc", "sqrtc", "pow", "accsin", "acccos", "acclog",
                                         "accabs", "accpow", "accsqrt", "abs")}
    addrs, entries = sorted(ins), set()
    for i, a in enumerate(addrs):
        if ins[a].startswith("s_swappc_b64"):
            lo = next(x for x in reversed(addrs[:i]) if ins[x].startswith("s_add_u32 s100, s100,"))
            d = int(ins[lo].split(",")[-1], 16)
            entries.add(lo + (d - (1 << 32) if d >> 31 else d))
    assert entries == {fn[f][1] for f in names}
    for f in names:
        assert ins[fn[f][0]] == "s_waitcnt vmcnt(0) expcnt(0) lgkmcnt(0)" and fn[f][1] == fn[f][0] + 4
        for a in fn[f]:
            t = ins[a]
            assert "scratch" not in t and "buffer" not in t and "m0" not in t and "swappc" not in t, (f, t)
            regs = re.findall(r"\b([sv])(?:\[(\d+):(\d+)\]|(\d+)\b)", t)
            most = 39 if f in scalar else 95      # (39 and 95: where prefetches land)
            for kind, lo, hi, one in regs:
                top = int(hi or one)
                if kind == "s" and (lo == "30" or (one == "27" and f not in scalar)):
                    continue                      # the return address, the immediate
                assert top < (26 if kind == "s" else most), (f, t)


def test_build_refuses_functions_its_calls_do_not_fit():
    """The build itself checks the functions that are entered past their first
    instruction: a listing with another first instruction, a longer one, a
    register the interpreter holds, scratch memory or no such function fails."""
    import importlib.util
    spec = importlib.util.spec_from_file_location("_b", os.path.join(ROOT, "paper_2607_03574_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    assert len(b.CALLED["wide.hip"]) == 27 and set(b.CALLED["walk.hip"]) == {"ndvm_walk_sin", "ndvm_walk_cos", "ndvm_walk_pow"}
    wait = "\ts_waitcnt vmcnt(0) expcnt(0) lgkmcnt(0)   // 000000001000: BF8C0000"
    end = "\ts_setpc_b64 s[30:31]   // 000000001010: BE801D1E"

    def listing(body):
        return "\n".join(f"0000000000001000 <{f}>:\n{body if f == 'ndvm_walk_pow' else wait}\n{end}" for f in b.CALLED["walk.hip"])

    b.check_called("walk.hip", listing(wait + "\n\tv_mul_f64 v[38:39], v[0:1], v[2:3]   // 000000001004: D2810000 00020500"))
    for bad in ("\ts_waitcnt lgkmcnt(0)   // 000000001000: BF8CC07F", wait + " 00000000",
                wait + "\n\tv_mul_f64 v[39:40], v[0:1], v[2:3]   // 000000001004: D2810000 00020500",
                wait + "\n\ts_mov_b32 s32, 0   // 000000001004: BEA00080",
                wait + "\n\tscratch_store_dword off, v0, s2   // 000000001004: DC704000 00020000"):
        with pytest.raises(RuntimeError):
            b.check_called("walk.hip", listing(bad))
    with pytest.raises(RuntimeError):
        b.check_called("walk.hip", listing(wait).replace("ndvm_walk_cos", "ndvm_walk_cot"))
