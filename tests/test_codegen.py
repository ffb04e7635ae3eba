"""Code-generation checks of the gfx950 kernels (CPU only: hipcc
cross-compiles to AMD assembly).

* No kernel spills to scratch.
* In the large-tile GEMM, the global->LDS loads of the next K step stay in
  flight while the current step's fragments are read: no `s_waitcnt vmcnt`
  immediately before a `ds_read_b128` (the compiler inserts one whenever it
  cannot tell the two LDS stages apart, which serialises load and compute).
* No packed fp32 arithmetic is emitted.
* No wave meets a barrier with LDS accesses of its own unfinished.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_09643_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                                reason="hipcc not available")


def _asm(src):
    from paper_2606_09643_amd.build import FLAGS, _hipcc
    out = subprocess.run([_hipcc(), *FLAGS, "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", "-"],
                         capture_output=True, text=True)
    assert out.returncode == 0, out.stderr[-2000:]
    return out.stdout


def _kernels(asm):
    """{kernel symbol: body text}"""
    res = {}
    for m in re.finditer(r"^(_Z\S+):\s*(?:;.*)?$", asm, re.M):
        name = m.group(1)
        end = asm.find(".Lfunc_end", m.end())      # early exits end the program too
        res[name] = asm[m.end():end]
    return res


@pytest.fixture(scope="module")
def all_asm():
    return {f: _asm(f) for f in sorted(os.listdir(CSRC)) if f.endswith(".hip")}


def test_no_scratch_spills(all_asm):
    for f, asm in all_asm.items():
        for name, size in re.findall(r"\.set (\S+)\.private_seg_size, (\d+)", asm):
            assert int(size) == 0, f"{f}: {name} uses {size} bytes of scratch"


def test_large_gemm_keeps_lds_dma_in_flight(all_asm):
    ks = {k: v for k, v in _kernels(all_asm["k_gemm.hip"]).items() if "gemm_bf16_large_kernel" in k}
    assert len(ks) == 24   # 4 epilogues x 3 tile shapes x packed / one-run LoRA steps
    for name, body in ks.items():
        lines = [l.strip() for l in body.splitlines() if l.strip() and not l.strip().startswith(";")]
        assert any(l.startswith("global_load_lds_dwordx4") for l in lines), name
        for prev, cur in zip(lines, lines[1:]):
            if cur.startswith("ds_read_b128"):
                assert "vmcnt" not in prev, f"{name}: DMA wait before a fragment read"


def test_no_packed_fp32(all_asm):
    for f, asm in all_asm.items():
        assert not re.search(r"\bv_pk_(add|mul|fma)_f32\b", asm), f


def test_lds_reads_stay_lds(all_asm):
    """LDS tiles are read with ds_* instructions and device tables' factors with
    global_*: a pointer that the compiler loses track of (one into LDS passed
    through an asm statement, one from a table indexed at run time) becomes a
    generic pointer, and its reads flat loads, which wait as both kinds."""
    for f, asm in all_asm.items():
        for name, body in _kernels(asm).items():
            assert not re.search(r"^\s+flat_(load|store)", body, re.M), f"{f}: {name} uses flat memory ops"


def test_gelu_polynomial_error_bound():
    """The bf16 GELU epilogue's polynomial (coefficients read from the kernel
    header, evaluated in float32 in the kernel's order) stays within its
    stated error against the exact erf form: <= 1e-4 for |x| <= 4 and
    5.4e-5 |x| beyond (the fit error at the clamp point plus the normal tail)."""
    import numpy as np
    from scipy.special import erf
    src = open(os.path.join(CSRC, "vfm_internal.h")).read()
    body = src[src.index("__device__ inline float gelu_fast"):]
    body = body[:body.index("\n}\n")]
    lits = [float(v) for v in re.findall(r"(-?\d+\.\d*(?:e-?\d+)?)f", body)]
    assert len(lits) == 2 + 8 + 1, lits      # clamp +-4, the 8 coefficients, 0.5
    assert lits[0] == -4.0 and lits[1] == 4.0 and lits[-1] == 0.5
    coef = [np.float32(c) for c in lits[2:-1]]  # highest power first, as evaluated
    x = np.linspace(-12, 12, 2_400_001).astype(np.float32)
    t = np.clip(x, np.float32(-4), np.float32(4))
    u = t * t
    p = np.full_like(x, coef[0])
    for c in coef[1:]:
        p = (p * u + c).astype(np.float32)
    g = (x * (p * t + np.float32(0.5))).astype(np.float32)
    xd = x.astype(np.float64)
    ref = 0.5 * xd * (1.0 + erf(xd / np.sqrt(2.0)))
    err = np.abs(g - ref)
    inner = np.abs(x) <= 4
    assert err[inner].max() <= 1e-4, err[inner].max()
    assert np.all(err[~inner] <= 5.4e-5 * np.abs(xd[~inner]))
    # GELU(0) = 0 exactly, and odd symmetry of the polynomial part
    x0 = np.zeros(1, np.float32)
    p0 = np.full_like(x0, coef[0])
    for c in coef[1:]:
        p0 = (p0 * x0 * x0 + c).astype(np.float32)
    assert float((x0 * (p0 * x0 + np.float32(0.5)))[0]) == 0.0


def _regs(op):
    """Registers named by an operand: v5 -> {5}, v[4:7] -> {4..7} (VGPRs only)."""
    m = re.fullmatch(r"v(\d+)", op)
    if m:
        return {int(m.group(1))}
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", op)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    return set()


def test_untracked_loads_not_touched_before_their_wait(all_asm):
    """Loads issued from inline asm are invisible to the compiler's wait
    insertion: the kernel's own s_waitcnt vmcnt must come before anything
    reads (or overwrites) their destination registers.  A register copy
    placed between such a load and its wait (for instance to carry the value
    around a loop) would read the register before the data landed.  The scan
    follows each kernel's instructions in program order, keeping the vector
    memory operations in flight; vmcnt(N) retires all but the last N."""
    vmem = re.compile(r"^(global_|buffer_|flat_|scratch_)")
    checked = 0
    for f, asm in all_asm.items():
        for name, body in _kernels(asm).items():
            inflight = []                                 # per VMEM op: its register set if untracked, else None
            in_asm = False
            for raw in body.splitlines():
                t = raw.strip()
                if t.startswith(";;#ASMSTART"):
                    in_asm = True
                    continue
                if t.startswith(";;#ASMEND"):
                    in_asm = False
                    continue
                l = t.split(";")[0].strip()
                if not l or l.endswith(":") or l.startswith("."):
                    continue
                mnem, _, rest = l.partition(" ")
                ops = [o.strip() for o in rest.split(",")] if rest else []
                if mnem == "s_waitcnt":
                    m = re.search(r"vmcnt\((\d+)\)", rest)
                    if m:
                        n = int(m.group(1))
                        inflight = inflight[len(inflight) - n:] if n else []
                    continue
                if not in_asm:
                    used = set().union(*(_regs(o) for o in ops)) if ops else set()
                    for regs in inflight:
                        if regs is not None:
                            assert not (used & regs), f"{f}: {name}: '{l}' touches an in-flight untracked load"
                if vmem.match(mnem):
                    if in_asm and mnem.startswith("global_load") and ops:
                        inflight.append(_regs(ops[0]))
                        checked += 1
                    else:
                        inflight.append(None)
    assert checked > 0


def _flow(body):
    """(basic blocks as instruction lists, {label: block}) of a kernel's text."""
    blocks, labels = [[]], {}
    for raw in body.splitlines():
        l = raw.split(";")[0].strip()
        if l.startswith(".L") and l.endswith(":"):
            if blocks[-1]:
                blocks.append([])
            labels[l[:-1]] = len(blocks) - 1
        elif l and not l.startswith(".") and not l.endswith(":"):
            blocks[-1].append(l)
            if re.match(r"s_(c?branch|endpgm)", l):
                blocks.append([])
    return blocks, labels


def _unfinished_at_barriers(body):
    """The LDS accesses (r / w) that a wave may still have in flight at each
    s_barrier, over every path: a walk of the control flow with the lgkmcnt
    operations in issue order.  lgkmcnt(N) retires all but the last N, except
    beside scalar loads (s), which complete in any order."""
    blocks, labels = _flow(body)
    rank = {"r": 3, "w": 2, "s": 1}

    def merge(a, b):                                      # the longer, the worse of each, from the newest back
        long, short = (a, b) if len(a) >= len(b) else (b, a)
        tail = [max(x, y, key=rank.get) for x, y in zip(long[len(long) - len(short):], short)]
        return long[:len(long) - len(short)] + tuple(tail)

    entry, todo, found = {0: ()}, [0], {}
    while todo:
        i = todo.pop()
        state, succ, falls = entry[i], [], True
        for j, l in enumerate(blocks[i]):
            mnem, _, rest = l.partition(" ")
            if mnem == "s_waitcnt" and "lgkmcnt" in rest:
                n = int(re.search(r"lgkmcnt\((\d+)\)", rest).group(1))
                state = () if n == 0 else state if "s" in state else state[-n:]
            elif mnem == "s_barrier":
                found[i, j] = merge(found.get((i, j), ()), state)
            elif mnem.startswith("ds_read") or mnem.startswith("flat_load"):
                state = (state + ("r",))[-64:]
            elif mnem.startswith(("ds_", "flat_")):
                state = (state + ("w",))[-64:]
            elif re.match(r"s_(buffer_)?load", mnem):
                state = (state + ("s",))[-64:]
            elif re.match(r"s_c?branch", mnem):
                succ.append(labels[rest.strip()])
                falls = mnem != "s_branch"
            elif mnem == "s_endpgm":
                falls = False
        if falls and i + 1 < len(blocks):
            succ.append(i + 1)
        for k in succ:
            new = merge(entry[k], state) if k in entry else state
            if entry.get(k) != new:
                entry[k] = new
                todo.append(k)
    return [set(v) & {"r", "w"} for v in found.values()]


def test_lds_accesses_finish_before_barriers(all_asm):
    """A wave's LDS reads and writes have finished when it meets a barrier:
    after it another wave may fill the stage that they touch (the GEMMs' raw
    barriers carry no wait of their own)."""
    barriers = 0
    for f, asm in all_asm.items():
        for name, body in _kernels(asm).items():
            found = _unfinished_at_barriers(body)
            barriers += len(found)
            assert not any(found), f"{f}: {name} passes a barrier with {found} unfinished"
    assert barriers > 100
