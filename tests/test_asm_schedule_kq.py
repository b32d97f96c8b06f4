"""Static checks of gemm_kq_kernel's machine code (CPU only), with the checkers
of test_asm_schedule.py: the MFMA wait states the compiler does not see, no
register that a load or an LDS read targets touched before it has landed, and,
since the kernel's own counted waits rely on it, the number of vector-memory
operations of an unrolled pass of its loop."""
import os
import re
import tempfile

import pytest

import test_asm_schedule as T

KERNEL = "gemm_kq_kernel"


def loop_code(body):
    """The instructions before the kernel's step loop, of one pass of it from
    its header on (the compiler may lay the header out last; every block marked
    as part of it), and after it, in the order they are laid out."""
    cur = ("entry", False, [])
    blocks = [(None, False, cur[2])]
    for line in body.splitlines():
        m = re.match(r"^\.LBB(\d+_\d+):(.*)", line)
        if m:
            head = "Loop Header" in m.group(2)
            part = head or "in Loop: Header" in m.group(2)
            cur = (m.group(1), head, [])
            blocks.append(cur if part else (None, False, cur[2]))
        cur[2].append(line)
    part = [k for k, b in enumerate(blocks) if b[0] is not None]
    heads = [k for k in part if blocks[k][1]]
    assert len(heads) == 1, "one loop, no waterfall loops"
    inside = [k for k in part if k >= heads[0]] + [k for k in part if k < heads[0]]
    before, after = range(part[0]), [k for k in range(part[0], len(blocks)) if k not in part]
    return [T.code(T.parse("\n".join(ln for k in ks for ln in blocks[k][2]))) for ks in (before, inside, after)]


@pytest.fixture(scope="module")
def fns():
    if not os.path.exists(T.B.HIPCC):
        pytest.skip("hipcc not available")
    with tempfile.TemporaryDirectory(prefix="tf_asm_") as tmp:
        out = T._compile_asm(os.path.join(T.B.CSRC, "tf_gemm_kq.hip"), os.path.join(tmp, "kq.s"))
        text = open(out).read()
    got = [(m.group(1), T.parse(m.group(2)), loop_code(m.group(2)))
           for m in re.finditer(r"^(_Z\S+):[^\n]*\n(.*?)^\.Lfunc_end", text, re.S | re.M) if KERNEL in m.group(1)]
    assert len(got) == 16      # both widths, both types, 128 x 128 and 64 x 64 tiles, whole chunks or any K
    return got


def _args(name):
    m = re.search(r"ILi(\d)ELb(\d)ELi(\d)ELi(\d)ELb(\d)E", name)
    return [int(v) for v in m.groups()]


def test_mfma_wait_states(fns):
    for name, ins, (_, loop, _) in fns:
        assert T.check_mfma_hazards(T.code(ins)) == [], name
        assert T.check_mfma_hazards(2 * loop) == [], name


def test_loads_land_before_use(fns):
    for name, ins, (_, loop, _) in fns:
        assert not any(op.startswith("scratch_") for op, _, _ in ins), name
        assert T.check_vm_waits(3 * loop) == [], name


def test_loads_per_pass(fns):
    for name, _, (_, loop, _) in fns:
        bits, _, rb, nb, g4 = _args(name)
        panels = 16 * nb // (64 if bits == 4 else 32)
        loads = [a for op, a in loop if op.startswith("buffer_load")]
        lds = sum(a.endswith(" lds") for a in loads)
        assert lds == 2 * 2 * rb, name
        assert len(loads) - lds == 4 * panels + (1 if g4 else 4) * 2 * panels, name
        assert sum(op.startswith("v_mfma") for op, _ in loop) == 4 * rb * nb, name


def test_direct_loads_land_before_their_reads(fns):
    """A step's fragments are read with at most the newest pair's direct loads
    in flight (the buffer being read is the older one): in the prologue, over
    three passes of the loop and over the steps that follow it."""
    for name, _, (before, loop, after) in fns:
        rb = _args(name)[2]
        end = next(k for k, (op, _) in enumerate(after) if op == "s_barrier")
        queue, reads = [], 0
        for op, a in before + 3 * loop + after[:end]:
            if op.startswith("buffer_load"):
                queue.append(a.endswith(" lds"))
            elif op == "s_waitcnt" and "vmcnt" in a:
                n = int(re.search(r"vmcnt\((\d+)\)", a).group(1))
                queue = queue[max(0, len(queue) - n):]
            elif op.startswith("ds_read"):
                reads += 1
                assert sum(queue) <= 2 * rb, name
        assert reads >= 13 * rb, name
