"""The matrix products of the attention kernel are inline asm: the compiler neither sees their results arrive nor puts the
waits of the hardware around them, and a wait that is missing shows as a wrong number now and then, with no error. Here
the assembly that the build's flags give is read for three rules, along every path:

  operands      a register that the vector ALU has just written is not an operand of a product within two wait states
  results       a result is touched by anything but a product at the earliest eight wait states on, and those are stated in the
                source: waits of settle_products and further products (the matrix pipe takes four wait states for each). Behind
                the first scheduling barrier that follows settle_products the order of the instructions is the source's too
  accumulators  the next product into the same accumulator has at least three others ahead of it
"""
import re
import subprocess

import pytest

from paper_2511_19835_amd import build

OPERAND_STATES, RESULT_STATES, PRODUCT_STATES, PRODUCTS_BETWEEN = 2, 8, 4, 3


def _registers(text):
    regs = set()
    for one, first, last in re.findall(r"\bv(?:(\d+)|\[(\d+):(\d+)\])(?![\w\[])", text):
        regs.update([int(one)] if one else range(int(first), int(last) + 1))
    return regs


class Instruction:
    def __init__(self, text, stated):
        self.text = text
        self.name, _, rest = text.partition(" ")
        operands = rest.split(",")
        self.product = self.name.startswith("v_mfma")
        self.vector = self.name.startswith("v_") and not self.product
        self.regs = [_registers(x) for x in operands]
        self.touched = set().union(*self.regs)
        self.written = set()
        if self.vector or self.product:
            both = "swap" in self.name
            self.written = set().union(*(self.regs if both else self.regs[:1]))
        nop = int(rest) + 1 if self.name == "s_nop" else 0
        self.states = nop or 1                       # wait states that pass, whoever put the instruction there
        self.stated = nop if stated else 0           # ... that the source asks for
        self.barrier = False


def _kernels(listing):
    """name -> (instructions, successors) of every function with products; a scheduling barrier is an instruction of no length."""
    bodies, body, stated = {}, None, False
    for line in listing.splitlines():
        if re.match(r"_Z\w+:", line):
            body = bodies.setdefault(line.split(":")[0], [])
        if body is None:
            continue
        if "#ASMSTART" in line or "#ASMEND" in line:
            stated = "#ASMSTART" in line
        if "; sched_barrier" in line:
            body.append("sched_barrier")
        text = line.split(";")[0].strip()
        if re.match(r"\.LBB\w+:", text):
            body.append(text)
        elif text and not text.startswith((".", "_Z")) and not text.endswith(":"):
            body.append((" ".join(text.split()), stated))
        if text.startswith(".Lfunc_end"):
            body = None
    out = {}
    for name, lines in bodies.items():
        code, labels = [], {}
        for x in lines:
            if isinstance(x, str) and x.endswith(":"):
                labels[x[:-1]] = len(code)
            elif x == "sched_barrier":
                code.append(Instruction("sched_barrier", False))
                code[-1].states, code[-1].barrier = 0, True
            else:
                code.append(Instruction(*x))
        if not any(i.product for i in code):
            continue
        assert not any(i.name.startswith(("s_setpc", "s_swappc")) for i in code), "paths are followed through branches only"
        after = []
        for k, i in enumerate(code):
            target = [labels[i.text.split()[-1]]] if re.match(r"s_c?branch", i.name) else []
            ends = i.name in ("s_branch", "s_endpgm") or k + 1 == len(code)
            after.append(target + ([] if ends else [k + 1]))
        out[name] = (code, after)
    return out


def _walk(after, start, state, step):
    """Follows every path from behind `start`; step(place, state) gives the state behind that instruction, or None to end."""
    seen, todo = set(), [(k, state) for k in after[start]]
    while todo:
        k, state = todo.pop()
        if (k, state) in seen:
            continue
        seen.add((k, state))
        state = step(k, state)
        if state is not None:
            todo += [(n, state) for n in after[k]]


def violations(listing):
    found = []
    for name, (code, after) in _kernels(listing).items():
        for start, first in enumerate(code):
            def operand(k, states):
                i = code[k]
                if i.product and first.written & i.touched:
                    found.append(("operand", name, first.text, i.text))
                states += i.states
                return states if states < OPERAND_STATES else None

            def result(k, state):
                states, settled = state
                i = code[k]
                if settled and i.barrier:
                    return None
                uses = set().union(*i.regs[1:3]) if i.product else i.touched
                if first.written & uses:
                    found.append(("result", name, first.text, i.text))
                    return None
                states += i.stated + PRODUCT_STATES * i.product
                return (states, settled or i.stated > 0) if states < RESULT_STATES else None

            def accumulator(k, between):
                i = code[k]
                if i.product and i.written & first.written:
                    found.append(("accumulator", name, first.text, i.text))
                between += i.product
                return between if between < PRODUCTS_BETWEEN else None

            if first.vector and first.written:
                _walk(after, start, 0, operand)
            if first.product:
                _walk(after, start, (0, False), result)
                _walk(after, start, 0, accumulator)
    return found


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("listing") / "attn.s")
    cmd = [build._hipcc(), *build.HIP_FLAGS, "-I", build.INCLUDE, "-I", build.CSRC, "-S", "--cuda-device-only",
           build.CSRC + "/attn_kernels.hip", "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read()


def test_every_product_of_the_attention_kernel_has_its_waits(listing):
    products = [sum(i.product for i in code) for code, _ in _kernels(listing).values()]
    assert len(products) == 5 and min(products) > 100
    found = violations(listing)
    assert not found, "\n".join(map(str, found[:20]))


PRODUCT = "\tv_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]\n"
OTHERS = "".join(f"\tv_mfma_f32_16x16x32_bf16 v[{r}:{r + 3}], v[8:11], v[12:15], 0\n" for r in (20, 24, 28))
STATED = "\t;;#ASMSTART\n\ts_nop 7\n\t;;#ASMEND\n"


@pytest.mark.parametrize("body,rules", [
    (PRODUCT + STATED + "\tv_mul_f32_e32 v4, v5, v2\n", []),
    (PRODUCT + "\ts_nop 7\n\tv_mul_f32_e32 v4, v5, v2\n", ["result"]),                    # not the source's wait
    (PRODUCT + STATED.replace("7", "6") + "\tv_mul_f32_e32 v4, v5, v2\n", ["result"]),
    (PRODUCT + OTHERS + "\tv_mul_f32_e32 v4, v5, v2\n", []),
    (PRODUCT + OTHERS + "\tglobal_store_dwordx4 v[40:41], v[28:31], off\n", ["result"]),
    (PRODUCT + STATED.replace("7", "0") + "\t; sched_barrier mask(0x00000000)\n\tv_mul_f32_e32 v4, v5, v2\n", []),
    (PRODUCT + "\ts_cbranch_scc1 .LBB0_2\n" + STATED + ".LBB0_2:\n\tv_mov_b32_e32 v2, 0\n", ["result"]),
    (PRODUCT + "\tv_mfma_f32_16x16x32_bf16 v[20:23], v[0:3], v[12:15], 0\n", ["result"]),
    (PRODUCT + OTHERS + PRODUCT, []),
    (PRODUCT + "\ts_nop 15\n" + PRODUCT, ["accumulator"]),
    ("\tv_mov_b32_e32 v9, v50\n" + PRODUCT, ["operand"]),
    ("\tv_mov_b64_e32 v[2:3], v[50:51]\n\ts_add_i32 s0, s0, 1\n" + PRODUCT, ["operand"]),
    ("\tv_permlane32_swap_b32_e32 v50, v12\n\ts_nop 0\n" + PRODUCT, ["operand"]),
    ("\tv_mov_b32_e32 v9, v50\n\ts_nop 1\n" + PRODUCT, []),
    ("\tv_mov_b32_e32 v16, v9\n" + PRODUCT, []),
    ("\tv_cmp_lt_i32_e64 s[8:9], v9, v10\n" + PRODUCT, []),
])
def test_the_rules_themselves(body, rules):
    found = violations("_Zkernel:\n" + body + "\ts_endpgm\n")
    assert [f[0] for f in found] == rules
