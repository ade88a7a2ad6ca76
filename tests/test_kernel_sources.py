"""CPU-only checks of the device sources themselves, for mistakes that no result shows on the machine at hand."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_15562_amd", "csrc")


def _asm_statements(text):
    """(line, text) of every asm statement, its parentheses balanced outside string literals."""
    for m in re.finditer(r"\basm volatile\s*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if quoted:
                i += c == "\\"
                quoted = c != '"'
            elif c == '"':
                quoted = True
            else:
                depth += (c == "(") - (c == ")")
            i += 1
        yield text.count("\n", 0, m.start()) + 1, text[m.start():i]


def test_wait_states_own_what_they_protect():
    """Wait states (s_nop) order nothing for the compiler by themselves: they stand in one statement with the instruction they
    belong to, or they name the registers that it wrote as operands ("+v"). Products issued in assembly are not known to the
    compiler as matrix instructions, so nothing else keeps a read of their results behind the wait."""
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        for line, stmt in _asm_statements(open(path).read()):
            if "s_nop" not in stmt:
                continue
            seen += 1
            assert re.search(r'v_mfma|global_store|"\+v"\(', stmt), f"{os.path.basename(path)}:{line}: {stmt}"
    assert seen >= 4


def test_wave_barriers_stand_between_fences():
    """A wave barrier keeps instructions in place, not memory accesses: what lanes leave each other in LDS is ordered by the fences around it
    (left out, a read may be moved to where only some lanes' writes have been seen; at wavefront scope they cost no instruction)."""
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        lines = [x.strip() for x in open(path).read().split("\n")]
        for i, x in enumerate(lines):
            if x.startswith("__builtin_amdgcn_wave_barrier()"):
                seen += 1
                assert lines[i - 1].startswith("__builtin_amdgcn_fence(__ATOMIC_RELEASE"), f"{os.path.basename(path)}:{i + 1}"
                assert lines[i + 1].startswith("__builtin_amdgcn_fence(__ATOMIC_ACQUIRE"), f"{os.path.basename(path)}:{i + 1}"
    assert seen >= 4


def test_mode_bits_are_put_back():
    """A bit of the mode register that a function clears is set again before it ends, by a statement that its last result passes through."""
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        text = open(path).read()
        state = {}
        for line, stmt in _asm_statements(text):
            for bit, value in re.findall(r"s_setreg_imm32_b32 hwreg\(HW_REG_MODE, (\d+), 1\), ([01])", stmt):
                where = f"{os.path.basename(path)}:{line}"
                if value == "0":
                    assert not state.get(bit), f"{where}: cleared twice"
                    state[bit] = where
                    seen += 1
                else:
                    assert state.pop(bit, None), f"{where}: set without having been cleared"
                    assert '"+v"(' in stmt, f"{where}: nothing keeps it behind what needs the bit off"
        assert not state, f"left cleared: {state}"
    assert seen >= 1
