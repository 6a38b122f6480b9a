"""Compile-time properties of the fitted projection tiles (no GPU needed): nothing spills, no compiler wait catches
the direct loads, and the accumulators stay where the matrix instructions find them: a move between the two
register files inside the main loop would run once per accumulator and slab."""
import re

from test_kernel_resources import _device_assembly, _innermost_loops, _waits_among_mfmas

FITTED = "_ZN4mvla18fitted_tile_kernelI"


def test_fitted_tile_main_loops(tmp_path):
    lines = _device_assembly("gemm.hip", tmp_path)
    names = [l.split(":")[0] for l in lines if re.match(r"^%s.*:" % FITTED, l)]
    assert len(names) == 48                                   # 12 tile shapes x 4 epilogues
    text = "\n".join(lines)
    for name in names:
        at = text.index(".amdhsa_kernel " + name)
        assert re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", text[at:]).group(1) == "0", name
    assert all(not w for w in _waits_among_mfmas(lines, FITTED).values())
    loops = {n: [b for b in bodies if sum("v_mfma" in x for x in b) >= 8]
             for n, bodies in _innermost_loops(lines, FITTED).items()}
    for name, bodies in loops.items():
        assert len(bodies) == 1, (name, len(bodies))
        moves = [x for x in bodies[0] if "v_accvgpr" in x]
        assert not moves, (name, moves[:3])
        assert not any("s_waitcnt" in x and "vmcnt" in x for x in _compiled(bodies[0])), name


def _compiled(body):
    """The instructions of a loop that the compiler placed itself (not those of inline asm)."""
    out, in_asm = [], False
    for x in body:
        if "ASMSTART" in x:
            in_asm = True
        elif "ASMEND" in x:
            in_asm = False
        elif not in_asm:
            out.append(x)
    return out
