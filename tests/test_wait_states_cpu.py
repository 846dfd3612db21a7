"""Wait states around the direct-to-LDS loads, counted in the code that is shipped.

The loads are written in inline assembly, where the compiler does not keep the distances that the hardware asks of
software: a vector-memory instruction may read a scalar register five wait states after a vector instruction (a lane read,
a compare) has written it, and a direct-to-LDS load may follow the write of M0 by one.  An instruction is a wait state,
s_nop N is N + 1.  The library's own gfx950 code is disassembled and every path into such an instruction is followed
backwards over as many wait states, across branches.
"""
import re

import paper_2605_12825_amd as orthrus
from built_code import functions, listings, needs_tool

LANE_TO_MEMORY, M0_TO_LDS_LOAD = 5, 1
_VMEM = ("global_", "buffer_", "flat_", "scratch_")


def _sgprs(operand):
    """Numbers of the scalar registers in an operand, M0 and VCC by name."""
    operand = operand.strip()
    if operand in ("m0", "vcc"):
        return {operand}
    hit = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if hit:
        return set(range(int(hit.group(1)), int(hit.group(2)) + 1))
    hit = re.fullmatch(r"s(\d+)", operand)
    return {int(hit.group(1))} if hit else set()


def _vector_writes(op, args):
    """Scalar registers that a vector instruction writes: the result of a lane read or compare, or a carry."""
    if not op.startswith("v_") or not args:
        return set()
    out = _sgprs(args[0])
    if len(args) > 1 and re.match(r"v_(add_co|sub_co|subrev_co|addc_co|subb_co|subbrev_co|div_scale|mad_u64_u32|mad_i64_i32)", op):
        out |= _sgprs(args[1])
    return out


def close_reads(listing):
    """([(function, index, text)] of the reads that come too soon, number of reads looked at)"""
    bad, seen = [], 0
    for name, code in functions(listing):
        into = {}   # index -> indices of the instructions that may run before it
        for i, (op, _, target) in enumerate(code):
            if target is not None:
                into.setdefault(target, []).append(i)
            if not op.startswith(("s_branch", "s_endpgm", "s_setpc")) and i + 1 < len(code):
                into.setdefault(i + 1, []).append(i)
        for i, (op, args, _) in enumerate(code):
            if not op.startswith(_VMEM):
                continue
            wanted = [(r, LANE_TO_MEMORY, _vector_writes) for x in args for r in _sgprs(x)]
            if "_lds_" in op:
                wanted.append(("m0", M0_TO_LDS_LOAD, lambda o, a: _sgprs(a[0]) if o.startswith("s_") and a else set()))
            for reg, need, writes in wanted:
                seen += 1
                todo, done = [(j, 0) for j in into.get(i, [])], {}
                while todo:
                    j, states = todo.pop()
                    if states >= need or done.get(j, need) <= states:
                        continue
                    done[j] = states
                    o, a, _ = code[j]
                    if reg in writes(o, a):
                        bad.append((name, i, "%s %s: %s written %d wait states before, %d needed"
                                    % (op, ", ".join(args), reg, states, need)))
                        break
                    if a and o.startswith("s_") and reg in _sgprs(a[0]) and not o.startswith(("s_cmp", "s_bitcmp")):
                        continue   # a scalar instruction has written it since
                    states += int(a[0], 0) + 1 if o == "s_nop" else 1
                    todo += [(k, states) for k in into.get(j, [])]
    return bad, seen


def test_scan_finds_a_planted_distance():
    """Two wait states between a lane read and the load, five, and two behind a branch back."""
    text = """
<f>:
\tv_readlane_b32 s3, v1, s4                                  // 000000000000: 00000000
\ts_mov_b32 m0, s9                                           // 000000000008: 00000000
\ts_nop %d                                                    // 00000000000C: 00000000
\tglobal_load_lds_dwordx4 v2, s[2:3] offset:1040 nt          // 000000000010: 00000000
\tv_readfirstlane_b32 s2, v5                                 // 000000000018: 00000000
\ts_branch 65530                                             // 00000000001C: 00000000 <f+0x%x>
\ts_endpgm                                                   // 000000000020: 00000000
"""
    assert len(close_reads(text % (0, 8))[0]) == 2
    assert len(close_reads(text % (1, 8))[0]) == 2
    assert len(close_reads(text % (3, 8))[0]) == 0
    assert len(close_reads(text % (3, 0xc))[0]) == 0
    assert len(close_reads(text % (3, 0x10))[0]) == 1      # straight to the load
    assert len(close_reads(text.replace("s_nop %d", "v_mov_b32 v9, 0") % 8)[0]) == 2
    assert len(close_reads(text.replace("s_mov_b32 m0, s9", "s_nop 3").replace("s_nop %d", "s_mov_b32 m0, s9") % 8)[0]) == 1


@needs_tool
def test_loads_keep_their_distance_from_lane_reads(tmp_path):
    total = 0
    for listing in listings(orthrus.library_path(), str(tmp_path)):
        bad, seen = close_reads(listing)
        total += seen
        assert not bad, "%d reads too soon, the first ones:\n%s" % (len(bad), "\n".join("%s[%d] %s" % x for x in bad[:8]))
    assert total > 1000   # the direct-to-LDS loads alone are more


@needs_tool
def test_page_ids_of_the_64_row_kernel_arrive_together(tmp_path):
    """Its waves fetch the page ids of many tiles with one or two vector loads and go on to tile loads.  A wait for an id
    behind a tile load would wait for the tile too, and two waits in a row are two round trips."""
    seen = 0
    for listing in listings(orthrus.library_path(), str(tmp_path)):
        for name, code in functions(listing):
            if "attn_wide_kernel" not in name:
                continue
            ids = [i for i, (op, _, _) in enumerate(code) if op == "global_load_dword"]
            while ids:
                first = ids[0]
                waits = [i for i in range(first, len(code)) if code[i][0] == "s_waitcnt" and "vmcnt(0)" in code[i][1][0]]
                tile = next(i for i in range(first, len(code)) if "load_lds" in code[i][0])
                group = [i for i in ids if i < waits[0]]
                assert waits[0] < tile and not any(i < tile for i in ids[len(group):]), name
                assert all(not (tile < x < tile + 16) for x in waits), name
                ids = ids[len(group):]
                seen += 1
    assert seen >= 2 * 11   # the fill and the loop of each instance
