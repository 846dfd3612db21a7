"""What the compiler made of the partials' way from the split kernel to the merge, read from the shipped code."""
import re

import paper_2605_12825_amd as orthrus
from built_code import functions, listings, needs_tool


def _forms(text, kernel):
    """{template arguments: code} of a kernel's instances."""
    out = {}
    for name, code in functions(text):
        if kernel in name:
            out[tuple(int(x) for x in re.findall(r"Li(\d+)E", name[name.index(kernel):]))] = code
    return out


@needs_tool
def test_merge_of_many_units_loads_live_pieces_only(tmp_path):
    """The four-wave form: a jump in front of every partial's load."""
    seen = 0
    for text in listings(orthrus.library_path(), str(tmp_path)):
        for (d, w, balanced, chunk, waves), code in _forms(text, "attn_combine_kernel").items():
            loads = [i for i, (op, _, _) in enumerate(code) if op == "global_load_dwordx4"]
            jumps = [i for i, (op, _, _) in enumerate(code) if op.startswith("s_cbranch")]
            gaps = [any(x < j < y for j in jumps) for x, y in zip(loads, loads[1:])]
            assert len(gaps) + 1 >= chunk
            if waves == 4 or not balanced:
                assert all(gaps) == (waves == 4), (d, w, balanced, chunk, waves)
            seen += 1
    assert seen == 2 * 8 * 4 * 2


@needs_tool
def test_partials_hint_with_fixed_splits_only(tmp_path):
    """The compiler folds a hinted and a plain store of the same value in two branches into a plain one, so the hint is a
    form of the kernel: 16 bytes of every accumulator block in the fixed-split form, none in the others."""
    seen = 0
    for text in listings(orthrus.library_path(), str(tmp_path)):
        for block in re.split(r"\n(?=[0-9a-f]* ?<_Z)", text):
            head = re.search(r"attn_split_kernelI((?:Li\d+E)+)E", block.split("\n")[0])
            if not head:
                continue
            d, _, _, mode, nt, probe = (int(x) for x in re.findall(r"Li(\d+)E", head.group(1)))
            hinted = len(re.findall(r"\tglobal_store_dwordx4 [^\n]* nt\b", block))
            assert hinted == (d // 8 if (mode, nt, probe) == (0, 1, 0) else 0), head.group(0)
            seen += 1
    assert seen == 2 * (8 * 3 + 4 + 4)
