"""What the compiler put into scratch memory, read from the metadata of the library's own gfx950 code, and which kernels lie together."""
import os
import re
import subprocess

import paper_2605_12825_amd as orthrus

from built_code import functions, listings, needs_tool, tool

BALANCED = 2   # the MODE argument of attn_split_kernel<D, W, NS, MODE, NT, PROBE>


def _spills(folder):
    """{mangled kernel: (vector registers spilled, bytes of scratch)}"""
    listings(orthrus.library_path(), folder)
    out = {}
    for f in sorted(f for f in os.listdir(folder) if f.endswith("gfx950")):
        notes = subprocess.run([os.path.join(os.path.dirname(tool()), "llvm-readelf"), "--notes", f], cwd=folder, check=True,
                               stdout=subprocess.PIPE, text=True).stdout
        for kernel in notes.split(".agpr_count:")[1:]:
            field = {k: re.search(r"\.%s:\s+(\S+)" % k, kernel).group(1) for k in ("name", "vgpr_spill_count", "private_segment_fixed_size")}
            out[field["name"]] = int(field["vgpr_spill_count"]), int(field["private_segment_fixed_size"])
    return out


@needs_tool
def test_only_the_balanced_kernel_spills(tmp_path):
    spills = _spills(str(tmp_path))
    forms = {name: re.search(r"attn_(split|by_size|thin)_kernelI((?:Li\d+E)+)E", name) for name in spills}
    forms = {name: (hit.group(1), tuple(int(x) for x in re.findall(r"Li(\d+)E", hit.group(2)))) for name, hit in forms.items() if hit}
    for kind, count in (("split", 2 * (8 * 3 + 4 + 4)), ("by_size", 2 * 8 * 2), ("thin", 2 * 5)):
        assert sum(k == kind for k, _ in forms.values()) == count, kind
    for name, (registers, scratch) in spills.items():
        kind, args = forms.get(name, (None, None))
        if kind == "split" and args[0] == 128 and args[3] == BALANCED:
            assert registers <= 5 and scratch <= 24, name
        else:
            assert registers == 0 and scratch == 0, name


@needs_tool
def test_the_forms_of_the_attention_kernel_lie_apart_from_its_split_and_merge(tmp_path):
    """A batch-1 step runs these two and the consensus; other kernels between them cost it time."""
    for listing in listings(orthrus.library_path(), str(tmp_path)):
        kinds = {hit.group(1) for name, _ in functions(listing) for hit in [re.search(r"attn_(split|combine|by_size|thin|wide)_kernel", name)] if hit}
        assert not ({"split", "combine"} & kinds and {"by_size", "thin", "wide"} & kinds), kinds
