"""The library's own gfx950 code, disassembled, for tests of what the compiler made of a kernel."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_12825_amd import build

_LINE = re.compile(r"^\t(\S+)(?:\s+(.*?))?\s*// ([0-9A-Fa-f]+):(.*)$")
_TARGET = re.compile(r"<[^>]*?(?:\+0x([0-9a-f]+))?>\s*$")


def tool():
    return os.path.join(os.path.dirname(os.path.dirname(build.hipcc_path())), "llvm", "bin", "llvm-objdump")


needs_tool = pytest.mark.skipif(not os.path.exists(tool()), reason="no llvm-objdump next to the compiler")


def functions(listing):
    """[(name, [(op, args, index of the branch's target or None)])]"""
    out, name, body, start = [], None, [], 0

    def close():
        if name is None:
            return
        at = {addr: i for i, (_, _, addr, _) in enumerate(body)}
        out.append((name, [(op, args, at.get(start + t) if t is not None else None) for op, args, _, t in body]))

    for line in listing.splitlines():
        head = re.match(r"^(?:[0-9a-f]+ )?<(.+)>:$", line)
        if head:
            close()
            name, body, start = head.group(1), [], None
            continue
        hit = _LINE.match(line)
        if not hit:
            continue
        op, rest, addr = hit.group(1), hit.group(2) or "", int(hit.group(3), 16)
        start = addr if start is None else start
        target = None
        if op.startswith("s_branch") or op.startswith("s_cbranch"):
            t = _TARGET.search(hit.group(4))
            assert t, "no branch target in: " + line
            target = int(t.group(1), 16) if t.group(1) else 0
        args = re.split(r",\s*", rest) if rest else []
        if args:   # modifiers follow the last operand
            args[-1] = args[-1].split(" ")[0]
        body.append((op, args, addr, target))
    close()
    return out


def listings(library, folder):
    """The disassembly of every gfx950 code object inside `library`."""
    lib = shutil.copy(library, os.path.join(folder, "lib.so"))
    subprocess.run([tool(), "--offloading", "lib.so"], cwd=folder, check=True, stdout=subprocess.DEVNULL)
    objects = sorted(f for f in os.listdir(folder) if f.endswith("gfx950"))
    assert os.path.exists(lib) and objects
    return [subprocess.run([tool(), "-d", f], cwd=folder, check=True, stdout=subprocess.PIPE, text=True).stdout for f in objects]
