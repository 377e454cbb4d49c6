"""Loads straight into LDS (global_load_lds) that may still be under way, found in the AMD assembly of a source of csrc/.

The compiler does not know of loads that asm statements request: a barrier does not wait for them, only a written
"s_waitcnt vmcnt(n)" does.  LDS that such a load can still reach must not be used for anything else, and a wavefront must
not end before it has arrived (its LDS may be another workgroup's by then).

    kernels(source)  ->  {kernel: [(line number, instruction), ...]}
"""
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
VMEM = re.compile(r"(global|buffer|flat|scratch)_(load|store|atomic)")


def kernels(source):
    from paper_2105_04246_amd import build
    with tempfile.TemporaryDirectory() as folder:
        out = os.path.join(folder, "kernel.s")
        flags = [f for f in build.FLAGS if f not in ("-shared", "-Wall")]
        r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["-S", "--offload-device-only", "-o", out,
                            os.path.join(ROOT, "paper_2105_04246_amd", "csrc", source)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        with open(out) as f:
            lines = f.read().splitlines()
    found, name = {}, None
    for number, line in enumerate(lines, 1):
        line = line.split(";")[0].strip()
        if re.match(r"_Z\w+:$", line):
            name = line[:-1]
            found[name] = []
        elif line.startswith(".section") or line.startswith(".end_amdhsa"):
            name = None
        elif name and line and (not line.startswith(".") or line.endswith(":")):
            found[name].append((number, line))
    return found


def under_way(code):
    """[(line number, instruction)] of `code` that some path reaches with a load into LDS possibly under way.

    Loads and stores retire in order, so one number says it all: how many others were requested after the youngest load into
    LDS, at the least over all paths (None: surely arrived).  Waiting until n are left leaves that load open if it is fewer."""
    starts = {line[:-1]: i for i, (_, line) in enumerate(code) if line.endswith(":")}
    young = {0: None}
    todo, seen = [0], {}

    def less(a, b):
        return a is not None and (b is None or a < b)

    while todo:
        i = todo.pop()
        d = young[i]
        while i < len(code):
            line = code[i][1]
            if i in seen and not less(d, seen[i]):
                break
            seen[i] = d
            op = line.split()[0]
            if op.startswith("global_load_lds"):
                d = 0
            elif VMEM.match(op):
                d = None if d is None else d + 1
            elif op == "s_waitcnt":
                n = re.search(r"vmcnt\((\d+)\)", line)
                if n and d is not None and d >= int(n.group(1)):
                    d = None
            target = starts.get(line.split()[-1]) if op.startswith("s_cbranch") or op == "s_branch" else None
            if target is not None and (target not in seen or less(d, seen[target])):
                young[target] = d
                todo.append(target)
            if op in ("s_branch", "s_endpgm"):
                break
            i += 1
    return [code[i] for i in sorted(seen) if seen[i] is not None]
