"""The GEMM's main loop waits for its activation slabs by counting: s_waitcnt vmcnt(n) leaves the n youngest vector-memory operations
outstanding, and n counts weight loads that the source issues and nobody reads in the last round.  A compiler that dropped or sank
one of them would make a wait too weak without an error.  So the built library is looked at: every path through every instance of the kernel is walked
with the queue of outstanding operations, and no slab may be read, no LDS re-used and no wavefront ended before its transfers have landed."""
import os
import re
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{template arguments: [(label, mnemonic, operands)]} of the instances of gemm_bf16_kernel in the library."""
    from paper_2604_26779_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    out = tmp_path_factory.mktemp("code")
    (out / "lib.so").symlink_to(binding.LIB_PATH)
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=out, check=True, capture_output=True)
    found, body = {}, None
    for part in sorted(out.glob("*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(part)], check=True, capture_output=True, text=True).stdout
        label = None
        for line in text.splitlines():
            head = re.match(r"^[0-9a-f]+ <(.+)>:", line)
            if head and head.group(1).startswith("_Z"):
                m = re.match(r"_ZN5specv16gemm_bf16_kernelI(.*?)EEv", head.group(1))
                body = found.setdefault(tuple(int(v) for v in re.findall(r"L[ib](\d+)E", m.group(1) + "E")), []) if m else None
            elif head:
                label = head.group(1)
            elif body is not None and line.startswith("\t"):
                words = line.split("//")[0].split(None, 1)
                body.append((label, words[0], words[1].strip() if len(words) > 1 else ""))
                label = None
    return found


def _walk(body, allowed):
    """The first fault on any path, or None.  `allowed`: transfers that may be outstanding at a barrier of the loop."""
    at = {label: i for i, (label, _, _) in enumerate(body) if label}
    todo, seen = [(0, "", 0)], set()                    # (instruction, queue of T = transfer into LDS / V = other, transfers outstanding at the last barrier)
    while todo:
        i, queue, at_barrier = todo.pop()
        while (i, queue, at_barrier) not in seen:
            seen.add((i, queue, at_barrier))
            _, op, args = body[i]
            if op.startswith(("global_store", "ds_write", "ds_store", "s_endpgm")):      # the epilogue, or the end
                if "T" in queue or at_barrier and op.startswith("ds_"):
                    return "%s %s with transfers outstanding (%s)" % (op, args, queue)
                break
            if op.startswith(("buffer_load", "global_load", "scratch_", "flat_", "global_atomic")):
                queue += "T" if args.split()[-1] == "lds" else "V"
            elif op == "s_waitcnt":
                n = re.search(r"vmcnt\((\d+)\)", args)
                if n:
                    queue = queue[max(0, len(queue) - int(n.group(1))):]
            elif op == "s_barrier":
                at_barrier = queue.count("T")
                if at_barrier > allowed:
                    return "s_barrier with %d transfers outstanding, %d allowed (%s)" % (at_barrier, allowed, queue)
            if op.startswith(("s_cbranch", "s_branch")):
                target = at[args.split()[0]]
                if op == "s_branch":
                    i = target
                    continue
                todo.append((target, queue, at_barrier))
            i += 1
    return None


def test_no_path_reads_a_slab_before_it_has_landed(kernels):
    assert len(kernels) > 100
    for args, body in sorted(kernels.items()):
        MB, XF, LA = args[0], args[6], args[8]
        assert sum(op.startswith("buffer_load") and ops.endswith("lds") for _, op, ops in body) >= 2 * MB * XF, args
        # a slab is MB * XF transfers per wavefront; those of the slabs beyond the next one stay outstanding
        assert _walk(body, (LA - 1) * MB * XF) is None, (args, _walk(body, (LA - 1) * MB * XF))


def test_the_walk_sees_a_dropped_load(kernels):
    """Any single weight load of the loop taken out of a listing makes a wait too weak."""
    for args in ((1, 1, 0, 0, 1, 0, 1, 2, 2), (2, 1, 1, 0, 1, 1, 1, 4, 2), (2, 2, 0, 0, 2, 0, 2, 2, 1)):
        body = kernels[args]
        MB, XF, LA = args[0], args[6], args[8]
        loop = next(i for i, (_, op, _) in enumerate(body) if op == "s_barrier")
        loads = [i for i, (_, op, ops) in enumerate(body) if i > loop and op.startswith("global_load_dwordx4")]
        assert loads
        for i in loads:
            gone = body[:i] + [(body[i][0], "s_nop", "0")] + body[i + 1:]
            assert _walk(gone, (LA - 1) * MB * XF) is not None, (args, body[i])
