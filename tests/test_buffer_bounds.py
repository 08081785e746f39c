"""Sizes of the kernels' buffer resources and their attributes, read from the sources.

The hardware accepts a raw buffer access when its per-lane offset is below the
resource's size minus the scalar offset, both unsigned.  A size below the scalar
offset (zero bytes to switch the loads off, say) wraps to a huge limit and bounds
nothing, so a resource's size is the buffer's, never a choice with a zero in it."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2311_08757_amd", "csrc")
CALL = "__builtin_amdgcn_make_buffer_rsrc("


def _arguments(src, start):
    """The top-level arguments of the call whose opening bracket ends at start."""
    depth, args, cur = 1, [], ""
    for ch in src[start:]:
        depth += (ch in "([{") - (ch in ")]}")
        if depth == 0:
            return [a.strip() for a in args + [cur]]
        if ch == "," and depth == 1:
            args.append(cur)
            cur = ""
        else:
            cur += ch
    raise ValueError("unbalanced call")


def _resources():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        src = open(path).read()
        for m in re.finditer(re.escape(CALL), src):
            yield "%s:%d" % (os.path.basename(path), src.count("\n", 0, m.start()) + 1), _arguments(src, m.end())


@pytest.mark.parametrize("where,args", list(_resources()))
def test_resources_have_their_buffers_size(where, args):
    assert len(args) == 4, where
    assert "?" not in args[2] and not re.fullmatch(r"0[uUlL]*", args[2]), (where, args[2])


def test_kernel_attributes_are_set_in_one_place():
    """The dynamic-LDS limit is the kernel's, shared by all problems and threads: it
    is set once to the most any launch takes, never by a launch to its own size."""
    srcs = {p: open(p).read() for p in glob.glob(os.path.join(CSRC, "*.hip"))}
    calls = [(p, m.start()) for p, s in srcs.items() for m in re.finditer(r"hipFuncSetAttribute\(", s)]
    assert len(calls) == 1, calls
    path, at = calls[0]
    assert "if (done.count(" in srcs[path][srcs[path].rindex("\nstatic ", 0, at):at]
