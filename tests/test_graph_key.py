"""A captured inference holds the addresses of the buffers its kernels read, so the key under which it is replayed
has to name every one of them.  Read from the sources: the buffers reached from the functions that enqueue the
sweeps, and those that the key and the context's list of buffers name."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2006_03512_amd", "csrc")
FILES = ("api.hip", "sweep_kernels.hip", "mrf_internal.hpp")


def _source(name):
    with open(os.path.join(CSRC, name)) as f:
        s = f.read()
    return re.sub(r"//[^\n]*", "", s)


def _functions():
    """{name: bodies of the functions of that name} of the host code: from a definition's line to the brace in column 0."""
    out = {}
    for f in FILES:
        for m in re.finditer(r"^[A-Za-z][^\n;{}=#]*?\b(\w+)\([^;{}]*\)(?:\n\{\n(.*?)^\}| \{([^\n]*)\}$)", _source(f),
                             re.M | re.S):
            out.setdefault(m.group(1), []).append(m.group(2) or m.group(3))
    return out


def _reached(funcs, name):
    seen, todo, bufs = set(), [name], set()
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        for body in funcs.get(f, ()):
            bufs |= set(re.findall(r"\bc->(b_\w+)", body))
            for lst in re.findall(r"\bc->(vox|pair)\b(?!\.cnt)", body):
                bufs |= {lst + ".desc", lst + ".hub"}
            todo += [g for g in re.findall(r"\b(\w+)\b", body) if g in funcs]
    return bufs, seen


def _declared():
    """Every buffer that a context has (the copies of host inputs, which only the traversal reads, apart)."""
    s = _source("mrf_internal.hpp")
    body = re.search(r"^struct mrf_ctx \{\n(.*?)^\};", s, re.M | re.S).group(1)
    bufs = set()
    for names in re.findall(r"mrf::DevBuf ([^;]*);", body):
        bufs |= set(re.findall(r"b_\w+", names))
    for name in re.findall(r"mrf::SegList (\w+);", body):
        bufs |= {name + ".desc", name + ".hub"}
    return bufs - {"b_host_in"}


def _named(funcs, name):
    bufs = set()
    for body in funcs[name]:
        bufs |= set(re.findall(r"&?c->(b_\w+|vox\.desc|vox\.hub|pair\.desc|pair\.hub)", body))
        if name != "context_buffers" and "context_buffers(" in body:
            bufs |= _named(funcs, "context_buffers")
    return bufs


@pytest.mark.parametrize("entry", ["enqueue_forward", "enqueue_forward_kf"])
def test_key_names_every_buffer_of_the_captured_sweeps(entry):
    funcs = _functions()
    bufs, seen = _reached(funcs, entry)
    # the search goes through the launches down to the kernels' arguments
    assert {"launch_first_sweep", "ray_phase", "seg_work", "run_sum", "small_tiles"} <= seen
    assert entry == "enqueue_forward" or "pair_weights" in seen
    assert {"b_col", "b_g", "b_theta", "b_runrow", "b_hubsum", "b_ray_list"} <= bufs
    assert bufs <= _named(funcs, "graph_key"), sorted(bufs - _named(funcs, "graph_key"))


def test_context_releases_every_buffer():
    funcs = _functions()
    assert _declared() <= _named(funcs, "mrf_destroy"), sorted(_declared() - _named(funcs, "mrf_destroy"))


@pytest.mark.parametrize("entry", ["mrf_infer_sensor", "mrf_infer_keyframe_avg"])
def test_a_failed_capture_overwrites_nothing(entry):
    """The sweeps are captured before the new prior and tables are written, so that an inference whose capture fails
    leaves the beliefs of the last one."""
    (body,) = _functions()[entry]
    assert body.index("capture_sweeps(") < body.index("launch_infer_inputs(") < body.index("launch_graph(")
