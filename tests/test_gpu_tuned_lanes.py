"""Lanes per operation by call size: a table whose tuning entry names one lane
per operation runs eight while a call's operations are all in flight at once."""
import ctypes
import json

import numpy as np
import pytest

import gen
import oracle
from gpu_util import check_stream_batches, check_table_invariants, dev_u32

pytestmark = pytest.mark.gpu


@pytest.fixture
def lhs(tmp_path):
    import torch
    assert torch.cuda.is_available()
    import paper_1004_2772_amd as m
    yield m
    m.tune_clear()


def tuned_table(lhs, tmp_path, ls, log2, W):
    """A table whose entry names `ls`-slot lines and one lane."""
    entry = {"kind": "table", "W": W, "log2_capacity": log2, "line_slots": ls, "probe": "double",
             "tps_find_or_put": 1, "tps_expand": 1}
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({"format": "lhs-tune-1", "device": "gfx950", "entries": [entry]}))
    assert lhs.tune_load(str(path)) == 1
    t = lhs.Table(1 << log2, W)
    assert t.config()["line_slots"] == ls and t.config()["tps_find_or_put"] == 1
    return t


@pytest.mark.parametrize("ls", [8, 16])
@pytest.mark.parametrize("W", [1, 9, 32])
def test_both_sides_of_the_rule_on_one_table(lhs, tmp_path, W, ls):
    """Calls around the line between eight lanes and one, in turn on one table
    that ends nearly full: what one kernel stores the other finds."""
    import torch
    line = torch.cuda.get_device_properties(0).multi_processor_count * 256
    sizes = [line, line + 1, 65, line - 1, line + 257, 1]
    print(f"\n[fop] tuned lanes W={W} ls={ls} sizes={sizes}", flush=True)
    log2 = 17
    n = sum(sizes)
    rows, order = gen.dup_stream(700 + W, (1 << log2) * 15 // 16, W, 3)
    stream = gen.gather(rows, order)[:n]
    assert len(stream) == n
    o_seen, o_id, distinct = oracle.stream(stream)
    dev = dev_u32(stream)
    seen = torch.empty(n, dtype=torch.uint8, device="cuda")
    idx = torch.empty(n, dtype=torch.int32, device="cuda")
    with tuned_table(lhs, tmp_path, ls, log2, W) as t:
        bounds, at = [], 0
        for k in sizes:
            t.find_or_put(dev[at:at + k], seen[at:at + k], idx[at:at + k])
            bounds.append((at, at + k))
            at += k
        t.check()
        check_stream_batches(o_id, distinct, seen.cpu().numpy(), idx.cpu().numpy().view(np.uint32), bounds)
        assert t.count() == distinct
        check_table_invariants(t, sample=5000)


class Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class KernelNodeParams(ctypes.Structure):
    _fields_ = [("block", Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", Dim3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def captured_grid(t, states, seen):
    """Workgroups of the one kernel that a call launches (captured, not run)."""
    import torch
    hip = ctypes.CDLL("libamdhip64.so")
    stream = torch.cuda.Stream()
    handle, graph, n, node = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t(1), ctypes.c_void_p()
    params = KernelNodeParams()
    assert hip.hipStreamBeginCapture(handle, 1) == 0      # thread-local mode
    t.find_or_put(states, seen, stream=stream)
    assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0 and n.value == 1
    assert hip.hipGraphGetNodes(graph, ctypes.byref(node), ctypes.byref(n)) == 0
    assert hip.hipGraphKernelNodeGetParams(node, ctypes.byref(params)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return params.grid.x


def test_the_rule_by_call_size(lhs, tmp_path):
    """A launch of eight lanes has a workgroup per 32 operations, one of a
    single lane a workgroup per 256; lanes that the caller chose stay."""
    import torch
    line = torch.cuda.get_device_properties(0).multi_processor_count * 256
    states = torch.zeros((line + 1, 4), dtype=torch.int32, device="cuda")
    seen = torch.empty(line + 1, dtype=torch.uint8, device="cuda")
    with tuned_table(lhs, tmp_path, 8, 17, 4) as t:
        assert [captured_grid(t, states[:n], seen) for n in (64, line, line + 1)] == [2, line // 32, line // 256 + 1]
        t.set_threads_per_state(1)
        assert [captured_grid(t, states[:n], seen) for n in (64, line)] == [1, line // 256]
    with lhs.Table(1 << 17, 4, lhs.config(8, "double", 1, 1)) as t:
        assert captured_grid(t, states[:64], seen) == 1
