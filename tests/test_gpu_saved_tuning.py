"""Choices of the autotuner's file are launched as they were recorded: the kernel's node format and workgroup
are read from a trace of the call, and the tuning reported is the one that runs."""
import json

import numpy as np
import pytest

import paper_2507_23700_amd as ax

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 30_000
SIZE = f"logn={N.bit_length() - 1} logm={N.bit_length() - 1}"


def line(key, defaults=None, **kw):
    t = dict(block=64, order=1, stack=8, schedule=0, seed=0, nodes=0, packet=0)
    t.update(kw)
    if defaults is not None:
        t["defaults"] = defaults
    return '{"key": "' + key + '", ' + ", ".join(f'"{k}": {v}' for k, v in t.items()) + ', "ms": 0.1}\n'


def launched(call, kernel, tmp_path):
    """(template arguments, workgroup) of the one launch of `kernel` in call()."""
    call()
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    out = str(tmp_path / "trace.json")
    p.export_chrome_trace(out)
    found = [e for e in json.load(open(out))["traceEvents"] if kernel + "<" in e.get("name", "") and "block" in e.get("args", {})]
    assert len(found) == 1, [e.get("name") for e in found]
    args = found[0]["name"].split(kernel + "<")[1].split(">")[0].split(", ")
    return args, found[0]["args"]["block"][0]


@pytest.fixture(autouse=True)
def _tuning_file(tmp_path, monkeypatch):
    monkeypatch.setenv("ARBORX_TUNING_CACHE", str(tmp_path / "tuning.jsonl"))
    yield
    ax.arborx_reset_tuning()


def points(dim, n=N):
    g = torch.Generator(device="cuda")
    g.manual_seed(dim)
    return torch.rand((n, dim), generator=g, device="cuda")


@pytest.mark.parametrize("old", [True, False])
@pytest.mark.parametrize("block,nodes", [(64, 0), (128, 0), (64, 1), (256, 1)])
def test_nearest_choice_runs_as_recorded(old, block, nodes, tmp_path):
    key = f"op=2 dim=3 kind=0 k=16 {SIZE}"
    (tmp_path / "tuning.jsonl").write_text(line(key, None if old else 0, block=block, nodes=nodes))
    v = points(3)
    t = ax.arborx_bvh_build(v)
    best, ms = ax.arborx_autotune(t, ax.OP_KNN, v, k=16)
    assert ms == -1.0 and best == ax.arborx_get_tuning_op(ax.OP_KNN)
    assert (best["block"], best["stack"], best["node_format"]) == (block, 8, nodes)
    args, group = launched(lambda: ax.arborx_query_knn(t, v, 16), "k_knn", tmp_path)
    assert args == ["3", "16", "false", str(nodes)] and group == block


def test_recorded_defaults_are_the_defaults(tmp_path):
    v = points(3)
    t = ax.arborx_bvh_build(v)
    base = ax.arborx_get_tuning_op(ax.OP_KNN)
    assert (base["block"], base["node_format"]) == (256, 1)  # what the defaults run over points
    plain = launched(lambda: ax.arborx_query_knn(t, v, 16), "k_knn", tmp_path)
    (tmp_path / "tuning.jsonl").write_text(line(f"op=2 dim=3 kind=0 k=16 {SIZE}", 1, block=256, nodes=1))
    best, ms = ax.arborx_autotune(t, ax.OP_KNN, v, k=16)
    assert ms == -1.0 and best == base
    assert launched(lambda: ax.arborx_query_knn(t, v, 16), "k_knn", tmp_path) == plain


def test_6d_lines_without_the_word_keep_their_walk(tmp_path):
    """They recorded the defaults' raw fields and ran 64 threads, 16 entries, format 1."""
    (tmp_path / "tuning.jsonl").write_text(line(f"op=2 dim=6 kind=0 k=8 {SIZE}"))
    v = points(6)
    t = ax.arborx_bvh_build(v)
    best, ms = ax.arborx_autotune(t, ax.OP_KNN, v, k=8)
    assert ms == -1.0 and (best["block"], best["stack"], best["node_format"]) == (64, 16, 1)
    args, group = launched(lambda: ax.arborx_query_knn(t, v, 8), "k_knn", tmp_path)
    assert args == ["6", "8", "false", "1"] and group == 64


@pytest.mark.parametrize("nodes,held,runs", [(0, True, 0), (1, True, 1), (2, False, 0), (1, False, 0)])
def test_forest_choice_runs_as_recorded_on_what_the_forest_holds(nodes, held, runs, tmp_path):
    (tmp_path / "tuning.jsonl").write_text(line(f"forest op=2 dim=3 kind=0 k=8 {SIZE}", 0, nodes=nodes))
    v = points(3)
    if not held:
        ax.arborx_set_tuning(node_format=0)
    fo = ax.arborx_forest_build(v, [0, N // 2, N])
    ax.arborx_reset_tuning()
    bo, bt = torch.tensor([0, N // 2, N], device="cuda"), torch.tensor([0, 1], dtype=torch.int32, device="cuda")
    best, ms = ax.arborx_autotune_forest(fo, ax.OP_KNN, v, bo, bt, None, k=8)
    assert ms == -1.0 and best["node_format"] == runs
    args, group = launched(lambda: ax.arborx_forest_query_knn(fo, v, bo, bt, 8), "k_forest_knn", tmp_path)
    assert args == ["3", "8", str(runs)] and group == 64


@pytest.mark.parametrize("dim", [3, 6])
def test_a_choice_made_here_is_the_one_loaded(dim, tmp_path):
    v = points(dim)
    t = ax.arborx_bvh_build(v)
    best, ms = ax.arborx_autotune(t, ax.OP_KNN, v, k=8)
    here = launched(lambda: ax.arborx_query_knn(t, v, 8), "k_knn", tmp_path)
    ax.arborx_reset_tuning()
    again, ms = ax.arborx_autotune(t, ax.OP_KNN, v, k=8)
    assert ms == -1.0 and again == best
    if best["schedule"] == 0:
        assert launched(lambda: ax.arborx_query_knn(t, v, 8), "k_knn", tmp_path) == here
