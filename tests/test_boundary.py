"""Host-side checks of the C ABI that need no GPU: the library loads, exports every
symbol the header declares, and rejects bad arguments with error codes."""
import ctypes as C
import os
import re

import pytest

from paper_2503_01330_amd import binding as wkv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_declared_symbol_is_exported():
    header = open(os.path.join(ROOT, "include", "wkv.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(wkv_[a-z_]+)\s*\(", header))
    assert declared == set(wkv.EXPORTS)
    lib = C.CDLL(wkv.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name
    assert wkv.wkv_version() >= 100


def test_header_constants_match_binding():
    header = open(os.path.join(ROOT, "include", "wkv.h")).read()
    for name, val in re.findall(r"#define\s+(WKV_[A-Z0-9_]+)\s+(-?\d+)", header):
        assert getattr(wkv, name) == int(val), name


def test_options_struct_layout():
    assert C.sizeof(wkv.wkv_options) == 16 * 4


@pytest.mark.parametrize("kw,code", [
    (dict(batch=0), wkv.WKV_EINVAL), (dict(heads=-1), wkv.WKV_EINVAL),
    (dict(head_dim=96), wkv.WKV_EINVAL), (dict(head_dim=256, dtype=wkv.WKV_FP32), wkv.WKV_EINVAL),
    (dict(dtype=7), wkv.WKV_EINVAL), (dict(budget=0), wkv.WKV_EINVAL),
    (dict(budget=wkv.WKV_MAX_BUDGET + 1), wkv.WKV_ESIZE),
    (dict(recent_window=0), wkv.WKV_EINVAL), (dict(recent_window=65), wkv.WKV_EINVAL),
    (dict(n_sink=-1), wkv.WKV_EINVAL), (dict(n_sink=60, recent_window=16), wkv.WKV_EINVAL),
    (dict(score_mode=3), wkv.WKV_EINVAL), (dict(merge_mode=2), wkv.WKV_EINVAL),
    (dict(score_mode=1, merge_mode=0), wkv.WKV_EINVAL), (dict(threads=128), wkv.WKV_EINVAL),
    (dict(log_capacity=-5), wkv.WKV_EINVAL), (dict(split=3), wkv.WKV_EINVAL), (dict(split=32), wkv.WKV_EINVAL),
    (dict(split=-1), wkv.WKV_EINVAL), (dict(streaming=3), wkv.WKV_EINVAL), (dict(streaming=-1), wkv.WKV_EINVAL),
])
def test_invalid_options_are_rejected_before_touching_the_gpu(kw, code):
    base = dict(batch=1, heads=4, head_dim=64, budget=64, recent_window=16, dtype=wkv.WKV_FP32)
    base.update(kw)
    opt = wkv.make_options(**base)
    assert wkv.wkv_workspace_bytes(opt) == 0
    with pytest.raises(wkv.WkvError) as e:
        wkv.wkv_create_ex(opt)
    assert e.value.code == code and wkv.wkv_last_error()


def test_null_arguments():
    lib = C.CDLL(wkv.LIB_PATH)
    assert lib.wkv_create_ex(None, None) == wkv.WKV_EINVAL
    assert lib.wkv_step(None, None, None, None, None, None) == wkv.WKV_EINVAL
    assert lib.wkv_state(None, 0, None, 0) == wkv.WKV_EINVAL
    assert lib.wkv_destroy(None) == wkv.WKV_OK


def test_size_arithmetic():
    # Llama-2-7B-shaped layer, batch 8, budget 410 (the stacked configuration)
    opt = wkv.make_options(8, 32, 128, 410, 32, wkv.WKV_FP16)
    units, L, row = 256, 411, 256
    assert wkv.wkv_step_bytes(opt) == units * (L * (2 * row + 20) + 7 * row)
    kv = 2 * units * L * row
    assert kv < wkv.wkv_workspace_bytes(opt) < kv * 1.1 + (1 << 22)


def test_workgroups_per_unit_are_chosen_by_shape():
    """Host-only: the scratch of the sliced kernel shows in the workspace size.  One sequence
    of a 32-head model with 819 slots is cut into 4 slices per unit by default; 256 units are
    not cut; short score rows are not cut; an explicit request wins."""
    def ws(batch, heads, m, **kw):
        return wkv.wkv_workspace_bytes(wkv.make_options(batch, heads, 128, m, 32, wkv.WKV_FP16, **kw))
    def scratch(units, m, S):     # exponentials per slot + S partial rows (8-byte cells) + 3 values per slice + counter
        return units * ((m + 1) * 8 + S * 128 * 8 + 3 * S * 8 + 4)
    assert ws(1, 32, 819) == ws(1, 32, 819, split=1) + scratch(32, 819, 4)
    assert ws(1, 32, 819, split=16) == ws(1, 32, 819, split=1) + scratch(32, 819, 16)
    assert ws(8, 32, 410) == ws(8, 32, 410, split=1)
    assert ws(1, 32, 256) == ws(1, 32, 256, split=1)
    assert ws(4, 32, 2048) == ws(4, 32, 2048, split=1) + scratch(128, 2048, 2)


def test_launch_shape_follows_the_unit_count():
    """Host-only: the grid wkv_step would launch.  256 units: one workgroup of 1024 threads each;
    one sequence of a 32-head model with 819 slots: 4 slices per unit in 512-thread workgroups;
    2048 units: 512 threads, one workgroup per unit; explicit requests win; bad options are refused."""
    def shape(batch, heads, m, **kw):
        return wkv.wkv_launch_shape(wkv.make_options(batch, heads, 128, m, 32, wkv.WKV_FP16, **kw))
    assert shape(8, 32, 410) == (256, 1024)
    assert shape(1, 32, 819) == (128, 512)
    assert shape(4, 32, 2048) == (256, 1024)
    assert shape(64, 32, 512) == (2048, 512)
    assert shape(8, 32, 410, threads=512, split=2) == (512, 512)
    with pytest.raises(wkv.WkvError):
        shape(8, 32, 410, threads=300)


def test_launches_stay_below_the_threads_a_grid_holds():
    """Host-only: a grid of 2^32 threads and more wraps without an error.  The default takes smaller workgroups there; what does not fit is refused."""
    def shape(units, d=128, **kw):
        return wkv.wkv_launch_shape(wkv.make_options(1, units, d, 2, 1, wkv.WKV_FP16, **kw))
    assert shape((1 << 23) - 1) == ((1 << 23) - 1, 512) and shape(1 << 23) == (1 << 23, 256)
    assert shape((1 << 24) - 1, d=64) == ((1 << 24) - 1, 256)
    assert shape(1 << 18, split=16)[0] == 1 << 22
    for units, kw in ((1 << 24, {}), (1 << 23, dict(threads=512)), (1 << 22, dict(threads=1024)), (1 << 20, dict(threads=256, split=16))):
        with pytest.raises(wkv.WkvError) as e:
            shape(units, **kw)
        assert e.value.code == wkv.WKV_ESIZE
    assert wkv._lib.wkv_probe_read(1 << 20, 16 << 22, 1 << 22, 1024, 0, None, None) == wkv.WKV_ESIZE


def test_kernels_of_a_prompt_need_no_stack():
    """Host-only: the runtime gives every queue stack memory for the whole chip when a kernel first wants some, hundreds of megabytes of device memory that
    wkv_prefill_noalloc promises not to take and wkv_workspace_bytes does not count.  The library's kernel descriptions say how much a lane wants."""
    data = open(wkv.LIB_PATH, "rb").read()
    found = {}
    for key in re.finditer(rb"\.private_segment_fixed_size([\x00-\x7f]|\xcc.|\xcd..|\xce....)", data, re.S):
        name = data[data.rindex(b".name", 0, key.start()):key.start()]                 # (keys of a kernel's description are sorted)
        value = key.group(1) if len(key.group(1)) == 1 else key.group(1)[1:]
        found[re.search(rb"\w*wkv_\w+", name).group().decode()] = int.from_bytes(value, "big")
    prompt = {n: v for n, v in found.items() if "wkv_prefill_" in n}
    assert len(prompt) > 20 and len(found) > len(prompt), "no descriptions found: has their format changed?"
    assert {n: v for n, v in prompt.items() if v} == {}


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures exactly one GPU: a larger --gpus exits with a message before anything is imported."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode == 2 and "one GPU" in r.stderr and r.stdout.strip() == ""


def test_launch_shape_follows_the_budget_of_few_units():
    """Host-only: up to 256 units, 512 threads while the budget is small, 1024 beyond; many units and slices are not affected."""
    def shape(units, m, **kw):
        return wkv.wkv_launch_shape(wkv.make_options(1, units, 64, m, 8, wkv.WKV_BF16, **kw))
    assert shape(60, 224) == (60, 512) and shape(60, 225) == (60, 1024)
    assert shape(256, 224) == (256, 512) and shape(257, 225) == (257, 512)
    assert shape(1024, 64) == (1024, 256)
    assert shape(60, 64, threads=1024) == (60, 1024)
