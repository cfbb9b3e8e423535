"""What the host side of the library launches, with the launches recorded instead of made
(host_launches.cpp): every visible key is in some launched split, and the route a call takes.
No test here computes anything on a GPU."""
import ctypes
import os
import re
import subprocess
import sys

import numpy as np
import pytest

from paper_2501_05408_amd import tempo as T

from test_gpu_prompt_shapes import FEW_GROUPS, ROPE_BY_BLOCKS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOMEWHERE = 1 << 20                       # pointers that are checked for NULL and alignment, never read


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return load(str(tmp_path_factory.mktemp("host") / "host_launches.so"))


def load(path, *flags, build=True):
    if build:
        compile_host(path, *flags)
    lib = ctypes.CDLL(path)
    for name, (res, args) in T.SIGNATURES.items():
        fn = getattr(lib, name)
        fn.restype, fn.argtypes = res, args
    lib.host_launches_take.restype = ctypes.c_char_p
    return lib


def compile_host(path, *flags):
    subprocess.check_call(
        ["g++", "-std=c++17", "-O1", "-w", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__", "-x", "c++",
         os.path.join(ROOT, "tests", "host_launches.cpp"), "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
         "-I", os.path.join(ROOT, "paper_2501_05408_amd", "csrc"), "-o", path, *flags])


def store(dtype, Hkv, D, Z, columns, ring=0):
    return T.make_kv(SOMEWHERE, SOMEWHERE, SOMEWHERE, 1 << 20, columns, Z, Hkv, D, dtype, ring)


def taken(lib):
    """The launches since the last call: (name, {field: number})."""
    out = []
    for line in lib.host_launches_take().decode().splitlines():
        name, *fields = line.split()
        out.append((name, {k: int(v) for k, v in (f.split("=") for f in fields)}))
    return out


def prefill(lib, kv, batch, Hq, t, count, window=0, workspace=1 << 50, rows=SOMEWHERE, out=SOMEWHERE):
    lib.host_launches_take()
    args = (ctypes.byref(kv), SOMEWHERE, rows, rows, out, batch, Hq, t, count, None)
    if window:
        rc = lib.tempo_prefill_window(*args, window, 0.125, SOMEWHERE, workspace, None)
    else:
        rc = lib.tempo_prefill_causal(*args, 0.125, SOMEWHERE, workspace, None)
    assert rc == T.TEMPO_OK
    return taken(lib)


def assert_all_keys_launched(launches, G, t, count):
    """Every step of the call is answered once, and the splits that are launched for the steps that
    share a workgroup reach from the first key of the first of them to the last step."""
    step = t
    for name, f in launches:
        if name not in ("prompt", "prompt_staged", "short_prompt", "block_bf16", "partial_bf16", "partial_f32", "step_f32"):
            continue
        assert f["t"] == step
        # the (step, head) columns that share a workgroup: a block may begin and end between the heads of a step
        columns = {"prompt": 32 * f["waves"], "prompt_staged": 32 * f["waves"], "short_prompt": 128}.get(name, f["queries"] * G)
        for k in range(0, f["queries"] * G, columns):
            lo, last = step + k // G, step + (min(k + columns, f["queries"] * G) - 1) // G
            first = max(0, lo - f["window"] + 1) if f["window"] else 0
            assert (last >> f["tps_log2"]) - (first >> f["tps_log2"]) + 1 <= f["grid_splits"], (name, f, first, last)
        step += f["queries"]
    assert step == t + count


@pytest.mark.parametrize("dtype,window,count", [(T.TEMPO_BF16, 40, 30), (T.TEMPO_BF16, 200, 1000), (T.TEMPO_F32, 40, 30),
                                                (T.TEMPO_F32, 200, 1000)])
@pytest.mark.parametrize("batch", [1, 64])
def test_prompts_whose_range_crosses_two_to_the_thirty(lib, dtype, window, count, batch):
    G, Z = 3, 32
    ring = T.tempo_ring_blocks(window, Z, min(count, 128 // G))
    t = (1 << 30) - 20
    launches = prefill(lib, store(dtype, 2, 128, Z, ring, ring), batch, 2 * G, t, count, window)
    assert_all_keys_launched(launches, G, t, count)


@pytest.mark.parametrize("Hq,Hkv,D,batch,t,ragged", [(24, 8, 128, 48, 8192, False), (32, 8, 128, 16, 17378, False),
                                                     (64, 1, 64, 16, 17378, True), (8, 2, 128, 64, 17378, False)])
def test_no_alloc_f32_step_takes_a_plan_that_fits_the_array(lib, Hq, Hkv, D, batch, t, ragged):
    kv = store(T.TEMPO_F32, Hkv, D, 64, t // 64 + 1)
    lib.host_launches_take()
    rc = lib.tempo_decode_step_causal_noalloc(ctypes.byref(kv), SOMEWHERE, SOMEWHERE, SOMEWHERE, SOMEWHERE, batch, Hq, t,
                                              SOMEWHERE if ragged else None, 0.125, None)
    assert rc == T.TEMPO_OK
    (name, f), *rest = taken(lib)
    assert name == "partial_f32" and f["num_splits"] * batch * Hq * (D + 2) * 4 <= 8 << 20
    assert f["grid_splits"] >= (t >> f["tps_log2"]) + 1
    assert [n for n, _ in rest] == (["combine"] if f["num_splits"] > 1 else [])


@pytest.mark.parametrize("G,Hkv,D,batch,t,ragged", [(17, 8, 64, 33, 16383, False), (33, 1, 64, 128, 40000, False),
                                                    (24, 4, 64, 17, 65535, False), (40, 8, 128, 20, 30000, True), (64, 8, 128, 3, 5000, False),
                                                    (100, 8, 128, 4, 30000, False), (70, 8, 64, 40, 700, False)])
def test_no_alloc_bf16_step_of_a_wide_group_takes_a_plan_that_fits_the_array(lib, G, Hkv, D, batch, t, ragged):
    """And the plan of the call with a workspace, if that one fits."""
    kv, plan, Hq = store(T.TEMPO_BF16, Hkv, D, 64, t // 64 + 1), T.tempo_plan(), G * Hkv
    lib.host_launches_take()
    rc = lib.tempo_decode_step_causal_noalloc(ctypes.byref(kv), SOMEWHERE, SOMEWHERE, SOMEWHERE, SOMEWHERE, batch, Hq, t,
                                              SOMEWHERE if ragged else None, 0.125, None)
    assert rc == T.TEMPO_OK
    _, (name, f), *rest = taken(lib)
    assert name == "block_bf16" and f["num_splits"] * batch * Hq * (D + 2) * 4 <= 8 << 20
    assert f["grid_splits"] >= (t >> f["tps_log2"]) + 1
    assert [n for n, _ in rest] == (["combine"] if f["num_splits"] > 1 else [])
    assert lib.tempo_attn_plan(ctypes.byref(kv), batch, Hq, t, 0, ragged, ctypes.byref(plan)) == T.TEMPO_OK
    fits = plan.num_splits * batch * Hq * (D + 2) * 4 <= 8 << 20
    assert (plan.num_splits == f["num_splits"]) == fits and fits == (batch == 3)


def test_no_alloc_bf16_step_that_does_not_fit_stays_refused(lib, capfd):
    kv = store(T.TEMPO_BF16, 8, 128, 256, 32)
    lib.host_launches_take()
    rc = lib.tempo_decode_step_causal_noalloc(ctypes.byref(kv), SOMEWHERE, SOMEWHERE, SOMEWHERE, SOMEWHERE, 64, 64, 8191,
                                              SOMEWHERE, 0.125, None)
    assert rc == T.TEMPO_ERR_WORKSPACE and not taken(lib)


@pytest.mark.parametrize("call", [
    "assert_all_keys_launched(prefill(lib, store(T.TEMPO_F32, 2, 64, 64, 100), 1, 8, 37, 300, (1 << 31) - 129), 4, 37, 300)",
    "assert_all_keys_launched(prefill(lib, store(T.TEMPO_BF16, 8, 128, 64, 100), 1, 8, 37, 3000, (1 << 31) - 129), 1, 37, 3000)",
    "lib.tempo_attn_block_plan(ctypes.byref(store(T.TEMPO_BF16, 8, 128, 64, 100)), 1, 8, 128, 37, (1 << 31) - 65, 0, "
    "ctypes.byref(T.tempo_plan()))"])
def test_windows_near_the_largest_integer_do_not_overflow(tmp_path, call):
    """In a process of its own: signed overflow ends it."""
    path = str(tmp_path / "checked.so")
    load(path, "-fsanitize=signed-integer-overflow", "-fno-sanitize-recover=all", "-static-libubsan")
    code = ("import ctypes, test_host_launches as H\nfrom test_host_launches import T, prefill, store, assert_all_keys_launched\n"
            f"lib = H.load({path!r}, build=False)\n{call}")
    run = subprocess.run([sys.executable, "-c", code], cwd=os.path.join(ROOT, "tests"),
                         env={**os.environ, "PYTHONPATH": ROOT}, capture_output=True, text=True)
    assert run.returncode == 0, run.stderr


@pytest.mark.parametrize("Hq,Hkv,D,batch,keys,kernel", [
    (24, 8, 128, 1, 192, "step_f32"), (24, 8, 128, 1, 193, "partial_f32"), (24, 8, 128, 16, 66, "step_f32"),
    (24, 8, 128, 16, 67, "partial_f32"), (8, 2, 64, 1, 24, "step_f32"), (8, 2, 64, 1, 25, "partial_f32"),
    (8, 8, 128, 16, 5000, "step_f32"), (16, 1, 128, 16, 192, "step_f32"), (8, 8, 64, 16, 5000, "partial_f32")])
@pytest.mark.parametrize("windowed", [False, True])
def test_kernel_of_an_f32_step(lib, Hq, Hkv, D, batch, keys, kernel, windowed):
    t = 20000 if windowed else keys - 1
    kv = store(T.TEMPO_F32, Hkv, D, 64, t // 64 + 1)
    lib.host_launches_take()
    rc = lib.tempo_attn_decode_window(ctypes.byref(kv), SOMEWHERE, SOMEWHERE, batch, Hq, t, None, keys, 0.125, SOMEWHERE,
                                      1 << 50, None)
    assert rc == T.TEMPO_OK
    (name, f), *_ = taken(lib)
    lo = t - keys + 1
    assert name == kernel and f["grid_splits"] >= (t >> f["tps_log2"]) - (lo >> f["tps_log2"]) + 1
    assert f["waves"] in (1, 2, 4, 8)


@pytest.mark.parametrize("Hq,Hkv,D,t,count,window,kernel", [
    (24, 8, 128, 0, 128, 0, "short_prompt"), (24, 8, 128, 0, 129, 0, "prompt"), (24, 8, 128, 86, 42, 0, "short_prompt"),
    (24, 8, 128, 500, 900, 87, "short_prompt"), (24, 8, 128, 500, 300, 87, "prompt"), (24, 8, 128, 500, 900, 88, "prompt"), (24, 8, 128, 0, 21, 0, "prompt"),
    (24, 8, 128, 0, 22, 0, "short_prompt"), (8, 2, 64, 0, 100, 0, "prompt"), (256, 2, 128, 0, 5, 0, "short_prompt")])
def test_kernel_of_a_bf16_prompt_over_a_short_range(lib, Hq, Hkv, D, t, count, window, kernel):
    launches = prefill(lib, store(T.TEMPO_BF16, Hkv, D, 64, 100), 2, Hq, t, count, window)
    assert [n for n, _ in launches][:2] == ["append", kernel]
    assert_all_keys_launched(launches, Hq // Hkv, t, count)


@pytest.mark.parametrize("dtype,Hq,Hkv,D,batch,t,count,window,blocks", [
    (T.TEMPO_BF16, 24, 8, 128, 1, 8000, 1, 0, 1), (T.TEMPO_BF16, 24, 8, 128, 16, 300, 5, 0, 1),    # the single-step kernel's
    (T.TEMPO_BF16, 24, 8, 128, 1, 32000, 21, 0, 1), (T.TEMPO_BF16, 24, 8, 128, 1, 2000, 21, 0, 0),  # long and short histories
    (T.TEMPO_BF16, 8, 1, 128, 1, 32000, 42, 0, 3), (T.TEMPO_BF16, 8, 2, 64, 1, 30000, 40, 0, 2),
    (T.TEMPO_BF16, 8, 1, 128, 1, 1000, 2, 0, 0), (T.TEMPO_BF16, 24, 8, 128, 64, 8000, 3, 0, 0),     # fills the part
    (T.TEMPO_BF16, 24, 8, 128, 1, 3000, 5, 64, 1), (T.TEMPO_BF16, 24, 8, 128, 4, 30000, 42, 64, 0),
    (T.TEMPO_F32, 24, 8, 128, 1, 2000, 16, 0, 1), (T.TEMPO_F32, 24, 8, 128, 1, 2000, 64, 0, 0)])
def test_prompts_behind_long_histories_go_block_by_block(lib, dtype, Hq, Hkv, D, batch, t, count, window, blocks):
    for ring in (False, True) if window else (False,):
        check_route(lib, dtype, Hq, Hkv, D, batch, t, count, window, blocks, ring)


def check_route(lib, dtype, Hq, Hkv, D, batch, t, count, window, blocks, ring):
    G, Z = Hq // Hkv, 64
    R = T.tempo_ring_blocks(window, Z, min(count, 128 // G)) if ring else 0
    launches = prefill(lib, store(dtype, Hkv, D, Z, R or (t + count) // Z + 1, R), batch, Hq, t, count, window)
    assert_all_keys_launched(launches, G, t, count)
    names = [n for n, _ in launches]
    answers = [f for n, f in launches if n in ("partial_bf16", "block_bf16", "partial_f32", "step_f32") and f["queries"] <= 128 // G]
    if blocks:
        assert len(answers) == blocks and names.count("append") == blocks
        assert [(f["t"], f["queries"]) for f in answers] == [(t + c, min(128 // G, count - c)) for c in range(0, count, 128 // G)]
    else:
        assert names[1] in ("prompt", "prompt_staged", "short_prompt", "partial_f32")
    bound = lib.tempo_prefill_launches(ctypes.byref(store(dtype, Hkv, D, Z, R or (t + count) // Z + 1, R)), batch, Hq, count)
    assert len(launches) <= bound


@pytest.mark.parametrize("Hq, Hkv, D, batch, t, count, window, split", [
    (24, 8, 128, 4, 3000, 21, 512, True), (24, 8, 128, 2, 4000, 42, 512, True), (32, 8, 64, 2, 3000, 21, 512, True),
    (8, 2, 64, 1, 1000, 64, 512, True), (1, 1, 128, 1, 4000, 42, 300, True), (24, 8, 128, 4, 3000, 21, 64, False)])
def test_key_ranges_of_windowed_prompts_are_split_where_that_is_faster(lib, Hq, Hkv, D, batch, t, count, window, split):
    for ring in (0, T.tempo_ring_blocks(window, 64, count)):
        launches = prefill(lib, store(T.TEMPO_BF16, Hkv, D, 64, ring or (t + count) // 64 + 1, ring), batch, Hq, t, count, window)
        assert_all_keys_launched(launches, Hq // Hkv, t, count)
        assert [n for n, _ in launches] == ["append", "prompt"] + (["prompt_combine"] if split else [])
        assert (launches[1][1]["grid_splits"] > 1) == split


def least_prompt_workspace(lib, kv, batch, Hq, t, count, window):
    """What the blocks of 128 columns need, and no byte more: the least a prompt is accepted with."""
    block, need = 128 // (Hq // kv.num_kv_heads), 0
    for c in range(0, count, block):
        n, plan = min(block, count - c), T.tempo_plan()
        assert lib.tempo_attn_block_plan(ctypes.byref(kv), batch, Hq, n, t + c, window, 0, ctypes.byref(plan)) == T.TEMPO_OK
        need = max(need, lib.tempo_attn_plan_workspace_bytes(ctypes.byref(kv), batch * n, Hq, ctypes.byref(plan)))
    return need


# (B, Hkv, G, D, Z, t, count, window) whose least workspace has no room to stage more than a chunk, and ...
CHUNKED = [(16, 32, 1, 64, 256, 0, 700, 100), (16, 32, 1, 64, 256, 77, 500, 100), (8, 64, 2, 64, 64, 13, 330, 40),
           (64, 8, 3, 128, 256, 0, 1100, 300)]
# ... some that has
STAGED = [(2, 2, 3, 128, 32, 0, 700, 100), (1, 4, 4, 64, 64, 0, 333, 33), (3, 1, 8, 128, 32, 77, 400, 64)]


@pytest.mark.parametrize("shape", CHUNKED + STAGED)
def test_ring_prompts_with_the_least_workspace(lib, shape):
    B, Hkv, G, D, Z, t, count, window = shape
    ring = T.tempo_ring_blocks(window, Z, min(count, 128 // G))
    kv = store(T.TEMPO_BF16, Hkv, D, Z, ring, ring)
    need = least_prompt_workspace(lib, kv, B, Hkv * G, t, count, window)
    # (rows that are not 16-byte aligned: else a prompt from step 0 on would be answered from them)
    launches = prefill(lib, kv, B, Hkv * G, t, count, window, need, rows=SOMEWHERE + 8, out=1 << 45)
    assert_all_keys_launched(launches, G, t, count)
    names = [n for n, _ in launches]
    if shape in STAGED:
        assert names.count("stage") >= 1 and "prompt_staged" in names
    else:
        assert "stage" not in names and names.count("append") >= 3
        at = t
        for (name, f), (_, answer) in zip(launches[::2], launches[1::2]):   # written, then answered, chunk by chunk
            assert name == "append" and (f["t"], f["count"]) == (answer["t"], answer["queries"]) == (at, f["count"])
            at += f["count"]
            # all that the chunk's steps see is still in the ring when it has been written
            oldest = max(0, f["t"] - window + 1)
            assert (at - 1) // Z - oldest // Z < ring
    assert lib.tempo_prefill_window(ctypes.byref(kv), SOMEWHERE, SOMEWHERE, SOMEWHERE, SOMEWHERE, B, Hkv * G, t, count, None,
                                    window, 0.125, SOMEWHERE, need - 256, None) == T.TEMPO_ERR_WORKSPACE


@pytest.mark.parametrize("Hq,Hkv,D,batch,t,count,window", [
    (24, 8, 128, 1, 1500, 100, 0), (24, 8, 128, 2, 4000, 42, 512), (5, 1, 64, 1, 2900, 70, 300), (40, 1, 64, 1, 1023, 11, 900)])
def test_splits_reach_over_blocks_that_begin_between_the_heads_of_a_step(lib, Hq, Hkv, D, batch, t, count, window):
    """A block is a run of (step, head) columns: all splits of the steps it touches are launched."""
    G = Hq // Hkv
    launches = prefill(lib, store(T.TEMPO_BF16, Hkv, D, 64, 100), batch, Hq, t, count, window)
    (_, f), = [l for l in launches if l[0] == "prompt"]
    assert f["grid_splits"] > 1
    assert_all_keys_launched(launches, G, t, count)


@pytest.mark.parametrize("what,Hq,Hkv,D,batch,t,count,window,ring,apart,names", [
    ("one launch", 24, 8, 128, 16, 0, 300, 0, False, 1 << 32, ["prompt"]),
    ("few columns behind few keys", 24, 8, 128, 1, 0, 3, 0, False, 1 << 32, ["prompt"]),
    ("split ranges", 8, 1, 128, 1, 0, 1000, 0, False, 1 << 32, ["prompt", "prompt_combine"]),
    ("a ring that does not hold the prompt", 24, 8, 128, 4, 0, 2048, 512, True, 1 << 32, ["prompt"]),
    ("a history", 24, 8, 128, 16, 1, 300, 0, False, 1 << 32, ["append", "prompt"]),
    ("long and causal", 24, 8, 128, 16, 0, 1300, 0, False, 1 << 32, ["append", "prompt"]),
    ("long and windowed", 24, 8, 128, 16, 0, 1300, 500, False, 1 << 32, ["prompt"]),
    ("out over the rows", 24, 8, 128, 16, 0, 300, 0, False, 16 * 300 * 24 * 128 * 2 - 16, ["append", "prompt"]),
    ("out right before the rows", 24, 8, 128, 16, 0, 300, 0, False, 16 * 300 * 24 * 128 * 2, ["prompt"]),
    ("rows not aligned", 24, 8, 128, 16, 0, 300, 0, False, (1 << 32) + 8, ["append", "prompt"]),
    ("fp32", 8, 2, 64, 1, 0, 512, 0, False, 1 << 32, ["partial_f32"]),
    ("fp32, one block", 8, 2, 64, 1, 0, 32, 0, False, 1 << 32, ["partial_f32"]),
    ("fp32, one block, few keys", 8, 2, 64, 1, 0, 5, 0, False, 1 << 32, ["step_f32"]),
    ("fp32, a ring that does not hold the prompt", 8, 2, 64, 4, 0, 2048, 512, True, 1 << 32, ["partial_f32"]),
    ("fp32, long at D = 128", 24, 8, 128, 4, 0, 1000, 0, False, 1 << 32, ["append", "partial_f32"]),
    ("fp32, a history", 8, 2, 64, 1, 1, 512, 0, False, 1 << 32, ["append", "partial_f32"]),
    ("fp32, out over the rows", 8, 2, 64, 1, 0, 512, 0, False, 512 * 8 * 64 * 4 - 16, ["append", "partial_f32"])])
def test_prompts_that_are_read_from_the_callers_rows(lib, what, Hq, Hkv, D, batch, t, count, window, ring, apart, names):
    R = T.tempo_ring_blocks(window, 256, 128 * Hkv // Hq) if ring else 0
    kv = store(T.TEMPO_F32 if what.startswith("fp32") else T.TEMPO_BF16, Hkv, D, 256, R or 100, R)
    out, k, v = 1 << 33, (1 << 33) + apart, (1 << 33) + 3 * (apart & ~15)
    args = (ctypes.byref(kv), SOMEWHERE, k, v, out, batch, Hq, t, count, None)
    for workspace in (1 << 50, least_prompt_workspace(lib, kv, batch, Hq, t, count, window)):
        lib.host_launches_take()
        rc = (lib.tempo_prefill_window(*args, window, 0.125, SOMEWHERE, workspace, None) if window else
              lib.tempo_prefill_causal(*args, 0.125, SOMEWHERE, workspace, None))
        assert rc == T.TEMPO_OK
        launches = taken(lib)
        assert [n for n, _ in launches if n != "prompt_combine"] == [n for n in names if n != "prompt_combine"]
        if workspace == 1 << 50:
            assert [n for n, _ in launches] == names
        assert launches[0][1]["k"] == k and all(f["k"] == 0 for n, f in launches[1:] if n != "prompt_combine")
        assert_all_keys_launched(launches, Hq // Hkv, t, count)


def assert_rows_are_read_before_answers_stand_over_them(launches, base, size, Hq, Hkv, D, esz, batch):
    """Plays the launches on the bytes base .. base+size-1: no launch may read a row that answers were written over."""
    over = np.zeros(size, dtype=bool)

    def spans(at, n, steps, heads):                      # n steps of each sequence, `steps` apart
        for b in range(batch):
            lo = at - base + b * steps * heads * D * esz
            yield max(lo, 0), max(min(lo + n * heads * D * esz, size), 0)

    for name, f in launches:
        if name == "stream_copy":
            lo = f["from"] - base
            assert not over[max(lo, 0):max(lo + f["bytes"], 0)].any(), (name, f)
            continue
        n = f["count"] if "count" in f else f["queries"]
        for rows in (f["k"], f["v"]):
            for lo, hi in spans(rows, n, f["steps"], Hkv) if rows else ():
                assert not over[lo:hi].any(), (name, f)
        if f.get("direct") or "combine" in name:
            for lo, hi in spans(f["out"], n, f["steps"], Hq):
                over[lo:hi] = True
            for rows in (f["k"], f["v"]):                # ... nor write answers over rows that it reads itself
                for lo, hi in spans(rows, n, f["steps"], Hkv) if rows else ():
                    assert not over[lo:hi].any(), (name, f)


# (dtype, batch, Hkv, G, D, t, count, window, ring): prompts of one launch, of several blocks and of several chunks of a ring
OVERLAPS = [(T.TEMPO_BF16, 1, 1, 3, 64, 16000, 70, 0, False), (T.TEMPO_BF16, 2, 1, 3, 128, 30000, 90, 0, False),
            (T.TEMPO_BF16, 2, 2, 3, 128, 0, 90, 0, False), (T.TEMPO_F32, 2, 2, 3, 64, 0, 90, 0, False),
            (T.TEMPO_BF16, 1, 2, 3, 128, 0, 900, 100, True), (T.TEMPO_BF16, 2, 2, 1, 64, 0, 700, 100, True),
            (T.TEMPO_BF16, 2, 1, 3, 64, 77, 500, 64, True), (T.TEMPO_F32, 2, 2, 3, 64, 0, 400, 50, True),
            (T.TEMPO_F32, 2, 2, 1, 64, 100, 500, 50, True), (T.TEMPO_F32, 1, 2, 4, 64, 5, 60, 20, True),
            (T.TEMPO_F32, 1, 2, 16, 64, 5, 20, 20, True)]


@pytest.mark.parametrize("dtype,batch,Hkv,G,D,t,count,window,ring", OVERLAPS)
@pytest.mark.parametrize("where", ["k", "v", "k's second half", "k's end", "between"])
def test_out_over_the_rows(lib, dtype, batch, Hkv, G, D, t, count, window, ring, where):
    """With the workspace the library asks for, and with the least that is accepted."""
    esz, Z = 2 if dtype == T.TEMPO_BF16 else 4, 64
    row, base = batch * count * Hkv * D * esz, 1 << 33
    R = T.tempo_ring_blocks(window, Z, min(count, 128 // G)) if ring else 0
    kv = store(dtype, Hkv, D, Z, R or (t + count) // Z + 1, R)
    k = base + row * G
    v = k + row + 4096
    out = {"k": k, "v": v, "k's second half": k + row // 2 // 256 * 256, "k's end": k + row - D * esz * Hkv,
           "between": k - row // 3 // 256 * 256}[where]
    most = T.tempo_prefill_workspace_bytes(kv, batch, Hkv * G, t + count - 1)
    args = (ctypes.byref(kv), SOMEWHERE, k, v, out, batch, Hkv * G, t, count, None)
    taken_at = []
    for workspace in (most, least_prompt_workspace(lib, kv, batch, Hkv * G, t, count, window)):
        lib.host_launches_take()
        rc = (lib.tempo_prefill_window(*args, window, 0.125, SOMEWHERE, workspace, None) if window else
              lib.tempo_prefill_causal(*args, 0.125, SOMEWHERE, workspace, None))
        launches = taken(lib)
        taken_at.append([n for n, _ in launches])
        if rc != T.TEMPO_OK:                             # only without room for a copy, and before anything is launched
            assert rc == T.TEMPO_ERR_WORKSPACE and workspace < most and ring and not launches
            continue
        assert_all_keys_launched(launches, G, t, count)
        assert_rows_are_read_before_answers_stand_over_them(launches, base - row * G, row * (3 * G + 3) + 8192, Hkv * G, Hkv, D,
                                                            esz, batch)
        for name, f in launches:                         # a copy lies in the workspace, behind the partials
            if name == "stream_copy":
                assert SOMEWHERE + least_prompt_workspace(lib, kv, batch, Hkv * G, t, count, window) <= f["to"]
                assert f["to"] + f["bytes"] <= SOMEWHERE + workspace and f["bytes"] == row
    if t and not ring:                                   # several blocks: all written first, or each before its answers
        blocks, apart = -(-count // (128 // G)), prefill(lib, kv, batch, Hkv * G, t, count, window, rows=k, out=1 << 45)
        assert blocks > 1 and taken_at[0].count("append") == blocks and taken_at[0][:blocks] == ["append"] * blocks
        assert [n for n, _ in apart] == ["append", "block_bf16", "combine"] * blocks


@pytest.mark.parametrize("D,G,t,count", ROPE_BY_BLOCKS)
def test_rope_prompts_by_blocks_go_by_blocks(lib, D, G, t, count):
    """The shapes that test_gpu_prompt_shapes.py answers on the GPU, two kv heads of one sequence."""
    kv, rope = store(T.TEMPO_BF16, 2, D, 32, (t + count) // 32 + 1), T.tempo_rope(SOMEWHERE, SOMEWHERE, t + count, D)
    lib.host_launches_take()
    assert lib.tempo_rope_prefill_causal(ctypes.byref(kv), ctypes.byref(rope), SOMEWHERE, SOMEWHERE, SOMEWHERE, 1 << 45, 1, 2 * G,
                                         t, count, None, 0.125, SOMEWHERE, 1 << 50, None) == T.TEMPO_OK
    launches, blocks = taken(lib), -(-count // (128 // G))
    assert [n for n, _ in launches] == ["append", "block_bf16" if G * count > 16 else "partial_bf16", "combine"] * blocks
    assert_all_keys_launched(launches, G, t, count)


@pytest.mark.parametrize("Hq,Hkv,D,batch,t,queries,window,stream", [
    (24, 8, 128, 1, 26, 6, 0, 0), (24, 8, 128, 1, 27, 6, 0, 1), (32, 1, 128, 1, 5, 1, 0, 0), (24, 8, 128, 26, 58, 6, 0, 1),
    (33, 1, 128, 1, 191, 1, 0, 0), (33, 1, 128, 1, 192, 1, 0, 1), (33, 1, 128, 1, 5000, 1, 192, 0), (24, 8, 128, 16, 4075, 21, 0, 1),
    (64, 1, 128, 1, 500, 1, 0, 1), (65, 1, 128, 1, 60000, 1, 0, 0), (24, 8, 128, 16, 4075, 42, 0, 0), (64, 1, 64, 1, 176, 1, 0, 1),
    (64, 1, 64, 1, 175, 1, 0, 0), (65, 1, 64, 1, 65535, 1, 0, 0), (65, 1, 64, 1, 65536, 1, 0, 1), (65, 8, 64, 2, 4095, 16, 100, 0),
    (32, 8, 64, 13, 225, 31, 0, 0), (32, 8, 64, 13, 226, 31, 0, 1),
    # more pairs than compute units, and than fill the part twice and four times
    (24, 8, 128, 33, 218, 6, 0, 0), (24, 8, 128, 33, 219, 6, 0, 1), (24, 8, 128, 64, 250, 6, 0, 0), (24, 8, 128, 64, 251, 6, 0, 1),
    (24, 8, 128, 128, 334, 6, 0, 0), (24, 8, 128, 128, 335, 6, 0, 1), (24, 8, 128, 33, 235, 21, 0, 0), (24, 8, 128, 33, 236, 21, 0, 1),
    (24, 8, 128, 64, 1179, 21, 0, 0), (24, 8, 128, 64, 1180, 21, 0, 1), (24, 8, 128, 70, 1779, 21, 0, 0), (24, 8, 128, 70, 1780, 21, 0, 1),
    (24, 8, 128, 97, 619, 21, 0, 0), (24, 8, 128, 97, 620, 21, 0, 1), (32, 8, 64, 64, 24, 8, 0, 0), (32, 8, 64, 33, 25, 8, 0, 1),
    (32, 8, 64, 65, 184, 8, 0, 0), (32, 8, 64, 65, 185, 8, 0, 1), (32, 8, 64, 128, 264, 8, 0, 0), (32, 8, 64, 128, 265, 8, 0, 1),
    (32, 8, 64, 63, 240, 16, 0, 0), (32, 8, 64, 63, 241, 16, 0, 1), (32, 8, 64, 64, 624, 16, 0, 0), (32, 8, 64, 64, 625, 16, 0, 1),
    (32, 8, 64, 70, 884, 16, 0, 0), (32, 8, 64, 70, 885, 16, 0, 1), (32, 8, 64, 97, 1084, 16, 0, 0), (32, 8, 64, 49, 993, 31, 0, 0),
    (32, 8, 64, 50, 226, 31, 0, 1), (32, 8, 64, 64, 1269, 31, 0, 0), (32, 8, 64, 64, 1270, 31, 0, 1), (32, 8, 64, 70, 2017, 31, 0, 0),
    (32, 8, 64, 97, 1770, 31, 0, 1)])
def test_kernel_of_a_wide_block(lib, Hq, Hkv, D, batch, t, queries, window, stream):
    Hq = Hq // Hkv * Hkv
    kv = store(T.TEMPO_BF16, Hkv, D, 64, (t + queries) // 64 + 1)
    lib.host_launches_take()
    args = (ctypes.byref(kv), SOMEWHERE, 1 << 45, batch, Hq, queries, t, None)
    rc = (lib.tempo_attn_block_window(*args, window, 0.125, SOMEWHERE, 1 << 50, None) if window else
          lib.tempo_attn_block_causal(*args, 0.125, SOMEWHERE, 1 << 50, None))
    assert rc == T.TEMPO_OK
    launches = taken(lib)
    assert launches[0][0] == "block_bf16" and launches[0][1]["stream"] == stream
    assert_all_keys_launched(launches, Hq // Hkv, t, queries)


@pytest.mark.parametrize("shape,blocks", FEW_GROUPS)
def test_prompts_of_few_columns_over_few_groups(lib, shape, blocks):
    B, Hkv, G, D, t, count, window = shape
    launches = prefill(lib, store(T.TEMPO_BF16, Hkv, D, 32, (t + count) // 32 + 1), B, Hkv * G, t, count, window)
    names = [n for n, _ in launches]
    assert names[0] == "append" and names[1] in (("block_bf16", "partial_bf16") if blocks else ("prompt",))
    assert_all_keys_launched(launches, G, t, count)


@pytest.mark.parametrize("Hq,Hkv,D,batch,count,window,rows", [
    (24, 8, 128, 1, 2800, 0, True), (24, 8, 128, 1, 2801, 0, False), (24, 8, 128, 4, 1700, 0, True), (24, 8, 128, 4, 1701, 0, False),
    (8, 8, 128, 3, 1320, 0, True), (8, 8, 128, 3, 1321, 0, False), (8, 8, 128, 6, 1700, 0, True), (8, 8, 128, 6, 1701, 0, False),
    (8, 8, 128, 2, 1920, 0, True), (8, 8, 128, 2, 1921, 0, False), (32, 4, 128, 1, 3700, 0, True), (16, 16, 64, 2, 2500, 0, True),
    (64, 8, 128, 10, 480, 52, False), (64, 8, 128, 10, 272, 52, True), (24, 8, 128, 10, 1088, 36, False), (24, 8, 128, 10, 1066, 36, True),
    (64, 8, 128, 10, 480, 200, True)])
def test_bf16_prompts_read_from_rows(lib, Hq, Hkv, D, batch, count, window, rows):
    launches = prefill(lib, store(T.TEMPO_BF16, Hkv, D, 64, count // 64 + 1), batch, Hq, 0, count, window, out=1 << 45)
    assert [n for n, _ in launches][0] == ("prompt" if rows else "append")
    assert bool(dict(launches[-1][1])["k"]) == rows or not rows
    assert_all_keys_launched(launches, Hq // Hkv, 0, count)


@pytest.mark.parametrize("ring,rows", [(8, False), (4, True)])  # holds 480 steps, or not
def test_prompts_on_a_ring_read_from_rows(lib, ring, rows):
    launches = prefill(lib, store(T.TEMPO_BF16, 8, 128, 64, ring, ring), 10, 64, 0, 480, 52, out=1 << 45)
    assert [n for n, _ in launches] == (["prompt"] if rows else ["append", "short_prompt"])


@pytest.mark.parametrize("Hq,Hkv,D,batch,count,rows", [
    (8, 2, 64, 1, 512, True), (8, 2, 64, 1, 529, True), (8, 2, 64, 1, 530, False), (8, 2, 64, 1, 1024, False), (8, 2, 64, 1, 1025, True),
    (8, 8, 64, 1, 700, False), (8, 8, 64, 1, 705, True), (8, 8, 64, 2, 700, True)])
def test_f32_prompts_read_from_rows(lib, Hq, Hkv, D, batch, count, rows):
    launches = prefill(lib, store(T.TEMPO_F32, Hkv, D, 64, count // 64 + 1), batch, Hq, 0, count, out=1 << 45)
    assert [n for n, _ in launches] == (["partial_f32"] if rows else ["append", "partial_f32"])


@pytest.mark.parametrize("batch,t,count,window,waves", [(2, 3993, 125, 107, 2), (3, 0, 122, 21, 2)])
def test_wavefronts_of_a_windowed_prompt(lib, batch, t, count, window, waves):
    """From the store, and from rows."""
    launches = prefill(lib, store(T.TEMPO_BF16, 8, 128, 64, (t + count) // 64 + 1), batch, 24, t, count, window, out=1 << 45)
    assert launches[-1][0] == "prompt" and launches[-1][1]["waves"] == waves
