"""GPU parity of prompts over the sizes at which the prompt kernel's launch changes shape (2, 4 or 8
wavefronts of 32 columns per workgroup, split key ranges, ring stores answered in chunks), against the
fp64 CPU oracle; and of block-store writes that begin or end inside a 32-slot group, bit for bit.
Tolerances are those of test_gpu_parity.py.
"""
import numpy as np
import pytest
import torch

from oracle import tempo_oracle as oracle
from paper_2501_05408_amd import tempo as T
from paper_2501_05408_amd.store import BlockStore

from test_gpu_parity import DEV, assert_close, dev, host_inputs, np64, random_table

pytestmark = pytest.mark.gpu


def run_prompt(B, Hkv, G, D, Z, t, count, window, ring, dtype, seed=70, least_workspace=False, aligned=True):
    Hq, steps = Hkv * G, t + count
    q, K, V = host_inputs(seed, B, steps, Hq, Hkv, D, dtype)
    if ring:
        block = 128 // G
        ring_blocks = T.tempo_ring_blocks(window, Z, min(count, block))
        table, nb = random_table(seed, B, ring_blocks)
        st = BlockStore(B, Hq, Hkv, D, Z, steps - 1, dtype, num_blocks=nb, block_table=table, fill="nan",
                        ring_blocks=ring_blocks)
    else:
        table, nb = random_table(seed, B, (steps - 1) // Z + 1)
        st = BlockStore(B, Hq, Hkv, D, Z, steps - 1, dtype, num_blocks=nb, block_table=table, fill="nan")
    Kd, Vd = dev(K, dtype), dev(V, dtype)
    at = 0
    while at < t:                                        # the history, in pieces a ring store accepts
        n = min(t - at, ring_blocks * Z) if ring else t
        st.append_block(Kd[:, at:at + n].contiguous(), Vd[:, at:at + n].contiguous(), at, n)
        at += n
    qd = dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))[:, t:]), dtype)
    out = torch.empty_like(qd)
    k_new, v_new = Kd[:, t:].contiguous(), Vd[:, t:].contiguous()
    if not aligned:                                      # to 16 bytes: not answered from the rows themselves
        k_new, v_new = (torch.cat([x.new_zeros(4), x.reshape(-1)])[4:].view(x.shape) for x in (k_new, v_new))
    if least_workspace:                                  # what the blocks of 128 columns need, and no byte more
        block = 128 // G
        need = max(T.tempo_attn_plan_workspace_bytes(st.kv, B * min(block, count - c), Hq, T.tempo_attn_block_plan(
            st.kv, B, Hq, min(block, count - c), t + c, window)) for c in range(0, count, block))
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=DEV)   # NaN, should anything of it be read unwritten
        T.tempo_prefill_window(st.kv, qd, k_new, v_new, out, B, Hq, t, count, None, window, st.scale, ws, need)
    else:
        st._prefill_ws = torch.full((T.tempo_prefill_workspace_bytes(
            st.kv, B, Hq, ring_blocks * Z + 128 if ring else st.max_t),), 0xFF, dtype=torch.uint8, device=DEV)
        st.prefill_attend(qd, k_new, v_new, out, t, count, window)
    got = np64(out)
    K64, V64 = K.astype(np.float64), V.astype(np.float64)
    picks = sorted({0, 1, count // 2, count - 2, count - 1} | set(range(0, count, max(1, count // 40))))
    for c in [c for c in picks if 0 <= c < count]:
        ref = oracle.attend(q[t + c].astype(np.float64), K64, V64, t + c, window, 1.0 / np.sqrt(D))
        assert_close(got[:, c], ref, dtype, f"prompt step {t + c} of {t}..{steps - 1} G={G} D={D} w={window} ring={ring}")
    # what the store must hold now: the last steps of a ring, everything of a linear store
    first = max(0, steps - ring_blocks * Z) if ring else 0
    kg, vg = st.gather(first, steps - first)
    assert torch.equal(kg, Kd[:, first:steps]) and torch.equal(vg, Vd[:, first:steps])


@pytest.mark.parametrize("B,Hkv,G,D,t,count,window", [
    (1, 8, 4, 64, 0, 499, 0), (1, 2, 3, 128, 1500, 37, 0), (1, 1, 8, 128, 700, 65, 300), (2, 4, 3, 128, 5, 700, 0),
    (1, 1, 128, 64, 40, 9, 0), (1, 2, 40, 128, 31, 33, 0), (2, 1, 20, 128, 0, 64, 31), (1, 1, 1, 128, 3000, 1, 0),
    (1, 1, 1, 64, 2047, 33, 0), (1, 2, 3, 128, 1023, 43, 1024), (4, 8, 3, 128, 0, 341, 0), (16, 8, 3, 128, 64, 171, 0)])
def test_prompt_shapes(B, Hkv, G, D, t, count, window):
    run_prompt(B, Hkv, G, D, 32, t, count, window, False, T.TEMPO_BF16)


@pytest.mark.parametrize("B,Hkv,G,D,Z,t,count,window", [
    (2, 2, 3, 128, 32, 0, 700, 100), (1, 4, 4, 64, 64, 0, 333, 33), (3, 1, 8, 128, 32, 77, 400, 64),
    (1, 2, 1, 64, 32, 1000, 129, 1), (1, 2, 3, 128, 256, 0, 900, 512), (2, 1, 3, 128, 256, 300, 513, 512)])
@pytest.mark.parametrize("least_workspace", [False, True])
def test_ring_prompt_shapes(B, Hkv, G, D, Z, t, count, window, least_workspace):
    """With the workspace tempo_prefill_workspace_bytes asks for the prompt is staged there; with the
    least that is accepted, the first three in several staged pieces.  (The last three fit the ring as
    one chunk either way; several chunks: test_ring_prompts_in_chunks.)"""
    run_prompt(B, Hkv, G, D, Z, t, count, window, True, T.TEMPO_BF16, least_workspace=least_workspace, aligned=False)


@pytest.mark.parametrize("D,G,t,count", [(128, 3, 1500, 37), (64, 2, 1021, 20), (128, 3, 1500, 5), (64, 3, 9000, 70)])
def test_rope_prompt_with_split_ranges(D, G, t, count):
    """Few unrotated columns behind a long history: the bits of rotating first."""
    B, Hkv, Z, dtype = 1, 2, 32, T.TEMPO_BF16
    q, K, V = host_inputs(74, B, t + count, Hkv * G, Hkv, D, dtype)
    half = D // 2
    angle = torch.arange(t + count, dtype=torch.float64)[:, None] * 500000.0 ** (-torch.arange(half, dtype=torch.float64) / half)
    Kd, Vd = dev(K, dtype), dev(V, dtype)
    qd = dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))[:, t:]), dtype)
    outs = []
    for fused in (True, False):
        st = BlockStore(B, Hkv * G, Hkv, D, Z, t + count - 1, dtype, fill="nan")
        st.set_rope(torch.cos(angle).float().to(DEV), torch.sin(angle).float().to(DEV))
        st.rope_append_block(Kd[:, :t].contiguous(), Vd[:, :t].contiguous(), 0, t)
        qr, kr = qd.clone(), Kd[:, t:].contiguous()
        if not fused:
            for c in range(count):
                qr[:, c] = st.rope_rotate(qr[:, c].contiguous(), torch.empty_like(qr[:, c]).contiguous(), t + c)
                kr[:, c] = st.rope_rotate(kr[:, c].contiguous(), torch.empty_like(kr[:, c]).contiguous(), t + c)
        out = torch.empty_like(qr)
        st.prefill_attend(qr, kr, Vd[:, t:].contiguous(), out, t, count, rope=fused)
        outs.append(out)
    assert torch.equal(outs[0], outs[1])


ROPE_BY_BLOCKS = [(128, 3, 1500, 1), (128, 3, 3000, 5), (128, 4, 3000, 8), (64, 4, 3000, 12), (64, 3, 16000, 70),
                  (128, 3, 16000, 60), (128, 20, 4000, 3)]


@pytest.mark.parametrize("D,G,t,count", ROPE_BY_BLOCKS)
def test_rope_prompt_by_blocks(D, G, t, count):
    """Those that go in blocks of columns (test_host_launches.py looks that they do): each size of kernel, two blocks, and
    groups wider than the single-step kernel."""
    test_rope_prompt_with_split_ranges(D, G, t, count)


# ((B, Hkv, G, D, t, count, window), by blocks): a few columns over a few groups, on both sides of the lines
FEW_GROUPS = [((2, 8, 3, 128, 26, 3, 0), False), ((2, 8, 3, 128, 29, 3, 0), False), ((2, 8, 3, 128, 30, 3, 0), True), ((1, 1, 8, 128, 30, 1, 0), True),
              ((1, 2, 7, 128, 62, 2, 0), False), ((1, 2, 7, 128, 63, 2, 0), True), ((3, 2, 12, 64, 31, 1, 0), False),
              ((3, 2, 11, 64, 31, 1, 0), True), ((3, 2, 4, 64, 30, 3, 0), True), ((1, 4, 3, 128, 24, 8, 0), False), ((1, 4, 3, 128, 25, 8, 0), True),
              ((1, 4, 3, 128, 55, 9, 0), False), ((1, 4, 3, 128, 56, 9, 0), True), ((2, 2, 1, 64, 15, 17, 0), False),
              ((2, 2, 1, 64, 16, 17, 0), True), ((2, 8, 4, 64, 1, 15, 0), False), ((1, 2, 4, 64, 240, 16, 0), False),
              ((1, 2, 4, 64, 400, 12, 244), False)]


@pytest.mark.parametrize("shape,blocks", FEW_GROUPS)
def test_prompts_of_few_columns_over_few_groups(shape, blocks):
    B, Hkv, G, D, t, count, window = shape
    run_prompt(B, Hkv, G, D, 32, t, count, window, False, T.TEMPO_BF16)


@pytest.mark.parametrize("dtype,B,Hkv,G,D,t,count,window,ring", [
    (T.TEMPO_BF16, 1, 1, 3, 64, 16000, 70, 0, False), (T.TEMPO_BF16, 1, 1, 8, 128, 32000, 42, 0, False),   # several blocks
    (T.TEMPO_BF16, 2, 2, 3, 128, 0, 90, 0, False), (T.TEMPO_F32, 2, 2, 3, 64, 0, 90, 0, False),            # one launch
    (T.TEMPO_BF16, 1, 2, 3, 128, 0, 900, 100, True), (T.TEMPO_BF16, 2, 2, 1, 64, 0, 700, 100, True),       # chunks of a ring
    (T.TEMPO_BF16, 2, 1, 3, 64, 77, 500, 64, True), (T.TEMPO_F32, 2, 2, 3, 64, 0, 400, 50, True),
    (T.TEMPO_F32, 2, 2, 1, 64, 100, 500, 50, True)])
@pytest.mark.parametrize("where", ["k", "v", "k's second half", "before k"])
def test_prompt_answered_over_its_rows(dtype, B, Hkv, G, D, t, count, window, ring, where):
    """out may lie over k_new and v_new: the answers and the store of a call whose buffers are apart.  (By which
    launches: test_host_launches.py.)"""
    torch.manual_seed(5)
    ty, n = (torch.bfloat16 if dtype == T.TEMPO_BF16 else torch.float32), B * count * Hkv * D
    q = torch.randn(B, count, Hkv * G, D, device=DEV).to(ty)
    k, v = (torch.randn(n, device=DEV).to(ty) for _ in range(2))
    R = T.tempo_ring_blocks(window, 64, min(count, 128 // G)) if ring else 0
    past = min(t, window) if ring else t
    K, V = (torch.randn(B, past, Hkv, D, device=DEV).to(ty) for _ in range(2))
    k_at = n * G                                         # in a buffer of k, v and `out` over them
    v_at = k_at + n + 64
    out_at = {"k": k_at, "v": v_at, "k's second half": k_at + n // 2 // 64 * 64, "before k": k_at - n // 3 // 64 * 64}[where]
    got = []
    for over in (False, True):
        st = BlockStore(B, Hkv * G, Hkv, D, 64, t + count - 1, dtype, fill="nan", ring_blocks=R)
        if t:
            st.append_block(K, V, t - past, past)
        room = torch.zeros(n * (2 * G + 3) + 64, dtype=ty, device=DEV)
        room[k_at:k_at + n], room[v_at:v_at + n] = k, v
        rows = [room[at:at + n].view(B, count, Hkv, D) for at in (k_at, v_at)]
        out = room[out_at:out_at + n * G].view(B, count, Hkv * G, D) if over else torch.empty_like(q)
        st.prefill_attend(q, *rows, out, t, count, window)
        got.append((out.float().cpu(), st.k_pool.cpu(), st.v_pool.cpu()))
    # another route may answer: weights rounded to bf16 against another reference, 2^-8 each way
    assert (got[1][0] - got[0][0]).abs().max() <= 2 ** -7 * got[0][0].abs().max()
    assert torch.equal(got[1][1].nan_to_num(7), got[0][1].nan_to_num(7))
    assert torch.equal(got[1][2].nan_to_num(7), got[0][2].nan_to_num(7))


@pytest.mark.parametrize("B,Hkv,G,D,Z,t,count,window,ring", [
    (1, 2, 4, 64, 64, 0, 300, 0, False), (2, 2, 3, 128, 4, 13, 70, 0, False), (1, 1, 1, 64, 8, 2500, 9, 0, False),
    (1, 1, 20, 128, 16, 37, 30, 33, False), (1, 1, 3, 128, 16, 3000, 5, 0, False), (2, 1, 3, 64, 8, 50, 260, 40, True)])
def test_f32_prompt_shapes(B, Hkv, G, D, Z, t, count, window, ring):
    run_prompt(B, Hkv, G, D, Z, t, count, window, ring, T.TEMPO_F32)


@pytest.mark.parametrize("D,G,window", [(64, 3, 0), (128, 1, 9)])
def test_f32_values_that_are_not_finite_reach_only_the_steps_that_see_them(D, G, window):
    """The steps of a prompt share key/value reads; an infinite value of key j may show in the
    outputs of steps that see j, in no other step's."""
    B, Hkv, Z, count, j = 1, 1, 16, 40, 21
    q, K, V = host_inputs(73, B, count, G, Hkv, D, T.TEMPO_F32)
    outs = []
    for bad in (False, True):
        Vx = V.copy()
        if bad:
            Vx[:, j, :, 3] = np.inf
        st = BlockStore(B, G, Hkv, D, Z, count - 1, T.TEMPO_F32, fill="nan")
        out = torch.empty((B, count, G, D), dtype=torch.float32, device=DEV)
        st.prefill_attend(dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))), T.TEMPO_F32), dev(K, T.TEMPO_F32),
                          dev(Vx, T.TEMPO_F32), out, 0, count, window)
        outs.append(np64(out))
    for t in range(count):
        sees = j <= t and (window == 0 or j > t - window)
        rest = [d for d in range(D) if d != 3]
        # bound: the two runs may take the products of a group in another order (32-bit sums of <= 40 terms)
        assert np.abs(outs[1][:, t][..., rest] - outs[0][:, t][..., rest]).max() <= 1e-5
        if sees:
            assert np.isposinf(outs[1][:, t][..., 3]).all()
        else:
            assert np.abs(outs[1][:, t] - outs[0][:, t]).max() <= 1e-5


@pytest.mark.parametrize("t,count", [(0, 32), (1, 32), (31, 33), (5, 59), (33, 95), (17, 64), (40, 200)])
def test_append_block_edges(t, count):
    """Writes that begin and end inside groups keep every other slot of those groups as it was."""
    B, Hkv, D, Z, steps = 2, 3, 128, 64, 256
    _, K, V = host_inputs(71, B, steps, Hkv, Hkv, D, T.TEMPO_BF16)
    Kd, Vd = dev(K, T.TEMPO_BF16), dev(V, T.TEMPO_BF16)
    st = BlockStore(B, Hkv, Hkv, D, Z, steps - 1, T.TEMPO_BF16)
    st.append_block(Kd, Vd, 0, steps)
    k2, v2 = -Kd[:, t:t + count].contiguous(), -Vd[:, t:t + count].contiguous()
    st.append_block(k2, v2, t, count)
    want_k, want_v = Kd.clone(), Vd.clone()
    want_k[:, t:t + count], want_v[:, t:t + count] = k2, v2
    kg, vg = st.gather(0, steps)
    assert torch.equal(kg, want_k) and torch.equal(vg, want_v)


def test_append_block_that_fills_a_ring_from_inside_a_group():
    B, Hkv, D, Z, R, t = 2, 2, 64, 32, 4, 45
    count = R * Z
    _, K, V = host_inputs(72, B, t + count, Hkv, Hkv, D, T.TEMPO_BF16)
    Kd, Vd = dev(K, T.TEMPO_BF16), dev(V, T.TEMPO_BF16)
    st = BlockStore(B, Hkv, Hkv, D, Z, 10 ** 6, T.TEMPO_BF16, ring_blocks=R)
    st.append_block(Kd[:, t:].contiguous(), Vd[:, t:].contiguous(), t, count)
    kg, vg = st.gather(t, count)
    assert torch.equal(kg, Kd[:, t:]) and torch.equal(vg, Vd[:, t:])


def run_from_first_visible_step(call, B, Hkv, G, D, Z, t, count, window, ring):
    """`call` answers steps t .. t+count-1 on a poisoned store whose history begins at the first step
    that step t sees; every step against the oracle."""
    Hq, steps, dtype = Hkv * G, t + count, T.TEMPO_BF16
    q, K, V = host_inputs(75, B, steps, Hq, Hkv, D, dtype)
    ring_blocks = T.tempo_ring_blocks(window, Z, min(count, 128 // G)) if ring else 0
    table, nb = random_table(75, B, ring_blocks if ring else (steps - 1) // Z + 1)
    st = BlockStore(B, Hq, Hkv, D, Z, steps - 1, dtype, num_blocks=nb, block_table=table, fill="nan", ring_blocks=ring_blocks)
    Kd, Vd, first = dev(K, dtype), dev(V, dtype), t - window + 1
    assert first > 0 and first % 32 != 0
    if window > 1:
        st.append_block(Kd[:, first:t].contiguous(), Vd[:, first:t].contiguous(), first, t - first)
    qd = dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))[:, t:]), dtype)
    out = torch.empty_like(qd)
    call(st, qd, Kd[:, t:].contiguous(), Vd[:, t:].contiguous(), out)
    got = np64(out)
    K64, V64 = K.astype(np.float64), V.astype(np.float64)
    for c in range(count):
        ref = oracle.attend(q[t + c].astype(np.float64), K64, V64, t + c, window, 1.0 / np.sqrt(D))
        assert_close(got[:, c], ref, dtype, f"step {t + c} of {t}..{steps - 1} G={G} D={D} w={window} ring={ring}")


FIRST_VISIBLE = [(1, 1, 3, 128, 32, 1000, 1, 64), (2, 2, 3, 128, 64, 1000, 5, 64), (1, 2, 3, 64, 32, 1000, 40, 64),
                 (1, 1, 3, 128, 256, 998, 400, 200), (1, 1, 20, 64, 32, 300, 3, 290), (2, 1, 1, 128, 32, 70, 1, 1)]


@pytest.mark.parametrize("B,Hkv,G,D,Z,t,count,window", FIRST_VISIBLE)
@pytest.mark.parametrize("ring", [False, True])
def test_prompt_behind_a_history_that_begins_inside_a_group(B, Hkv, G, D, Z, t, count, window, ring):
    """Slots of the first group before the window's start were never written and hold NaN."""
    run_from_first_visible_step(lambda st, q, k, v, out: st.prefill_attend(q, k, v, out, t, count, window),
                                B, Hkv, G, D, Z, t, count, window, ring)


@pytest.mark.parametrize("B,Hkv,G,D,Z,t,count,window", [
    (1, 2, 20, 64, 32, 300, 1, 290), (1, 1, 3, 128, 32, 1000, 5, 64), (2, 2, 3, 128, 64, 1000, 10, 64),
    (1, 1, 3, 128, 256, 998, 21, 200), (1, 1, 3, 64, 32, 1000, 42, 600), (1, 2, 1, 128, 32, 70, 20, 1)])
@pytest.mark.parametrize("ring", [False, True])
def test_block_behind_a_history_that_begins_inside_a_group(B, Hkv, G, D, Z, t, count, window, ring):
    def call(st, q, k, v, out):
        st.append_block(k, v, t, count)
        st.attend_block(q, out, t, count, window)
    run_from_first_visible_step(call, B, Hkv, G, D, Z, t, count, window, ring)


@pytest.mark.parametrize("dtype,B,count", [(T.TEMPO_BF16, 1, 40), (T.TEMPO_BF16, 1, 300), (T.TEMPO_F32, 16, 40)])
def test_ring_prompt_whose_range_crosses_two_to_the_thirty(dtype, B, count):
    """A ring store answers any step; the oracle sees the same rows counted from the first visible step."""
    Hkv, G, D, Z, window = 8, 3, 128, 32, 50
    t = (1 << 30) - 20
    first, n = t - window + 1, window - 1 + count
    q, K, V = host_inputs(76, B, n, Hkv * G, Hkv, D, dtype)
    ring_blocks = T.tempo_ring_blocks(window, Z, min(count, 128 // G))
    st = BlockStore(B, Hkv * G, Hkv, D, Z, t + count - 1, dtype, fill="nan", ring_blocks=ring_blocks)
    Kd, Vd = dev(K, dtype), dev(V, dtype)
    st.append_block(Kd[:, :window - 1].contiguous(), Vd[:, :window - 1].contiguous(), first, window - 1)
    qd = dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))[:, window - 1:]), dtype)
    out = torch.empty_like(qd)
    st.prefill_attend(qd, Kd[:, window - 1:].contiguous(), Vd[:, window - 1:].contiguous(), out, t, count, window)
    got = np64(out)
    K64, V64 = K.astype(np.float64), V.astype(np.float64)
    for c in range(0, count, 3):
        at = window - 1 + c
        ref = oracle.attend(q[at].astype(np.float64), K64, V64, at, window, 1.0 / np.sqrt(D))
        assert_close(got[:, c], ref, dtype, f"prompt step 2^30 {t + c - (1 << 30):+d}")


def test_appends_to_the_same_groups_on_two_streams_keep_each_others_rows():
    """Two calls that are not ordered write different slots of the same 32-slot groups: neither may
    write a slot of the other's back as it was."""
    B, Hkv, D, Z, steps = 16, 8, 128, 64, 128
    _, K, V = host_inputs(77, B, steps, Hkv, Hkv, D, T.TEMPO_BF16)
    Kd, Vd = dev(K, T.TEMPO_BF16), dev(V, T.TEMPO_BF16)
    st = BlockStore(B, Hkv, Hkv, D, Z, steps - 1, T.TEMPO_BF16)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for first in (33, 40, 47, 50, 62):
        parts = [(0, first), (first, steps - first)]
        rows = [(Kd[:, t:t + n].contiguous(), Vd[:, t:t + n].contiguous()) for t, n in parts]
        for _ in range(10):
            st.k_pool.zero_(), st.v_pool.zero_()
            torch.cuda.synchronize()
            for s, (t, n), (k, v) in zip(streams, parts, rows):
                with torch.cuda.stream(s):
                    st.append_block(k, v, t, n)
            torch.cuda.synchronize()
            kg, vg = st.gather(0, steps)
            assert torch.equal(kg, Kd) and torch.equal(vg, Vd)


@pytest.mark.parametrize("B,Hkv,G,D,Z,steps,window", [(1, 2, 3, 128, 16, 200, 0), (2, 1, 1, 128, 64, 420, 0), (3, 2, 4, 64, 8, 40, 0),
                                                      (1, 1, 17, 128, 4, 210, 0), (2, 2, 3, 128, 32, 260, 70), (16, 2, 8, 128, 64, 110, 0)])
@pytest.mark.parametrize("rope", [False, True])
def test_f32_steps_where_the_kernel_changes(B, Hkv, G, D, Z, steps, window, rope):
    """Every step of sequences that grow past the ranges the vector kernel takes (24 keys at D = 64,
    192 at D = 128 or fewer for many heads, all where no head shares a read), with the write fused in."""
    Hq, dtype = Hkv * G, T.TEMPO_F32
    q, K, V = host_inputs(78, B, steps, Hq, Hkv, D, dtype)
    table, nb = random_table(78, B, (steps - 1) // Z + 1)
    st = BlockStore(B, Hq, Hkv, D, Z, steps - 1, dtype, num_blocks=nb, block_table=table, fill="nan")
    qd, Kd, Vd = dev(q, dtype), dev(K, dtype), dev(V, dtype)
    half = D // 2
    angle = np.arange(steps)[:, None] * 500000.0 ** (-np.arange(half) / half)
    if rope:
        st.set_rope(torch.from_numpy(np.cos(angle)).float().to(DEV), torch.from_numpy(np.sin(angle)).float().to(DEV))
    out = torch.empty((steps, B, Hq, D), dtype=torch.float32, device=DEV)
    for t in range(steps):
        k_t, v_t = Kd[:, t].contiguous(), Vd[:, t].contiguous()
        if rope:
            st.rope_step(qd[t], k_t, v_t, out[t], t, window)
        elif window:
            st.step_window(qd[t], k_t, v_t, out[t], t, window)
        else:
            st.step_causal(qd[t], k_t, v_t, out[t], t)
    got = np64(out)

    def turned(x, at):                                   # [..., D] rows of steps `at`, in 64 bits
        c, s = np.cos(angle).astype(np.float32).astype(np.float64)[at], np.sin(angle).astype(np.float32).astype(np.float64)[at]
        lo, hi = x[..., :half], x[..., half:]
        return np.concatenate([lo * c - hi * s, hi * c + lo * s], axis=-1)

    q64, K64, V64 = q.astype(np.float64), K.astype(np.float64), V.astype(np.float64)
    if rope:
        q64 = np.stack([turned(q64[t], t) for t in range(steps)])
        K64 = np.stack([turned(K64[:, t], t) for t in range(steps)], axis=1)
    for t in range(0, steps, 3):
        assert_close(got[t], oracle.attend(q64[t], K64, V64, t, window, 1.0 / np.sqrt(D)), dtype, f"fp32 step {t} w={window} rope={rope}")
    kg, vg = st.gather(0, steps)
    assert torch.equal(vg, Vd) and (rope or torch.equal(kg, Kd))


@pytest.mark.parametrize("B,Hkv,G,D,t,count,window", [
    (16, 8, 3, 128, 0, 64, 0), (2, 2, 3, 128, 60, 43, 0), (1, 1, 3, 128, 0, 128, 0), (2, 1, 3, 128, 900, 300, 64),
    (1, 2, 128, 128, 31, 5, 0), (3, 1, 20, 128, 7, 33, 1), (1, 1, 1, 128, 0, 128, 0), (1, 1, 1, 128, 33, 400, 1)])
def test_prompts_over_short_ranges(B, Hkv, G, D, t, count, window):
    run_prompt(B, Hkv, G, D, 32, t, count, window, False, T.TEMPO_BF16)


def test_prompts_over_short_ranges_rotated_and_of_different_lengths():
    test_rope_prompt_with_split_ranges(128, 3, 20, 70)
    B, Hkv, G, D, count = 4, 2, 3, 128, 100
    q, K, V = host_inputs(79, B, count, Hkv * G, Hkv, D, T.TEMPO_BF16)
    st = BlockStore(B, Hkv * G, Hkv, D, 32, count - 1, T.TEMPO_BF16, fill="nan")
    lengths = torch.tensor([0, 1, 43, 100], dtype=torch.int32, device=DEV)
    qd = dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))), T.TEMPO_BF16)
    out = torch.full_like(qd, 7.0)
    st.prefill_attend(qd, dev(K, T.TEMPO_BF16), dev(V, T.TEMPO_BF16), out, 0, count, count_per_seq=lengths)
    got = np64(out)
    for b, n in enumerate(lengths.tolist()):
        assert (got[b, n:] == 7.0).all()
        for c in range(0, n, 6):
            ref = oracle.attend(q[c].astype(np.float64), K.astype(np.float64), V.astype(np.float64), c, 0, 1.0 / np.sqrt(D))
            assert_close(got[b, c], ref[b], T.TEMPO_BF16, f"sequence {b} of {n} steps, step {c}")


@pytest.mark.parametrize("B,Hkv,G,D,t,count,window", [
    (1, 8, 3, 128, 0, 4, 0), (1, 1, 16, 128, 100, 4, 0), (2, 2, 1, 128, 100, 16, 0), (1, 2, 3, 128, 900, 5, 70),
    (1, 2, 4, 64, 0, 4, 0), (1, 2, 4, 64, 20, 4, 0), (1, 2, 4, 64, 22, 4, 0), (1, 1, 1, 128, 33, 9, 1)])
def test_f32_blocks_where_the_kernel_changes(B, Hkv, G, D, t, count, window):
    """Small blocks over short ranges (vector kernel) and just past them, unrotated and with rotated queries."""
    dtype = T.TEMPO_F32
    q, K, V = host_inputs(80, B, t + count, Hkv * G, Hkv, D, dtype)
    st = BlockStore(B, Hkv * G, Hkv, D, 16, t + count - 1, dtype, fill="nan")
    first = max(0, t - window + 1) if window else 0
    Kd, Vd = dev(K, dtype), dev(V, dtype)
    st.append_block(Kd[:, first:].contiguous(), Vd[:, first:].contiguous(), first, t + count - first)
    qd = dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))[:, t:]), dtype)
    out = st.attend_block(qd, torch.empty_like(qd), t, count, window)
    for c in range(count):
        ref = oracle.attend(q[t + c].astype(np.float64), K.astype(np.float64), V.astype(np.float64), t + c, window, 1.0 / np.sqrt(D))
        assert_close(np64(out)[:, c], ref, dtype, f"fp32 block step {t + c} w={window}")
    half = D // 2
    angle = torch.arange(t + count, dtype=torch.float64)[:, None] * 500000.0 ** (-torch.arange(half, dtype=torch.float64) / half)
    st.set_rope(torch.cos(angle).float().to(DEV), torch.sin(angle).float().to(DEV))
    turned = torch.stack([st.rope_rotate(qd[:, c].contiguous(), torch.empty_like(qd[:, c]).contiguous(), t + c)
                          for c in range(count)], dim=1)
    got = st.attend_block(qd, torch.empty_like(qd), t, count, window, rope=True)
    assert torch.equal(got, st.attend_block(turned, torch.empty_like(qd), t, count, window))


@pytest.mark.parametrize("B,Hkv,G,D,Z,t,count,window", [
    (16, 32, 1, 64, 256, 0, 700, 100), (16, 32, 1, 64, 256, 77, 500, 100), (8, 64, 2, 64, 64, 13, 330, 40),
    (64, 8, 3, 128, 256, 0, 1100, 300)])
def test_ring_prompts_in_chunks(B, Hkv, G, D, Z, t, count, window):
    """Shapes whose least workspace has no room to stage the prompt (test_host_launches.py checks that
    they take this path): each chunk written into the ring and answered from it."""
    run_prompt(B, Hkv, G, D, Z, t, count, window, True, T.TEMPO_BF16, least_workspace=True, aligned=False)


@pytest.mark.parametrize("B,Hkv,G,D,t,count,window", [
    (1, 2, 3, 128, 1500, 130, 0), (1, 1, 5, 64, 2900, 70, 300), (2, 1, 40, 64, 1023, 11, 129), (1, 8, 3, 128, 0, 1100, 0),
    (2, 2, 3, 128, 0, 43, 0), (2, 1, 23, 128, 0, 90, 40), (1, 1, 127, 64, 3, 5, 0)])
def test_blocks_that_begin_between_the_heads_of_a_step(B, Hkv, G, D, t, count, window):
    run_prompt(B, Hkv, G, D, 64, t, count, window, False, T.TEMPO_BF16)


@pytest.mark.parametrize("dtype", [T.TEMPO_BF16, T.TEMPO_F32])
@pytest.mark.parametrize("B,Hkv,G,D,Z,count,window,ring", [
    (1, 2, 3, 128, 32, 1, 0, False), (2, 2, 3, 128, 64, 31, 0, False), (2, 1, 4, 64, 32, 33, 0, False),
    (1, 3, 1, 64, 64, 97, 0, False), (2, 2, 3, 128, 32, 171, 40, False), (1, 1, 128, 128, 32, 37, 0, False),
    (2, 8, 3, 128, 256, 700, 0, False), (1, 2, 5, 64, 32, 1000, 0, False), (2, 2, 3, 128, 32, 403, 33, True),
    (1, 4, 1, 64, 32, 129, 64, True), (2, 2, 8, 128, 64, 650, 100, True), (1, 2, 3, 128, 32, 64, 1, True)])
def test_prompts_read_from_the_callers_rows(B, Hkv, G, D, Z, count, window, ring, dtype):
    """From step 0 on the prompt kernels read the call's rows and write the store themselves; rows that are not
    16-byte aligned take the way through the store.  Same store, bit for bit (slots nobody writes included),
    same outputs within the tolerance against the oracle."""
    Hq = Hkv * G
    q, K, V = host_inputs(91, B, count, Hq, Hkv, D, dtype)
    R = T.tempo_ring_blocks(window, Z, min(count, 128 // G)) if ring else 0
    table, nb = random_table(91, B, R or (count - 1) // Z + 1)
    Kd, Vd = dev(K, dtype), dev(V, dtype)
    qd = dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))), dtype)
    got = []
    for shift in (0, 4 if dtype == T.TEMPO_BF16 else 2):
        st = BlockStore(B, Hq, Hkv, D, Z, count - 1, dtype, num_blocks=nb, block_table=table, fill="nan", ring_blocks=R)
        rows = []
        for x in (Kd, Vd):
            room = torch.full((x.numel() + shift,), float("nan"), dtype=x.dtype, device=DEV)
            room[shift:] = x.reshape(-1)
            rows.append(room[shift:].reshape(x.shape))
        out = torch.empty_like(qd)
        st.prefill_attend(qd, rows[0], rows[1], out, 0, count, window)
        got.append((out, st.k_pool.view(torch.int16), st.v_pool.view(torch.int16)))
    assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][2], got[1][2])
    assert_close(np64(got[0][0]), np64(got[1][0]), dtype, f"{(B, Hkv, G, D, Z, count, window, ring)}")
    for c in sorted({0, count // 2, count - 1}):
        ref = oracle.attend(q[c].astype(np.float64), K.astype(np.float64), V.astype(np.float64), c, window, 1.0 / np.sqrt(D))
        assert_close(np64(got[0][0])[:, c], ref, dtype, f"step {c}")


@pytest.mark.parametrize("D,G", [(128, 3), (64, 8)])
def test_rows_beyond_a_sequences_own_count_are_not_read(D, G):
    B, Hkv, Z, count = 4, 2, 64, 150
    Hq, counts = Hkv * G, [150, 1, 0, 77]
    q, K, V = host_inputs(92, B, count, Hq, Hkv, D, T.TEMPO_BF16)
    st = BlockStore(B, Hq, Hkv, D, Z, count - 1, T.TEMPO_BF16, fill="nan")
    Kd, Vd = dev(K, T.TEMPO_BF16), dev(V, T.TEMPO_BF16)
    for b, n in enumerate(counts):
        Kd[b, n:], Vd[b, n:] = float("nan"), float("nan")
    qd = dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))), T.TEMPO_BF16)
    out = torch.full_like(qd, 7.0)
    st.prefill_attend(qd, Kd, Vd, out, 0, count, count_per_seq=torch.tensor(counts, dtype=torch.int32, device=DEV))
    kg, vg = st.gather(0, count)
    for b, n in enumerate(counts):
        assert torch.equal(kg[b, :n], Kd[b, :n]) and torch.equal(vg[b, :n], Vd[b, :n])
        assert torch.isnan(kg[b, n:]).all() and torch.isnan(vg[b, n:]).all() and (out[b, n:] == 7.0).all()
        for c in sorted({0, n // 2, n - 1} & set(range(n))):
            ref = oracle.attend(q[c].astype(np.float64), K.astype(np.float64), V.astype(np.float64), c, 0, 1.0 / np.sqrt(D))
            assert_close(np64(out)[b:b + 1, c], ref[b:b + 1], T.TEMPO_BF16, f"sequence {b} step {c}")


@pytest.mark.parametrize("B,Hkv,G,D,first,steps,window", [
    (2, 2, 3, 128, 60, 75, 0), (1, 1, 8, 128, 700, 34, 97), (3, 2, 4, 64, 90, 12, 0), (1, 1, 16, 64, 1530, 12, 0),
    (2, 1, 1, 64, 1700, 5, 1536), (1, 2, 3, 128, 250, 60, 0)])
@pytest.mark.parametrize("rope", [False, True])
def test_steps_around_the_ranges_whose_last_group_stands_apart(B, Hkv, G, D, first, steps, window, rope):
    """bf16 steps first .. first + steps - 1 (96 keys; 1536 at D = 64), the write fused in."""
    Hq, dtype, T_ = Hkv * G, T.TEMPO_BF16, first + steps
    q, K, V = host_inputs(93, B, T_, Hq, Hkv, D, dtype)
    table, nb = random_table(93, B, (T_ - 1) // 32 + 1)
    st = BlockStore(B, Hq, Hkv, D, 32, T_ - 1, dtype, num_blocks=nb, block_table=table, fill="nan")
    angle = np.arange(T_)[:, None] * 500000.0 ** (-np.arange(D // 2) / (D // 2))
    st.set_rope(torch.from_numpy(np.cos(angle)).float().to(DEV), torch.from_numpy(np.sin(angle)).float().to(DEV))
    qd, Kd, Vd = dev(q, dtype), dev(K, dtype), dev(V, dtype)
    write = st.rope_append_block if rope else st.append_block
    write(Kd[:, :first].contiguous(), Vd[:, :first].contiguous(), 0, first)
    out = torch.empty((steps, B, Hq, D), dtype=torch.bfloat16, device=DEV)
    for i in range(steps):
        t = first + i
        row = (qd[t], Kd[:, t].contiguous(), Vd[:, t].contiguous(), out[i], t)
        if rope:
            st.rope_step(*row, window)
        elif window:
            st.step_window(*row, window)
        else:
            st.step_causal(*row)
    kg, vg = st.gather(0, T_)                            # (rotated keys: as stored, which the rotary tests pin)
    assert torch.equal(vg, Vd) and (rope or torch.equal(kg, Kd))
    K64, V64, got = np64(kg), V.astype(np.float64), np64(out)
    for i in range(steps):
        qt = qd[first + i]
        if rope:
            qt = st.rope_rotate(qt, torch.empty_like(qt), first + i)
        ref = oracle.attend(np64(qt), K64, V64, first + i, window, 1.0 / np.sqrt(D))
        assert_close(got[i], ref, dtype, f"step {first + i} w={window} rope={rope}")


# (Hkv, G, D, count, window, j): the value of step j is infinite; and the steps that see it or share a block of columns
# with one that does.  Blocks have 128 columns here, or (few columns) 64.
@pytest.mark.parametrize("Hkv,G,D,count,window,j,touched", [
    (8, 3, 128, 700, 0, 50, range(42, 700)), (8, 3, 64, 700, 0, 50, range(42, 700)),       # later than the block's last step
    (2, 8, 64, 100, 0, 17, range(16, 100)), (8, 4, 128, 700, 40, 10, range(0, 64)),        # earlier than its first key
    (8, 3, 128, 700, 5, 35, range(0, 43)), (1, 16, 64, 200, 3, 4, range(0, 8)),            # in a group that it writes
    (8, 3, 64, 700, 1, 36, range(0, 43)), (1, 1, 128, 130, 2, 126, range(64, 128))])
@pytest.mark.parametrize("aligned", [True, False])
def test_values_that_are_not_finite_stay_in_the_blocks_that_see_them(Hkv, G, D, count, window, j, touched, aligned):
    """Read from the call's rows as through the store: the same store, and nothing of such a value in other blocks."""
    B, Hq, dtype = 2, Hkv * G, T.TEMPO_BF16
    q, K, V = host_inputs(94, B, count, Hq, Hkv, D, dtype)
    qd = dev(np.ascontiguousarray(np.transpose(q, (1, 0, 2, 3))), dtype)
    got = []
    for bad in (False, True):
        rows = [dev(K, dtype), dev(V, dtype)]
        if bad:
            rows[1][:, j] = float("inf")
        if not aligned:
            rows = [torch.cat([x.new_zeros(4), x.reshape(-1)])[4:].view(x.shape) for x in rows]
        st = BlockStore(B, Hq, Hkv, D, 32, count - 1, dtype, fill="nan")
        out = torch.empty_like(qd)
        st.prefill_attend(qd, rows[0], rows[1], out, 0, count, window)
        kg, vg = st.gather(0, count)
        assert torch.equal(kg, rows[0]) and torch.equal(vg, rows[1])
        got.append(out)
    for c in range(count):
        sees = c >= j and (window == 0 or c - j < window)
        assert not sees or not torch.isfinite(got[1][:, c]).any(), c
        assert c in touched or torch.equal(got[1][:, c], got[0][:, c]), c
