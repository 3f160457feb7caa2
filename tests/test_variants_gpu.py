"""GPU parity of the general entry points (avion_attn_fwd_ex / avion_attn_bwd_ex): every combination of
element format (bf16, fp16), masking (none, causal) and packing ([B,N,H,d] x 3, or [B,N,3,H,d]) against
the fp64 oracle, and bit for bit against the specific entry points where those exist."""
import itertools

import numpy as np
import pytest

import synth_inputs as si
from tests import gpu_harness as gh

pytestmark = pytest.mark.gpu


def _upload(bits, f16):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda()
    return t.view(torch.float16 if f16 else torch.bfloat16)


def run_ex(w, x, f16, causal, packed):
    """fwd + bwd through the general entry points; x holds bit patterns of the chosen format."""
    import torch
    import paper_2309_16669_amd as av
    dO = _upload(x["dO"], f16)
    o = torch.full_like(dO, float("nan"))
    lse = torch.full((w.B, w.H, w.N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(av.attn_bwd_workspace_bytes(w.B, w.H, w.N, w.d), dtype=torch.uint8, device="cuda").fill_(255)
    if packed:
        qkv = _upload(np.stack([x["q"], x["k"], x["v"]], axis=2), f16)
        dqkv = torch.full_like(qkv, float("nan"))
        av.attn_fwd_ex(qkv, None, None, o, lse, w.scale, causal)
        av.attn_bwd_ex(qkv, None, None, o, lse, dO, dqkv, None, None, w.scale, ws, causal)
        torch.cuda.synchronize()
        return dict(o=o, lse=lse, dq=dqkv[:, :, 0], dk=dqkv[:, :, 1], dv=dqkv[:, :, 2])
    q, k, v = (_upload(x[n], f16) for n in ("q", "k", "v"))
    dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(3))
    av.attn_fwd_ex(q, k, v, o, lse, w.scale, causal)
    av.attn_bwd_ex(q, k, v, o, lse, dO, dq, dk, dv, w.scale, ws, causal)
    torch.cuda.synchronize()
    return dict(o=o, lse=lse, dq=dq, dk=dk, dv=dv)


def check(w, x, out, f16, causal):
    """Against the oracle on the exactly widened inputs.  Bounds: those of the format (fp16: eight
    times tighter than bf16); the absolute bound follows one unit in the last place of the largest
    reference value where that exceeds it (causal rows over few keys carry weights near one)."""
    import oracle
    widen = si.f16_bits_to_f64 if f16 else si.bf16_bits_to_f64
    q, k, v, dO = (widen(x[n]) for n in ("q", "k", "v", "dO"))
    ro, rl = oracle.fwd_f64(q, k, v, w.scale, causal=causal)
    refs = oracle.bwd_f64(q, k, v, dO, w.scale, causal=causal)
    max_abs_tol, rel_tol, ulp = (gh.MAX_ABS_F16, gh.REL_FRO_F16, 2.0 ** -10) if f16 else (gh.MAX_ABS, gh.REL_FRO, 2.0 ** -7)
    # fewer than 16 keys: the gradients' relative bound of tests/test_tolerance_model.py (an eighth of it in fp16)
    grad_tol = rel_tol if w.N >= 16 else (gh.REL_FRO_TINY_N / 8 if f16 else gh.REL_FRO_TINY_N)
    assert float(np.abs(out["lse"].double().cpu().numpy() - rl).max()) <= gh.LSE_ABS
    for name, key, ref in (("O", "o", ro), ("dQ", "dq", refs[0]), ("dK", "dk", refs[1]), ("dV", "dv", refs[2])):
        got = out[key].contiguous().double().cpu().numpy()
        assert np.all(np.isfinite(got)), name
        max_abs, rel = gh.errors(got, ref)
        assert max_abs <= max(max_abs_tol, float(np.abs(ref).max()) * ulp), (name, max_abs)
        assert rel <= (rel_tol if name == "O" else grad_tol), (name, rel)


# the last three run as windows of several problems per wavefront (N <= 32), with a ragged last window
SHAPES = [(2, 3, 197, 64), (3, 8, 77, 64), (1, 2, 300, 80), (1, 2, 785, 64), (7, 3, 12, 64), (5, 2, 5, 80), (9, 2, 32, 64)]


@pytest.mark.parametrize("f16,causal,packed", [c for c in itertools.product((False, True), repeat=3)])
@pytest.mark.parametrize("B,H,N,d", SHAPES)
def test_every_combination_matches_the_oracle(B, H, N, d, f16, causal, packed):
    w = si.small_workload(B, H, N, d, seed=9000 + N + d)
    x = si.make_inputs(w, fmt="f16" if f16 else "bf16")
    check(w, x, run_ex(w, x, f16, causal, packed), f16, causal)


def _same_bits(a, b):
    import torch
    for n in ("o", "dq", "dk", "dv"):
        assert torch.equal(a[n].contiguous().view(torch.int16), b[n].contiguous().view(torch.int16)), n
    assert torch.equal(a["lse"], b["lse"])


@pytest.mark.parametrize("B,H,N,d", [(2, 3, 197, 64), (1, 2, 300, 80), (2, 2, 100, 64)])
def test_general_entry_points_give_the_bits_of_the_specific_ones(B, H, N, d):
    w = si.small_workload(B, H, N, d, seed=9100 + N)
    x = si.make_inputs(w)
    _same_bits(run_ex(w, x, False, False, False), gh.run_hip(w, x))
    _same_bits(run_ex(w, x, False, True, False), gh.run_hip(w, x, causal=True))
    _same_bits(run_ex(w, x, False, False, True), gh.run_hip_packed(w, x))
    x16 = si.make_inputs(w, fmt="f16")
    _same_bits(run_ex(w, x16, True, False, False), gh.run_hip_f16(w, x16))
    # packing never changes the bits, whatever the format and the mask
    _same_bits(run_ex(w, x16, True, True, True), run_ex(w, x16, True, True, False))
    _same_bits(run_ex(w, x, False, True, True), run_ex(w, x, False, True, False))


def test_general_entry_points_reject_unknown_flags_and_mixed_packing():
    import ctypes
    import paper_2309_16669_amd as av
    lib = av.load_library()
    fake, null, f = ctypes.c_void_p(0x1000), ctypes.c_void_p(None), ctypes.c_float(0.125)
    assert lib.avion_attn_fwd_ex(fake, fake, fake, fake, fake, 1, 2, 64, 64, f, 8, None) == av.EINVAL
    assert lib.avion_attn_fwd_ex(fake, fake, null, fake, fake, 1, 2, 64, 64, f, av.FLAG_QKVPACKED, None) == av.EINVAL
    assert lib.avion_attn_bwd_ex(fake, null, null, fake, fake, fake, fake, fake, null, 1, 2, 64, 64, f,
                                 av.FLAG_QKVPACKED, fake, 1 << 20, None) == av.EINVAL
    assert lib.avion_attn_bwd_ex(fake, fake, fake, fake, fake, fake, fake, fake, fake, 1, 2, 64, 64, f, 16,
                                 fake, 1 << 20, None) == av.EINVAL


def test_autograd_front_end_covers_the_combinations():
    # loss = sum(O * W): fp16 + causal, and packed + causal, through torch.autograd
    import torch
    import oracle
    from paper_2309_16669_amd import autograd as ag
    w = si.small_workload(2, 3, 150, 64, seed=9200)
    x16 = si.make_inputs(w, fmt="f16")
    q, k, v = (_upload(x16[n], True).requires_grad_() for n in ("q", "k", "v"))
    dO = _upload(x16["dO"], True)
    o = ag.attention(q, k, v, w.scale, causal=True)
    (o.float() * dO.float()).sum().backward()
    check(w, x16, dict(o=o.detach(), lse=_lse_of(w, x16, True, True), dq=q.grad, dk=k.grad, dv=v.grad), True, True)
    x = si.make_inputs(w)
    qkv = _upload(np.stack([x["q"], x["k"], x["v"]], axis=2), False).requires_grad_()
    o = ag.attention_qkvpacked(qkv, w.scale, causal=True)
    (o.float() * _upload(x["dO"], False).float()).sum().backward()
    check(w, x, dict(o=o.detach(), lse=_lse_of(w, x, False, True), dq=qkv.grad[:, :, 0], dk=qkv.grad[:, :, 1],
                     dv=qkv.grad[:, :, 2]), False, True)
    # the classes keep the workspace of the backward per (device, stream): a second backward of theirs allocates none
    q2, k2, v2 = (_upload(x[n], False).requires_grad_() for n in ("q", "k", "v"))
    ag._Attention.apply(q2, k2, v2, w.scale, False).float().sum().backward()
    before = {k_: v_.data_ptr() for k_, v_ in ag._workspaces.items()}
    assert (q2.device, torch.cuda.current_stream().cuda_stream) in before
    ag._Attention.apply(q2, k2, v2, w.scale, False).float().sum().backward()
    assert {k_: v_.data_ptr() for k_, v_ in ag._workspaces.items()} == before
    # the native calls take theirs from torch's allocator and keep none
    held = torch.cuda.memory_allocated()
    for _ in range(2):
        g = torch.autograd.grad(ag.attention(q2, k2, v2, w.scale).float().sum(), [q2, k2, v2])
        del g
    assert torch.cuda.memory_allocated() == held


def _lse_of(w, x, f16, causal):
    """LSE of the forward (the autograd front end keeps it to itself), recomputed through the binding."""
    import torch
    import paper_2309_16669_amd as av
    q, k, v = (_upload(x[n], f16) for n in ("q", "k", "v"))
    o = torch.empty_like(q)
    lse = torch.empty((w.B, w.H, w.N), dtype=torch.float32, device="cuda")
    av.attn_fwd_ex(q, k, v, o, lse, w.scale, causal)
    torch.cuda.synchronize()
    return lse


# Launches small enough that several groups of wavefronts share a workgroup's rows (forward and backward): two to
# four groups over 64- and 128-row blocks, key tiles that do not divide among the groups, groups without a tile, and
# the first size beyond each line of the rule.  Bounds as everywhere in this file.
@pytest.mark.parametrize("B,H,N,d,f16,causal", [
    (1, 2, 65, 64, False, False), (1, 2, 65, 80, True, True), (1, 3, 129, 64, False, True), (1, 2, 161, 80, False, False),
    (2, 64, 128, 64, False, False), (2, 64, 129, 64, True, True), (1, 86, 321, 64, False, False), (1, 64, 385, 64, False, True),
    (1, 52, 321, 80, True, False), (1, 17, 961, 64, False, False), (1, 17, 1025, 64, False, True), (1, 16, 1025, 80, False, False),
    (1, 43, 321, 64, False, True), (1, 32, 1025, 64, True, False)])
def test_launches_split_into_groups_match_the_oracle(B, H, N, d, f16, causal):
    w = si.small_workload(B, H, N, d, seed=9300 + N + d)
    x = si.make_inputs(w, fmt="f16" if f16 else "bf16")
    check(w, x, run_ex(w, x, f16, causal, False), f16, causal)


# The same kernels with one group per workgroup, as every full-size launch runs them: at least 257 blocks of 128 rows.
@pytest.mark.parametrize("B,H,N,d,f16,causal,packed", [
    (2, 43, 321, 80, False, True, False), (2, 43, 321, 80, True, True, True), (1, 86, 321, 80, False, False, True),
    (2, 43, 321, 64, True, True, False), (1, 86, 321, 64, False, False, True)])
def test_launches_of_one_group_match_the_oracle(B, H, N, d, f16, causal, packed):
    w = si.small_workload(B, H, N, d, seed=9350 + N + d)
    x = si.make_inputs(w, fmt="f16" if f16 else "bf16")
    check(w, x, run_ex(w, x, f16, causal, packed), f16, causal)


# The running-maximum fallback of the forward in launches of one group (130 heads x 2 blocks).  Keys from 64 on are 16
# (fp16: 4) times larger and scale = 1, so later scores overflow the fixed reference by far.  Bounds: one unit in the last
# place of the largest reference value for O (near one-hot rows), fp32 rounding of LSE at its magnitude.
@pytest.mark.parametrize("d", [64, 80])
@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("causal", [False, True])
def test_the_running_maximum_fallback_in_launches_of_one_group(d, f16, causal):
    import oracle
    import torch
    import paper_2309_16669_amd as av
    w = si.small_workload(10, 13, 200, d, seed=9370 + d, scale=1.0)
    x = si.make_inputs(w, fmt="f16" if f16 else "bf16")
    widen, narrow = (si.f16_bits_to_f64, si.f32_to_f16_bits) if f16 else (si.bf16_bits_to_f64, si.f32_to_bf16_bits)
    x["k"][:, 64:] = narrow((widen(x["k"][:, 64:]) * (4 if f16 else 16)).astype(np.float32))     # exact: powers of two
    q, k, v = (_upload(x[n], f16) for n in ("q", "k", "v"))
    o = torch.full_like(q, float("nan"))
    lse = torch.full((w.B, w.H, w.N), float("nan"), dtype=torch.float32, device="cuda")
    av.attn_fwd_ex(q, k, v, o, lse, w.scale, causal)
    ro, rl = oracle.fwd_f64(*(widen(x[n]) for n in ("q", "k", "v")), w.scale, causal=causal)
    og, lg = o.double().cpu().numpy(), lse.double().cpu().numpy()
    assert np.all(np.isfinite(og)) and np.abs(og - ro).max() <= 2.0 ** (-10 if f16 else -7) * np.abs(ro).max()
    assert np.abs(lg - rl).max() <= 2e-6 * np.abs(rl).max() + 1e-3


# cuts (blocks of 32 rows, groups): (2, 2) twice, (3, 4), (2, 4) with the last and with the first group overflowing, (4, 4) likewise
@pytest.mark.parametrize("H,N,sink", [(2, 300, 250), (2, 300, 40), (17, 1025, 1000), (2, 900, 890), (2, 900, 40), (24, 1153, 1100), (24, 1153, 40)])
def test_a_group_whose_reference_overflows_redoes_the_block(H, N, sink):
    # keys from `sink` on carry scores far above the first 32 keys of their group: 2^15 in fp16 is passed
    w = si.small_workload(1, H, N, 64, seed=9400 + N, scale=1.0)
    x = si.make_inputs(w, fmt="f16")
    k = x["k"].copy()
    k[:, sink:sink + 4] = (si.f16_bits_to_f64(k[:, sink:sink + 4]) * 6).astype(np.float16).view(np.uint16)
    x["k"] = k
    out = run_ex(w, x, True, False, False)
    import oracle
    ro, rl = oracle.fwd_f64(*(si.f16_bits_to_f64(x[n]) for n in ("q", "k", "v")), w.scale)
    o, lse = out["o"].double().cpu().numpy(), out["lse"].double().cpu().numpy()
    # forward only: rows are near one-hot, and the rounding of O inside delta alone moves dQ beyond the general bound
    # (tests/test_tolerance_model.py).  O within one unit in the last place of its largest value, LSE in fp32.
    assert np.all(np.isfinite(o)) and np.abs(o - ro).max() <= 2.0 ** -10 * np.abs(ro).max()
    assert np.abs(lse - rl).max() <= 2e-6 * np.abs(rl).max() + 1e-3


# Whole heads per workgroup (64 channels, 33..256 tokens): both sides of every 32-token block, 64-row slot and instance
# boundary, one block to eight, more heads than compute units (workgroups that walk several heads, with heads left over),
# every format, mask and packing.  The two phases give the same bits (the workspace of the first feeds the second).
@pytest.mark.parametrize("B,H,N,f16,causal,packed", [
    (1, 3, 33, False, False, False), (2, 3, 64, True, True, True), (3, 2, 65, False, True, False), (1, 2, 95, True, False, True),
    (1, 5, 96, False, False, True), (2, 2, 97, False, True, False), (1, 3, 128, True, False, False), (1, 3, 129, False, True, True),
    (2, 2, 160, False, False, False), (1, 2, 161, True, True, False), (1, 3, 192, False, False, True), (1, 3, 193, False, True, False),
    (1, 2, 224, True, False, False), (1, 2, 225, False, False, True), (2, 1, 256, False, True, True), (1, 2, 257, False, False, False),
    (27, 10, 130, False, False, True), (3, 172, 196, False, True, False), (45, 6, 256, True, False, False), (33, 16, 49, False, False, False)])
def test_whole_heads_match_the_oracle_and_the_two_phases(B, H, N, f16, causal, packed):
    import torch
    import paper_2309_16669_amd as av
    w = si.small_workload(B, H, N, 64, seed=9500 + N)
    x = si.make_inputs(w, fmt="f16" if f16 else "bf16")
    out = run_ex(w, x, f16, causal, packed)
    check(w, x, out, f16, causal)
    if f16 or causal or packed:
        return                                            # the phases are bf16, unmasked and unpacked entry points
    q, k, v, dO = (_upload(x[n], False) for n in ("q", "k", "v", "dO"))
    dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(3))
    ws = torch.empty(av.attn_bwd_workspace_bytes(B, H, N, 64), dtype=torch.uint8, device="cuda").fill_(255)
    av.attn_bwd_dq(q, k, v, out["o"], out["lse"], dO, dq, w.scale, ws)
    av.attn_bwd_dkdv(q, k, v, out["lse"], dO, dk, dv, w.scale, ws)
    for n, t in (("dq", dq), ("dk", dk), ("dv", dv)):
        assert torch.equal(out[n].contiguous().view(torch.int16), t.view(torch.int16)), n


# Every instance of the whole-head kernel (blocks of 32 tokens 2..8, mask, format) at its shortest and its longest length
@pytest.mark.parametrize("blocks", range(2, 9))
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("f16", [False, True])
def test_every_whole_head_instance_at_both_ends_of_its_lengths(blocks, causal, f16):
    for N in (32 * blocks - 31, 32 * blocks):
        test_whole_heads_match_the_oracle_and_the_two_phases(1, 3, N, f16, causal, False)


# Cuts of small launches into blocks of 64, 96 and 128 rows with four groups (fwd_cut, bwd_cut): both sides of the lines in tiles, groups of
# unequal and of no tiles (11 tiles in four groups: 3, 3, 3, 2; 13: 4, 4, 4, 1), ragged last rows and keys
@pytest.mark.parametrize("B,H,N,f16,causal,packed", [
    (1, 3, 640, False, False, False), (1, 3, 641, True, False, True), (1, 2, 705, False, True, False), (1, 2, 833, False, False, True),
    (1, 2, 896, True, True, False), (1, 2, 897, False, False, False), (2, 2, 1281, False, True, True), (1, 12, 1409, False, False, False),
    (1, 16, 1025, True, False, True), (1, 15, 1024, False, True, False), (1, 12, 1569, False, True, False),
    # 128 rows: beyond the line of 96-row blocks
    (1, 16, 1568, False, False, False), (1, 24, 1153, True, True, True), (1, 32, 1000, False, True, False), (2, 16, 961, True, False, False)])
def test_small_launches_cut_into_four_groups(B, H, N, f16, causal, packed):
    w = si.small_workload(B, H, N, 64, seed=9700 + N)
    x = si.make_inputs(w, fmt="f16" if f16 else "bf16")
    check(w, x, run_ex(w, x, f16, causal, packed), f16, causal)


# Cuts of launches around one and two workgroups per compute unit (fwd_cut, bwd_cut): 96 rows in two groups within one per
# unit (forward from 6 tiles, backward from 5) and, forward, within two; causal 64 and 128 rows in two groups beyond one; both
# sides of the lines in tiles (7, 8, 10) and workgroups.  Ragged last rows and keys, groups with a tile less.
@pytest.mark.parametrize("B,H,N,d,f16,causal", [
    (1, 43, 385, 64, False, False), (1, 43, 385, 64, True, True), (1, 43, 385, 80, False, True), (2, 26, 321, 64, False, False),
    (1, 64, 384, 64, True, False), (1, 65, 385, 64, False, False), (2, 40, 448, 64, True, False), (1, 65, 512, 64, False, True),
    (1, 52, 600, 64, False, False), (1, 53, 610, 64, False, True), (1, 56, 640, 64, True, True), (1, 57, 577, 64, False, True),
    (1, 75, 577, 64, False, False), (2, 43, 620, 64, True, False), (3, 27, 639, 80, False, False),
    # backward in 96 rows that end half way through the last 64, at 5 tiles and 8
    (2, 30, 270, 64, False, False), (2, 30, 270, 64, True, True), (2, 30, 270, 80, True, False), (2, 30, 270, 80, False, True),
    (1, 48, 480, 64, False, False), (1, 48, 480, 64, False, True)])
def test_cuts_around_one_and_two_workgroups_per_compute_unit(B, H, N, d, f16, causal):
    import torch
    w = si.small_workload(B, H, N, d, seed=9750 + N + d)
    gen = torch.Generator(device="cuda").manual_seed(N)
    dt = torch.float16 if f16 else torch.bfloat16
    x = {n: torch.randn(B, N, H, d, device="cuda", generator=gen).to(dt).view(torch.int16).cpu().numpy().view(np.uint16)
         for n in ("q", "k", "v", "dO")}
    out = run_ex(w, x, f16, causal, False)
    for n in ("o", "lse", "dq", "dk", "dv"):
        assert bool(torch.isfinite(out[n]).all()), n
    if causal:
        check(w, x, out, f16, causal)
    else:
        (gh.check_f16_against_oracle if f16 else gh.check_against_oracle)(w, x, out, [(0, 0), (B // 2, H // 2), (B - 1, H - 1)])


# dK and dV of the pipelined form (by_flow): 64, 96 and 128 rows, both sides of the lines in tiles (8, 15), one tile per group to
# many, groups with a tile less (odd numbers of tiles: its zero rows must add nothing), last tiles of one unit and two, keys past the end
@pytest.mark.parametrize("B,H,N,f16,packed", [
    (1, 3, 257, False, False), (2, 2, 320, True, True), (1, 2, 385, False, True), (1, 3, 833, True, False), (1, 2, 1025, False, False),
    (1, 28, 449, False, False), (1, 28, 448, True, False), (1, 30, 481, True, True), (1, 16, 1030, False, True), (1, 9, 1569, False, False),
    (1, 30, 897, False, False), (1, 29, 896, False, True), (1, 20, 1250, True, False), (1, 24, 1024, False, False)])
def test_pipelined_dk_dv_of_small_launches(B, H, N, f16, packed):
    w = si.small_workload(B, H, N, 64, seed=9770 + N)
    x = si.make_inputs(w, fmt="f16" if f16 else "bf16")
    check(w, x, run_ex(w, x, f16, False, packed), f16, False)


# The per-query scalars that dQ leaves in the workspace for dK and dV, LSE * log2(e) and -delta, reach to the end of the last 64 queries with
# +inf and 0, whatever block of rows ends there: 64, 96 (also half way through the last 64) and 128 rows, two groups, four and one, and pairs.
@pytest.mark.parametrize("B,H,N,d", [(1, 3, 300, 64), (1, 2, 1025, 64), (2, 30, 270, 64), (2, 30, 270, 80), (1, 48, 480, 64), (1, 16, 1030, 64),
                                     (1, 16, 1025, 80), (1, 32, 785, 64), (1, 86, 321, 64), (1, 51, 1025, 64), (1, 51, 1060, 64), (2, 3, 100, 64)])
def test_the_scalars_left_for_dk_and_dv_reach_to_the_end_of_the_last_tile(B, H, N, d):
    import math
    import torch
    import paper_2309_16669_amd as av
    gen = torch.Generator(device="cuda").manual_seed(N + d)
    q, k, v, dO = (torch.randn(B, N, H, d, device="cuda", generator=gen).bfloat16() for _ in range(4))
    o, dq, lse = torch.empty_like(q), torch.empty_like(q), torch.empty(B, H, N, device="cuda")
    ws = torch.empty(av.attn_bwd_workspace_bytes(B, H, N, d), dtype=torch.uint8, device="cuda").fill_(255)
    av.attn_fwd(q, k, v, o, lse, 0.125)
    av.attn_bwd_dq(q, k, v, o, lse, dO, dq, 0.125, ws)
    npad = (N + 63) // 64 * 64
    got = ws[:B * H * 2 * npad * 4].view(torch.float32).view(B, H, 2, npad)
    assert bool((got[:, :, 0, N:] == math.inf).all()) and bool((got[:, :, 1, N:] == 0).all())
    delta = (o.double() * dO.double()).sum(-1).transpose(1, 2)
    # one rounding of the product; delta: d additions in fp32 of products of about 0.1
    assert float((got[:, :, 0, :N].double() - lse.double() * math.log2(math.e)).abs().max()) <= 2.0 ** -22 * float(lse.abs().max()) * 1.5
    assert float((got[:, :, 1, :N].double() + delta).abs().max()) <= d * 2.0 ** -24 * float((o.double() * dO.double()).abs().sum(-1).max())


# Units of 32 queries that lie wholly past the end, in tiles past the end (an odd number of tiles in two groups) and in half tiles, are
# left out: a key with an infinite component that no query sees (weights of exactly 0, as for a finite one far below the others) gets dK and
# dV of 0 and changes nothing of the other keys'.  64, 96 and 128 rows, pipelined; then the other kernels.
@pytest.mark.parametrize("H,N,f16", [(3, 320, False), (3, 352, True), (30, 576, True), (30, 544, False), (34, 480, False), (30, 960, False),
                                     (28, 992, True), (48, 480, True), (65, 448, False), (90, 640, True), (3, 160, False)])
def test_units_past_the_end_leave_keys_with_infinite_components_alone(H, N, f16):
    import torch
    import paper_2309_16669_amd as av
    dt = torch.float16 if f16 else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(N + H)
    q, k, v, dO = (torch.randn(1, N, H, 64, device="cuda", generator=gen).to(dt) for _ in range(4))
    q[..., 0] = 1.0
    ws = torch.empty(av.attn_bwd_workspace_bytes(1, H, N, 64), dtype=torch.uint8, device="cuda").fill_(255)
    outs = []
    for low in (-30000.0, float("-inf")):
        k[:, [40, N - 3], :, 0] = low
        o, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
        lse = torch.full((1, H, N), float("nan"), device="cuda")
        av.attn_fwd_ex(q, k, v, o, lse, 0.125, False)
        av.attn_bwd_ex(q, k, v, o, lse, dO, dq, dk, dv, 0.125, ws, False)
        torch.cuda.synchronize()
        outs.append((o, lse, dq[..., 1:], dk, dv))      # (dQ of channel 0 is a product of that component with 0)
    for name, a, b in zip(("o", "lse", "dq", "dk", "dv"), *outs):
        assert (int((~torch.isfinite(b)).sum()), torch.equal(a, b)) == (0, True), name
    assert [int(t[:, [40, N - 3]].count_nonzero()) for t in outs[1][3:]] == [0, 0]


# The running-maximum fallback where the last and where the first of two groups of 96 and of 128 rows overflows
@pytest.mark.parametrize("H,N,sink", [(43, 385, 370), (43, 385, 40), (50, 600, 590), (50, 600, 40), (70, 448, 440)])
def test_an_overflowing_group_of_two_redoes_the_block(H, N, sink):
    test_a_group_whose_reference_overflows_redoes_the_block(H, N, sink)


# dQ in two blocks per wavefront (by_pair): last workgroups of one and two blocks (shared by four and two wavefronts) to eight,
# last tiles of one unit and two, ragged and full, both layouts (packed: Q, K, V, dQ rows three times as far apart as those of O,
# dO), one round of workgroups and several.  Oracle on a first, a middle and a last head; dK, dV read the scalars it leaves.
# (The first six rows are just beyond the line in workgroups.)
@pytest.mark.parametrize("B,H,N,f16,packed", [
    (31, 4, 1025, False, False), (30, 4, 1088, False, False), (39, 3, 1119, True, False), (55, 2, 1153, False, False),
    (35, 3, 1248, False, False), (3, 32, 1300, True, False),
    (16, 4, 1000, False, False), (16, 4, 1024, True, True), (17, 3, 1060, False, True), (17, 3, 1060, True, False),
    (17, 3, 1119, True, False), (17, 3, 1124, False, True), (25, 2, 1153, False, False), (17, 3, 1185, True, True),
    (17, 3, 1248, False, False), (14, 3, 1300, True, True), (14, 3, 1312, False, False), (61, 3, 1200, False, True)])
def test_dq_in_pairs_of_blocks(B, H, N, f16, packed):
    import torch
    w = si.small_workload(B, H, N, 64, seed=9800 + N)
    gen = torch.Generator(device="cuda").manual_seed(N)
    dt = torch.float16 if f16 else torch.bfloat16
    bits = lambda: torch.randn(B, N, H, 64, device="cuda", generator=gen).to(dt).view(torch.int16).cpu().numpy().view(np.uint16)
    x = {n: bits() for n in ("q", "k", "v", "dO")}
    out = run_ex(w, x, f16, False, packed)
    for n in ("dq", "dk", "dv"):
        assert bool(torch.isfinite(out[n]).all()), n
    slices = [(0, 0), (B // 2, H // 2), (B - 1, H - 1)]
    (gh.check_f16_against_oracle if f16 else gh.check_against_oracle)(w, x, out, slices)


# The shortest sequences that take it, with one or two and with several workgroups per compute unit, and the ones below them
@pytest.mark.parametrize("B,H,N,f16,packed", [
    (16, 5, 500, False, False), (16, 5, 499, True, False), (17, 5, 540, True, True), (80, 3, 700, False, False), (80, 3, 699, False, True),
    (120, 2, 736, True, False)])
def test_dq_in_pairs_of_blocks_at_its_shortest(B, H, N, f16, packed):
    test_dq_in_pairs_of_blocks(B, H, N, f16, packed)


# On the other side of by_pair's lines dQ is avion_dq_kernel's, whose bits do not depend on the other heads of the launch; the
# pair form adds up a last block that wavefronts share in another order.  Heads whose short last workgroup would open another
# round have the former's bits (those of a launch that fills the chip badly in blocks too), heads within the lines have not.
@pytest.mark.parametrize("heads,more,N,paired", [(52, 78, 1050, False), (44, 66, 1300, False), (33, 50, 1800, False),
                                                 (68, 80, 1800, False), (42, 66, 1300, True), (51, 78, 1060, True)])
def test_short_last_workgroups_do_not_open_another_round(heads, more, N, paired):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(N + heads)
    q, k, v, dO = (torch.randn(more, N, 1, 64, device="cuda", generator=gen).bfloat16() for _ in range(4))
    # one forward for both launches: its own cut of the rows is not what is looked at
    import paper_2309_16669_amd as av
    o, lse = torch.empty_like(q), torch.empty(more, 1, N, device="cuda")
    av.attn_fwd_ex(q, k, v, o, lse, 0.125, False)
    got = [_dq_of(*(t[:h] for t in (q, k, v, o, lse, dO))) for h in (heads, more)]
    assert torch.equal(got[0].view(torch.int16), got[1][:heads].view(torch.int16)) != paired


def _dq_of(q, k, v, o, lse, dO):
    import torch
    import paper_2309_16669_amd as av
    B, N, H, d = q.shape
    dq = torch.full_like(q, float("nan"))
    ws = torch.empty(av.attn_bwd_workspace_bytes(B, H, N, d), dtype=torch.uint8, device="cuda").fill_(255)
    av.attn_bwd_dq(q, k, v, o, lse, dO, dq, 0.125, ws)
    torch.cuda.synchronize()
    return dq
