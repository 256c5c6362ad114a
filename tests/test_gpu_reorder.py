"""GPU parity of the spatio-temporal token reordering: the row gather/scatter kernels and
the reordered attention entry point, called through the C ABI, against the CPU oracle.

* Row moves are data movement only, so they must match the oracle's numpy gather/scatter
  bit for bit (16-byte and 4-byte paths, ragged sizes, out-of-range index entries).
* Reordered attention is compared in the reordered frame: the oracle runs the rule on
  inputs permuted by ``oracle.reorder`` (teacher-forced on the GPU's reordered mask), and
  the GPU output, returned in the original query order, is permuted the same way before
  the comparison.  With identity maps the entry point must reproduce the plain call bit
  for bit.
"""

import math
import sys

import numpy as np
import pytest

import oracle
from oracle.reorder import block_order, gather_rows, scatter_rows
from synth import make_random_qkv, make_video_qkv

from _parity import (DeviceRun, RULE_NAMES, TILE_K, TILE_Q, assert_parity, compare,
                     expected_stats_from_mask, from_device_bf16, run_gpu, to_device)

pytestmark = pytest.mark.gpu

SCALE = 1.0 / math.sqrt(128)


@pytest.fixture(scope="module", autouse=True)
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_16317_amd as dsa

    dsa.lib()
    return torch


def announce(msg):
    print(f"\n[case] {msg}", flush=True)
    sys.stdout.flush()


def dev_index(perm):
    import torch

    return torch.from_numpy(np.ascontiguousarray(perm, dtype=np.int32)).cuda()


# ---- row moves ------------------------------------------------------------------------

@pytest.mark.parametrize("grid,block,B,H", [((2, 32, 32), (2, 8, 8), 1, 2),
                                            ((3, 10, 13), (1, 8, 8), 2, 3),
                                            ((5, 7, 9), (2, 3, 4), 1, 1)])
def test_gather_scatter_bf16_rows_bit_exact(grid, block, B, H):
    import torch
    import paper_2606_16317_amd as dsa

    announce(f"gather/scatter bf16 grid={grid} block={block} B={B} H={H}")
    N = int(np.prod(grid))
    x, _, _ = make_random_qkv(B, H, N, 128, seed=N)
    perm = block_order(grid, block)
    xd = to_device(x)
    idx = dev_index(perm)
    g = dsa.dsattn_gather_rows(xd, idx)
    s = dsa.dsattn_scatter_rows(xd, idx)
    torch.cuda.synchronize()
    assert np.array_equal(from_device_bf16(g), gather_rows(x, perm))
    assert np.array_equal(from_device_bf16(s), scatter_rows(x, perm))


@pytest.mark.parametrize("width", [1, 3, 4, 5])
def test_gather_scatter_narrow_rows_bit_exact(width):
    """Rows of 4, 12, 16 and 20 bytes; 16-byte rows are given a 4-byte-misaligned source so
    that the word-per-lane path is taken."""
    import torch
    import paper_2606_16317_amd as dsa

    announce(f"gather/scatter float rows width={width}")
    rng = np.random.default_rng(width)
    BH, N = 3, 777
    x = rng.standard_normal((BH, N, width)).astype(np.float32)
    perm = rng.permutation(N)
    big = torch.zeros(BH * N * width + 1, dtype=torch.float32, device="cuda")
    xd = big[1:].view(BH, N, width)              # starts 4 bytes past a 256-byte boundary
    xd.copy_(torch.from_numpy(x))
    idx = dev_index(perm)
    g = dsa.dsattn_gather_rows(xd, idx)
    s = dsa.dsattn_scatter_rows(xd, idx)
    torch.cuda.synchronize()
    assert np.array_equal(g.cpu().numpy(), gather_rows(x, perm))
    assert np.array_equal(s.cpu().numpy(), scatter_rows(x, perm))


def test_out_of_range_index_entries_touch_nothing():
    import torch
    import paper_2606_16317_amd as dsa

    announce("gather/scatter with out-of-range index entries")
    BH, N = 2, 300
    x, _, _ = make_random_qkv(1, BH, N, 128, seed=5)
    index = np.arange(N, dtype=np.int64)[::-1].copy()
    bad = [0, 17, 299]
    index[0], index[17], index[299] = -1, N, 2**31 - 1
    xd = to_device(x)
    idx = dev_index(index)
    g = dsa.dsattn_gather_rows(xd, idx)
    sentinel = torch.full_like(xd, 3.0)
    s = dsa.dsattn_scatter_rows(xd, idx, dst=sentinel)
    torch.cuda.synchronize()
    gh, sh = from_device_bf16(g), from_device_bf16(s)
    ok = np.setdiff1d(np.arange(N), bad)
    assert np.array_equal(gh[..., ok, :], x[..., index[ok], :])
    assert not gh[..., bad, :].any()                           # zero rows
    assert np.array_equal(sh[..., index[ok], :], x[..., ok, :])
    three = np.uint16(0x4040)                                   # bf16 bits of 3.0
    untouched = np.setdiff1d(np.arange(N), index[ok])
    assert (sh[..., untouched, :] == three).all()               # dropped rows


# ---- reordered attention ----------------------------------------------------------------

def run_reordered(qd, kd, vd, rule, param, q_perm, kv_perm):
    import torch
    import paper_2606_16317_amd as dsa

    B, H, N, d = qd.shape
    n_qt, n_kt = -(-N // TILE_Q), -(-N // TILE_K)
    o = torch.empty_like(qd)
    stats = torch.full((B * H * 4,), -7, dtype=torch.int64, device="cuda")
    mask = torch.full((B * H * n_qt * n_kt,), 7, dtype=torch.uint8, device="cuda")
    lse = torch.full((B * H * N,), float("nan"), dtype=torch.float32, device="cuda")
    dsa.dsattn_attn_fwd_reordered(RULE_NAMES[rule], param, qd, kd, vd, dev_index(q_perm),
                                  dev_index(kv_perm), o, scale=SCALE, stats_out=stats,
                                  mask_out=mask, lse_out=lse)
    torch.cuda.synchronize()
    return DeviceRun(from_device_bf16(o), mask.cpu().numpy().reshape(B, H, n_qt, n_kt),
                  lse.cpu().numpy().reshape(B, H, N), stats.cpu().numpy().reshape(B, H, 4))


REORDER_CASES = [
    # grid, q block, kv block, a, rule, param
    ((2, 32, 32), (2, 8, 8), (1, 8, 8), 6.0, "dynsparse_lambda", -6.0),
    ((2, 32, 32), (2, 8, 8), (1, 8, 8), 6.0, "dynsparse_lambda", -8.0),
    ((2, 32, 32), (2, 8, 8), (1, 8, 8), 6.0, "dense", 0.0),
    ((2, 32, 32), (1, 8, 16), (1, 8, 16), 4.0, "blasst", 1e-2),
    ((3, 21, 26), (2, 8, 8), (1, 8, 8), 5.0, "dynsparse_recall", 0.95),
    ((3, 21, 26), (2, 8, 8), (1, 8, 8), 5.0, "dynsparse_lambda", -7.0),
]


@pytest.mark.parametrize("grid,qb,kb,a,rule,param", REORDER_CASES)
def test_reordered_attention_matches_oracle(grid, qb, kb, a, rule, param):
    announce(f"reordered {rule}={param} grid={grid} qb={qb} kb={kb} a={a}")
    q, k, v, _ = make_video_qkv(1, 2, grid, a, a, True, 11)
    N = q.shape[2]
    qp, kp = block_order(grid, qb), block_order(grid, kb)
    g = run_reordered(to_device(q), to_device(k), to_device(v), rule, param, qp, kp)
    # the same problem in the reordered frame, on the oracle side
    qr, kr, vr = gather_rows(q, qp), gather_rows(k, kp), gather_rows(v, kp)
    g_frame = DeviceRun(gather_rows(g.o, qp), g.mask, gather_rows(g.lse[..., None], qp)[..., 0],
                     g.stats)
    rep = compare(qr, kr, vr, g_frame, rule, param, SCALE)
    print(f"[case] {rep}", flush=True)
    assert_parity(rep)
    assert np.array_equal(g.stats, expected_stats_from_mask(g.mask, N))
    assert (g.mask[..., 0] == 0).all()


def test_identity_maps_reproduce_the_plain_call_bit_for_bit():
    announce("reordered with identity maps vs plain call")
    grid = (3, 21, 26)
    q, k, v, _ = make_video_qkv(1, 3, grid, 5.0, 5.0, True, 12)
    N = q.shape[2]
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    ident = np.arange(N)
    for rule, param in (("dynsparse_lambda", -7.0), ("dense", 0.0)):
        r = run_reordered(qd, kd, vd, rule, param, ident, ident)
        p = run_gpu(qd, kd, vd, rule, param, SCALE)
        assert np.array_equal(r.o, p.o)
        assert np.array_equal(r.mask, p.mask)
        assert np.array_equal(r.stats, p.stats)
        assert np.array_equal(r.lse.view(np.uint32), p.lse.view(np.uint32))


@pytest.mark.parametrize("rule,param,tile_q,tile_k,order,N", [
    ("dense", 0.0, 128, 64, 0, 129), ("dynsparse_lambda", -4.0, 32, 64, 1, 1000),
    ("dynsparse_recall", 0.95, 128, 128, 0, 640), ("blasst", 0.05, 128, 32, 0, 65),
    ("dynsparse_lambda", -4.0, 128, 128, 1, 777), ("mask", 0.0, 32, 64, 0, 1000),
    ("mask", 0.0, 128, 128, 0, 300)])
def test_reordered_call_equals_gathers_plain_call_and_scatters(rule, param, tile_q, tile_k,
                                                               order, N):
    """Queries read and outputs written in place through q_index have the bits of moving
    q, k and v first, the plain call, and moving o and the LSE back; entries outside the
    sequence stand for a zero query and leave their output rows alone."""
    check_in_place(rule, param, tile_q, tile_k, order, N, 2, 2)


@pytest.mark.parametrize("tile_q,tile_k", [(32, 64), (128, 128)])
@pytest.mark.parametrize("B,H,N", [(2, 52, 600), (1, 14, 37 * 128 - 5), (1, 2, 257 * 128 + 1)])
def test_reordered_mask_reuse_with_interleaved_heads(B, H, N, tile_q, tile_k):
    """The same above 512 workgroups, where a reused mask's launch interleaves its heads: the
    gather map belongs to the tile, not to the place in the grid."""
    check_in_place("mask", 0.0, tile_q, tile_k, 0, N, B, H)


def check_in_place(rule, param, tile_q, tile_k, order, N, B, H):
    import ctypes

    import torch
    import paper_2606_16317_amd as dsa

    announce(f"reordered in place {rule}={param} {tile_q}x{tile_k} B={B} H={H} N={N}")
    qd, kd, vd = (to_device(x) for x in make_random_qkv(B, H, N, 128, N, q_std=2.0, k_std=2.0))
    rng = np.random.default_rng(N)
    qi, ki = rng.permutation(N), rng.permutation(N)
    qi[5], qi[N - 1], qi[N // 2] = -1, N, 2 ** 31 - 1
    ki[3] = -7
    qi, ki = dev_index(qi), dev_index(ki)
    n_qu, n_kd = -(-N // tile_q), -(-N // tile_k)
    mask_in = torch.from_numpy((rng.random((B, H, n_qu, n_kd)) < 0.6).astype(np.uint8)).cuda()
    rule_id = dsa.RULE_MASK if rule == "mask" else RULE_NAMES[rule]

    def outputs():
        return {"stats_out": torch.full((B * H * 4,), -7, dtype=torch.int64, device="cuda"),
                "mask_out": torch.full((B * H * n_qu * n_kd,), 7, dtype=torch.uint8,
                                       device="cuda"),
                "lse_out": torch.full((B, H, N, 1), 9.0, dtype=torch.float32, device="cuda")}

    plain, o_plain, o_back = outputs(), torch.empty_like(qd), torch.full_like(qd, 3.0)
    dsa.dsattn_attn_fwd_ex(rule_id, param, *(dsa.dsattn_gather_rows(x, i) for x, i in
                                             ((qd, qi), (kd, ki), (vd, ki))), o_plain,
                           tile_q=tile_q, tile_k=tile_k, key_order=order, mask_in=mask_in, **plain)
    dsa.dsattn_scatter_rows(o_plain, qi, o_back)
    lse_back = torch.full((B, H, N, 1), 9.0, dtype=torch.float32, device="cuda")
    dsa.dsattn_scatter_rows(plain["lse_out"], qi, lse_back)

    got, o = outputs(), torch.full_like(qd, 3.0)
    ws = torch.empty(dsa.dsattn_reordered_workspace_bytes(B, H, N, 128, True), dtype=torch.uint8,
                     device="cuda")
    a = dsa.DsAttnArgs(rule_id, param, qd.data_ptr(), kd.data_ptr(), vd.data_ptr(), o.data_ptr(),
                       B, H, N, 128, SCALE, tile_q, tile_k,
                       torch.cuda.current_stream().cuda_stream, got["stats_out"].data_ptr(),
                       got["mask_out"].data_ptr(), got["lse_out"].data_ptr(), order,
                       mask_in.data_ptr())
    rc = dsa.lib().dsattn_attn_fwd_reordered(ctypes.byref(a), qi.data_ptr(), ki.data_ptr(),
                                             ws.data_ptr(), ws.numel())
    assert rc == 0, dsa.last_error()
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), o_back.view(torch.int16))
    assert torch.equal(got["lse_out"], lse_back)
    assert torch.equal(got["stats_out"], plain["stats_out"])
    assert torch.equal(got["mask_out"], plain["mask_out"])


def test_reordering_raises_sparsity_on_video_inputs():
    """Blocked order gathers spatial neighbours into tiles: on these video-shaped inputs the
    reordered run skips more tiles than the row-major one at the same lambda (the oracle
    gives 0.028 against 0.000 on this seed)."""
    announce("reordered sparsity >= row-major sparsity")
    grid = (4, 24, 32)
    q, k, v, _ = make_video_qkv(1, 4, grid, 2.0, 3.0, True, 13)
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    plain = run_gpu(qd, kd, vd, "dynsparse_lambda", -8.0, SCALE)
    r = run_reordered(qd, kd, vd, "dynsparse_lambda", -8.0, block_order(grid, (2, 8, 8)),
                      block_order(grid, (1, 8, 8)))
    print(f"[case] sparsity row-major {plain.mask.mean():.3f} reordered {r.mask.mean():.3f}",
          flush=True)
    assert r.mask.mean() > plain.mask.mean()


@pytest.mark.slow
def test_reordered_wan720p_sampled():
    """The 720p layer regrouped into (2, 8, 8) query and (1, 8, 8) key/value blocks, in
    the launch shape the reorder sweep times: sampled query tiles of three heads against
    the oracle in the reordered frame."""
    from synth import WORKLOADS, workload_inputs

    from _parity import sample_tiles

    w = WORKLOADS["wan720p"]
    announce(f"generate {w.describe()}")
    q, k, v, _ = workload_inputs("wan720p")
    qp, kp = block_order(w.grid, (2, 8, 8)), block_order(w.grid, (1, 8, 8))
    dev = (to_device(q), to_device(k), to_device(v))
    qr, kr, vr = gather_rows(q, qp), gather_rows(k, kp), gather_rows(v, kp)
    tiles = sample_tiles(w.B, w.H, w.N, per_head=3, heads=[(0, 2), (0, 21), (0, 39)], seed=7)
    for rule, param in [("dynsparse_lambda", -8.0), ("dynsparse_recall", 0.95)]:
        announce(f"reordered wan720p rule={rule} param={param} tiles={len(tiles)}")
        g = run_reordered(*dev, rule, param, qp, kp)
        g_frame = DeviceRun(gather_rows(g.o, qp), g.mask,
                            gather_rows(g.lse[..., None], qp)[..., 0], g.stats)
        rep = compare(qr, kr, vr, g_frame, rule, param, SCALE, tiles=tiles)
        print(rep, f"full-run tile sparsity={float(g.mask.mean()):.4f}", flush=True)
        assert_parity(rep)
        assert np.array_equal(g.stats, expected_stats_from_mask(g.mask, w.N))


@pytest.mark.parametrize("lse", [False, True])
def test_side_stream_call_keeps_its_own_workspace(lse):
    """A call on a side stream without a workspace: memory that the current stream allocates
    and overwrites right after the call returns, with the side stream still busy ahead of the
    call's kernels, is not the call's scratch."""
    import torch
    import paper_2606_16317_amd as dsa

    announce(f"reordered on a side stream lse={lse}")
    B, H, grid = 1, 2, (3, 21, 26)
    q, k, v, _ = make_video_qkv(B, H, grid, 5.0, 5.0, True, 13)
    N = q.shape[2]
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    qi, ki = dev_index(block_order(grid, (2, 8, 8))), dev_index(block_order(grid, (1, 8, 8)))
    need = dsa.dsattn_reordered_workspace_bytes(B, H, N, 128, lse)

    def call(o, ls, **more):
        dsa.dsattn_attn_fwd_reordered(dsa.RULE_DYNSPARSE_LAMBDA, -6.0, qd, kd, vd, qi, ki, o,
                                      scale=SCALE, lse_out=ls if lse else None, **more)

    want, want_ls = torch.empty_like(qd), torch.zeros(B, H, N, device="cuda")
    call(want, want_ls, workspace=torch.empty(need, dtype=torch.uint8, device="cuda"))
    o, ls = torch.zeros_like(qd), torch.zeros(B, H, N, device="cuda")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for _ in range(3):
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)                 # some milliseconds
        call(o, ls, stream=side)
        grabbed = [torch.empty(need, dtype=torch.uint8, device="cuda").fill_(0x7f)
                   for _ in range(4)]
        torch.cuda.synchronize()
        del grabbed
        assert torch.equal(o.view(torch.int16), want.view(torch.int16))
        assert torch.equal(ls, want_ls)
