"""Launches that interleave their heads (of mask reuse and MX-FP8, above 512 workgroups) against
the same heads called a few at a time, which run in grid order: workgroups do not depend on
each other, so every output is the same bit for bit, whatever the order."""

import pytest

pytestmark = pytest.mark.gpu

# (heads, tokens): groups of 8, 4, 2 and 1 with ragged last tiles; one query tile a head;
# a leftover single head; tile counts that the group size does not divide.
SHAPES = [(15, 36 * 128 - 5), (43, 13 * 128 - 100), (130, 4 * 128), (520, 100), (2, 257 * 128 + 1)]
# Groups of 8, 4 and 2 and leftover single heads above 320 query tiles, where a reused mask's
# launch interleaves whatever it reports.
MASK_SHAPES = SHAPES + [(14, 37 * 128 - 5), (3, 321 * 128 - 70), (5, 320 * 128 + 1)]
# MX-FP8 rules interleave up to 64 query tiles, and up to 256 if the last round of 512 workgroups
# is at least 0.8 full: the same groups on both sides of these lines.
MXFP8_SHAPES = SHAPES + [(15, 64 * 128 - 5), (15, 65 * 128 - 5), (11, 64 * 128 + 1),
                         (8, 115 * 128 - 9), (5, 193 * 128 + 1), (4, 256 * 128), (2, 300 * 128)]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_16317_amd as dsa

    dsa.lib()
    return torch


def outputs(torch, heads, n, tile_q, tile_k):
    return {"lse_out": torch.zeros(1, heads, n, device="cuda"),
            "stats_out": torch.zeros(1, heads, 4, dtype=torch.int64, device="cuda"),
            "mask_out": torch.full((1, heads, -(-n // tile_q), -(-n // tile_k)), 9,
                                   dtype=torch.uint8, device="cuda")}


def check(torch, call, heads, n, tile_q, tile_k):
    """`call(heads slice, outputs)` over all heads and over runs that stay in grid order."""
    whole = outputs(torch, heads, n, tile_q, tile_k)
    o = call(slice(0, heads), whole)
    step = max(1, 512 // -(-n // 128))
    for h in range(0, heads, step):
        part = slice(h, min(heads, h + step))
        got = outputs(torch, part.stop - h, n, tile_q, tile_k)
        assert torch.equal(call(part, got).view(torch.int16), o[:, part].view(torch.int16))
        for name, x in got.items():
            assert torch.equal(x, whole[name][:, part]), name


@pytest.mark.parametrize("heads,n", MASK_SHAPES)
@pytest.mark.parametrize("tile_q,tile_k", [(128, 64), (32, 128), (32, 64)])
def test_mask_reuse(gpu, heads, n, tile_q, tile_k):
    import paper_2606_16317_amd as dsa

    torch = gpu
    print(f"\n[case] mask heads={heads} n={n} tile_q={tile_q} tile_k={tile_k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(heads)
    q, k, v = (torch.randn(1, heads, n, 128, generator=g, device="cuda").to(torch.bfloat16)
               for _ in range(3))
    mask = (torch.rand(1, heads, -(-n // tile_q), -(-n // tile_k), generator=g,
                       device="cuda") < 0.8).to(torch.uint8)

    def call(part, out):
        qp, kp, vp, mp = (x[:, part].contiguous() for x in (q, k, v, mask))
        return dsa.dsattn_attn_fwd_ex(dsa.RULE_MASK, 0.0, qp, kp, vp, mask_in=mp, tile_q=tile_q,
                                      tile_k=tile_k, **out)

    check(torch, call, heads, n, tile_q, tile_k)


@pytest.mark.parametrize("heads,n", MXFP8_SHAPES)
@pytest.mark.parametrize("rule,param,tile_q,tile_k", [
    ("RULE_DYNSPARSE_LAMBDA", -7.5, 128, 64), ("RULE_DYNSPARSE_LAMBDA", -8.0, 32, 32),
    ("RULE_BLASST", 1e-2, 128, 128), ("RULE_DENSE", 0.0, 128, 64)])
def test_mxfp8(gpu, heads, n, rule, param, tile_q, tile_k):
    import paper_2606_16317_amd as dsa

    torch = gpu
    print(f"\n[case] mxfp8 heads={heads} n={n} {rule} {tile_q}x{tile_k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(heads)
    q, k, v = (torch.randn(1, heads, n, 128, generator=g, device="cuda").mul(s).to(torch.bfloat16)
               for s in (2.0, 2.0, 1.0))
    q8, qs = dsa.dsattn_quantize_mxfp8(q)
    k8, ks = dsa.dsattn_quantize_mxfp8(k)

    def call(part, out):
        a = [x[:, part].contiguous() for x in (q8, qs, k8, ks, v)]
        return dsa.dsattn_attn_fwd_mxfp8(getattr(dsa, rule), param, *a, tile_q=tile_q,
                                         tile_k=tile_k, **out)

    check(torch, call, heads, n, tile_q, tile_k)
