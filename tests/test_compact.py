"""GPU: the compact path (GDN in bf16: calls with more walks than half the compute
units, and segmented calls) against the general path.

A batch of short sequences with enough value heads takes the compact path, in
each of its three walks (four waves on one column tile or two, up to 256 and 512
tiles; beyond them a whole head per workgroup); the same sequences one by one
(few walks, one segment) take the affine factors.
Both round the operands of every product to bf16 and accumulate in fp32, and
each is held to 2e-2 of the fp64 oracle elsewhere, so they agree to the sum.
In the 2-norm they are held closer: a value passes about eight roundings to 8 bits
on either side, of 2^-9 / sqrt(3) each, which add up to 4.5e-3 for the difference;
three times that is allowed (4.4e-3 seen, 6.9e-3 for the outputs of single tokens).
Lengths sit on the edges of 16-token tiles and 64-token chunks."""

import numpy as np
import pytest

from gpu_harness import TOL, check_against_oracle, oracle_threads, relerr, run_gpu, to_device
from paper_2609_32114_amd.inputs import Inputs, make_case

pytestmark = pytest.mark.gpu

LENS = (1, 15, 16, 17, 63, 64, 65, 0, 128, 129, 193)


def _alone(inp, n):
    a, b = int(inp.cu_seqlens[n]), int(inp.cu_seqlens[n + 1])
    cut = lambda x: np.ascontiguousarray(x[a:b])  # noqa: E731
    return Inputs(kind=inp.kind, dtype=inp.dtype, q=cut(inp.q), k=cut(inp.k), v=cut(inp.v), g=cut(inp.g),
                  beta=cut(inp.beta), s0=None if inp.s0 is None else inp.s0[n:n + 1],
                  cu_seqlens=np.array([0, b - a], dtype=np.int32), scale=inp.scale, meta=dict(inp.meta))


def _close(got, ref, what):
    d = np.max(np.abs(got - ref)) / max(np.max(np.abs(ref)), 1e-30)
    assert np.all(np.isfinite(got)) and d <= 4e-2, f"{what}: {d:.3e}"
    r = np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-30)
    assert r <= 1.4e-2, f"{what}: 2-norm {r:.3e}"


@pytest.mark.parametrize("raw", [False, True], ids=["plain", "raw"])
@pytest.mark.parametrize("heads", [2, 4, 6])
@pytest.mark.parametrize("dims", [(128, 128), (64, 64), (64, 128), (128, 64)], ids=lambda d: f"{d[0]}x{d[1]}")
def test_batch_matches_single_sequences(dims, heads, raw):
    import paper_2609_32114_amd as P
    Dk, Dv = dims
    Hv = heads * (128 // Dv)
    Hqk = Hv // 2
    inp = make_case("gdn", LENS, Hqk, Hv, Dk, Dv, "bf16", with_s0=not raw, seed=51, scale=Dk ** -0.5, raw=raw)
    pre = P.PRE_ALL if raw else 0
    assert 128 < len(LENS) * Hv * Dv // 16
    o, s = run_gpu(inp, preprocess=pre)
    for n, length in enumerate(LENS):
        if length == 0:
            np.testing.assert_array_equal(s[n], inp.s0[n] if inp.s0 is not None else np.zeros_like(s[n]))
            continue
        o1, s1 = run_gpu(_alone(inp, n), preprocess=pre)
        a = int(inp.cu_seqlens[n])
        _close(o[a:a + length], o1, f"o of sequence {n}")
        _close(s[n], s1[0], f"state of sequence {n}")


@pytest.mark.parametrize("variant", ["lm", "ks", "fg"])
def test_segments_of_every_count(variant):
    """2 to 6 segments per sequence (with and without a scan of the maps), the
    last one ragged, against the oracle."""
    import paper_2609_32114_amd as P
    try:
        P.set_segment_chunks(2)
        inp = make_case("gdn", (129, 257, 300, 385, 700), 2, 4, 128, 128, "bf16", with_s0=True, variant=variant, seed=52)
        check_against_oracle(inp, label=f"compact-segments-{variant}")
    finally:
        P.set_segment_chunks(0)


@pytest.mark.parametrize("lens", [(700,), (129, 0, 300)], ids=["one", "batch"])
@pytest.mark.parametrize("heads", [1, 6, 12], ids=["tile", "pair", "head"])
@pytest.mark.parametrize("dims", [(128, 128), (64, 64), (64, 128), (128, 64)], ids=lambda d: f"{d[0]}x{d[1]}")
def test_segments_on_each_walk(dims, heads, lens):
    """Segments of two chunks whose column tiles, one or two to a workgroup, fit 256
    compute units (row walk) or do not (head walk), against the oracle and with
    the final state written over the initial one."""
    import torch
    import paper_2609_32114_amd as P
    Dk, Dv = dims
    Hv, segs = heads * (128 // Dv), (sum(lens) // 64 + len(lens)) // 2 + len(lens)
    tiles = -(-segs * Hv // 8) * 8 * (Dv // 16)
    assert tiles <= 256 if heads == 1 else 256 < tiles <= 512 if heads == 6 else tiles > 512
    inp = make_case("gdn", lens, Hv, Hv, Dk, Dv, "bf16", with_s0=True, variant="s0", seed=54, scale=Dk ** -0.5)
    try:
        P.set_segment_chunks(2)
        check_against_oracle(inp, label="compact-segments")
        d = to_device(inp)
        run = lambda s0, out: P.gdn_prefill(d["q"], d["k"], d["v"], d["g"], d["beta"], initial_state=s0,  # noqa: E731
                                            cu_seqlens=d["cu"], scale=inp.scale, final_out=out)
        o1, s1 = run(d["s0"], None)
        state = d["s0"].clone()
        o2, _ = run(state, state)
        torch.cuda.synchronize()
    finally:
        P.set_segment_chunks(0)
    assert torch.equal(o1, o2) and torch.equal(state, s1)


LONG = [  # lengths, value heads at d_v = 128 (twice as many at 64)
    ((20,) * 7 + (3000,) + (20,) * 8, 4),               # tile pairs beside one long sequence
    ((20,) * 30 + (2000, 0, 1500, 65), 4),              # whole heads beside two
    ((2,) * 299 + (2500,), 1),                          # more sequences than the index kernel's threads
]
SHORT = [  # the same, on either side of the 12 chunks from which long sequences are walked apart
    ((3,) * 6 + (674,) + (3,) * 4, 4, 11),
    ((3,) * 6 + (675,) + (3,) * 4, 4, 12),
    ((3,) * 17 + (653,), 4, 11),
    ((3,) * 17 + (654,), 4, 12),
]


@pytest.mark.parametrize("case", LONG, ids=["pairs", "heads", "many"])
@pytest.mark.parametrize("dims", [(128, 128), (64, 64), (64, 128), (128, 64)], ids=lambda d: f"{d[0]}x{d[1]}")
def test_long_sequences_among_short_ones(dims, case):
    """Batches with more column tiles than 256 compute units in which some
    sequences are so much longer than the others that they are walked apart,
    against the oracle and with the final state written over the initial one."""
    import torch
    import paper_2609_32114_amd as P
    Dk, Dv = dims
    lens, Hv = case[0], case[1] * (128 // Dv)
    chunks = [-(-n // 64) for n in lens]
    share, tiles = Hv * Dv // 16, -(-len(lens) * Hv // 8) * 8 * (Dv // 16)
    assert tiles > 256 and sum(lens) >= 64 * (48 if tiles <= 512 else 32) - 63
    assert (tiles <= 512) == (len(lens) == 16) and max(chunks) * 256 > share * sum(chunks)
    inp = make_case("gdn", lens, Hv, Hv, Dk, Dv, "bf16", with_s0=True, variant="s0", seed=55, scale=Dk ** -0.5)
    check_against_oracle(inp, label="compact-long")
    d = to_device(inp)
    run = lambda s0, out: P.gdn_prefill(d["q"], d["k"], d["v"], d["g"], d["beta"], initial_state=s0,  # noqa: E731
                                        cu_seqlens=d["cu"], scale=inp.scale, final_out=out)
    o1, s1 = run(d["s0"], None)
    state = d["s0"].clone()
    o2, _ = run(state, state)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(state, s1)


@pytest.mark.parametrize("case", SHORT, ids=lambda c: f"N{len(c[0])}-{c[2]}chunks")
@pytest.mark.parametrize("dims", [(128, 128), (64, 64), (64, 128), (128, 64)], ids=lambda d: f"{d[0]}x{d[1]}")
def test_long_sequence_in_a_batch_of_few_chunks(dims, case):
    Dk, Dv = dims
    lens, Hv = case[0], case[1] * (128 // Dv)
    tiles = -(-len(lens) * Hv // 8) * 8 * (Dv // 16)
    assert tiles > 256 and (tiles <= 512) == (len(lens) == 11) and -(-sum(lens) // 64) == case[2]
    inp = make_case("gdn", lens, Hv, Hv, Dk, Dv, "bf16", with_s0=True, variant="s0", seed=60, scale=Dk ** -0.5)
    check_against_oracle(inp, label="compact-long-short")


def test_workspace_regions_of_a_compact_call():
    import paper_2609_32114_amd as P
    for T, Hv, held in ((200, 2, True), (32768, 16, False), (4096, 64, False)):
        for r in (P.WS_NM, P.WS_B, P.WS_QP, P.WS_OLOC, P.WS_DECAY):
            assert (P.workspace_region("gdn", 1, T, Hv, Hv, 128, 128, P.HAGDN_BF16, r)[1] > 0) == held


@pytest.mark.parametrize("dims,lens,heads", [((64, 64), (40,) * 7 + (4000,), 8), ((128, 128), (40,) * 15 + (5500,), 2)],
                         ids=["64x64", "128x128"])
def test_batch_that_may_hold_one_long_sequence_keeps_the_affine_factors(dims, lens, heads):
    """129 to 256 column tiles: a long batch keeps the affine factors, whose walk has
    the shorter step; a short one takes the compact form."""
    import paper_2609_32114_amd as P
    Dk, Dv = dims
    assert 128 < len(lens) * heads * Dv // 16 <= 256
    nm = lambda T: P.workspace_region("gdn", len(lens), T, heads, heads, Dk, Dv, P.HAGDN_BF16, P.WS_NM)[1]  # noqa: E731
    assert nm(1000) == 0 and nm(sum(lens)) > 0
    inp = make_case("gdn", lens, heads, heads, Dk, Dv, "bf16", with_s0=True, variant="s0", seed=56, scale=Dk ** -0.5)
    check_against_oracle(inp, label="affine-batch")


@pytest.mark.parametrize("raw", [False, True], ids=["plain", "raw"])
@pytest.mark.parametrize("T", [1, 64, 65, 700])
@pytest.mark.parametrize("dims", [(128, 128), (64, 64), (64, 128), (128, 64)], ids=lambda d: f"{d[0]}x{d[1]}")
def test_single_sequence_one_tile_walk(dims, T, raw):
    """129 to 256 column tiles of one sequence (the row walk's one-tile instance that
    derives its tables itself), against the oracle."""
    import oracle
    import paper_2609_32114_amd as P
    Dk, Dv = dims
    Hv = 20 * (128 // Dv)
    assert 128 < Hv * Dv // 16 <= 256
    assert P.workspace_region("gdn", 1, T, Hv // 2, Hv, Dk, Dv, P.HAGDN_BF16, P.WS_NM)[1] == 0
    inp = make_case("gdn", (T,), Hv // 2, Hv, Dk, Dv, "bf16", with_s0=True, seed=57, scale=Dk ** -0.5, raw=raw)
    if not raw:
        check_against_oracle(inp, label="compact-single")
        return
    o, s = run_gpu(inp, preprocess=P.PRE_ALL)
    ro, rs = oracle.run_inputs(inp, nthreads=oracle_threads(), pre=P.PRE_ALL)
    for what, got, ref in (("o", o, ro), ("s_final", s, rs)):
        assert np.all(np.isfinite(got)) and relerr(got, ref) <= TOL["bf16"], (what, relerr(got, ref))


@pytest.mark.parametrize("Hqk,Hv,T,forced", [(1, 256, 32704, 0), (1, 256, 32832, 0), (1, 256, 32832, 32),
                                             (1, 64, 131008, 2047)],
                         ids=["head-walk", "capped", "short-segments", "tile-pairs"])
def test_output_up_to_and_beyond_2gib(Hqk, Hv, T, forced):
    """One sequence whose output rows span just under 2 GiB, walked whole by heads or
    tile pairs, or more, in segments of at most 511 chunks: the walks' 32-bit byte
    offsets.  Inputs are drawn on the GPU; the oracle checks the last head."""
    import torch
    import oracle
    import paper_2609_32114_amd as P
    D = 128
    gen = torch.Generator(device="cuda").manual_seed(58)
    unit = lambda: torch.nn.functional.normalize(  # noqa: E731
        torch.randn(T, Hqk, D, device="cuda", generator=gen), dim=-1).bfloat16()
    q, k = unit(), unit()
    v = torch.empty(T, Hv, D, device="cuda", dtype=torch.bfloat16)
    for part in v.split(16384):
        part.copy_(torch.randn(part.shape, device="cuda", generator=gen))
    g = -0.01 * torch.nn.functional.softplus(torch.randn(T, Hv, device="cuda", generator=gen))
    beta = torch.sigmoid(torch.randn(T, Hv, device="cuda", generator=gen))
    rows = 64 * Hv * D * 2  # bytes of a chunk's
    try:
        P.set_segment_chunks(forced)
        L = P.segment_chunks(1, T, Hv, D, torch.bfloat16)
        assert L * rows < 2 ** 31 and (forced == 32 or (L + 1) * rows >= 2 ** 31)
        assert (T <= 64 * L) == (T * Hv * D * 2 < 2 ** 31)
        o, s = P.gdn_prefill(q, k, v, g, beta)
        torch.cuda.synchronize()
    finally:
        P.set_segment_chunks(0)
    h = [Hv - 1]
    host = lambda x: x.float().cpu().numpy()  # noqa: E731
    ro, rs = oracle.prefill("gdn", host(q), host(k), host(v[:, h]), host(g[:, h]), host(beta[:, h]),
                            nthreads=oracle_threads())
    assert relerr(host(o[:, h]), ro) <= TOL["bf16"] and relerr(host(s[:, h]), rs) <= TOL["bf16"]


@pytest.mark.parametrize("Hqk,Hv", [(1, 3), (4, 20)], ids=["tile", "head"])
def test_in_place_state_of_whole_chains(Hqk, Hv):
    import torch
    import paper_2609_32114_amd as P
    lens = (70, 64, 1, 200, 33, 129, 0, 31)
    assert 128 < -(-len(lens) * Hv // 8) * 64 <= 256 if Hv == 3 else len(lens) * Hv * 8 > 512
    assert P.workspace_region("gdn", len(lens), sum(lens), Hqk, Hv, 128, 128, P.HAGDN_BF16, P.WS_NM)[1] == 0
    inp = make_case("gdn", lens, Hqk, Hv, 128, 128, "bf16", with_s0=True, variant="s0", seed=59)
    d = to_device(inp)
    o1, s1 = P.gdn_prefill(d["q"], d["k"], d["v"], d["g"], d["beta"], initial_state=d["s0"], cu_seqlens=d["cu"])
    state = d["s0"].clone()
    o2, _ = P.gdn_prefill(d["q"], d["k"], d["v"], d["g"], d["beta"], initial_state=state, cu_seqlens=d["cu"],
                          final_out=state)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(state, s1)


def test_in_place_state_batch():
    import torch
    import paper_2609_32114_amd as P
    inp = make_case("gdn", (70, 64, 1, 200, 33, 129, 0, 31), 4, 8, 128, 128, "bf16", with_s0=True, variant="s0", seed=53)
    d = to_device(inp)
    o1, s1 = P.gdn_prefill(d["q"], d["k"], d["v"], d["g"], d["beta"], initial_state=d["s0"], cu_seqlens=d["cu"])
    state = d["s0"].clone()
    o2, _ = P.gdn_prefill(d["q"], d["k"], d["v"], d["g"], d["beta"], initial_state=state, cu_seqlens=d["cu"],
                          final_out=state)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(state, s1)
