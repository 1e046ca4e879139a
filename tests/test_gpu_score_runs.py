"""GPU parity of scoring where the launch shortens its runs of tiles (few heads over a short context) and where a
wavefront of the shared-K kernel holds a single row block (head_dim 256), against the fp64 oracle.

Bar: 1e-4 relative, as everywhere for chunk masses and densities (fp32 sums of fp32 exponentials)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2403_11805_amd as kvs
from paper_2403_11805_amd import synth

from gpu_util import DEV, both_shapes, gpu_score
from test_score_run_rule import runs_of

pytestmark = pytest.mark.gpu


def score_with(ks, q, kv, n_valid, ws_bytes):
    cm = torch.full((ks.n_layers, ks.n_q_heads, ks.n_chunks), float("nan"), dtype=torch.float32, device=DEV)
    d = torch.full((ks.n_chunks,), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.full((ws_bytes,), 0xff, dtype=torch.uint8, device=DEV)
    kvs.kv_score_chunks_valid(ks, q.to(DEV), kv.to(DEV), n_valid, oracle.NORM_VISIBLE, ws, cm, d)
    torch.cuda.synchronize()
    return cm.cpu().numpy(), d.cpu().numpy()


def check(got, want):
    for g, w in zip(got, want):
        assert np.all(np.isfinite(g))
        np.testing.assert_allclose(g, w, rtol=1e-4, atol=1e-30)


def exact_masses(q, k, T):
    """Chunk masses of query rows q [heads][R][D] (the newest tokens) over keys k [N][D] in 64 bits, columns averaged over
    the rows that see them."""
    R, N = q.shape[1], k.shape[0]
    s = q.double() @ k.double().T / q.shape[2] ** 0.5
    seen = torch.arange(N, device=DEV) <= torch.arange(N - R, N, device=DEV)[:, None]
    a = torch.softmax(s.masked_fill(~seen, float("-inf")), -1).sum(1) / seen.sum(0)
    return a.view(q.shape[0], N // T, T).sum(-1)


@pytest.mark.parametrize("geom,R,n_valid", [
    ((1, 1, 3, 256, 1056, 16, 64), 32, 1056),    # head_dim 256, three row blocks: one wavefront of four without work
    ((2, 1, 8, 256, 544, 8, 64), 23, 471),       # eight blocks in two workgroups, 17 tiles, the last two padding only
    ((1, 1, 2, 256, 256, 32, 256), 33, 97),      # two heads of two blocks; most of the cache is padding
    ((1, 1, 4, 128, 160, 32, 64), 5, 160),       # 5 tiles: a run of four and one of one
    ((1, 1, 4, 64, 128, 16, 64), 32, 128),       # 4 tiles: nothing to shorten
    ((3, 1, 1, 64, 96, 16, 64), 9, 70),          # four runs side by side, 3 tiles: runs of two and one, padding behind
    ((200, 1, 4, 64, 256, 16, 64), 32, 250),     # enough heads: two runs of four tiles
])
def test_short_runs(geom, R, n_valid):
    ks, os_ = both_shapes(synth.Geometry(*geom))
    kv = synth.make_kv(synth.Geometry(*geom), 61, "cpu", 1, 4.0)
    q = (synth.make_q(synth.Geometry(*geom), 61, R).float() * 6).to(torch.float16)
    want = oracle.score_chunks_valid(os_, q.numpy(), kv.numpy(), n_valid, oracle.NORM_VISIBLE)
    kv[:, :, :, n_valid:] = float("nan")
    check(score_with(ks, q, kv, n_valid, kvs.kv_score_workspace_bytes(ks, R)), want)


@pytest.mark.parametrize("D,hot_token", [(256, 3), (256, 140), (256, 900), (128, 140)])
def test_huge_logit_in_a_short_run(D, hot_token):
    """A key far above the row references of its run: the run is redone through the general pass."""
    g = synth.Geometry(1, 1, 4, D, 1024, 16, 64)
    ks, os_ = both_shapes(g)
    kv = (synth.make_kv(g, 29, "cpu").float() * 0.05).to(torch.float16)
    kv[0, 0, 0, hot_token] = 20.0
    q = torch.full((1, 4, 32, D), 2.0, dtype=torch.float16)
    check(gpu_score(ks, q.to(DEV), kv.to(DEV), oracle.NORM_NONE),
          oracle.score_chunks(os_, q.numpy(), kv.numpy(), oracle.NORM_NONE))


def longest_runs_bytes(g, R, longest):
    rows, tiles = (R + 31) // 32 * 32, g.N // 32
    runs = (tiles + longest - 1) // longest
    least = 4 * g.L * g.Hq * rows * (tiles + g.N // min(g.T, 32) + 3 * runs)
    return (least + 255) // 256 * 256


@pytest.mark.parametrize("T", [8, 16, 32])
@pytest.mark.parametrize("D", [64, 128, 256])
@pytest.mark.parametrize("n_valid", [2048, 2015, 1983, 1951])
def test_long_runs_of_the_shared_kernel(D, T, n_valid):
    """63, 62, 61 and 60 tiles of one run below the causal diagonal, so that the loop over pairs of tiles turns many
    times and ends in each of its ways; six row blocks per kv head: a wavefront (at head_dim 256 two) without work.  The
    workspace holds the longest runs only, or these heads would be scored in runs of seven tiles."""
    g = synth.Geometry(1, 1, 6, D, 2048, T, 64)
    ks, os_ = both_shapes(g)
    kv = synth.make_kv(g, 43, "cpu", 1, 4.0)
    q = (synth.make_q(g, 43, 32).float() * 6).to(torch.float16)
    want = oracle.score_chunks_valid(os_, q.numpy(), kv.numpy(), n_valid, oracle.NORM_VISIBLE)
    kv[:, :, :, n_valid:] = float("nan")
    check(score_with(ks, q, kv, n_valid, longest_runs_bytes(g, 32, 64)), want)


@pytest.mark.parametrize("D,T", [(64, 8), (64, 16), (128, 8), (256, 8), (256, 16), (256, 32)])
@pytest.mark.parametrize("hot_token", [1000, 1980])
def test_huge_logit_late_in_a_long_run(D, T, hot_token):
    g = synth.Geometry(1, 1, 6, D, 2048, T, 64)
    ks, os_ = both_shapes(g)
    kv = (synth.make_kv(g, 47, "cpu").float() * 0.05).to(torch.float16)
    kv[0, 0, 0, hot_token] = 20.0
    q = torch.full((1, 6, 32, D), 2.0, dtype=torch.float16)
    check(score_with(ks, q, kv, g.N, longest_runs_bytes(g, 32, 64)),
          oracle.score_chunks(os_, q.numpy(), kv.numpy(), oracle.NORM_VISIBLE))


@pytest.mark.parametrize("geom,R,longest", [
    ((1, 1, 4, 128, 2048, 16, 64), 32, 64),
    ((1, 1, 1, 64, 2048, 16, 64), 32, 8),
])
def test_workspace_that_holds_the_longest_runs_only(geom, R, longest):
    """A workspace without room for the run planes of shorter runs is served with the longest ones; one byte less
    than these need is refused."""
    g = synth.Geometry(*geom)
    ks, os_ = both_shapes(g)
    least = longest_runs_bytes(g, R, longest)
    assert least < kvs.kv_score_workspace_bytes(ks, R)
    kv = synth.make_kv(g, 67, "cpu", 1, 4.0)
    q = (synth.make_q(g, 67, R).float() * 6).to(torch.float16)
    check(score_with(ks, q, kv, g.N, least), oracle.score_chunks(os_, q.numpy(), kv.numpy(), oracle.NORM_VISIBLE))
    with pytest.raises(kvs.KvError) as err:
        score_with(ks, q, kv, g.N, least - 1)
    assert err.value.code == kvs.KV_ENOMEM


@pytest.mark.parametrize("per,D,R,hot_block", [
    (1, 256, 256, 2), (1, 256, 256, 6),      # one head of eight blocks in two workgroups of four
    (2, 256, 96, 3), (2, 256, 96, 5),        # the second head: its first block in one workgroup, two in the next
    (4, 128, 96, 7), (4, 128, 96, 8),        # the third head: two blocks in one workgroup of eight, one in the next
    (4, 64, 96, 6), (4, 64, 96, 8),
])
@pytest.mark.parametrize("norm", [oracle.NORM_VISIBLE, oracle.NORM_NONE])
def test_reference_left_by_one_row_block(per, D, R, hot_block, norm):
    """A head whose row blocks lie in two workgroups, and a key that the queries of only one block answer to, far
    above the reference of its run: one workgroup redoes the run, the other does not, and every row has to be
    combined with the references of its own workgroup."""
    hot_token = 200
    g = synth.Geometry(1, 1, per, D, 1024, 16, 64)
    ks, os_ = both_shapes(g)
    kv = (synth.make_kv(g, 37, "cpu").float() * 0.05).to(torch.float16)
    kv[0, 0, 0, hot_token] = 20.0
    q = torch.full((1, per, R, D), 2.0, dtype=torch.float16)
    q[..., ::2] = -2.0                       # nothing to the hot key: its channels are all alike
    blocks = (R + 31) // 32
    rows = slice(hot_block % blocks * 32, min(hot_block % blocks * 32 + 32, R))
    q[0, hot_block // blocks, rows] = 2.0
    want = oracle.score_chunks(os_, q.numpy(), kv.numpy(), norm)
    ws = torch.full((kvs.kv_score_workspace_bytes(ks, R),), 0xff, dtype=torch.uint8, device=DEV)
    cm = torch.full((1, per, ks.n_chunks), float("nan"), dtype=torch.float32, device=DEV)
    d = torch.full((ks.n_chunks,), float("nan"), dtype=torch.float32, device=DEV)
    kvs.kv_score_chunks(ks, q.to(DEV), kv.to(DEV), norm, ws, cm, d)
    torch.cuda.synchronize()
    check((cm.cpu().numpy(), d.cpu().numpy()), want)


def test_static_array_gives_the_same_bits():
    """A shape whose longest runs just fit the static array's promised size, and whose shorter ones need more: the
    call without a workspace still gives the bits of the call with one."""
    # (128 000 tokens in chunks of 32 are scored in the longest runs, which are the fastest there: 46.0 us, runs of 33 tiles 52.2)
    g = synth.Geometry(1, 1, 8, 64, 86016, 16, 64)
    ks, _ = both_shapes(g)
    R = 128
    assert longest_runs_bytes(g, R, 64) <= kvs.KV_SCORE_STATIC_BYTES
    assert kvs.kv_score_workspace_bytes(ks, R) > kvs.KV_SCORE_STATIC_BYTES
    kv = synth.make_kv(g, 41, DEV)
    q = synth.make_q(g, 41, R, DEV)
    cm = torch.full((1, 8, ks.n_chunks), float("nan"), dtype=torch.float32, device=DEV)
    d = torch.full((ks.n_chunks,), float("nan"), dtype=torch.float32, device=DEV)
    kvs.kv_score_chunks_static(ks, q, kv, oracle.NORM_VISIBLE, cm, d)
    torch.cuda.synchronize()
    want_cm, want_d = gpu_score(ks, q, kv, oracle.NORM_VISIBLE)
    assert np.array_equal(cm.cpu().numpy(), want_cm) and np.array_equal(d.cpu().numpy(), want_d)


@pytest.mark.parametrize("R", [16, 64, 96, 160])
def test_many_runs_and_row_blocks(R):
    """69, 74, 52 and 36 runs and one, two, three and five row blocks per head; the rows of one block of the second head
    meet a key far above their run's reference."""
    g = synth.Geometry(1, 1, 4, 64, 32768, 16, 64)
    ks, os_ = both_shapes(g)
    kv = (synth.make_kv(g, 53, "cpu").float() * 0.5).to(torch.float16)
    kv[0, 0, 0, 20007] = 20.0
    q = (synth.make_q(g, 53, R).float() * 6).to(torch.float16)
    q -= q.float().mean(-1, keepdim=True).to(torch.float16)       # hardly anything to the hot key
    q[0, 1, max(R - 32, 0):] = 2.0
    check(gpu_score(ks, q.to(DEV), kv.to(DEV), oracle.NORM_VISIBLE),
          oracle.score_chunks(os_, q.numpy(), kv.numpy(), oracle.NORM_VISIBLE))


@pytest.mark.parametrize("R,N,more_than", [(16, 1060864, 512), (64, 532480, 256), (96, 270336, 128), (160, 270336, 128)])
def test_more_runs_than_one_pass_of_the_combine_kernel(R, N, more_than):
    """The combine kernel collects the runs' bits `more_than` at a time, for one, two and three to eight row blocks per
    head: a key far above its run's reference in the first runs and in the last, met by the rows of one block only."""
    g = synth.Geometry(1, 1, 4, 64, N, 16, 64)
    ks, _ = both_shapes(g)
    assert runs_of(*g[:6], R) > more_than
    gen = torch.Generator(device=DEV)
    gen.manual_seed(59)
    kv = (torch.randn(ks.kv_dims, generator=gen, device=DEV) * 0.5).half()
    kv[0, 0, 0, 20007] = 20.0
    kv[0, 0, 0, N - 1000] = 20.0
    q = (torch.randn((1, 4, R, 64), generator=gen, device=DEV) * 6).half()
    q -= q.float().mean(-1, keepdim=True).half()                  # hardly anything to the hot keys
    q[0, 1, max(R - 32, 0):] = 2.0
    cm, d = gpu_score(ks, q, kv, oracle.NORM_VISIBLE)
    want = exact_masses(q[0], kv[0, 0, 0], 16)
    check((cm[0], d), (want.cpu().numpy(), (want.mean(0) / 16).cpu().numpy()))


@pytest.mark.parametrize("geom,R,n_valid", [
    ((18, 1, 8, 256, 1600, 16, 64), 23, 1589),   # 36 workgroups a run: seven runs of eight tiles, the last of two
    ((20, 5, 20, 128, 1600, 32, 64), 9, 1600),   # 100: five runs of ten tiles
    ((4, 4, 16, 128, 4096, 8, 64), 40, 4075),    # 16: runs of nine tiles, 128 tiles, the last of two
    ((1, 1, 6, 64, 2080, 16, 64), 32, 2017),     # one workgroup a run: runs of four tiles, 65 tiles, the last of one is padding
    ((10, 1, 8, 256, 2464, 16, 64), 23, 2300),   # 20: runs of nine tiles at head_dim 256, 77 tiles, the last of five is padding
    ((18, 1, 8, 256, 2272, 16, 64), 23, 2250),   # 36: seven runs of eleven tiles, the last of five
])
def test_runs_of_any_length(geom, R, n_valid):
    """Runs of other lengths too than powers of two: the combine kernel finds a tile's run by a product with 1 / length."""
    ks, os_ = both_shapes(synth.Geometry(*geom))
    kv = synth.make_kv(synth.Geometry(*geom), 71, "cpu", 1, 4.0)
    q = (synth.make_q(synth.Geometry(*geom), 71, R).float() * 6).to(torch.float16)
    want = oracle.score_chunks_valid(os_, q.numpy(), kv.numpy(), n_valid, oracle.NORM_VISIBLE)
    kv[:, :, :, n_valid:] = float("nan")
    check(score_with(ks, q, kv, n_valid, kvs.kv_score_workspace_bytes(ks, R)), want)


@pytest.mark.parametrize("L,D,N,T", [(4, 64, 65536, 8), (4, 64, 65536, 16), (4, 64, 65536, 32), (2, 128, 65536, 8),
                                     (2, 128, 65536, 16), (2, 128, 65536, 32), (2, 256, 32768, 8), (2, 256, 32768, 16),
                                     (2, 256, 32768, 32)])
def test_keys_read_past_the_caches(L, D, N, T):
    """256 MiB of keys, the least that is read past the caches, against a call per layer, which reads its share through
    them: the same runs (256 workgroups of the longest in all, and a workspace for the longest in a layer), the same sums,
    the same bits; and some heads against 64 bits.  Four row blocks per kv head, so that the fast pass, which alone reads
    past the caches, takes every tile below the diagonal."""
    Hkv, Hq, R = 8, 32, 5
    gen = torch.Generator(device=DEV)
    gen.manual_seed(73)
    kv = torch.empty((L, 2, Hkv, N, D), dtype=torch.float16, device=DEV)
    for l in range(L):
        kv[l] = torch.randn((2, Hkv, N, D), generator=gen, device=DEV)
    q = torch.randn((L, Hq, R, D), generator=gen, device=DEV).half()
    assert L * Hkv * N * D * 2 == 256 << 20

    def masses(layers, qs, kvs_):
        ks = kvs.Shape(layers, Hkv, Hq, D, N, T, 64)
        cm = torch.full((layers, Hq, ks.n_chunks), float("nan"), dtype=torch.float32, device=DEV)
        d = torch.zeros(ks.n_chunks, dtype=torch.float32, device=DEV)
        ws = torch.full((longest_runs_bytes(synth.Geometry(layers, Hkv, Hq, D, N, T, 64), R, 64),), 0xff, dtype=torch.uint8,
                        device=DEV)
        kvs.kv_score_chunks(ks, qs, kvs_, oracle.NORM_VISIBLE, ws, cm, d)
        torch.cuda.synchronize()
        return cm

    together = masses(L, q, kv)
    assert torch.isfinite(together).all()
    for l in range(L):
        assert torch.equal(together[l], masses(1, q[l:l + 1].contiguous(), kv[l:l + 1].contiguous())[0])
    for l, kvh in ((0, 0), (L - 1, Hkv - 1)):
        heads = slice(kvh * 4, kvh * 4 + 4)
        np.testing.assert_allclose(together[l, heads].cpu().numpy(), exact_masses(q[l, heads], kv[l, 0, kvh], T).cpu().numpy(),
                                   rtol=1e-4, atol=1e-30)
