"""GPU parity of the recompute attention where a row's softmax reference has to move late (keys far above all earlier
ones) and where the rows of a workgroup see very different key ranges, against the oracle's recompute procedure with
the bars of test_gpu_recompute."""
import numpy as np
import pytest
import torch

import oracle.recompute as orc
import paper_2403_11805_amd as kvs
from paper_2403_11805_amd import binding, synth

from gpu_util import DEV
from test_gpu_recompute import close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv,Hq,D,N,missing,hot", [
    (1, 4, 128, 1024, [3, 40, 62, 63], {20: 2.0, 300: 8.0, 701: 30.0, 990: 60.0}),   # maxima that grow along the keys
    (1, 4, 128, 1024, [60, 61, 62, 63], {5: 60.0}),                                  # one key takes it all at once
    (8, 8, 64, 2048, [0, 1, 2, 3, 124, 125, 126, 127], {64: 20.0, 1500: 60.0}),      # rows at both ends of the cache
    (8, 16, 64, 512, [0], {}),                                                       # one key tile for every share
])
def test_reference_moves_and_ranges_differ(Hkv, Hq, D, N, missing, hot):
    T, d_model, d_ff = 16, 256, 512
    shape = kvs.Shape(1, Hkv, Hq, D, N, T, 64)
    dims_o = orc.LayerDims(d_model, Hq, Hkv, D, d_ff)
    dims = binding.LayerDims(d_model, d_ff, dims_o.rope_base, dims_o.rms_eps)
    w = synth.make_layer_weights(d_model, Hq, Hkv, D, d_ff, 83)
    kv = (synth.make_kv(synth.Geometry(1, Hkv, Hq, D, N, T, 64), 83, "cpu").float() * 0.2)
    for token, scale in hot.items():
        kv[0, 0, :, token] *= scale
    kv = kv.to(torch.float16)
    rows = np.concatenate([np.arange(c * T, (c + 1) * T) for c in missing])
    x = synth.make_hidden(len(rows), d_model, 83)
    k_ref, v_ref = kv[0, 0].numpy().copy(), kv[0, 1].numpy().copy()
    y_ref = orc.recompute_layer(x.numpy(), missing, T, k_ref, v_ref, {k: v.numpy() for k, v in w.items()}, dims_o)
    kv_dev = kv.to(DEV)
    y = torch.full((len(rows), d_model), float("nan"), dtype=torch.float16, device=DEV)
    ws = torch.empty(kvs.kv_recompute_workspace_bytes(shape, dims, len(missing)), dtype=torch.uint8, device=DEV)
    rc = kvs.Recompute()
    rc.layer(shape, dims, {k: v.to(DEV) for k, v in w.items()}, 0,
             torch.tensor(missing, dtype=torch.int32, device=DEV), x.to(DEV), kv_dev, y, ws)
    torch.cuda.synchronize()
    rc.close()
    err = close(y.cpu().numpy(), y_ref, 1e-2, 1e-2, "layer output")
    assert err < 3e-3


@pytest.mark.parametrize("Hkv,Hq,D,N,T,missing", [
    (1, 4, 128, 128, 8, [2, 5]),             # undivided; the last row is token 47 of tile 32..63
    (1, 2, 64, 96, 16, [0, 2]),              # undivided; token 47 again, the cache ends a tile later
    (1, 4, 128, 1024, 16, [3, 20, 40]),      # divided: token 655 of tile 640..671
    (8, 8, 64, 1024, 8, [1, 64, 100]),       # divided, kv heads dealt to the XCDs: token 807 of tile 800..831
])
def test_nothing_behind_the_last_token_is_used(Hkv, Hq, D, N, T, missing):
    """The cache has to hold what lies before the last recomputed token; what lies behind it, in the last tile of keys
    too, may be anything (NaN here)."""
    d_model, d_ff = 256, 512
    shape = kvs.Shape(1, Hkv, Hq, D, N, T, 64)
    dims_o = orc.LayerDims(d_model, Hq, Hkv, D, d_ff)
    dims = binding.LayerDims(d_model, d_ff, dims_o.rope_base, dims_o.rms_eps)
    w = synth.make_layer_weights(d_model, Hq, Hkv, D, d_ff, 89)
    kv = synth.make_kv(synth.Geometry(1, Hkv, Hq, D, N, T, 64), 89, "cpu")
    rows = np.concatenate([np.arange(c * T, (c + 1) * T) for c in missing])
    x = synth.make_hidden(len(rows), d_model, 89)
    k_ref, v_ref = kv[0, 0].numpy().copy(), kv[0, 1].numpy().copy()
    y_ref = orc.recompute_layer(x.numpy(), missing, T, k_ref, v_ref, {k: v.numpy() for k, v in w.items()}, dims_o)
    kv_dev = kv.to(DEV)
    kv_dev[:, :, :, rows[-1] + 1:] = float("nan")
    y = torch.full((len(rows), d_model), float("nan"), dtype=torch.float16, device=DEV)
    ws = torch.empty(kvs.kv_recompute_workspace_bytes(shape, dims, len(missing)), dtype=torch.uint8, device=DEV)
    rc = kvs.Recompute()
    rc.layer(shape, dims, {k: v.to(DEV) for k, v in w.items()}, 0,
             torch.tensor(missing, dtype=torch.int32, device=DEV), x.to(DEV), kv_dev, y, ws)
    torch.cuda.synchronize()
    rc.close()
    err = close(y.cpu().numpy(), y_ref, 1e-2, 1e-2, "layer output")
    assert err < 3e-3


@pytest.mark.parametrize("Hkv,Hq,D,N,T,missing", [
    (1, 1, 64, 64, 8, [2]),                      # one pair of 8 rows, one tile: three wavefronts have none
    (1, 1, 128, 96, 8, [0, 3, 11]),              # one pair of 24 rows, three tiles, undivided
    (1, 1, 128, 1024, 16, [63]),                 # one pair, divided in eight: four tiles a share, one a wavefront
    (16, 16, 64, 512, 8, [10]),                  # 16 tiles, undivided, kv heads dealt to the XCDs
    (16, 16, 64, 1024, 8, [10]),                 # divided, kv heads dealt to the XCDs; the row sees less than a share
    (32, 32, 64, 1024, 16, [3, 62]),             # divided in four: eight tiles a share, two a wavefront
    (2, 2, 128, 640, 16, [0, 39]),               # 20 tiles, the most that are not divided: five a wavefront
    (2, 2, 128, 672, 16, [0, 41]),               # 21 tiles, divided in five, the last share of one
    (2, 2, 128, 1184, 16, [1, 30, 73]),          # two pairs: 32 rows and 16; 37 tiles, shares of five, the last of two
    (8, 16, 128, 224, 8, [0, 27]),               # two heads on a kv head, undivided, rows at both ends
    (3, 3, 64, 2048, 16, [5, 64, 100, 127]),     # two pairs of 32 rows, kv heads in plain order
])
def test_few_pairs_share_a_workgroup(Hkv, Hq, D, N, T, missing):
    """One or two (row block, head) pairs per kv head: the wavefronts of a workgroup take the key tiles of one pair in
    turn, some of them none, and their outputs are merged."""
    d_model, d_ff = 256, 512
    shape = kvs.Shape(1, Hkv, Hq, D, N, T, 64)
    dims_o = orc.LayerDims(d_model, Hq, Hkv, D, d_ff)
    dims = binding.LayerDims(d_model, d_ff, dims_o.rope_base, dims_o.rms_eps)
    w = synth.make_layer_weights(d_model, Hq, Hkv, D, d_ff, 97)
    kv = (synth.make_kv(synth.Geometry(1, Hkv, Hq, D, N, T, 64), 97, "cpu").float() * 0.2).to(torch.float16)
    rows = np.concatenate([np.arange(c * T, (c + 1) * T) for c in missing])
    x = synth.make_hidden(len(rows), d_model, 97)
    k_ref, v_ref = kv[0, 0].numpy().copy(), kv[0, 1].numpy().copy()
    y_ref = orc.recompute_layer(x.numpy(), missing, T, k_ref, v_ref, {k: v.numpy() for k, v in w.items()}, dims_o)
    y = torch.full((len(rows), d_model), float("nan"), dtype=torch.float16, device=DEV)
    ws = torch.empty(kvs.kv_recompute_workspace_bytes(shape, dims, len(missing)), dtype=torch.uint8, device=DEV)
    rc = kvs.Recompute()
    rc.layer(shape, dims, {k: v.to(DEV) for k, v in w.items()}, 0,
             torch.tensor(missing, dtype=torch.int32, device=DEV), x.to(DEV), kv.to(DEV), y, ws)
    torch.cuda.synchronize()
    rc.close()
    err = close(y.cpu().numpy(), y_ref, 1e-2, 1e-2, "layer output")
    assert err < 3e-3
