"""Lazy projection in several passes against the float64 oracle: the listing of
the later passes, their size classes, counts on the device and waited for, the
walk through a pass over several layers, exact ties, normalized rows. The
shapes are those of lazy_walks.py, which do walk (test_host_calls.py)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_36452_amd import binding as rpd
from paper_2609_36452_amd.workload import CONFIGS, make_workload, round_bf16_bits
from tests.gpu_util import gain_tensor, gpu_params, note, run_gpu, to_device
from tests.lazy_walks import WALKS, lazy_from_eager, stop_early
from tests.parity import compare
from tests.test_gpu_parity import _duplicate_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("name,K,B,n,d,V,dtype,every,norm,ties", WALKS, ids=[c[0] for c in WALKS])
def test_walks_in_several_passes(name, K, B, n, d, V, dtype, every, norm, ties):
    w = make_workload(CONFIGS["llada_late"].with_(name=name, B=B, L=n + 9, K=K, d=d, V=V, n_masked=n, masked_frac=None,
                                                  dtype=dtype, sharp=("calibrated", -0.5, 2.5), unstable_frac=0.1), K * n)
    stop_early(w, K + n)
    if ties:
        _duplicate_rows(w, (1, 3, -2) if ties == "near" else (V // 2 + 7, -(V // 2) - 5))
    gain = None
    if norm:
        g = np.random.default_rng(n).uniform(0.75, 1.25, d)
        gain = (round_bf16_bits(g) if dtype == "bf16" else g.astype(np.float32), 1e-5, False)
    # four equal tops have a probability of at most a quarter each
    P = dataclasses.replace(O.LLADA, lazy=True, lazy_all=every, theta_c=0.2 if ties else O.LLADA.theta_c)
    pos, layer = O.layer_stats_masked(w.hidden, w.w_u, w.mask, dtype,
                                      norm=gain and (gain[0], float(np.float32(gain[1])), False))
    o = lazy_from_eager(w.mask, pos, layer, P)
    depth = o["layers_projected"]
    assert (depth > 1).sum() > 0.1 * len(pos) and len(set(depth)) >= 3
    if ties:
        assert (layer["gap"] == 0.0).mean() > 0.9
    tensors = to_device(w)
    a = run_gpu(w, P, tensors=tensors, norm=gain)
    rep = compare(a, o, w.mask, P, d)
    note("  " + rep.summary()[:300])
    assert rep.ok(), rep.summary()
    assert sum(rep.excused.values()) <= max(2, 0.05 * len(pos) * (K + 3)), rep.summary()
    # without a bound the call plans for the same count; without pinned memory it copies the counts it waits for
    kw = {} if gain is None else dict(norm_weight=gain_tensor(w, gain[0]), norm_eps=gain[1])
    b = [rpd.score_commit(*tensors, gpu_params(P), layer_stats=True, **kw)]
    if rpd.workspace_size(K, B, n + 9, d, V, tensors[0].dtype, max_masked=-1, norm=norm) <= rpd.NOALLOC_SCRATCH_BYTES:
        b.append(rpd.score_commit_noalloc(*tensors, gpu_params(P), layer_stats=True, **kw))
    torch.cuda.synchronize()
    m = w.mask != 0
    for other in b:
        for k in a:
            x, y = a[k], other[k].cpu().numpy()
            np.testing.assert_array_equal(x[..., m] if k.startswith("layer_") else x,
                                          y[..., m] if k.startswith("layer_") else y, err_msg=k)


def test_captured_walks_decode_as_eager_launches():
    # a decode whose calls walk: graph replays give what the same calls give launch by launch
    w = make_workload(CONFIGS["llada_late"].with_(name="walkdecode", B=1, L=256, K=4, d=2048, V=30011, n_masked=256,
                                                  masked_frac=None, sharp=("calibrated", -0.5, 2.5),
                                                  unstable_frac=0.1), 5)
    stop_early(w, 6)
    P = gpu_params(dataclasses.replace(O.LLADA, lazy=True, beta=1.0))
    tensors = to_device(w)
    res = []
    for graph in (True, False):
        dec = rpd.Decoder(*tensors, P, graph=graph)
        for _ in range(2):                  # the second decode replays the plans of the first
            dec.reset()
            r = dec.run(max_iter=24)
            torch.cuda.synchronize()
            res.append({k: r[k].cpu().numpy().copy() for k in ("canvas", "step", "mask")})
        assert dec.captures > 0 or not graph
    for r in res[1:]:
        for k in r:
            np.testing.assert_array_equal(res[0][k], r[k], err_msg=k)
    assert 1 < (res[0]["step"].max() + 1) <= 24
