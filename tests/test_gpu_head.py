"""Classifier head and its backward for every number of classes that has a kernel of its own, and for ones that do not; row counts around
the stages of the weight gradient.  fp32 sums of at most 517 products: 1e-5 relative to the largest, sums over rows 1e-4."""
import numpy as np
import pytest
import torch

from paper_1809_00832_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [3, 37, 64, 516])
@pytest.mark.parametrize("C", [1, 2, 3, 4, 5, 6, 7, 8, 9, 16, 17, 32])
def test_every_number_of_classes(C, H):
    print("case head", C, H, flush=True)
    net = binding.TreeNet(synth.make_rnn_params(1, synth.CELL_TREERNN, 10, H))
    try:
        for n in (1, 31, 129, 700):
            rng = np.random.default_rng(n)
            h = rng.standard_normal((n, H)).astype(np.float32)
            w = (rng.standard_normal((H, C)) / H ** 0.5).astype(np.float32)
            b = rng.standard_normal(C).astype(np.float32)
            label = rng.integers(-1, C + 1, n).astype(np.int32)
            dh, dw, db, dl = (torch.from_numpy(x).cuda() for x in (h, w, b, label))
            # the reference in 64 bits on the host
            z = h.astype(np.float64) @ w.astype(np.float64) + b
            z -= z.max(axis=1, keepdims=True)
            probs = np.exp(z) / np.exp(z).sum(axis=1, keepdims=True)
            got = binding.tl_classify(net.ctx, dh, dw, db, torch.full((n, C), float("nan"), device="cuda")).cpu().numpy()
            np.testing.assert_allclose(got, probs, rtol=1e-4, atol=1e-6, err_msg="probs n=%d" % n)
            live = np.flatnonzero((label >= 0) & (label < C))
            d = np.zeros_like(probs)
            d[live] = probs[live]
            d[live, label[live]] -= 1
            back = {k: v.cpu().numpy() for k, v in binding.tl_classify_backward(net.ctx, dh, dw, db, dl).items()}
            loss = -np.log(probs[live, label[live]]).sum().reshape(1)
            for key, want in (("d_logits", d), ("g_h", d @ w.T.astype(np.float64)), ("d_w_s", h.T.astype(np.float64) @ d), ("d_b_s", d.sum(0)), ("loss", loss)):
                top = max(1.0, float(np.abs(want).max()))
                atol = (1e-4 if key in ("d_w_s", "d_b_s", "loss") else 1e-5) * top
                np.testing.assert_allclose(back[key].reshape(want.shape), want, rtol=1e-4, atol=atol, err_msg="%s n=%d" % (key, n))
    finally:
        net.close()
