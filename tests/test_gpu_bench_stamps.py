"""The benchmark's time stamps see every layer of a forward pass, whichever way the walker makes its calls."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_every_layer_is_stamped():
    import bench
    from paper_2506_17870_amd import binding, network
    ops = [dict(op="conv", src=0, dst=1, residual=None, relu=True, cin=16, cout=32, k=3, stride=1, pad=1),
           dict(op="conv", src=1, dst=2, residual=1, relu=True, cin=32, cout=32, k=1, stride=1, pad=0),
           dict(op="avgpool", src=2, dst=3, cout=32),
           dict(op="fc", src=3, dst=4, residual=None, relu=False, cin=32, cout=10)]
    model = network.NestedCNN(ops, network.plan_float_weights(ops, seed=0), 8, 2)
    x = torch.ones((2, 8, 8, 16), dtype=torch.int8, device="cuda")
    model.calibrate(x, 0.05)
    before = {n: getattr(binding, n) for n in ("run_layer", "nq_conv_full", "nq_gemm_full")}
    plain = model.forward(x, 0.05, full=True).clone()
    recs = bench.stamped_forward(model, binding, x, 0.05, True)
    assert [r["layer"] for r in recs] == ["3x3 s1 8x8 16->32", "1x1 s1 8x8 32->32 + residual", "fc 32->10"]
    assert all(r["us"] > 0 for r in recs)
    assert torch.equal(model.forward(x, 0.05, full=True), plain)
    assert before == {n: getattr(binding, n) for n in before}
