"""Rows with an infinity or NaN in the sketch encoders: their sign bits are all
zero (no residual can be told), for every width and bit width of the
matrix-core encoder and, beside it, the VALU encoder (fp32); the other rows of
the same tile are what they are without them.  The logit call that writes -inf
accepts caches without blocks through the C entry, and max_len in any integer
type through the binding.  Needs an MI355X."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_28430_amd as iq  # noqa: E402


@pytest.mark.parametrize("variant,d,bits,m,dtype", [("full", 64, 2, 64, "f16"), ("fast", 64, 4, 128, "f16"),
                                                    ("full", 128, 3, 128, "f16"), ("2d", 128, 4, 128, "f16"),
                                                    ("full", 256, 3, 64, "f16"), ("fast", 128, 3, 128, "f32")])
def test_signs_of_nonfinite_rows(variant, d, bits, m, dtype):
    print(f"case {variant} d={d} b={bits} m={m} {dtype}", flush=True)
    n, heads = 333, 3
    p = iq.isoq_params_init(variant, d, bits, 1)
    sk = iq.isoq_sketch_init(p, m)
    g = torch.Generator(device="cuda").manual_seed(d + bits)
    x = torch.randn((n * heads, d), generator=g, device="cuda").to(torch.float16 if dtype == "f16" else torch.float32)
    bad = x.clone()
    rows = torch.arange(0, n * heads, 11, device="cuda")
    for i, v in enumerate((float("inf"), float("-inf"), float("nan"))):
        bad[rows[i::3], (7 * i) % d] = v
    keep = torch.ones(n * heads, dtype=torch.bool, device="cuda")
    keep[rows] = False
    ref, got = iq.isoq_quantize_qjl(p, sk, x), iq.isoq_quantize_qjl(p, sk, bad)
    for a, b in zip(ref, got):
        assert torch.equal(a[keep], b[keep])
    assert (got[2][rows] == 0).all()
    # the append writes the same signs
    bs, nb = 16, 21
    cache = [torch.zeros((nb, heads, bs, p.record_bytes), dtype=torch.uint8, device="cuda"),
             torch.zeros((nb, heads, bs), device="cuda"),
             torch.full((nb, heads, bs, m // 8), 255, dtype=torch.uint8, device="cuda"),
             torch.zeros((nb, heads, bs), device="cuda")]
    iq.isoq_kv_append_qjl(p, sk, bad.view(n, heads, d), torch.arange(n, device="cuda"), *cache)
    signs = cache[2].transpose(1, 2).reshape(nb * bs * heads, m // 8)[:n * heads]
    assert torch.equal(signs, got[2])


@pytest.mark.parametrize("d,group", [(128, 1), (128, 2), (100, 1)])
def test_logits_without_blocks_and_integer_lengths(d, group):
    print(f"case d={d} group={group}", flush=True)
    p = iq.isoq_params_init("fast", d, 3, 2)
    q = torch.randn((2, 2 * group, d), device="cuda").half()
    rec = torch.zeros((4, 2, 16, p.record_bytes), dtype=torch.uint8, device="cuda")
    rho = torch.ones((4, 2, 16), device="cuda")
    table = torch.arange(4, dtype=torch.int32, device="cuda").view(2, 2)
    lens = torch.tensor([20, 3], dtype=torch.int32, device="cuda")
    assert torch.equal(iq.isoq_kv_scores(p, q, rec, rho, table, lens, max_len=np.int64(40)),
                       iq.isoq_kv_scores(p, q, rec, rho, table, lens, max_len=40))
    out = torch.zeros((2, 2 * group, 50), device="cuda")
    for blocks, per_seq in ((0, 2), (4, 0)):
        out.zero_()
        st = iq.isoquant.lib.isoq_kv_scores_filled(
            p.handle, None, 0, q.data_ptr(), 2, 2 * group, 2, None, None, None, None, blocks, 16, None, per_seq,
            lens.data_ptr(), 1.0, out.data_ptr(), 50, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert st == 0 and (out == float("-inf")).all()
