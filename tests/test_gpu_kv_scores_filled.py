"""The filled logit call (isoq_kv_scores_filled, which the binding uses where it
allocates the logits): every position that has a key holds exactly what the
plain call writes, every other one -inf, for the table, matrix-core and generic
kernels, with and without the sketch, at lengths around their 64-, 256- and
512-key steps, invalid block-table entries, empty sequences, max_len short of
and past the table's blocks, and caches without blocks.  Needs an MI355X."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_28430_amd as iq  # noqa: E402


@pytest.mark.parametrize("d,bits,group,m", [(128, 3, 1, 0), (128, 4, 1, 128), (64, 2, 1, 64), (512, 4, 1, 0),
                                            (128, 3, 2, 0), (96, 4, 4, 64), (128, 2, 5, 128), (100, 3, 1, 0),
                                            (44, 4, 3, 0)])
def test_filled_equals_plain(d, bits, group, m):
    rng = np.random.default_rng(d + group)
    n_kv, bs = 2, 16
    lens = [0, 1, 64, 255, 513, 700]
    blocks = 44
    p = iq.isoq_params_init("fast", d, bits, n_kv)
    sk = iq.isoq_sketch_init(p, m) if m else None
    n_blocks = len(lens) * blocks
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rec = T(rng.integers(0, 256, (n_blocks, n_kv, bs, p.record_bytes), dtype=np.uint8))
    rho = T(rng.uniform(0.5, 2.0, (n_blocks, n_kv, bs)).astype(np.float32))
    table = rng.permutation(n_blocks).reshape(len(lens), blocks).astype(np.int32)
    table[4, 3], table[5, 40] = -1, n_blocks   # blocks without keys
    q = T(rng.standard_normal((len(lens), n_kv * group, d)).astype(np.float16))
    kw = dict(sketch=sk, k_signs=T(rng.integers(0, 256, (n_blocks, n_kv, bs, m // 8), dtype=np.uint8)),
              k_gamma=rho * 0.2) if m else {}
    args = (p, q, rec, rho, T(table), T(np.asarray(lens, np.int32)), 0.1)
    for max_len in (None, 600, blocks * bs + 333, 1):
        print(f"case d={d} b={bits} group={group} m={m} max_len={max_len}", flush=True)
        got = iq.isoq_kv_scores(*args, max_len=max_len, **kw)
        ref = torch.full_like(got, float("-inf"))
        iq.isoq_kv_scores(*args, max_len=max_len, scores=ref, **kw)
        assert torch.equal(got, ref)
        assert got.isfinite().sum() > 0
    # a cache or a table without blocks
    none = iq.isoq_kv_scores(p, q, rec[:0], rho[:0], T(table), T(np.asarray(lens, np.int32)), 0.1, max_len=50,
                             **({} if not m else dict(kw, k_signs=kw["k_signs"][:0], k_gamma=kw["k_gamma"][:0])))
    assert none.shape[-1] == 50 and (none == float("-inf")).all()
    none = iq.isoq_kv_scores(p, q, rec, rho, T(table[:, :0]), T(np.asarray(lens, np.int32)), 0.1, max_len=50, **kw)
    assert (none == float("-inf")).all()
