"""Logit launches large enough for whole workgroups (1,024 positions, 4,096 on
the matrix cores with the sketch: several rounds of 256 keys each, the next
round's records, block-table entries, signs and gammas loaded ahead), for the
matrix-core and the table kernels.  A key's logit does not depend on how the
positions are cut, so every sequence of the large launch must give bit for bit
what it gives alone, where the positions are cut into the smallest workgroups
(the size that the oracle tests of the other files run); one case is compared
with the oracle directly.  Ragged lengths around the ends of workgroups and
rounds, block-table entries out of range, and the filled call on a buffer of
NaN.  Needs an MI355X."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2603_28430_amd as iq  # noqa: E402
import test_gpu_kv_scores as plain  # noqa: E402
import test_gpu_kv_scores_groups as groups  # noqa: E402

CANARY = -12345.0


def run_case(d, bits, group, m, n_seqs, n_kv, ctx, bs=16, codebook=None):
    print(f"case d={d} b={bits} group={group} m={m} seqs={n_seqs} heads={n_kv} ctx={ctx}", flush=True)
    rng = np.random.default_rng(d + group + m)
    p = iq.isoq_params_init("fast", d, bits, n_kv, codebook=codebook)
    sk = iq.isoq_sketch_init(p, m) if m else None
    per = (ctx + bs - 1) // bs
    n_blocks = n_seqs * per + 2
    gen = torch.Generator(device="cuda").manual_seed(d + bits)

    def rand_bytes(*shape):
        return torch.randint(0, 256, shape, generator=gen, dtype=torch.uint8, device="cuda")

    rec = rand_bytes(n_blocks, n_kv, bs, p.record_bytes)
    rho = torch.rand((n_blocks, n_kv, bs), generator=gen, device="cuda") + 0.5
    table = rng.permutation(n_blocks)[:n_seqs * per].reshape(n_seqs, per).astype(np.int32)
    table[::3, per // 2], table[1::3, per - 1] = -1, n_blocks
    edges = [ctx, 1, 256, 257, 512, 1023, 1025, 1281, ctx - 1, 4097, 4096 + 257, 2048]
    lens = np.array([min(ctx, edges[s % len(edges)]) for s in range(n_seqs)], np.int32)
    q = torch.randn((n_seqs, n_kv * group, d), generator=gen, device="cuda").half()
    table, lens = torch.from_numpy(table).cuda(), torch.from_numpy(lens).cuda()
    sg = rand_bytes(n_blocks, n_kv, bs, m // 8) if m else None
    gam = rho * 0.2
    ml = per * bs + 5   # past the table's blocks
    kw = dict(sketch=sk, k_signs=sg, k_gamma=gam) if m else {}
    got = torch.full((n_seqs, n_kv * group, ml), CANARY, device="cuda")
    iq.isoq_kv_scores(p, q, rec, rho, table, lens, 0.1, max_len=ml, scores=got, **kw)
    for s in range(n_seqs):
        one = torch.full((1, n_kv * group, ml), CANARY, device="cuda")
        iq.isoq_kv_scores(p, q[s:s + 1], rec, rho, table[s:s + 1], lens[s:s + 1], 0.1, max_len=ml, scores=one, **kw)
        assert torch.equal(got[s], one[0]), s
        assert (one[0, :, :lens[s].item()] != CANARY).sum() > 0
    filled = torch.full_like(got, float("nan"))
    st = iq.isoquant.lib.isoq_kv_scores_filled(
        p.handle, sk.handle if m else None, iq.ISOQ_F16, q.data_ptr(), n_seqs, n_kv * group, n_kv, rec.data_ptr(),
        rho.data_ptr(), sg.data_ptr() if m else None, gam.data_ptr() if m else None, n_blocks, bs, table.data_ptr(),
        per, lens.data_ptr(), 0.1, filled.data_ptr(), ml, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    assert torch.equal(filled, torch.where(got == CANARY, torch.full_like(got, float("-inf")), got))


# (d, bits, group, m, sequences, key heads, context): the grid has at least 1,024
# workgroups of 1,024 positions (matrix cores, small tables), 512 (sketch of
# 4,096 on the matrix cores, large tables)
@pytest.mark.parametrize("case", [(128, 3, 4, 0, 24, 16, 3000), (128, 4, 8, 0, 24, 16, 3000), (80, 3, 4, 0, 16, 32, 2100),
                                  (128, 2, 2, 0, 24, 16, 3000), (256, 2, 9, 0, 13, 16, 5000), (128, 3, 4, 128, 12, 24, 4500),
                                  (64, 4, 8, 64, 12, 24, 4500), (80, 3, 2, 128, 12, 24, 4500), (192, 2, 5, 128, 12, 24, 4500),
                                  (512, 4, 1, 64, 12, 24, 4500), (128, 2, 1, 0, 24, 16, 3000), (128, 3, 1, 128, 12, 16, 3000),
                                  (256, 4, 1, 64, 12, 16, 3000), (80, 3, 1, 0, 24, 16, 3000), (64, 4, 1, 0, 16, 32, 2100)])
def test_scores_of_large_launches(case):
    run_case(*case)


@pytest.mark.parametrize("group", [2, 4, 9])
def test_scores_of_large_launches_wide_codebook(group):
    run_case(128, 3, group, 0, 24, 16, 3000, codebook=groups.wide_codebook(3, 1e5))


def test_scores_of_large_launches_oracle():
    plain.run_case("full", 128, 3, "f16", n_seqs=16, n_q=256, n_kv=64, bs=16, seq_lens=[513] * 4 + [257] * 6 + [300] * 6,
                   seed=3)
