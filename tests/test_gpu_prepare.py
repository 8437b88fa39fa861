"""Rotation and projection tables at the edges of their tiles, against fp64 sums rounded once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# d: below one chunk of 16, with and without a rest to the chunks of 64 that four waves take; dsub: 1, the sizes held in
# registers (16, 32, 48) and one past each; rows: around the tiles of 16 and 32, past the line between them, and on both sides
# of the 2,048 workgroups up to which a table entry is one thread's (2,048, 1,024 and 512 rows of 16, 32 and 64 subspaces)
@pytest.mark.parametrize("d,P,rows", [(4, 4, (1, 17)), (12, 1, (33,)), (68, 4, (1, 16, 31)), (260, 20, (5, 600)),
                                      (512, 16, (15, 513, 2100)), (768, 16, (1, 340, 352)), (784, 16, (64,)),
                                      (1024, 64, (250, 256, 257)), (1280, 8, (40,)), (3072, 64, (3, 90)),
                                      (16, 16, (2048, 2049)), (132, 4, (7, 2048, 2049, 70000)), (272, 16, (2048, 2050)), (784, 16, (2049,)),
                                      (384, 24, (1024, 1025)), (1024, 32, (1024, 1031)), (1056, 32, (1025,)), (3072, 64, (512, 513))])
def test_prepare_against_fp64(d, P, rows):
    import torch
    from paper_2603_06660_amd import PagIndex
    rng = np.random.default_rng(d)
    ix = PagIndex.build(torch.from_numpy(rng.standard_normal((80, d), dtype=np.float32)).cuda(), metric="l2", max_degree=8,
                        num_subspaces=P, ef_construction=20, seed=3)
    ex = ix.export()
    rot, cb = torch.from_numpy(ex["rotation"]).cuda().double(), torch.from_numpy(ex["codebooks"]).cuda().double()
    for n in rows:
        q = torch.from_numpy(rng.standard_normal((n, d), dtype=np.float32)).cuda()
        qr, tab = ix.prepare_queries(q)
        want = (q.double() @ rot.T)
        # one rounding to fp32, and the rounding of the fp64 sums, which is 2^-29 of it per term
        bound = want.abs() * 2.0 ** -24 * 1.001 + (q.double().abs() @ rot.abs().T) * d * 2.0 ** -52
        assert torch.all((qr.double() - want).abs() <= bound), (d, n)
        parts = qr.double().reshape(n, P, d // P)
        want = torch.matmul(parts.transpose(0, 1).contiguous(), cb.transpose(1, 2).contiguous()).transpose(0, 1)
        scale = torch.matmul(parts.abs().transpose(0, 1).contiguous(), cb.abs().transpose(1, 2).contiguous()).transpose(0, 1)
        assert torch.all((tab.double() - want).abs() <= want.abs() * 2.0 ** -24 * 1.001 + scale * d * 2.0 ** -52), (d, n)
    ix.close()
