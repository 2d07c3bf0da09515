"""Short reduction lengths with fp32 weights have a kernel of their own whose additions are the streaming kernel's: the
logits of a vocabulary small enough for it against those of a larger one (which the streaming kernel takes) on the same
rows, bit for bit, at the edges of the 256-element blocks; and the ids are the top of these logits."""
import numpy as np
import pytest
import torch

from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [8, 248, 256, 264, 512, 520, 768, 1016, 1024])
@pytest.mark.parametrize("norm", [0, 1])
def test_short_rows_are_the_streaming_kernels_bit_exact(K, norm):
    gen = torch.Generator().manual_seed(K + norm)
    head = torch.randn(8200, K, generator=gen).cuda()          # 2050 sets of 4 rows: more than 512 workgroups of 4 waves
    h = (3 * torch.randn(K, generator=gen) + 1).cuda()
    g = (1 + 0.1 * torch.randn(K, generator=gen)).cuda()
    b = (0.1 * torch.randn(K, generator=gen)).cuda() if norm == 0 else None
    _, _, big = binding.ppd_early_topk(h, g, b, head, 8, norm, 1e-5, want_logits=True)
    big = np.asarray(big.cpu() if torch.is_tensor(big) else big)
    for vocab in (8, 9, 1001, 8189):
        ids, vals, z = binding.ppd_early_topk(h, g, b, head[:vocab].contiguous(), 8, norm, 1e-5, want_logits=True)
        z = np.asarray(z.cpu() if torch.is_tensor(z) else z)
        ids = np.asarray(ids.cpu() if torch.is_tensor(ids) else ids)
        np.testing.assert_array_equal(z.view(np.uint32), big[:vocab].view(np.uint32))
        np.testing.assert_array_equal(ids, np.argsort(-z, kind="stable")[:8])
