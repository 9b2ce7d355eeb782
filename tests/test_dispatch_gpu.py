"""Rules that send a call to one kernel or launch shape rather than another: both sides of each line give the same result."""
import pytest
import torch

import paper_2605_21325_amd as tri

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
GATES = [tri.GATE_SCALAR, tri.GATE_PER_CHANNEL, tri.GATE_NONE]


def make_inputs(T, H, d_k, gate, k_dtype=torch.bfloat16, seed=0, B=1):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rand = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    K = torch.nn.functional.normalize(rand(B, T, H, d_k), dim=-1).to(k_dtype)
    beta = torch.sigmoid(rand(B, T, H))
    shape = {tri.GATE_SCALAR: (B, T, H), tri.GATE_PER_CHANNEL: (B, T, H, d_k)}.get(gate)
    g = None if shape is None else -0.01 * (torch.arange(T, device=DEV) % 64).view(1, T, *[1] * (len(shape) - 2)) * torch.rand(
        1, 1, *shape[2:], generator=gen, device=DEV).expand(B, 1, *shape[2:])
    return K, beta, None if g is None else g.expand(*shape).contiguous()


# Up to 512 matrices a workgroup holds one wavefront, above four: a matrix does not depend on the others of its call, so the same
# chunks give the same bits on either side.
@pytest.mark.parametrize("gate", GATES)
@pytest.mark.parametrize("H", [1, 3, 4, 8])
@pytest.mark.parametrize("C", [16, 32, 64])
def test_few_matrices_give_the_bits_of_a_larger_call(C, H, gate):
    most = 512 // H                                   # chunks of the largest call with one wavefront to a workgroup
    T = (most + 1) * C - 5                            # ends inside a chunk
    K, beta, g = make_inputs(T, H, 64, gate)
    X = torch.randn(1, T, H, 72, device=DEV).bfloat16()
    part = lambda x, n: None if x is None else x[:, :n * C].contiguous()
    many = [tri.gdn_chunk_tri_inv_ex(K, beta, g, C, gate_kind=gate, method=m) for m in (tri.BLOCK_RECURSIVE, tri.NEWTON_SCHULZ)]
    W = tri.gdn_chunk_tri_solve(K, beta, g, X, C, row_scale=beta, gate_kind=gate)
    for n in (1, 2, most):
        k, b, gg, x = part(K, n), part(beta, n), part(g, n), part(X, n)
        for m, T_many in zip((tri.BLOCK_RECURSIVE, tri.NEWTON_SCHULZ), many):
            few = tri.gdn_chunk_tri_inv_ex(k, b, gg, C, gate_kind=gate, method=m)
            assert few.shape[0] <= 512 < T_many.shape[0]
            assert torch.equal(few, T_many[:few.shape[0]])
        w = tri.gdn_chunk_tri_solve(k, b, gg, x, C, row_scale=b, gate_kind=gate)
        assert torch.equal(w, W[:, :n * C])
        w1, w2 = tri.gdn_chunk_tri_solve_multi(k, b, gg, [x, x], C, row_scales=[b, None], gate_kind=gate)
        assert torch.equal(w1, w)
