"""Transition probabilities and log-sum-exps at the sizes where their loops end: a row of one piece, one short of / exactly /
just over a round trip (512 pieces of 16 bytes; 256 vocabulary tiles), rows without 16-byte pieces.  Against 64 bits."""
import pytest
import torch

from paper_2402_11131_amd import api

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, n) for n in (64, 4032, 4096, 4160, 8256)] + [(torch.float32, n) for n in (64, 1984, 2048, 2112)])
def test_transition_probs(dtype, d):
    torch.manual_seed(d)
    B, T, V = 2, 7, 300
    h, W = torch.randn(B, T, d).to(dtype), (torch.randn(V, d) / d ** 0.5).to(dtype)
    parent = torch.tensor([[-1, 0, 0, 1, 1, 2, 5]] * B, dtype=torch.int32)
    tok = torch.randint(0, V, (B, T), dtype=torch.int32)
    tok[0, 3], tok[1, 4] = -1, V
    logits = h.double() @ W.double().T
    lse = torch.logsumexp(logits, -1).float()
    got = api.ss_transition_probs(h.cuda(), W.cuda(), tok.cuda(), parent.cuda(), lse.reshape(-1).cuda()).cpu().double()
    for b in range(B):
        assert got[b, 0] == 1.0
        for i in range(1, T):
            p, c = int(parent[b, i]), int(tok[b, i])
            if not 0 <= c < V:
                assert got[b, i] == 0.0
                continue
            x = float(logits[b, p, c]) - float(lse[b, p])
            # a thread's chain of d / 256 + 16 products, ten additions across threads, the subtraction and expf (2 ulp)
            size = float((h[b, p].double() * W[c].double()).abs().sum())
            bound = (d / 256 + 26) * U * size + 2 * U * abs(x) + 8 * U
            assert abs(float(got[b, i]) / float(torch.tensor(x).double().exp()) - 1) <= bound, (b, i)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("V", [1, 130, 32640, 32768, 32769, 65537])
def test_logsumexp_tiles(dtype, V):
    torch.manual_seed(V)
    N, d = 3, 64
    h, W = torch.randn(N, d).to(dtype), torch.randn(V, d).to(dtype)
    got = api.ss_lm_head_logsumexp(h.cuda(), W.cuda()).cpu().double()
    logits = h.double() @ W.double().T
    # a logit is off by d roundings of sum |x w|; the sum by V / 64 + 20 roundings, expf's and logf's ulps
    bound = (d + 2) * U * float((h.double().abs() @ W.double().abs().T).max()) + (V / 64 + 40) * U
    assert float((got - torch.logsumexp(logits, -1)).abs().max()) <= bound
