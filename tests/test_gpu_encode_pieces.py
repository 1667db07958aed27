"""The separate encoding on a batch whose samples x levels pass 2^32, which no
single launch holds: the samples around every multiple of 2^27 and at both ends
against a call on those alone.  Forward bit for bit; backward with one-hot
gradients on samples of their own cells' weights, summed as the small call sums."""
import pytest
import torch

pytestmark = pytest.mark.gpu

L = 16
N = (1 << 28) + 1003
RES = [[2, 2, 2, 2]] * (L - 1) + [[40, 40, 40, 40]]  # the last level is past the LDS image


@pytest.fixture(scope="module")
def batch():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2507_03836_amd import _lib as fl
    fl.lib()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GB of device memory")
    pos = torch.empty(N, 4, device="cuda").uniform_(
        generator=torch.Generator(device="cuda").manual_seed(3))
    edge = [0, *range(1 << 27, N, 1 << 27), N]
    at = torch.cat([torch.arange(max(0, e - 700), min(N, e + 700)) for e in edge]).unique().cuda()
    yield fl, pos, at
    del pos
    torch.cuda.empty_cache()


def test_forward(batch):
    fl, pos, at = batch
    idx, counts = fl.fhash_dense_index(fl.grid_desc(RES, 1))
    table = torch.rand(sum(counts), device="cuda")
    enc = torch.full((N, L), -1.0, device="cuda")
    fl.fhash_encode_fwd(idx, pos, N, table, enc)
    want = torch.empty(len(at), L, device="cuda")
    fl.fhash_encode_fwd(idx, pos[at].contiguous(), len(at), table, want)
    assert torch.equal(enc[at], want)
    assert all((enc[i:i + (1 << 24)] >= 0).all() for i in range(0, N, 1 << 24))


def test_backward(batch):
    fl, pos, at = batch
    idx, counts = fl.fhash_dense_index(fl.grid_desc(RES, 1))
    g = torch.zeros(N, L, device="cuda")
    ga = 1.0 + torch.rand(len(at), L, device="cuda")
    g[at] = ga
    got, want = (torch.zeros(sum(counts), device="cuda") for _ in range(2))
    fl.fhash_encode_bwd(idx, pos, N, g, got)
    fl.fhash_encode_bwd(idx, pos[at].contiguous(), len(at), ga, want)
    # every sum has positive terms only: within 1e-5 of itself in any order (the
    # first levels' 16 vertices take len(at) terms each, error below len(at) 2^-24 of
    # it in the worst order; every order here adds in chunks)
    assert torch.allclose(got, want, rtol=1e-5, atol=1e-12)
    for l in range(L):  # and nothing is left out: the weights of a sample sum to 1
        lo = int(idx.slot_offset[l])
        s = got[lo:lo + counts[l]].double().sum().item()
        assert abs(s - ga[:, l].double().sum().item()) <= 1e-5 * s
