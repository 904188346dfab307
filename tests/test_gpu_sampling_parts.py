"""Rows that are shared by several work-groups, against the oracle: vocabularies at the edges of the shares (2048
tokens each, at most 16), nucleus cuts whose bin holds more tokens than the kernel keeps in LDS (4096), rows of one
value only, and a row without a nucleus."""
import numpy as np
import pytest
import torch

from test_gpu_sampling import _ctx_for_vocab, _oracle_decisions

pytestmark = pytest.mark.gpu


def _rows(rng, rows, vocab, kind):
    z = rng.standard_normal((rows, vocab))
    if kind == "equal":                       # one bin, one key: the cut is by id
        z[:] = 1.25
    elif kind == "crowded":                   # one far token, the others within one bin of 256 but with different keys
        z = z * 1e-3
        z[:, vocab // 3] = -40.0
    elif kind == "far":                       # every weight but one rounds to nothing
        z[:, vocab - 1] = 90.0
    return np.ascontiguousarray(z, dtype=np.float32)


@pytest.mark.parametrize("vocab", [37, 1023, 2047, 2048, 2049, 4098, 12289, 32767, 32768, 32773])
def test_shared_rows_decide_as_the_oracle(vocab):
    ctx, _ = _ctx_for_vocab(vocab)
    rng = np.random.default_rng(vocab)
    for kind in ("plain", "equal", "crowded", "far"):
        for T, top_p in [(1.0, 1.0), (0.6, 0.95), (0.7, 0.3)]:
            gamma = 2
            pl = _rows(rng, gamma + 1, vocab, kind)
            ql = _rows(rng, gamma, vocab, kind)
            un = (rng.integers(0, 1 << 24, 2 * gamma + 1) / float(1 << 24)).tolist()
            got = ctx.spec_sample(ql, pl, gamma, T, top_p, un)
            assert (got[0], got[1], got[2]) == _oracle_decisions(ql, pl, gamma, T, top_p, un), (kind, T, top_p)


def test_static_entry_point_in_a_replayed_graph():
    """The captured launches, replayed with other logits and with an eager call of another size between the replays,
    give what the eager call gives."""
    from paper_2504_05598_amd.binding import del_spec_sample_static
    vocab, gamma = 9000, 5
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    q = torch.empty(gamma, vocab, device="cuda")
    p = torch.empty(gamma + 1, vocab, device="cuda")
    un = torch.empty(2 * gamma + 1, device="cuda")
    out = torch.zeros(3 + gamma, dtype=torch.int32, device="cuda")
    want = torch.zeros_like(out)

    def call(o, v, g, stream=0):
        del_spec_sample_static(q.data_ptr(), p.data_ptr(), vocab, v, g, 0.6, 0.9, un.data_ptr(), o.data_ptr(), stream)

    def refill():
        p.normal_(0.0, 2.0, generator=gen)
        q.copy_(p[:gamma])
        q.add_(torch.empty_like(q).normal_(0.0, 0.5, generator=gen))
        un.uniform_(0.0, 1.0, generator=gen).clamp_(max=0.999)

    refill()
    torch.cuda.synchronize()
    call(want, vocab, gamma)                     # the array's address is looked up outside the capture
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(out, vocab, gamma, side.cuda_stream)
    for _ in range(4):
        refill()
        torch.cuda.synchronize()
        call(want, vocab, gamma)
        torch.cuda.synchronize()
        eager = want.tolist()
        call(want, 3001, 2)                      # other contents in the scratch array
        torch.cuda.synchronize()
        out.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert out.tolist() == eager
