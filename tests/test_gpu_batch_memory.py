"""Device memory of batched calls and Jacobian columns: what a call takes follows the
members it has, not the largest group, and calls of any size after one another give
the single calls' results bit for bit, also a captured graph that is replayed after a
larger call took other buffers, and a call captured with buffers for fewer members."""
import pytest

from gpu_util import BOX, say, to_dev
from paper_1804_05087_amd import SP_OP_PHI, synth

pytestmark = pytest.mark.gpu

DIMS = (16, 17, 16)
MIB = 1 << 20


def _plan_and_fields(count):
    import torch
    from paper_1804_05087_amd import Plan
    P = Plan(*DIMS, *BOX, 400.0, 10.0)
    few = torch.stack([to_dev(synth.perturbation_field(*DIMS, *BOX, seed=i)) for i in range(3)])
    u = few.repeat((count + 2) // 3, 1, 1, 1, 1)[:count].contiguous()
    u *= torch.linspace(0.5, 1.0, count, dtype=torch.float64, device=u.device)[:, None, None, None, None]
    return P, u


def _taken(call):
    import torch
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    call()
    torch.cuda.synchronize()
    return (free - torch.cuda.mem_get_info()[0]) / MIB


@pytest.mark.parametrize("kind", ["step", "jvp", "columns"])
def test_memory_of_small_calls(kind):
    """A member's intermediates are 0.45 MiB and a column's unit field and image 0.22 MiB:
    1.3 MiB for two. The bound of 16 MiB leaves room for the granularity of allocations;
    the largest group, of 256 members, takes 115 MiB and more."""
    import torch
    say("memory", kind)
    P, u = _plan_and_fields(600)
    P.befe_step_batch(u)  # the process' streams and queues
    P.close()
    Q, u = _plan_and_fields(2)
    Q.linearize(u[0].contiguous())
    out = torch.empty_like(u)
    J = torch.empty(2, Q.packed_n, dtype=torch.float64, device=u.device)
    call = {"step": lambda: Q.befe_step_batch(u, out=out),
            "jvp": lambda: Q.jvp_lin_batch(u, SP_OP_PHI, out=out),
            "columns": lambda: Q.jacobian_columns(SP_OP_PHI, first=0, count=2, out=J)}[kind]
    assert _taken(call) < 16
    assert _taken(call) < 1  # kept


def test_sizes_after_one_another():
    import torch
    say("sizes")
    P, u = _plan_and_fields(300)
    P.linearize(u[0].contiguous())
    single = torch.stack([P.befe_step(v.contiguous()) for v in u])
    eye = torch.zeros(P.packed_n, dtype=torch.float64, device=u.device)
    for count in (2, 3, 40, 300, 1, 7):
        assert torch.equal(P.befe_step_batch(u[:count].contiguous()), single[:count]), count
        cols = P.jacobian_columns(SP_OP_PHI, first=5, count=count)
        for i in {0, count // 2, count - 1}:
            eye.zero_()
            eye[5 + i] = 1.0
            assert torch.equal(cols[i], P.pack(P.jvp_lin(P.unpack(eye), SP_OP_PHI))), (count, i)


def test_captured_calls():
    import torch
    say("captured")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        P, u = _plan_and_fields(40)
        single = torch.stack([P.befe_step(v.contiguous()) for v in u])
        two, five = u[:2].contiguous(), u[:5].contiguous()
        out2, out5 = P.befe_step_batch(two), torch.empty_like(five)
        torch.cuda.synchronize()
        graphs = []
        for v, out in ((two, out2), (five, out5)):  # the second with buffers for two members
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                P.befe_step_batch(v, out=out)
            graphs.append(g)
        for _ in range(3):
            assert torch.equal(P.befe_step_batch(u), single)  # 40 members: larger buffers
            for g, out in zip(graphs, (out2, out5)):
                out.zero_()
                g.replay()
                torch.cuda.synchronize()
                assert torch.equal(out, single[:out.shape[0]])
    P.close()
