"""The slots kernel at the edges of its blocks and on both sides of the line up to which it counts the tokens itself,
against the integer oracle; and the dense gate at one, two and three k-steps."""
import numpy as np
import pytest

from oracle import locmoe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,N,free_map", [(4, 2, False), (12, 5, True), (300, 3, False)])
@pytest.mark.parametrize("T", [1, 1023, 1024, 1025, 2049, 5119, 5120, 5121, 8191, 8192, 8193])
def test_dispatch_counts_at_block_edges(T, E, N, free_map):
    rng = np.random.default_rng(T * 31 + E)
    check_dispatch((rng.zipf(1.3, T) % E).astype(np.int32), E, N, free_map)


# the counting adds up the tokens of a wave that share the first one's expert: all, none but one, runs, and a last wave
# that is not full
@pytest.mark.parametrize("kind", ["one", "two", "runs", "first differs"])
@pytest.mark.parametrize("T", [1, 63, 65, 1000, 5119, 5120, 5121])
def test_dispatch_counts_of_skewed_tokens(T, kind):
    E, m, rng = 16, np.arange(T), np.random.default_rng(T)
    eid = {"one": np.full(T, E - 1), "two": rng.integers(0, 2, T) * 9, "runs": m // 50 % E,
           "first differs": np.where(m % 64 == 0, 3, 4 + m % 2)}[kind]
    check_dispatch(eid.astype(np.int32), E, 4, False)


def check_dispatch(eid, E, N, free_map):
    import torch
    from paper_2401_13920_amd import locmoe as lm
    assert torch.cuda.is_available(), "this test needs the MI355X"
    T = len(eid)
    e2n = (np.arange(E) * 7 % N if free_map else np.arange(E) // (E // N)).astype(np.int32)
    C = max(1, T // (2 * E))
    d = 8 * E
    desc = lm.make_desc(T, d, E, N, 8, C, "bf16")
    b = lm.alloc_buffers(desc)
    x = torch.randn(T, d, device="cuda").to(torch.bfloat16)
    print(f"[dispatch] T={T} E={E} N={N} C={C}", flush=True)
    lm.locmoe_dispatch(desc, x, torch.from_numpy(eid).cuda(), torch.from_numpy(e2n).cuda() if free_map else None, b.pos,
                       b.slot, b.kept, b.seg_off, b.node_off, b.buf_expert, b.row_token, b.send, b.ws, b.ws_bytes)
    torch.cuda.synchronize()
    ref = orc.slots(eid, E, C, e2n, N)
    for name in ("pos", "slot", "kept", "seg_off", "node_off", "buf_expert"):
        assert np.array_equal(getattr(b, name).cpu().numpy(), ref[name]), name
    kept = torch.from_numpy(ref["slot"] >= 0).cuda()
    assert torch.equal(b.send[b.slot[kept].long()], x[kept])


@pytest.mark.parametrize("E,d", [(32, 64), (32, 128), (32, 192), (32, 320), (128, 128), (128, 256), (128, 384), (128, 640)])
def test_dense_gate_k_steps(E, d):
    import torch
    from paper_2401_13920_amd import locmoe as lm
    T = 130
    gen = torch.Generator(device="cuda").manual_seed(d)
    x = torch.randn(T, d, generator=gen, device="cuda").to(torch.bfloat16)
    Wg = torch.randn(E, d, generator=gen, device="cuda").to(torch.bfloat16)
    g = torch.full((T, E), float("nan"), device="cuda")
    lm.locmoe_gate_dense(lm.make_desc(T, d, E, 1, 8, 8, "bf16"), x, Wg, g)
    torch.cuda.synchronize()
    ref = x.double() @ Wg.double().T
    bound = d * 2.0 ** -23 * (x.double().abs() @ Wg.double().abs().T)  # d exact products summed in fp32
    assert ((g.double() - ref).abs() <= bound).all()
