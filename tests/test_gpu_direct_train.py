"""GPU parity of the direct sum at sampled targets and of the selector's training
step at the edges of their blocks, against the oracle.

Bars: the direct sum 1e-12 of the field's RMS (FP64 sums of up to a few thousand
terms, ~1e-16 each); loss 1e-5 relative, gradient 1e-4 relative RMS (FP32 sums),
as for the network elsewhere.
"""
import numpy as np
import pytest

from paper_0810_0233_amd import ccfmm, inputs, selector

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ref():
    import oracle

    return oracle


def rel_rms(a, b):
    return float(np.sqrt(np.sum((a - b) ** 2) / np.sum(b ** 2)))


# one target per block up to 256, two up to 512, four beyond; sources around one
# and two strides of a block's 1,024 threads
@pytest.mark.parametrize("n,nt", [(2, 2), (1023, 256), (1024, 257), (1025, 512), (2048, 513), (2049, 1027), (3100, 1)])
def test_direct_targets_block_edges(ref, n, nt):
    import torch

    rng = np.random.default_rng(n + nt)
    pos = rng.random((n, 3)) * 10.0
    if n > 10:
        pos[7] = pos[3]  # coincident dipoles leave each other out
    m = inputs.random_moments(n, nt)
    idx = rng.integers(0, n, nt).astype(np.int64)
    bad = nt > 300
    if bad:
        idx[[0, nt // 2, nt - 1]] = [-1, n, n + 5]  # out of range: NaN there, nothing else touched
    d_pos, d_m, d_idx = (torch.from_numpy(v).cuda() for v in (pos, m, idx))
    d_H = torch.zeros((nt + 1, 3), dtype=torch.float64, device="cuda")
    print("case n=%d nt=%d" % (n, nt), flush=True)
    ccfmm.direct_targets_device(n, d_pos.data_ptr(), d_m.data_ptr(), nt, d_idx.data_ptr(), d_H.data_ptr(),
                                torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    H = d_H.cpu().numpy()
    assert np.all(H[nt] == 0.0)
    good = (idx >= 0) & (idx < n)
    assert np.all(np.isnan(H[:nt][~good]))
    R = ref.bruteforce_targets(pos, m, idx[good])
    assert rel_rms(H[:nt][good], R) <= 1e-12


# a dipole so far away that its squared distance leaves FP64 adds nothing, as by the
# definition (1 / r^3 is zero); one whose place is no number makes no number
@pytest.mark.parametrize("nt", [1, 300, 1100])
@pytest.mark.parametrize("place,ok", [(1e200, True), (-1e155, True), (1e140, True), (np.nan, False), (np.inf, False)])
def test_direct_targets_far_away(ref, place, ok, nt):
    import torch

    rng = np.random.default_rng(nt)
    n = 1500
    pos = rng.random((n, 3)) * 10.0
    pos[n - 1, 1] = place
    m = inputs.random_moments(n, nt)
    idx = rng.integers(0, n - 1, nt).astype(np.int64)
    d_pos, d_m, d_idx = (torch.from_numpy(v).cuda() for v in (pos, m, idx))
    d_H = torch.zeros((nt, 3), dtype=torch.float64, device="cuda")
    print("case place=%g nt=%d" % (place, nt), flush=True)
    ccfmm.direct_targets_device(n, d_pos.data_ptr(), d_m.data_ptr(), nt, d_idx.data_ptr(), d_H.data_ptr(),
                                torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    H = d_H.cpu().numpy()
    if ok:
        assert rel_rms(H, ref.bruteforce_targets(pos[:n - 1], m[:n - 1], idx)) <= 1e-12
    else:
        assert np.isnan(H).all()


def train_inputs(rows, seed):
    rng = np.random.default_rng(seed)
    x = rng.normal(size=(rows, ccfmm.MLP_IN)).astype(np.float32)
    t = (-5.0 + rng.normal(size=(rows, ccfmm.MLP_OUT))).astype(np.float32)
    mask = (rng.random((rows, ccfmm.MLP_OUT)) < 0.9).astype(np.float32)
    return x, t, mask, selector.init_params(seed)


@pytest.mark.parametrize("rows", [1, 31, 32, 33, 500, 1025])
def test_training_step_block_edges(ref, rows):
    import torch

    x, t, mask, P = train_inputs(rows, rows)
    dx, dt, dm, dP = (torch.from_numpy(v).cuda() for v in (x, t, mask, P))
    dg = torch.empty_like(dP)
    dl = torch.empty(1, device="cuda")
    print("case rows=%d" % rows, flush=True)
    st = torch.cuda.current_stream().cuda_stream
    ccfmm.mlp_loss_grad(dP.data_ptr(), rows, dx.data_ptr(), dt.data_ptr(), dm.data_ptr(), dg.data_ptr(), dl.data_ptr(),
                        st)
    torch.cuda.synchronize()
    loss, g = ref.mlp_loss_grad(P.astype(np.float64), x.astype(np.float64), t.astype(np.float64),
                                mask.astype(np.float64), ccfmm.MLP_IN, ccfmm.MLP_HIDDEN, ccfmm.MLP_HIDDEN, ccfmm.MLP_OUT)
    assert abs(float(dl[0]) - loss) <= 1e-5 * abs(loss)
    assert rel_rms(dg.cpu().numpy(), g) <= 1e-4


def test_training_loops_on_several_streams():
    """Six loops queued side by side (more than the kept buffers), each with the
    result it has alone."""
    import torch

    rows, loops = 3000, 6
    sets = [[torch.from_numpy(v).cuda() for v in train_inputs(rows, 40 + k)] for k in range(loops)]
    streams = [torch.cuda.Stream() for _ in range(loops)]
    grads = [torch.empty_like(s[3]) for s in sets]
    alone = []
    for s in sets:
        g = torch.empty_like(s[3])
        ccfmm.mlp_loss_grad(s[3].data_ptr(), rows, s[0].data_ptr(), s[1].data_ptr(), s[2].data_ptr(), g.data_ptr(),
                            None, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        alone.append(g.clone())
    torch.cuda.synchronize()
    for rep in range(5):
        for s, g, st in zip(sets, grads, streams):
            ccfmm.mlp_loss_grad(s[3].data_ptr(), rows, s[0].data_ptr(), s[1].data_ptr(), s[2].data_ptr(), g.data_ptr(),
                                None, st.cuda_stream)
        torch.cuda.synchronize()
        for g, a in zip(grads, alone):
            assert torch.equal(g, a)


def test_captured_step_keeps_its_buffer():
    """A step captured on a third stream, after smaller and equal ones on two others,
    gives the eager gradient on every replay, with larger eager steps between."""
    import torch

    def step(s, rows, g, st):
        ccfmm.mlp_loss_grad(s[3].data_ptr(), rows, s[0].data_ptr(), s[1].data_ptr(), s[2].data_ptr(), g.data_ptr(), None,
                            st.cuda_stream)

    sets = {r: [torch.from_numpy(v).cuda() for v in train_inputs(r, r)] for r in (64, 5000, 9000)}
    grads = {r: torch.empty_like(sets[r][3]) for r in sets}
    a, b, c, d, e = (torch.cuda.Stream() for _ in range(5))
    torch.cuda.synchronize()
    step(sets[64], 64, grads[64], a)
    step(sets[5000], 5000, grads[5000], b)
    torch.cuda.synchronize()
    want = grads[5000].clone()
    torch.cuda.synchronize()
    graphs = []
    for st in (c, d):
        g, out = torch.cuda.CUDAGraph(), torch.empty_like(want)
        with torch.cuda.graph(g, stream=st):
            step(sets[5000], 5000, out, st)
        graphs.append((g, out))
        torch.cuda.synchronize()
        step(sets[5000], 5000, grads[5000], e)  # (a buffer for the next capture)
        torch.cuda.synchronize()
    for rep in range(4):
        for st in (a, b, c, d, e):
            step(sets[9000], 9000, grads[9000], st)
            torch.cuda.synchronize()
        for g, out in graphs:
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            print("case replay %d" % rep, flush=True)
            assert torch.equal(out, want)
