"""GPU parity of dpsgd_grad in fp32 arithmetic (least squares, softmax regression, ReLU MLP)
against the CPU oracle: Algorithm 1 step 3, minibatch mean (footnote [a]).  1e-5 relative."""
import numpy as np
import pytest
import torch

import oracle
from paper_1705_09056_amd import binding as B
from paper_1705_09056_amd import synth
from paper_1705_09056_amd.configs import CONFIGS, MODEL_LSQ, MODEL_MLP, MODEL_SOFTMAX, shrink

from conftest import ELEM, check_close, max_err, rel_err
from gpu_util import bf16_dev, from_dev, oracle_topo_for, to_dev, topo_for

pytestmark = pytest.mark.gpu
TOL = 1e-5


def grad_case(cfg, ld, k=0, spread=0.5, bf16_inputs=False):
    d = synth.model_dim(cfg.model_kind, cfg.widths)
    X = synth.make_replicas(cfg, spread=spread, key=k)
    if cfg.model_kind in (MODEL_LSQ, MODEL_SOFTMAX):
        X = X + synth.rng(cfg.index, 99, k).standard_normal(X.shape).astype(np.float32) * np.float32(0.1)
    inp, tgt = synth.make_batch(cfg, k)
    if bf16_inputs:
        inp = synth.round_to_bf16(inp)
    Gref, lref = oracle.grad_all(cfg.model_kind, cfg.widths, X, inp, tgt)
    Xd = to_dev(X, ld)
    Gd = torch.full_like(Xd, 777.0)
    loss = torch.zeros(cfg.n, device="cuda")
    inp_d = bf16_dev(inp) if bf16_inputs else torch.from_numpy(inp).cuda()
    tgt_d = torch.from_numpy(tgt).cuda()
    model = B.Model(cfg.model_kind, cfg.widths, compute_bf16=False)
    print(f"grad f32 {cfg.name} widths={cfg.widths} n={cfg.n} B={cfg.batch} ld={ld}", flush=True)
    with B.Dpsgd(cfg.n, d, topo_for(cfg), cfg.gamma, ld=ld) as ctx:
        ctx.grad(model, Xd, inp_d, tgt_d, cfg.batch, Gd, loss, input_is_bf16=bf16_inputs)
        torch.cuda.synchronize()
    check_close(from_dev(Gd, d), Gref, TOL, "G")
    assert rel_err(loss.cpu().numpy(), lref) < TOL


def test_lsq_config0():
    grad_case(CONFIGS[0], 64)


@pytest.mark.parametrize("feat,batch,n", [(1, 1, 1), (65, 33, 5), (1000, 70, 3)])
def test_lsq_ragged(feat, batch, n):
    cfg = shrink(CONFIGS[0], widths=(feat,), batch=batch, n=n)
    grad_case(cfg, synth.padded_stride(feat))
    grad_case(cfg, feat)


def test_softmax_config1():
    cfg = CONFIGS[1]
    grad_case(cfg, synth.padded_stride(30730))


@pytest.mark.parametrize("widths,batch,n", [((70, 3), 9, 4), ((129, 10), 65, 2), ((64, 1), 64, 3),
                                            # 256 inputs or more and at most 16 outputs: the forward that splits a pair of
                                            # sample rows over four waves (odd minibatch: a last row alone; 259 inputs:
                                            # no 16-byte loads; 1100: a ragged last 1 KB piece) and the bias gradient
                                            # with a wave per output
                                            ((300, 7), 33, 3), ((259, 16), 5, 2), ((1100, 10), 64, 2)])
def test_softmax_ragged(widths, batch, n):
    cfg = shrink(CONFIGS[1], widths=widths, batch=batch, n=n)
    d = synth.model_dim(MODEL_SOFTMAX, widths)
    grad_case(cfg, d)
    grad_case(cfg, synth.padded_stride(d))


@pytest.mark.parametrize("widths,batch,n", [((256, 16), 1, 2), ((1025, 10), 17, 3), ((2049, 3), 33, 2), ((3139, 10), 16, 2),
                                            ((300, 257, 1), 18, 2), ((300, 12, 5), 9, 2)])
def test_class_layer_contractions_of_every_length(widths, batch, n):
    """One, two and three pieces of 64 elements per wave, a second round of pieces, ragged last pieces and sample tiles;
    a hidden layer of as few outputs keeps its own kernel."""
    cfg = shrink(CONFIGS[2 if len(widths) > 2 else 1], widths=widths, batch=batch, n=n, bf16=False)
    d = synth.model_dim(cfg.model_kind, widths)
    grad_case(cfg, d)
    grad_case(cfg, synth.padded_stride(d))


@pytest.mark.parametrize("widths,batch,n", [((48, 40, 10), 16, 3), ((100, 70, 33, 5), 37, 4), ((3072, 128, 10), 128, 2)])
def test_mlp_fp32(widths, batch, n):
    cfg = shrink(CONFIGS[2], widths=widths, batch=batch, n=n, bf16=False)
    d = synth.model_dim(MODEL_MLP, widths)
    grad_case(cfg, synth.padded_stride(d), spread=0.3)


@pytest.mark.parametrize("widths,batch,n", [
    ((3, 2, 3), 5, 2),            # extents below the 4 elements of a load
    ((5, 4, 4), 1, 1),            # exactly 4, one sample
    ((64, 32, 16), 32, 2),        # whole tiles, few of them: 32 x 32, four waves each
    ((515, 130, 7), 40, 9),       # a long ragged contraction on small tiles
    ((640, 97, 70, 33), 33, 160), # 32-row tiles and 64-row tiles side by side, a contraction of 640 in two waves
    ((513, 1030, 10), 65, 16),    # a multiple of 8 workers (tiles of a worker on one XCD), every extent ragged
])
def test_mlp_fp32_tiles_and_remainders(widths, batch, n):
    """The matrix-instruction product behind forward, data and weight gradient: every tile shape of its dispatch, with
    remainders in all three directions, on padded and on odd row strides."""
    cfg = shrink(CONFIGS[2], widths=widths, batch=batch, n=n, bf16=False)
    d = synth.model_dim(MODEL_MLP, widths)
    grad_case(cfg, synth.padded_stride(d), spread=0.3)
    grad_case(cfg, d | 1, spread=0.3)


@pytest.mark.parametrize("widths,batch,n", [((5, 191, 10), 33, 130), ((67, 255, 10), 65, 60), ((100, 64, 10), 64, 400)])
def test_forward_of_many_tiles_of_64_by_64(widths, batch, n):
    """A hidden layer whose 64 x 64 tiles fill the chip more than once and in half the rounds of 64 x 32 ones: a contraction
    shorter than a chunk, and ones with a remainder; rows and columns that end inside a tile, and whole tiles."""
    cfg = shrink(CONFIGS[2], widths=widths, batch=batch, n=n, bf16=False)
    d = synth.model_dim(MODEL_MLP, widths)
    grad_case(cfg, synth.padded_stride(d), spread=0.3)
    grad_case(cfg, d | 1, spread=0.3)


@pytest.mark.parametrize("widths,batch,n", [
    ((64, 300, 2), 70, 3),        # data gradient of two classes: a contraction of 2
    ((20, 65, 3), 64, 2),         # ... of 3, an input more than a tile
    ((9, 3, 4), 33, 2),           # three inputs of the data gradient
])
def test_two_and_three_classes(widths, batch, n):
    cfg = shrink(CONFIGS[2], widths=widths, batch=batch, n=n, bf16=False)
    d = synth.model_dim(MODEL_MLP, widths)
    grad_case(cfg, synth.padded_stride(d), spread=0.3)
    grad_case(cfg, d | 1, spread=0.3)


def test_weight_gradient_of_more_rows_than_32_row_tiles_fit_a_grid():
    """A hidden layer of 2 097 153 outputs on 3 inputs: its weight gradient has more rows than 65535 tiles of 32.  No
    unit's input lies within 1e-5 of zero (bias 1, weights of 0.1), so no sign hangs on a rounding.  Tolerance: a logit is a sum of 2^21 terms of
    1e-4 (0.15 in all) in chains of 2^21 / (16 waves x 4) and errs by about sqrt(2^15) 2^-24 of that, 1.6e-6; softmax and
    the bias gradients add a few roundings."""
    I, O, C, batch = 3, 32 * 65535 + 33, 2, 4
    d = O * I + O + C * O + C
    g = torch.Generator().manual_seed(17)
    x = torch.cat([0.1 * torch.randn(O * I, generator=g), torch.ones(O), 1e-4 * torch.randn(C * O, generator=g), torch.zeros(C)])
    a = torch.randn(batch, I, generator=g)
    y = torch.tensor([0, 1, 1, 0], dtype=torch.int32)
    xr = x.double().requires_grad_(True)
    h = torch.relu(a.double() @ xr[:O * I].view(O, I).t() + xr[O * I:O * I + O])
    assert float((a.double() @ xr[:O * I].view(O, I).t() + 1).abs().min()) > 1e-5
    z = h @ xr[O * I + O:O * I + O + C * O].view(C, O).t() + xr[d - C:]
    ref = torch.nn.functional.cross_entropy(z, y.long())
    ref.backward()
    X, G, loss = x.cuda()[None], torch.full((1, d), 777.0, device="cuda"), torch.zeros(1, device="cuda")
    print("launching", flush=True)
    with B.Dpsgd(1, d, B.Topology.complete(), 0.1, ld=d) as ctx:
        ctx.grad(B.Model(MODEL_MLP, (I, O, C), compute_bf16=False), X, a.cuda()[None], y.cuda()[None], batch, G, loss)
        torch.cuda.synchronize()
    assert abs(float(loss) - float(ref)) < 1e-5
    got, want = G[0].cpu().double(), xr.grad
    for lo, hi in ((0, O * I), (O * I, O * I + O), (O * I + O, d - C), (d - C, d)):
        assert float((got[lo:hi] - want[lo:hi]).norm() / want[lo:hi].norm()) < 2e-5


def test_bf16_inputs_with_fp32_arithmetic():
    cfg = shrink(CONFIGS[2], widths=(96, 50, 10), batch=24, n=3, bf16=True)
    d = synth.model_dim(MODEL_MLP, cfg.widths)
    grad_case(cfg, synth.padded_stride(d), bf16_inputs=True)


def test_dimension_mismatch_is_rejected():
    cfg = CONFIGS[0]
    Xd = to_dev(np.zeros((cfg.n, 64), np.float32))
    Gd = torch.zeros_like(Xd)
    inp = torch.zeros(cfg.n * 32 * 64, device="cuda")
    tgt = torch.zeros(cfg.n * 32, device="cuda")
    with B.Dpsgd(cfg.n, 64, B.Topology.ring(), 0.1) as ctx:
        with pytest.raises(B.DpsgdError) as e:
            ctx.grad(B.Model(B.MODEL_LSQ, [32]), Xd, inp[: cfg.n * 32 * 32], tgt, 32, Gd)
        assert e.value.status == B.EINVAL
        with pytest.raises(B.DpsgdError) as e:
            ctx.grad(B.Model(B.MODEL_LSQ, [64]), Xd, inp, tgt, 32, Xd)   # G aliases X
        assert e.value.status == B.EINVAL


def run_trajectory(cfg, K, ld):
    """Both gates: (i) single step from the oracle's X_k every iteration; (ii) free-running."""
    d = synth.model_dim(cfg.model_kind, cfg.widths)
    topo_o = oracle_topo_for(cfg)
    model = B.Model(cfg.model_kind, cfg.widths)
    Xo = synth.make_replicas(cfg).astype(np.float64)
    Xfree = to_dev(Xo, ld)
    Gd = torch.full_like(Xfree, 777.0)
    worst_step = worst_traj = worst_elem = 0.0
    with B.Dpsgd(cfg.n, d, topo_for(cfg), cfg.gamma, ld=ld) as ctx:
        for k in range(K):
            inp, tgt = synth.make_batch(cfg, k)
            inp_d, tgt_d = torch.from_numpy(inp).cuda(), torch.from_numpy(tgt).cuda()
            Xn, _, _ = oracle.iteration(cfg.model_kind, cfg.widths, topo_o, np.float32(cfg.gamma), Xo, inp, tgt)
            # (i) one GPU step from the oracle's iterate
            Xs = to_dev(Xo, ld)
            ctx.grad(model, Xs, inp_d, tgt_d, cfg.batch, Gd)
            ctx.mix_step(Xs, Gd, Xs)
            worst_step = max(worst_step, rel_err(from_dev(Xs, d), Xn))
            worst_elem = max(worst_elem, max_err(from_dev(Xs, d), Xn))
            # (ii) the GPU's own trajectory
            ctx.grad(model, Xfree, inp_d, tgt_d, cfg.batch, Gd)
            ctx.mix_step(Xfree, Gd, Xfree)
            if k % 10 == 9 or k == K - 1:
                worst_traj = max(worst_traj, rel_err(from_dev(Xfree, d), Xn))
                worst_elem = max(worst_elem, max_err(from_dev(Xfree, d), Xn))
            Xo = Xn
        xbar = torch.zeros(d, device="cuda")
        ctx.mean(Xfree, xbar)
        torch.cuda.synchronize()
    print(f"{cfg.name}: K={K} worst single-step {worst_step:.2e}, worst trajectory {worst_traj:.2e}, worst element "
          f"{worst_elem:.2e} rms", flush=True)
    assert worst_step < TOL
    assert worst_traj < TOL
    assert worst_elem < ELEM * TOL
    check_close(xbar.cpu().numpy(), oracle.mean(Xo), TOL, "xbar")


def test_trajectory_config0_full():
    run_trajectory(CONFIGS[0], CONFIGS[0].iters, 64)


def test_trajectory_config1_full():
    run_trajectory(CONFIGS[1], CONFIGS[1].iters, synth.padded_stride(30730))


@pytest.mark.parametrize("feat,batch,n", [(3, 70, 5),      # less than 4 features: a kernel of their own
                                          (4, 9, 3), (7, 8, 2),     # one and two quads of features, the second clamped
                                          (63, 17, 4), (257, 1, 2), (1023, 40, 3), (300, 1000, 2),
                                          (64, 335, 3), (64, 336, 3),     # the last of one launch, the first of two
                                          (511, 46, 2), (512, 46, 2),     # eight lanes per sample, a wave from 512 features on
                                          (64, 8, 2), (64, 9, 2), (300, 24, 2), (300, 25, 2),     # ... and for few samples
                                          (64, 11, 2), (64, 12, 2),       # the last of a thread per feature, the first of eight waves
                                          (4, 2731, 2), (7, 2729, 2), (63, 141, 4), (9700, 1, 2)])
def test_lsq_gradient_of_every_length(feat, batch, n):
    cfg = shrink(CONFIGS[0], widths=(feat,), batch=batch, n=n)
    grad_case(cfg, feat)


def test_lsq_gradient_of_more_workers_than_a_grid_holds():
    """65 537 workers whose samples do not fit LDS: the two launches of any other number of workers, in two parts.  Tolerance: a
    residual is 64 lanes' chains of 52 products of a random sign, an error of about sqrt(26) 2^-25 = 1.5e-7, and a few roundings;
    one chain over the 3200 features errs by sqrt(1600) 2^-25 = 1.2e-6."""
    n, batch, feat = 65537, 8, 3200
    g = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randn(n, feat, generator=g, device="cuda")
    A = torch.randn(n, batch, feat, generator=g, device="cuda")
    y = torch.randn(n, batch, generator=g, device="cuda")
    G, loss = torch.full_like(X, 777.0), torch.zeros(n, device="cuda")
    print("launching", flush=True)
    with B.Dpsgd(n, feat, B.Topology.ring(), 0.1, ld=feat) as ctx:
        ctx.grad(B.Model(MODEL_LSQ, [feat]), X, A, y, batch, G, loss)
        torch.cuda.synchronize()
    for w in (0, 1, 32768, 65534, 65535, 65536):
        a, r = A[w].double(), A[w].double() @ X[w].double() - y[w].double()
        want = a.t() @ r / batch
        assert float((G[w].double() - want).norm() / want.norm()) < 4e-7, w
        assert float(loss[w]) == pytest.approx(float(0.5 * (r * r).mean()), rel=1e-6)
    assert not bool((G == 777.0).any())


@pytest.mark.parametrize("feat,batch,n,topo", [(64, 32, 8, "ring"), (5, 3, 3, "ring"), (73, 20, 16, "complete"), (16, 9, 12, "torus"),
                                               (120, 31, 9, "ring"),      # 35 919 floats of LDS of 36 864
                                               (120, 32, 9, "ring"),      # one sample more does not fit: two launches and the mix
                                               # the consensus distance by groups of rows: of unequal size, one row or two each, at most
                                               # half as many as rows, 224 columns
                                               (8, 2, 33, "ring"), (4, 1, 256, "ring"), (31, 3, 33, "complete"), (32, 1, 32, "ring"), (17, 2, 48, "torus"),
                                               (224, 1, 32, "ring"),
                                               # elements of a thread, the most that one launch takes and one more: by a row's non-zeros, by the
                                               # workers of a ring, by themselves
                                               (160, 9, 12, "complete"), (73, 3, 15, "complete"), (16, 2, 128, "complete"), (17, 2, 128, "complete"),
                                               (30, 2, 136, "ring"), (31, 2, 136, "ring"), (896, 2, 8, "ring"), (897, 2, 8, "ring")])
def test_lsq_step_in_one_launch(feat, batch, n, topo):
    """dpsgd_step of a problem that fits one workgroup: update, gradient, loss and consensus distance against the oracle, at
    both sides of what fits, and the gradient it leaves against dpsgd_grad's."""
    cfg = shrink(CONFIGS[0], widths=(feat,), batch=batch, n=n)
    X = synth.make_replicas(cfg, spread=0.5) + synth.rng(0, 98).standard_normal((n, feat)).astype(np.float32) * np.float32(0.1)
    inp, tgt = synth.make_batch(cfg, 0)
    W = {"ring": oracle.ring, "complete": oracle.complete, "torus": lambda n: oracle.torus(3, n // 3)}[topo](n).with_fp32_values()
    Xref, Gref, lref = oracle.iteration(MODEL_LSQ, cfg.widths, W, np.float32(cfg.gamma), X, inp, tgt)
    tb = {"ring": B.Topology.ring, "complete": B.Topology.complete, "torus": lambda: B.Topology.torus(3, n // 3)}[topo]()
    Xd, inp_d, tgt_d = to_dev(X, feat + 3), torch.from_numpy(inp).cuda(), torch.from_numpy(tgt).cuda()
    G1, G2 = torch.full_like(Xd, 777.0), torch.full_like(Xd, 777.0)
    loss, cons = torch.zeros(n, device="cuda"), torch.zeros(1, device="cuda")
    model = B.Model(MODEL_LSQ, [feat])
    print(f"lsq step {feat} x {batch} x {n} {topo}", flush=True)
    with B.Dpsgd(n, feat, tb, cfg.gamma, ld=feat + 3) as ctx:
        ctx.grad(model, Xd, inp_d, tgt_d, batch, G1)
        ctx.step(model, Xd, inp_d, tgt_d, batch, G2, loss, cons)
        torch.cuda.synchronize()
    check_close(from_dev(Xd, feat), Xref, TOL, "X")
    check_close(from_dev(G2, feat), Gref, TOL, "G")
    check_close(from_dev(G2, feat), from_dev(G1, feat), TOL, "G of step and grad")
    assert rel_err(loss.cpu().numpy(), lref) < TOL
    m = float(((Xref - Xref.mean(0)) ** 2).sum() / n)
    assert float(cons) == pytest.approx(m, rel=TOL)


@pytest.mark.parametrize("feat,batch,n", [(4, 2000, 2), (9, 700, 2), (5, 1003, 3), (64, 32, 8)])
def test_lsq_step_adds_long_minibatches_in_64_bits(feat, batch, n):
    """The gradient that the one-launch step leaves is as near to the oracle's as dpsgd_grad's: sums of eight products in fp32, the
    rest in fp64.  Tolerance: the result is rounded twice and every residual once (2^-24 each at most, 6e-8, the latter averaging
    out), the eight-term sums add 8 * 2^-24 of a partial sum at random signs, less than 1e-7 of the norm over 32 samples and more;
    an fp32 chain over N samples errs by about sqrt(N / 2) 2^-25, 9e-7 at 2000."""
    cfg = shrink(CONFIGS[0], widths=(feat,), batch=batch, n=n)
    X = synth.make_replicas(cfg, spread=0.5) + synth.rng(0, 98).standard_normal((n, feat)).astype(np.float32) * np.float32(0.1)
    inp, tgt = synth.make_batch(cfg, 0)
    Gref, _ = oracle.grad_all(MODEL_LSQ, cfg.widths, X, inp, tgt)
    Xd, inp_d, tgt_d = to_dev(X), torch.from_numpy(inp).cuda(), torch.from_numpy(tgt).cuda()
    Gd = torch.full_like(Xd, 777.0)
    print(f"lsq step {feat} x {batch} x {n}", flush=True)
    with B.Dpsgd(n, feat, B.Topology.complete(), cfg.gamma, ld=feat) as ctx:
        ctx.step(B.Model(MODEL_LSQ, [feat]), Xd, inp_d, tgt_d, batch, Gd)
        torch.cuda.synchronize()
    err = rel_err(from_dev(Gd, feat), Gref)
    print(f"  rel err G {err:.2e}", flush=True)
    assert err < 3e-7


@pytest.mark.parametrize("widths,batch,n", [((4, 2), 1, 2), ((5, 17), 17, 3), ((63, 16), 16, 2), ((257, 26), 31, 3), ((1100, 32), 33, 2),
                                            ((300, 33), 20, 2), ((3, 26), 9, 2), ((2100, 26), 70, 9), ((130, 70, 26), 40, 3)])
def test_class_layers_of_every_width(widths, batch, n):
    """The two kernels of a class layer at the edges of what they take: 4 inputs, one and two tiles of outputs (33 outputs and 3
    inputs go to the tiled products), ragged sample tiles, pieces and last inputs."""
    cfg = shrink(CONFIGS[1], widths=widths, batch=batch, n=n) if len(widths) == 2 else \
        shrink(CONFIGS[2], widths=widths, batch=batch, n=n, bf16=False)
    grad_case(cfg, synth.model_dim(cfg.model_kind, widths))


@pytest.mark.parametrize("widths,batch,n", [((70, 1, 5), 9, 3), ((70, 1, 5), 4, 3), ((70, 1, 5), 3, 2), ((600, 1, 1, 5), 70, 300), ((3, 1, 2), 8, 2),
                                            ((70, 3, 10), 1, 2), ((129, 65, 33, 7), 67, 3), ((2, 130, 10), 33, 2),
                                            ((520, 1030, 64, 3), 200, 9)])
def test_hidden_bias_gradients_of_every_width(widths, batch, n):
    """A hidden layer's bias gradient comes from the last column of workgroups of its weight gradient: one output (whose deltas lie
    contiguously along the samples as well, in tiles that load four of them at a time from four samples on), part tiles, more samples than a thread's loads in flight."""
    grad_case(shrink(CONFIGS[2], widths=widths, batch=batch, n=n, bf16=False), synth.model_dim(MODEL_MLP, widths))
