"""The matrix exponential of the calibration and its gradient over the norms that change its form: fewer and more
polynomial blocks, one to eight applications per column block with up to two squarings, and squarings alone beyond that.

exp(S) carries a relative error of a few ||S|| 2^-53 on either side (S is skew, so ||exp(S)|| = 1 and an error of S adds at
most its own norm; the library's halvings double theirs back), and the reference's eigenvectors and the product with R0 some
50 x 2^-53 more: _exp_rtol. A polynomial one block short errs by 2e-14 to 1e-9 at the smaller norms here (the norm estimate
leaves a block to spare at the larger ones). A loss is an average of smooth functions of logits of order one: its relative
error is a few times that of the rotation; the gradient goes through both factors of the rotated products, the
exponential's derivative and differences of probabilities, some ten times that. No code flips at such errors (a rotated
value would have to lie within them of a rounding boundary)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import optr_oracle as P
from paper_2608_02691_amd import int2kv as K
from paper_2608_02691_amd import workloads as W

from _helpers import dev

pytestmark = pytest.mark.gpu


def _exp_rtol(A):
    return 6e-15 + 2.0 ** -52 * np.linalg.norm(A - A.T, 2)


def _rotation(A, R0):
    """R0 exp(A - A^T) in fp64, from the eigenvectors of the Hermitian i (A - A^T)."""
    w, U = np.linalg.eigh(1j * (A - A.T))
    return R0.astype(np.float64) @ ((U * np.exp(-1j * w)) @ U.conj().T).real


@pytest.mark.parametrize("scale", [1e-4, 0.003, 0.01, 0.03, 0.06, 0.1, 0.2, 0.4, 0.7, 3.0, 30.0])
def test_rotation_over_generator_norms(scale):
    """The rotation itself, as the key objective leaves it in the workspace (after the Gram matrices)."""
    H, Hq = 3, 3
    w = W.make_workload(1, batch=1, ctx=16, num_q_heads=Hq, num_kv_heads=H, d_model=64)
    rng = np.random.default_rng([8, int(1e4 * scale)])
    bits = lambda *s: dev(W.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32)))
    tr = K.OptrTraces(bits(20, H, 128), bits(20, H, 128), bits(20, Hq, 128), np.array([0, 20], np.int32))
    cfg = K.optr_config(H, Hq, 64, group_size=32, n_last=4, sink=0, recent=0)
    A = rng.standard_normal((H, 128, 128)) * scale
    A[1] *= 0.4
    A[2] *= 0.01  # the heads of one launch take different forms
    R0, mu, Wo, Ad = dev(w.R_k), torch.zeros((H, 128), device="cuda"), dev(w.W_o), dev(A)
    loss = torch.empty(H, dtype=torch.float64, device="cuda")
    n = K.int2kv_optr_workspace_bytes(cfg, tr)
    ws = torch.empty(n + 256, dtype=torch.uint8, device="cuda")
    ws = ws[-ws.data_ptr() % 256:]
    st = K.load_library().int2kv_optr_key_loss(
        ctypes.byref(cfg), ctypes.byref(tr.desc), R0.data_ptr(), mu.data_ptr(), Wo.data_ptr(), Ad.data_ptr(),
        loss.data_ptr(), None, ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    assert st == K.INT2KV_OK
    mat = 128 * 128 * 8
    R = ws[Hq * mat:(Hq + H) * mat].view(torch.float64).view(H, 128, 128).cpu().numpy()
    for h in range(H):
        ref = _rotation(A[h], w.R_k[h])
        err, tol = np.linalg.norm(R[h] - ref) / np.linalg.norm(ref), _exp_rtol(A[h])
        print(f"scale {scale} head {h}: {err:.1e} of {tol:.1e}", flush=True)
        assert err <= tol, (scale, h, err, tol)


@pytest.mark.parametrize("scale", [1e-4, 0.01, 0.1, 0.2, 0.7, 3.0, 30.0])
def test_objectives_and_gradients_over_generator_norms(scale):
    H, Hq = 2, 4
    print(f"\n[optr norms] {scale}", flush=True)
    w = W.make_workload(1, batch=1, ctx=16, num_q_heads=Hq, num_kv_heads=H, d_model=64)
    rng = np.random.default_rng(5)
    bits = lambda *s: W.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
    k, v, q, st = bits(70, H, 128), bits(70, H, 128), bits(70, Hq, 128), np.array([0, 40, 70], np.int32)
    mu = P.key_mean(k)
    cfg = K.optr_config(H, Hq, 64, group_size=32, n_last=12, sink=0, recent=0)
    A, Av = rng.standard_normal((2, H, 128, 128)) * scale
    Av[1] *= 0.01  # the heads of one launch take different forms
    tr = K.OptrTraces(dev(k), dev(v), dev(q), st)
    lk, gk = K.int2kv_optr_key_loss(cfg, tr, dev(w.R_k), dev(mu), dev(w.W_o), dev(A))
    lv, gv = K.int2kv_optr_value_loss(cfg, tr, dev(w.R_k), dev(A), dev(mu), dev(w.R_v), dev(w.W_o), dev(Av))
    kw = dict(group=32, n_last=12)
    for h in range(H):
        for got_l, got_g, gen, loss in (
                (lk, gk, A, lambda x: P.key_loss(x, w.R_k, k, v, q, st, mu, w.W_o, h, 2, clip=0.96, **kw)),
                (lv, gv, Av, lambda x: P.value_loss(x, w.R_v, v, st, P.key_probs(w.R_k, A[h], k, q, st, mu, h, 2,
                                                                                  clip=0.96, **kw),
                                                    w.W_o, h, 2, clip=0.92, **kw))):
            x = torch.from_numpy(gen[h].copy()).requires_grad_(True)
            ref = loss(x)
            ref.backward()
            g = x.grad.numpy()
            dl = abs(float(got_l[h]) / float(ref.detach()) - 1.0)
            dg = np.linalg.norm(got_g[h].cpu().numpy() - g) / np.linalg.norm(g)
            print(f"head {h}: loss {dl:.1e}, gradient {dg:.1e}", flush=True)
            e = _exp_rtol(A[h]) + _exp_rtol(gen[h])
            assert dl <= 4 * e and dg <= 32 * e, (scale, h, dl, dg, e)


@pytest.mark.parametrize("lens,sink,recent", [([40, 30], 0, 1000), ([50, 3, 41], 7, 30), ([64, 33], 16, 0)])
def test_few_or_no_int2_tokens(lens, sink, recent):
    """Only the tokens some query reads from INT2 are rotated and differentiated: windows that leave none at all, none in
    some sequences, or a count that is not a multiple of the sixteen tokens of a unit."""
    H, Hq = 2, 4
    w = W.make_workload(1, batch=1, ctx=16, num_q_heads=Hq, num_kv_heads=H, d_model=64)
    rng = np.random.default_rng(6)
    T = sum(lens)
    bits = lambda *s: W.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
    k, v, q, st = bits(T, H, 128), bits(T, H, 128), bits(T, Hq, 128), np.cumsum([0] + lens).astype(np.int32)
    mu = P.key_mean(k)
    cfg = K.optr_config(H, Hq, 64, group_size=128, n_last=12, sink=sink, recent=recent)
    A, Av = rng.standard_normal((2, H, 128, 128)) * 0.02
    tr = K.OptrTraces(dev(k), dev(v), dev(q), st)
    lk, gk = K.int2kv_optr_key_loss(cfg, tr, dev(w.R_k), dev(mu), dev(w.W_o), dev(A))
    lv, gv = K.int2kv_optr_value_loss(cfg, tr, dev(w.R_k), dev(A), dev(mu), dev(w.R_v), dev(w.W_o), dev(Av))
    kw = dict(group=128, n_last=12, sink=sink, recent=recent)
    for h in range(H):
        probs = P.key_probs(w.R_k, A[h], k, q, st, mu, h, 2, clip=0.96, **kw)
        for got_l, got_g, gen, loss in (
                (lk, gk, A, lambda x: P.key_loss(x, w.R_k, k, v, q, st, mu, w.W_o, h, 2, clip=0.96, **kw)),
                (lv, gv, Av, lambda x: P.value_loss(x, w.R_v, v, st, probs, w.W_o, h, 2, clip=0.92, **kw))):
            x = torch.from_numpy(gen[h].copy()).requires_grad_(True)
            ref = loss(x)
            ref.backward()
            g = x.grad.numpy()
            # absolute terms: with no INT2 token both are zero up to the rounding of the softmaxes' sums
            assert abs(float(got_l[h]) - float(ref.detach())) <= 1e-9 * abs(float(ref.detach())) + 1e-14
            assert np.linalg.norm(got_g[h].cpu().numpy() - g) <= 1e-7 * np.linalg.norm(g) + 1e-13


def test_inputs_of_any_alignment():
    """q, R^0, A, mu and W_O need no alignment beyond their types': one element past an aligned address, the losses and
    gradients are the same bits."""
    H, Hq, lens = 2, 4, [50, 41]
    w = W.make_workload(1, batch=1, ctx=16, num_q_heads=Hq, num_kv_heads=H, d_model=64)
    rng = np.random.default_rng(7)
    T = sum(lens)
    bits = lambda *s: W.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32))
    k, v, q, st = bits(T, H, 128), bits(T, H, 128), bits(T, Hq, 128), np.cumsum([0] + lens).astype(np.int32)
    mu = P.key_mean(k)
    cfg = K.optr_config(H, Hq, 64, group_size=32, n_last=12, sink=4, recent=9)
    A, Av = rng.standard_normal((2, H, 128, 128)) * 0.02

    def run(put):
        tr = K.OptrTraces(dev(k), dev(v), put(q), st)
        key = K.int2kv_optr_key_loss(cfg, tr, put(w.R_k), put(mu), put(w.W_o), put(A))
        value = K.int2kv_optr_value_loss(cfg, tr, put(w.R_k), put(A), put(mu), put(w.R_v), put(w.W_o), put(Av))
        return [x.cpu() for x in key + value]

    def shifted(a):
        x = dev(a)
        at = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")[1:].view(x.shape)
        at.copy_(x)
        assert at.data_ptr() % 16 == x.element_size()
        return at

    for aligned, odd in zip(run(dev), run(shifted)):
        assert torch.equal(aligned, odd)
