"""Scene dynamics (Sec. 3.4) and model expansion (Sec. 3.3) through the C
ABI: rigid object transforms and DC relighting within one FP32 rounding of
the oracle's FP64 results (static Gaussians and unit gains untouched bit for
bit), on ragged sizes and on the 3M-Gaussian model with the dynamics
harness's own object motion; appending to the active pool bit-exact for
parameters, moments and ID columns, and an optimizer that grows keeps
rendering like the oracle and trains the new Gaussians."""
import math

import numpy as np
import pytest
import torch

from gpu_util import compare_images, renderer_for
from paper_2604_02851_amd import native as N
from paper_2604_02851_amd import scenes as S
from paper_2604_02851_amd.native import DeviceParams

pytestmark = pytest.mark.gpu
F32 = np.float32


def _ulp_close(got, ref):
    """|got - ref| within one FP32 spacing of ref (both rounded from FP64)."""
    got, ref = np.asarray(got, F32), np.asarray(ref, F32)
    return np.abs(got.astype(np.float64) - ref) <= np.spacing(np.abs(ref)).astype(np.float64)


def _moves(rng, n_obj):
    out = []
    for _ in range(n_obj):
        q = rng.normal(size=4) * rng.uniform(0.5, 2.0)          # not normalised: the kernel normalises
        out.append((q, rng.normal(size=3), rng.normal(0, 0.3, size=3)))
    return out


@pytest.mark.parametrize("n,n_obj", [(1, 1), (1000, 7), (70001, 40)])
def test_object_transform_matches_oracle(oracle, n, n_obj):
    rng = np.random.default_rng(n)
    sc = S.draw_scene(rng, n, 3.0, 1)
    obj = rng.integers(-2, n_obj + 2, n).astype(np.int32)        # some static, some beyond the table
    moves = _moves(rng, n_obj)
    P = DeviceParams.from_scene(sc)
    ctx = N.Context(0)
    ctx.object_transform(P, torch.from_numpy(obj).cuda(), N.transforms_tensor(moves), n_obj)
    torch.cuda.synchronize()
    ref_m, ref_q = oracle.object_transform(sc.mean, sc.quat, obj, [(np.asarray(q, F32), np.asarray(p, F32),
                                                                   np.asarray(t, F32)) for q, p, t in moves])
    got = P.to_scene()
    assert _ulp_close(got.mean, ref_m).all() and _ulp_close(got.quat, ref_q).all()
    static = (obj < 0) | (obj >= n_obj)
    assert np.array_equal(got.mean[:, static], sc.mean[:, static])
    assert np.array_equal(got.quat[:, static], sc.quat[:, static])
    for a, b in ((got.log_scale, sc.log_scale), (got.opacity_logit, sc.opacity_logit), (got.sh, sc.sh)):
        assert np.array_equal(a, b)                               # scales, opacity, SH untouched


def test_object_transform_full_size_harness_motion(oracle):
    """The 3M-Gaussian dynamics workload: the harness's 20 object moves
    (rotation about each object's centroid, translation) as engine
    transforms."""
    w = S.workload(5)
    sc = w.scene
    dyn = S.Dynamics(np.random.default_rng(77), sc)
    moved = sc.copy()
    moves, _ = dyn.step([moved])
    obj = np.full(sc.n, -1, np.int32)
    tf = []
    for k, (idx, axis, ang, tr) in enumerate(moves):
        obj[idx] = k
        c = sc.mean[:, idx].astype(np.float64).mean(1)
        tf.append((np.r_[math.cos(ang / 2), math.sin(ang / 2) * axis].astype(F32), c.astype(F32), tr.astype(F32)))
    P = DeviceParams.from_scene(sc)
    ctx = N.Context(0)
    ctx.object_transform(P, torch.from_numpy(obj).cuda(), N.transforms_tensor(tf), len(tf))
    torch.cuda.synchronize()
    ref_m, ref_q = oracle.object_transform(sc.mean, sc.quat, obj, tf)
    got = P.to_scene()
    assert _ulp_close(got.mean, ref_m).all() and _ulp_close(got.quat, ref_q).all()
    # and the harness's own host update agrees to FP32 accuracy
    assert np.allclose(got.mean, moved.mean, atol=1e-5) and np.allclose(got.quat, moved.quat, atol=1e-5)


@pytest.mark.parametrize("channels", [1, 3])
@pytest.mark.parametrize("n", [1, 777, 100003])
def test_relight_dc_matches_oracle(oracle, channels, n):
    rng = np.random.default_rng(n + channels)
    sc = S.draw_scene(rng, n, 1.0, 2)
    gain = rng.uniform(0.3, 1.8, (channels, n)).astype(F32)
    gain[:, rng.random(n) < 0.4] = 1.0
    P = DeviceParams.from_scene(sc)
    ctx = N.Context(0)
    ctx.relight_dc(P, torch.from_numpy(gain).cuda(), channels)
    torch.cuda.synchronize()
    ref = oracle.relight_dc(sc.sh, gain)
    got = P.to_scene().sh
    assert _ulp_close(got, ref).all()
    unit = gain == 1.0
    for c in range(3):
        g = unit[c if channels == 3 else 0]
        assert np.array_equal(got[c, g], sc.sh[c, g])
    assert np.array_equal(got[3:], sc.sh[3:])


@pytest.mark.parametrize("n,na,k", [(1000, 600, 300), (513, 513, 1), (400, 0, 77), (300, 120, 0), (0, 0, 50)])
def test_append_bit_exact(oracle, n, na, k):
    rng = np.random.default_rng(n + k)
    old = S.draw_scene(rng, n, 1.0, 3)
    add = S.draw_scene(rng, k, 1.0, 3)
    rows = lambda sc, m: [a.reshape(int(np.prod(a.shape[:-1])), m) for _, a in sc.tensors()]
    mk = lambda m: DeviceParams(*[torch.from_numpy(rng.normal(size=t.shape[:-1] + (m,)).astype(F32)).cuda()
                                  for _, t in old.tensors()], 3)
    Po, Pa = DeviceParams.from_scene(old), DeviceParams.from_scene(add)
    mo, vo = mk(na), mk(na)
    Pn = DeviceParams.zeros(n + k, 3)
    mn, vn = DeviceParams.zeros(na + k, 3), DeviceParams.zeros(na + k, 3)
    mn.mean.fill_(5.0)                                              # must be overwritten with zeros
    ids_o = torch.arange(n, dtype=torch.int32, device="cuda") * 3
    ids_a = torch.arange(k, dtype=torch.int32, device="cuda") - 1000
    ids_n = torch.full((n + k,), -7, dtype=torch.int32, device="cuda")
    ctx = N.Context(0)
    ctx.append(Po, Pa, Pn, na, moments=(mo, vo, mn, vn), cols=[(ids_o, ids_a, ids_n)])
    torch.cuda.synchronize()
    for a, b, c in zip(rows(Pn.to_scene(), n + k), rows(old, n), rows(add, k)):
        assert np.array_equal(a, oracle.append_rows(b, c, na))
    for got, src in ((mn, mo), (vn, vo)):
        for a, b in zip(rows(got.to_scene(), na + k), rows(src.to_scene(), na)):
            assert np.array_equal(a, oracle.append_rows(b, np.zeros((b.shape[0], k), F32), na))
    assert np.array_equal(ids_n.cpu().numpy(), oracle.append_rows(ids_o.cpu().numpy(), ids_a.cpu().numpy(), na))


@pytest.mark.parametrize("n,na,k", [(4099, 1030, 5), (2050, 2050, 1), (1024, 0, 1024), (3, 1, 2), (2047, 1023, 3)])
def test_append_across_quads_of_shifted_rows(n, na, k):
    """Rows whose 16-byte quads straddle row ends and the seams between old,
    added and frozen elements, into destinations off a 16-byte boundary."""
    g = torch.Generator(device="cuda").manual_seed(n + na + k)
    ctx = renderer_for(S.small_workload(1, 8, 1.0, 0, [(16, 16)], dist=3.0)).ctx

    def mk(m, shift=0):
        rows = [(3,), (3,), (4,), (), (12,)]
        return DeviceParams(*[torch.randn(int(np.prod(r, dtype=int)) * m + shift, device="cuda", generator=g)[shift:]
                              .view(*r, m) for r in rows], 1)
    old, add, new = mk(n), mk(k, 1), mk(n + k, 3)
    mo, vo, mn, vn = mk(na, 2), mk(na), mk(na + k, 1), mk(na + k)
    ctx.append(old, add, new, na, moments=(mo, vo, mn, vn))
    torch.cuda.synchronize()
    for o, a, d in zip(old.tensors(), add.tensors(), new.tensors()):
        assert torch.equal(d, torch.cat([o[..., :na], a, o[..., na:]], -1))
    for src, dst in ((mo, mn), (vo, vn)):
        for o, d in zip(src.tensors(), dst.tensors()):
            assert torch.equal(d, torch.cat([o, torch.zeros_like(d[..., :k])], -1))


def test_invalid_append_is_refused():
    rng = np.random.default_rng(1)
    Po = DeviceParams.from_scene(S.draw_scene(rng, 10, 1.0, 1))
    Pa = DeviceParams.from_scene(S.draw_scene(rng, 4, 1.0, 1))
    ctx = N.Context(0)
    with pytest.raises(N.GsError):
        ctx.append(Po, Pa, DeviceParams.zeros(13, 1), 5)            # wrong new size
    with pytest.raises(N.GsError):
        ctx.append(Po, Pa, DeviceParams.zeros(14, 1), 11)           # n_active beyond n
    with pytest.raises(N.GsError):
        ctx.append(Po, Pa, DeviceParams.zeros(14, 2), 5)            # SH degree differs
    m = DeviceParams.zeros(5, 1)
    with pytest.raises(N.GsError):                                  # moments of the wrong size
        ctx.append(Po, Pa, DeviceParams.zeros(14, 1), 5, moments=(m, m, DeviceParams.zeros(8, 1), m))


def test_growing_optimizer_renders_and_trains_new_gaussians(oracle):
    w = S.small_workload(160, 2500, 1.0, 3, [(96, 64), (64, 80)], dist=3.0)
    rng = np.random.default_rng(161)
    extra = S.draw_scene(rng, 400, 1.0, 3)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        _grow_and_train(oracle, w, extra, s)


def _grow_and_train(oracle, w, extra, s):
    from paper_2604_02851_amd.renderer import Optimizer
    r = renderer_for(w, tile=(32, 32), batch=128, ppt=4, wave_w=16, loss_mode=1)
    P = DeviceParams.from_scene(w.scene)
    r.fit_capacity(P)
    tgt = r.forward(DeviceParams.from_scene(w.extra["perturbed"]))[0].clone()
    opt = Optimizer(r, P, tgt, n_active=2000, stream=s)
    opt.ids = torch.arange(2500, dtype=torch.int32, device="cuda")
    opt.step()
    before = opt.params.to_scene()
    newp = opt.append(DeviceParams.from_scene(extra))
    assert opt.params is newp and newp.n == 2900 and opt.n_active == 2400 and r.n == 2900
    ids = opt.ids.cpu().numpy()
    assert ids[:2000].tolist() == list(range(2000)) and ids[2000:2400].tolist() == list(range(2500, 2900))
    assert ids[2400:].tolist() == list(range(2000, 2500))
    grown = newp.to_scene()
    # the grown model renders like the oracle's render of it
    img = r.forward(newp)[0].clone()
    s.synchronize()
    compare_images(oracle, S.Workload("grown", grown, w.cams, 16, {}), img.cpu().numpy())
    for _ in range(2):
        opt.step()
    s.synchronize()
    after = opt.params.to_scene()
    # the appended Gaussians train, the frozen pool does not move
    assert not np.array_equal(after.mean[:, 2000:2400], grown.mean[:, 2000:2400])
    assert np.array_equal(after.mean[:, 2400:], before.mean[:, 2000:])
    assert np.array_equal(after.sh[:, 2400:], before.sh[:, 2000:])
    # the captured graph path works at the new size
    opt.capture()
    opt.replay()
    s.synchronize()
    assert np.isfinite(opt.loss.item())
