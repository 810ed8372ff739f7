"""The build without allocation (ac_alpha_complex_noalloc) through the C ABI
against ac_alpha_complex_device, the entry point whose kernels it shares:
two calls in a row on one device (the second with a smaller input) give
exactly the rows and Sizes of the allocating call; the smaller one is also
checked against the oracle. Output buffers that are too small are reported
with the counts needed and left untouched.
"""
import numpy as np
import pytest

import oracle
import synth
from parity import assert_same_complex

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def acx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1908_05944_amd as m
    return m


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to("cuda:0")


def _buffers(caps, fill=-7):
    import torch
    simp = [torch.full((c, d + 1), fill, dtype=torch.int32, device="cuda:0") for d, c in enumerate(caps)]
    size = [torch.full((c,), float(fill), dtype=torch.float64, device="cuda:0") for c in caps]
    return simp, size


def _reference(acx, X, R, alpha, opts):
    c = acx.ac_alpha_complex_device(X, R, alpha, options=opts)
    out = [(c.simplices(d), c.sizes(d)) for d in range(4)]
    c.close()
    return out


def _check_same(counts, simp, size, ref, what):
    import torch
    torch.cuda.synchronize()
    for d in range(4):
        rows, sz = ref[d]
        assert counts[d] == len(rows), (what, d, counts[d], len(rows))
        got = simp[d][: counts[d]].cpu().numpy()
        assert np.array_equal(got, rows), (what, d)
        # the same kernels compute the Sizes: bit-identical
        assert np.array_equal(size[d][: counts[d]].cpu().numpy().view(np.int64), sz.view(np.int64)), (what, d)


@pytest.mark.parametrize("sas", [False, True])
def test_two_calls_against_allocating_entry(acx, sas):
    # solvent-accessible radii give about ten times the candidates per ball:
    # a smaller molecule keeps the build within the fixed scratch
    big = synth.molecule(6000 if sas else 20000, 71, sas=sas)
    small = synth.molecule(3000, 72, sas=sas)
    for alpha, opts in ((0.0, None), (1.0, {"cell_order": 1})):
        refs = []
        for m in (big, small):
            X, R = _dev(m.xyz), _dev(m.radii)
            refs.append((X, R, _reference(acx, X, R, alpha, opts)))
        # one set of output buffers, sized for the larger result plus slack
        caps = [max(len(refs[0][2][d][0]), len(refs[1][2][d][0])) + 5 for d in range(4)]
        simp, size = _buffers(caps)
        for k, (X, R, ref) in enumerate(refs):
            print(f"[case] noalloc call {k}: n={X.shape[0]} sas={sas} alpha={alpha} opts={opts}", flush=True)
            counts = acx.ac_alpha_complex_noalloc(X, R, alpha, simp, size, options=opts)
            _check_same(counts, simp, size, ref, f"call {k}")
        # the smaller input against the oracle as well
        got_rows = [simp[d][: counts[d]].cpu().numpy() for d in range(4)]
        got_size = [size[d][: counts[d]].cpu().numpy() for d in range(4)]
        want = oracle.alpha_complex(small.xyz, small.radii, alpha)

        class _Got:
            def simplices(self, d):
                return got_rows[d]

            def sizes(self, d):
                return got_size[d]

            def counts(self):
                return [len(r) for r in got_rows]

        assert_same_complex(_Got(), want, f"noalloc small sas={sas} alpha={alpha}")


def test_too_small_output_is_reported_and_untouched(acx):
    import torch
    m = synth.molecule(2000, 73)
    X, R = _dev(m.xyz), _dev(m.radii)
    ref = _reference(acx, X, R, 0.0, None)
    need = [len(ref[d][0]) for d in range(4)]
    caps = list(need)
    caps[2] -= 1  # one triangle short
    simp, size = _buffers(caps)
    print("[case] noalloc with a short triangle buffer", flush=True)
    with pytest.raises(acx.CapacityError) as ei:
        acx.ac_alpha_complex_noalloc(X, R, 0.0, simp, size)
    assert ei.value.counts == need
    torch.cuda.synchronize()
    for d in range(4):
        assert bool((simp[d] == -7).all()) and bool((size[d] == -7.0).all()), d
    # then a call with room for the result succeeds on the same scratch
    simp, size = _buffers(need)
    counts = acx.ac_alpha_complex_noalloc(X, R, 0.0, simp, size)
    _check_same(counts, simp, size, ref, "after a capacity error")


def test_argument_errors(acx):
    m = synth.molecule(500, 74)
    X, R = _dev(m.xyz), _dev(m.radii)
    simp, size = _buffers([600, 2000, 2000, 1000])
    with pytest.raises(acx.AlphaCxError) as ei:
        acx.ac_alpha_complex_noalloc(X, R, 0.0, simp, size, options={"profile": 1})
    assert ei.value.status == 1
    with pytest.raises(acx.AlphaCxError) as ei:
        acx.ac_alpha_complex_noalloc(X, R, float("nan"), simp, size)
    assert ei.value.status == 1


def test_input_beyond_the_scratch_is_refused(acx):
    """A build that needs more than the fixed scratch stops with a capacity
    error (nothing written to the outputs), and the next call works."""
    import torch
    big = synth.molecule(60000, 75, sas=True)
    X, R = _dev(big.xyz), _dev(big.radii)
    simp, size = _buffers([64, 64, 64, 64])
    print("[case] noalloc beyond the scratch: 60000 solvent-accessible balls", flush=True)
    with pytest.raises(acx.AlphaCxError) as ei:
        acx.ac_alpha_complex_noalloc(X, R, 0.0, simp, size)
    assert ei.value.status == 6 and "scratch" in ei.value.detail
    torch.cuda.synchronize()
    for d in range(4):
        assert bool((simp[d] == -7).all()), d
    m = synth.molecule(1000, 76)
    X, R = _dev(m.xyz), _dev(m.radii)
    ref = _reference(acx, X, R, 0.0, None)
    simp, size = _buffers([len(ref[d][0]) for d in range(4)])
    counts = acx.ac_alpha_complex_noalloc(X, R, 0.0, simp, size)
    _check_same(counts, simp, size, ref, "after a scratch overflow")


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_outputs_aligned_as_their_elements_only(acx, shift):
    """Output arrays that start `shift` int32 (one float64) past a 16-byte line, as
    slices of one buffer do; what lies around the rows is not touched."""
    import torch
    m = synth.molecule(4000, 77)
    X, R = _dev(m.xyz), _dev(m.radii)
    ref = _reference(acx, X, R, 1.0, None)
    simp, size, around = [], [], []
    for d in range(4):
        k = len(ref[d][0])
        a = torch.full((k * (d + 1) + 8,), -7, dtype=torch.int32, device="cuda:0")
        z = torch.full((k + 2,), -7.0, dtype=torch.float64, device="cuda:0")
        simp.append(a[shift:shift + k * (d + 1)].view(k, d + 1))
        size.append(z[1:1 + k])
        around.append((a, z, shift + k * (d + 1)))
        assert simp[d].data_ptr() % 16 == 4 * shift and size[d].data_ptr() % 16 == 8
    print(f"[case] noalloc outputs {shift} int32 past a line", flush=True)
    counts = acx.ac_alpha_complex_noalloc(X, R, 1.0, simp, size)
    _check_same(counts, simp, size, ref, f"shift {shift}")
    for a, z, end in around:
        assert bool((a[:shift] == -7).all()) and bool((a[end:] == -7).all())
        assert float(z[0]) == -7.0 and float(z[-1]) == -7.0


@pytest.mark.parametrize("k", [500, 4000, 5000])
def test_many_pairs_and_few_triangles(acx, k):
    """A ball with thousands of small ones around it, the least and the last by id:
    more pairs of its edges than the scratch has room for, and few triangles."""
    i = np.arange(k) + 0.5
    phi, z = np.pi * (1 + 5 ** 0.5) * i, 1 - 2 * i / k
    p = np.stack([np.cos(phi) * np.sqrt(1 - z * z), np.sin(phi) * np.sqrt(1 - z * z), z], -1) * 8.2
    p += np.random.RandomState(k).uniform(-0.02, 0.02, p.shape)
    for last in (False, True):
        xyz, rad = np.vstack([[0, 0, 0], p]), np.append(7.9, np.full(k, 0.33))
        if last:
            xyz, rad = xyz[::-1], rad[::-1]
        X, R = _dev(xyz), _dev(rad)
        ref = _reference(acx, X, R, 0.0, None)
        simp, size = _buffers([len(ref[d][0]) for d in range(4)])
        print(f"[case] noalloc hub of {k}, last={last}", flush=True)
        counts = acx.ac_alpha_complex_noalloc(X, R, 0.0, simp, size)
        _check_same(counts, simp, size, ref, f"hub {k}")


@pytest.mark.parametrize("n,large,radius", [(416000, 1, 2.75), (416000, 1, 5.0), (9001, 200, 2.75), (9001, 8, 3.4)])
def test_few_large_balls(acx, n, large, radius):
    """One large ball does not take the scratch of many atoms; some side by side whose
    rows outgrow their slots."""
    m = synth.molecule(n, 36)
    rad = m.radii.copy()
    rad[np.argsort(((m.xyz - m.xyz.mean(0)) ** 2).sum(1))[:large]] = radius
    X, R = _dev(m.xyz), _dev(rad)
    ref = _reference(acx, X, R, 0.0, None)
    simp, size = _buffers([len(ref[d][0]) for d in range(4)])
    print(f"[case] noalloc {n} with {large} of {radius} A", flush=True)
    counts = acx.ac_alpha_complex_noalloc(X, R, 0.0, simp, size)
    _check_same(counts, simp, size, ref, f"{large} of {radius}")
