"""The library's host code against a stand-in for the HIP runtime
(fake_hip.cpp): what it launches, allocates and keeps at sizes, limits and
errors that a GPU test cannot bring about. No kernel runs, and every case is a
process of its own."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = '''
import ctypes as C
import sys
F = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
for f in ("fake_live", "fake_peak", "fake_threads", "fake_arg"):
    getattr(F, f).restype = C.c_uint64
F.fake_name.restype = C.c_char_p
F.fake_limit.argtypes = [C.c_uint64]
F.fake_is_device.argtypes = [C.c_uint64]
F.fake_arg.argtypes = F.fake_threads.argtypes = [C.c_int, C.c_int]
from paper_2106_03287_amd import stein_icp as S
L = S.lib()
assert "torch" not in sys.modules

def malloc(n):
    p = C.c_void_p()
    assert F.hipMalloc(C.byref(p), C.c_size_t(n)) == 0
    return p

def init(n_src, n_ref, pairs=1, shared=False, **cfg):
    """(status, context) of a batch of equal pairs."""
    cfg.setdefault("use_graph", 0)
    c = S.stein_icp_default_config(**cfg)
    src = [malloc(12 * n_src)] * pairs if shared else [malloc(12 * n_src) for _ in range(pairs)]
    ref = [malloc(12 * n_ref)] * pairs if shared else [malloc(12 * n_ref) for _ in range(pairs)]
    vp, i64 = C.c_void_p * pairs, C.c_int64 * pairs
    sched = malloc(4 * c.schedule_rows * c.batch_size)
    ctx = C.c_void_p()
    rc = L.stein_icp_batch_init(C.byref(ctx), C.byref(c), pairs, vp(*[s.value for s in src]), i64(*[n_src] * pairs),
                                vp(*[r.value for r in ref]), i64(*[n_ref] * pairs), None,
                                vp(*[sched.value] * pairs), None)
    return rc, ctx

def names():
    return [F.fake_name(i).decode() for i in range(F.fake_launches())]

def ran(part):
    return sum(part in n for n in names())

def ok(rc):
    assert rc == 0, (rc, S.stein_icp_last_error())
'''


@pytest.fixture(scope="session")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"),
                           "-o", out])
    return out


def run(fake, body, *args):
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), fake, *map(str, args)], cwd=ROOT,
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


def test_a_context_launches_its_three_stages(fake):
    run(fake, """
        rc, ctx = init(500, 2000, batch_size=100, num_particles=100)
        ok(rc)
        F.fake_clear()
        ok(L.stein_icp_step(ctx, 2, None))
        assert len(names()) == 6 and ran("index_nn_kernel") == 2, names()
        L.stein_icp_destroy(ctx)
    """)


def test_a_shape_that_does_not_fit_leaves_the_context_as_it_was(fake):
    """The search's buffers after a refused change of shape: those of the
    shape before, and a step launches on them. Where even these cannot be had
    again, a step is refused and launches nothing, until a shape fits."""
    run(fake, """
        for nn_mode in (S.NN_FP32, S.NN_F16_RERANK):
            rc, ctx = init(500, 2000, batch_size=100, num_particles=100, nn_mode=nn_mode)
            ok(rc)
            if nn_mode != S.NN_FP32:   # the screen's fragments are built
                ok(L.stein_icp_set_nn_tiling(ctx, 1, 4, 32, 0, None))
                ok(L.stein_icp_set_nn_tiling(ctx, 1, 4, 2016, 0, None))
            F.fake_limit(F.fake_live() + 1000)
            assert L.stein_icp_set_nn_tiling(ctx, 1, 4, 32, 0, None) == S.E_NOMEM
            F.fake_clear()
            ok(L.stein_icp_step(ctx, 1, None))
            if nn_mode == S.NN_FP32:
                assert "index_nn_kernel" in names()[0] and F.fake_is_device(F.fake_arg(0, 4))
            else:
                chunk = C.c_int32()
                ok(L.stein_icp_nn_tiling(ctx, None, None, C.byref(chunk), None, None, None))
                assert chunk.value == 2016 and "nn_bf16_kernel" in names()[0]
            F.fake_limit(1)
            assert L.stein_icp_set_nn_tiling(ctx, 1, 4, 32, 0, None) == S.E_NOMEM
            F.fake_clear()
            ms = (C.c_double * 3)()
            for rc in (L.stein_icp_step(ctx, 1, None), L.stein_icp_stage_times(ctx, 1, ms, None),
                       L.stein_icp_time_nn(ctx, 1, ms, None)):
                assert rc == S.E_NOMEM
            assert not names()
            F.fake_limit(1 << 62)
            ok(L.stein_icp_set_nn_tiling(ctx, 1, 4, 32, 0, None))
            ok(L.stein_icp_step(ctx, 1, None))
            L.stein_icp_destroy(ctx)
    """)


def test_a_screen_whose_build_failed_is_built_again(fake):
    """Every copy and launch of a screen's build in turn fails; the next
    request of a brute-force shape builds the fragments anew."""
    run(fake, """
        for what in ("hipMemcpyAsync", "hipLaunchKernel", "hipMalloc"):
            for nth in range(1, 12):
                rc, ctx = init(500, 2000, batch_size=100, num_particles=100, nn_mode=S.NN_F16_RERANK)
                ok(rc)
                F.fake_clear()
                F.fake_fail(what.encode(), nth, 1)
                rc = L.stein_icp_set_nn_tiling(ctx, 1, 4, 32, 0, None)
                F.fake_no_failures()
                if rc == 0:   # past the last call of the build and the upload
                    break
                ok(L.stein_icp_set_nn_tiling(ctx, 1, 4, 32, 0, None))
                ok(L.stein_icp_step(ctx, 1, None))
                assert ran("pack_f16_refs") >= 1, (what, nth)
                assert ran("nn_bf16_kernel") == 1
                L.stein_icp_destroy(ctx)
            assert nth < 11
    """)


def test_searches_too_large_for_an_indexed_launch_take_the_brute_force_one(fake):
    """A launch takes fewer than 2^32 threads. The indexed search needs 4 or 16
    a query, the brute-force one one or two by default: contexts and stand-alone
    searches just below and at the line are launched either way, in every mode."""
    run(fake, """
        for nn_mode in (S.NN_FP32, S.NN_BF16_RERANK, S.NN_F16_RERANK):
            for K, m, autotune, indexed in ((1000, 1 << 20, 0, True), (1024, 1 << 20, 0, False),
                                            (1024, 1 << 21, 0, False), (256, 1 << 20, 1, True),
                                            (1000, 1 << 20, 1, True)):
                if nn_mode != S.NN_FP32 and K * m == 1 << 31:
                    continue   # the screens take two threads a query: too many
                rc, ctx = init(m, 100, num_particles=K, batch_size=m, nn_mode=nn_mode, autotune=autotune)
                ok(rc)
                F.fake_clear()
                ok(L.stein_icp_step(ctx, 1, None))
                assert len(names()) == 3 and ("index_nn" in names()[0]) == indexed, (nn_mode, K, m, names())
                L.stein_icp_destroy(ctx)
            ref = malloc(12 * 100000)
            for nq, indexed in ((1000 << 20, True), (1 << 30, False), ((1 << 31) - 64, False)):
                if nn_mode != S.NN_FP32 and nq > 1 << 30:
                    continue
                q, idx = malloc(12 * nq), malloc(4 * nq)
                F.fake_clear()
                ok(L.stein_icp_nn(q, nq, ref, 2000, nn_mode, idx, None, None))
                assert ran("index_nn") == indexed, (nn_mode, nq, names())
                assert ran("nn_finish") == 1
                F.hipFree(q), F.hipFree(idx)
    """)


def test_an_index_keeps_no_scratch_and_yields_its_room(fake):
    """What an indexed context keeps: the packed references (16 bytes each) and
    the index; its build scratch, of clouds of some size, goes when init ends. And
    where the index, its scratch or what follows it does not fit, the context
    searches without, in no more memory than it needs then."""
    run(fake, """
        for metric in (S.METRIC_POINT, S.METRIC_PLANE):
            kept = []
            for n_ref in (500000, 1000000):
                F.fake_limit(1 << 62)
                cfg = dict(batch_size=300, num_particles=100, metric=metric)
                rc, ctx = init(500, n_ref, **cfg)
                ok(rc)
                kept.append(F.fake_live() - 12 * n_ref)
                before = F.fake_live()
                L.stein_icp_destroy(ctx)
                kept[-1] -= F.fake_live() - 12 * n_ref
            per_ref = (kept[1] - kept[0]) / 500000
            assert per_ref < 40 + (32 if metric == S.METRIC_PLANE else 0), per_ref

        for nn_mode in (S.NN_FP32, S.NN_F16_RERANK):
            cfg = dict(batch_size=300, num_particles=100, nn_mode=nn_mode)
            need = None   # of the search without an index
            for nth, times in ((2, 1), (3, 1), (4, 2)):   # the index, its scratch, the keys (tried twice)
                F.fake_clear()
                F.fake_fail(b"hipMalloc", nth + 3, times)   # after the three inputs
                live = F.fake_live()
                F.fake_peak_reset()
                rc, ctx = init(500, 500000, **cfg)
                F.fake_no_failures()
                ok(rc)
                need = F.fake_peak() - live if need is None else need
                F.fake_clear()
                ok(L.stein_icp_step(ctx, 1, None))
                assert len(names()) == 3 and not ran("index_nn"), names()
                L.stein_icp_destroy(ctx)
            for more in range(0, 40 << 20, 1 << 19):
                F.fake_limit(F.fake_live() + need + more)
                rc, ctx = init(500, 500000, **cfg)
                ok(rc)
                L.stein_icp_destroy(ctx)
            F.fake_limit(1 << 62)
    """)


def test_tuned_shapes_are_shared_by_contexts_alike_only(fake):
    """A tuned shape goes to the next context of the same sizes, mode, particles
    and metric, and to no other: a screen cannot take the FP32 search's four
    queries per lane, and where the bandwidths are selected depends on the
    particles and the lanes of an indexed search."""
    run(fake, """
        def tuned(n_src, n_ref, **cfg):
            F.fake_clear()
            rc, ctx = init(n_src, n_ref, autotune=1, **cfg)
            ok(rc)
            nn = ran("nn_fp32") + ran("nn_bf16") + ran("index_nn")
            q = C.c_int32()
            ok(L.stein_icp_nn_tiling(ctx, C.byref(q), None, None, None, None, None))
            ok(L.stein_icp_step(ctx, 1, None))
            L.stein_icp_destroy(ctx)
            return nn, q.value

        small = dict(n_src=500, n_ref=900, batch_size=100, num_particles=10)   # searched by brute force
        assert tuned(**small, nn_mode=S.NN_FP32)[1] == 4   # the fewest workgroups, which the stand-in takes for time
        for mode in (S.NN_BF16_RERANK, S.NN_F16_RERANK):
            n, q = tuned(**small, nn_mode=mode)
            assert n > 0 and q <= 2, (mode, n, q)
        assert tuned(**small, nn_mode=S.NN_FP32) == (0, 4)
        big = dict(n_src=500, n_ref=20000)
        for other in (dict(num_particles=100, batch_size=300), dict(num_particles=300, batch_size=100),
                      dict(num_particles=100, batch_size=300, metric=S.METRIC_PLANE),
                      dict(num_particles=100, batch_size=300, bandwidth_mode=S.BW_FIXED)):
            assert tuned(**big, **other)[0] > 0, other
            assert tuned(**big, **other)[0] == 0, other
    """)


def test_outputs_past_their_allocation_are_refused(fake):
    """Several outputs in one kernel launch, as long as each lies inside its
    allocation: one that does not is left to a copy, which refuses it, and no
    kernel writes past it."""
    run(fake, """
        rc, ctx = init(500, 2000, batch_size=100, num_particles=100)
        ok(rc)
        n = 8 * 100 * 6
        whole, short = malloc(n), malloc(n - 8)
        for a, b, code in ((whole, malloc(n), 0), (whole, short, S.E_DEVICE), (short, whole, S.E_DEVICE),
                           (C.c_void_p(whole.value + 8), malloc(n), S.E_DEVICE)):
            F.fake_clear()
            assert L.stein_icp_get_diagnostics(ctx, a, b, None, None, None) == code
            assert ran("copy_out") == (code == 0)
            F.fake_clear()
            assert L.stein_icp_get_state(ctx, a, b, None, None, None) == code
            assert ran("copy_out") == (code == 0)
    """)


def test_outputs_on_another_devices_stream_are_copied(fake):
    """A copy on a stream of another device than the context's reads and writes
    where it is told; a kernel would run on that other device."""
    run(fake, """
        rc, ctx = init(500, 2000, batch_size=100, num_particles=100)
        ok(rc)
        n = 8 * 100 * 6
        a, b = malloc(n), malloc(n)
        for device in (0, 1):
            s = malloc(8)
            F.fake_stream_device(s, device)
            F.fake_clear()
            ok(L.stein_icp_get_diagnostics(ctx, a, b, None, None, s))
            assert ran("copy_out") == (device == 0)
    """)


def test_the_stand_alone_set_loss_is_one_launch(fake):
    """One workgroup a sample writes the sample's loss: nothing is left for a
    second launch, which would read the losses where it writes them."""
    run(fake, """
        B, K = 3, 100
        x, y, out = malloc(48 * B * K), malloc(48 * B * K), malloc(8 * B)
        sigma = (C.c_double * 6)(*[0.1] * 6)
        F.fake_clear()
        ok(L.stein_icp_proposal_mmd(x, y, B, K, 1, sigma, out, None))
        assert len(names()) == 1, names()
    """)


def test_which_contexts_build_an_index(fake):
    """Either side of the lines: few FP32 queries need more evaluations to
    repay an index, unless normals come from it too; the screens do not."""
    run(fake, """
        def indexed(K, m, n_ref, **cfg):
            rc, ctx = init(4000, n_ref, num_particles=K, batch_size=m, **cfg)
            ok(rc)
            F.fake_clear()
            ok(L.stein_icp_step(ctx, 1, None))
            L.stein_icp_destroy(ctx)
            return ran("index_nn") == 1

        for K, m, n_ref, fp32, plane, screen in (
                (16, 32, 29000, False, False, False), (16, 32, 30000, False, True, True),
                (16, 32, 58000, False, True, True), (16, 32, 59000, True, True, True),
                (64, 32, 7400, False, True, True), (64, 32, 14700, True, True, True),
                (64, 64, 3600, False, False, True), (64, 64, 3700, True, True, True)):
            assert indexed(K, m, n_ref) == fp32, (K, m, n_ref)
            assert indexed(K, m, n_ref, metric=S.METRIC_PLANE) == plane, (K, m, n_ref)
            for mode in (S.NN_BF16_RERANK, S.NN_F16_RERANK):
                assert indexed(K, m, n_ref, nn_mode=mode) == screen, (K, m, n_ref)
    """)


def test_lanes_of_an_indexed_search(fake):
    """Either side of the line, for a context (all its pairs together) and for a
    stand-alone search."""
    run(fake, """
        def lanes(found):
            assert found == 1
            return 4 if ran("index_nn_kernelILi4") else 16

        for pairs, K, m, want in ((1, 100, 491, 16), (1, 100, 492, 4), (3, 100, 163, 16), (3, 100, 164, 4)):
            rc, ctx = init(500, 20000, pairs=pairs, num_particles=K, batch_size=m)
            ok(rc)
            F.fake_clear()
            ok(L.stein_icp_step(ctx, 1, None))
            assert lanes(ran("index_nn")) == want, (pairs, K, m)
            L.stein_icp_destroy(ctx)
        ref = malloc(12 * 20000)
        for nq, want in ((49151, 16), (49152, 4)):
            F.fake_clear()
            ok(L.stein_icp_nn(malloc(12 * nq), nq, ref, 20000, S.NN_FP32, malloc(4 * nq), None, None))
            assert lanes(ran("index_nn")) == want, nq
    """)


def test_a_failed_indexed_search_waits_for_its_uploads(fake):
    """Whichever launch of a stand-alone search's index fails, the call returns
    only after the copy of the build's plan from its own host memory."""
    run(fake, """
        nq, n_ref = 100000, 100000
        q, ref, idx = malloc(12 * nq), malloc(12 * n_ref), malloc(4 * nq)
        for call in (L.stein_icp_nn, L.stein_icp_nn_noalloc):
            failed = 0
            for nth in range(1, 30):
                F.fake_clear()
                F.fake_fail(b"hipLaunchKernel", nth, 1)
                rc = call(q, nq, ref, n_ref, S.NN_FP32, idx, None, None)
                F.fake_no_failures()
                assert not F.fake_in_flight(), nth
                if rc == 0:
                    break
                failed += 1
            assert failed >= 8 and ran("index_nn") == 1
    """)
