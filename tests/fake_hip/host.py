"""Loads liblt.so on the stand-in of the HIP runtime (fake_hip.cpp) in a
process of its own: `python host.py SCENARIO`, LD_LIBRARY_PATH leading to the
stand-in.  torch is replaced by the two names that the binding uses here, so
that nothing else of a HIP runtime is loaded."""
import ctypes as C
import os
import sys
import types

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(os.path.dirname(HERE)))


class _Device:
    def __init__(self, kind, index=0):
        self.type, self.index = kind, index


STREAM = {"now": 0x1000}
torch = types.ModuleType("torch")
torch.device = _Device
torch.Tensor = type("Tensor", (), {})
torch.autograd = types.SimpleNamespace(Function=object)
torch.cuda = types.SimpleNamespace(current_stream=lambda d: types.SimpleNamespace(cuda_stream=STREAM["now"]))
sys.modules["torch"] = torch

from paper_2609_32920_amd import lt, scenes  # noqa: E402

lt.library()
fake = C.CDLL("libamdhip64.so.7")
fake.fake_held.restype = fake.fake_alloc.restype = C.c_size_t
fake.fake_launch.restype = C.c_char_p
fake.fake_limit.argtypes = [C.c_size_t]
fake.fake_capture.argtypes = [C.c_void_p, C.c_int]


def launches():
    """What was launched since the last call."""
    out = []
    for i in range(fake.fake_launches()):
        dev, stream = C.c_int(), C.c_void_p()
        lds, threads, groups, arg = C.c_uint64(), C.c_uint64(), C.c_uint64(), (C.c_uint64 * 4)()
        name = fake.fake_launch(i, C.byref(dev), C.byref(stream), C.byref(lds), C.byref(threads), C.byref(groups), arg)
        out.append(types.SimpleNamespace(name=name.decode(), device=dev.value, stream=stream.value or 0, lds=lds.value,
                                         threads=threads.value, groups=groups.value, arg=list(arg)))
    fake.fake_clear_launches()
    return out


def named(ls, part):
    return [l for l in ls if part in l.name]


class Calls:
    """A context with a scene and (never read) buffers, called through the C ABI."""

    def __init__(self, sc, device=0):
        self.ctx = lt.Context(device).scene_upload(sc)
        self.lib, self.h = self.ctx.lib, self.ctx.h
        self.buf = (C.c_char * 64)()
        at = C.addressof(self.buf)
        hf = sc.get("hf") is not None
        self.p = lt.Params(at, at, at if hf else None, None, None)
        self.g = lt.Grads(at, at, at if hf else None, None)
        self.at = at

    def args(self, n, depth, flags=0):
        return self.ctx.args(1, n, depth, flags)

    def ok(self, st):
        self.ctx._status(st)

    def trace(self, n, depth=4, flags=0):
        a = self.args(n, depth, flags)
        nb = self.lib.lt_side_state_bytes(self.h, C.byref(a))
        self.ctx._stream()
        self.ok(self.lib.lt_trace(self.h, C.byref(a), C.byref(self.p), self.at, self.at if nb else None, nb))

    def loss(self, n=300):
        self.ctx._stream()
        self.ok(self.lib.lt_loss_l2(self.h, self.at, self.at, n, self.at, self.at))

    def backward(self, mode, n, depth=4, flags=0):
        rec = {"naive": lt.RECORD_TAPE, "reslrb": lt.RECORD_RESERVOIR, "lrb2": lt.RECORD_SPLATS}.get(mode, 0)
        a = self.args(n, depth, flags | rec)
        nb = self.lib.lt_side_state_bytes(self.h, C.byref(a))
        self.ctx._stream()
        f = getattr(self.lib, "lt_backward_" + mode)
        side = (self.at, nb) if rec else ()
        self.ok(f(self.h, C.byref(a), C.byref(self.p), self.at, *side, C.byref(self.g)))


# ------------------------------------------------------------ scenarios
def loss_sums():
    """Every loss adds to sums that are zero, whatever the loss before it left there."""
    c = Calls(scenes.box_scene(32, 32))

    def check(want, clears=None):
        ls = launches()
        got = named(ls, "k_loss")
        assert len(got) == want and all(l.arg[1] for l in got), [(l.name, l.arg) for l in ls]
        if clears is not None:
            assert len(named(ls, "k_begin")) == clears

    c.loss()
    c.loss()
    check(2)
    c.trace(4096)
    c.loss()
    check(1, clears=1)               # a step pays nothing for it
    c.loss()
    c.backward("lrb3", 4096)
    c.loss()
    check(2)
    c.trace(4096)                    # a pass on another stream than the loss
    STREAM["now"] = 0x2000
    c.loss()
    check(1, clears=2)
    c.trace(4096)                    # a pass before the capture of a loss alone
    fake.fake_capture(0x2000, 1)
    c.loss()
    check(1)
    c.trace(4096)                    # a captured step, and a loss before it has run
    c.loss()
    c.trace(4096)
    check(1)
    fake.fake_capture(0x2000, 0)
    c.loss()
    check(1)


def height_range():
    """Nothing is counted between the workgroups that form the height range:
    up to 64x64 heights one forms it, of more a launch before the pass does,
    from parts that all were written by the pass's own start."""
    for G, parts in ((2, 0), (33, 0), (64, 0), (65, 1), (128, 1)):
        c = Calls(scenes.caustic_scene(G=G, width=16, height=16))
        for call in (lambda: c.trace(1000), lambda: c.backward("lrb3", 1000), lambda: c.backward("lrb3", 1000, flags=lt.ATTACHED)):
            launches()
            call()
            ls = [l.name for l in launches()]
            assert "k_begin" in ls[0]
            assert ["k_hf_whole" in n for n in ls[1:]] == [True] * parts + [False] * (len(ls) - 1 - parts), (G, ls)


def devices():
    """Two contexts on two devices in one thread: each call allocates and
    launches on its own context's device and leaves the thread's current one."""
    for mine, other in ((1, 0), (0, 1)):
        for flags in (0, lt.GUIDE_DIFFUSE):
            c = Calls(scenes.box_scene(64, 64), device=mine)
            if flags:
                c.p.guide_w = c.at
            lib, h, at = c.lib, c.h, c.at
            a = lambda n, fl=0: C.byref(c.args(n, 3, fl))
            calls = [
                ("trace", lambda: c.trace(1 << 17, flags=flags)),
                ("loss", c.loss),
                ("naive", lambda: c.backward("naive", 1000, flags=flags)),
                ("reslrb", lambda: c.backward("reslrb", 1000, flags=flags)),
                ("lrb2", lambda: c.backward("lrb2", 1000, flags=flags)),
                ("lrb3", lambda: c.backward("lrb3", 1000, flags=flags)),
                ("lrb3 in two kernels", lambda: (c.ctx.set_tuning(lrb3_split=1), c.backward("lrb3", 1000, flags=flags))),
                ("camera", lambda: c.ok(lib.lt_camera_trace(h, a(4096), C.byref(c.p), at))),
                ("camera backward", lambda: c.ok(lib.lt_camera_backward_prb(h, a(4096), C.byref(c.p), at, C.byref(c.g)))),
                ("guide eval", lambda: c.ok(lib.lt_guide_eval(h, at, at, at, 5, at))),
                ("guide grad", lambda: c.ok(lib.lt_guide_grad(h, at, at, 5, at, at))),
                ("adam", lambda: c.ok(lib.lt_guide_adam(h, at, at, at, at, 1, 0.1, 0.9, 0.9, 1e-8))),
                ("train", lambda: c.ok(lib.lt_guide_train_step(h, a(100), at, at, at, 100, at, at, at, at, 1, 0.1, 0.9, 0.9, 1e-8))),
            ]
            if flags:
                calls += [("emit", lambda: c.ok(lib.lt_guide_emit(h, a(100), C.byref(c.p), at, at))),
                          ("vertex samples", lambda: c.ok(lib.lt_guide_vertex_samples(h, a(100), C.byref(c.p), at)))]
            else:
                calls += [("noalloc", lambda: c.ok(lib.lt_backward_lrb3_noalloc(h, a(1000), C.byref(c.p), at, C.byref(c.g))))]
            fake.fake_set_current(other)
            for name, call in calls:
                launches()
                before = sum(fake.fake_alloc_device(i) == other for i in range(fake.fake_allocs()))
                call()
                assert sum(fake.fake_alloc_device(i) == other for i in range(fake.fake_allocs())) == before, name
                ls = launches()
                assert ls and all(l.device == mine for l in ls), (name, [(l.name, l.device) for l in ls])
                assert fake.fake_current() == other, name


def soup(sc, n):
    """sc with n small random triangles more."""
    import numpy as np
    rng = np.random.default_rng(n)
    v = rng.uniform(0.0, 1.0, size=(n, 1, 3)) + rng.uniform(-0.01, 0.01, size=(n, 3, 3))
    return dict(sc, tri_v=np.concatenate([sc["tri_v"], v]), tri_uv=np.concatenate([sc["tri_uv"], np.zeros((n, 3, 2))]),
                tri_mat=np.concatenate([sc["tri_mat"], np.zeros(n, np.int32)]))


def scene_bytes():
    """The bytes that lt_workspace_bytes reports and the memory cap is held
    against are those that a context and its scene hold."""
    box, glass = scenes.box_scene(16, 16), scenes.caustic_scene(G=96, width=16, height=16)
    for sc in (box, soup(box, 20000), glass, soup(glass, 20000), scenes.plane_point_light_scene(8, 8)):
        before = fake.fake_held()
        c = Calls(sc)
        held = fake.fake_held() - before
        a = c.args(1, 1)
        # 512 bytes more by definition, the guide's packed weights (51200) and one emission record
        said = c.ctx.workspace_bytes(a) - 512 - 51200 - 16
        assert held <= said <= held + 256, (sc["name"], held, said)
        for cap, fits in ((said + 64, True), (said + 63, False)):
            c.ctx.set_memory_cap(cap)
            try:
                c.trace(1, 1)
                assert fits
            except lt.LTError as e:
                assert not fits and e.status == lt.LT_ERR_OOM
        del c  # its memory goes back before the next is measured


def batch_of(calls, n_paths, depth, flags=0):
    tab = (lt.Instance * len(calls))()
    for k, c in enumerate(calls):
        tab[k].ctx, tab[k].args, tab[k].params, tab[k].grads = c.h, c.args(n_paths, depth, flags), c.p, c.g
        tab[k].target = tab[k].image = tab[k].d_image = tab[k].loss = c.at
    return tab


def new_batch(lib):
    b = C.c_void_p()
    assert lib.lt_batch_create(0, None, C.byref(b)) == lt.LT_OK
    return b


def batch_cells():
    """A batch's film cells keep under its contexts' memory caps and take no
    memory that the step cannot do without."""
    sc = scenes.caustic_scene(G=16, width=256, height=256)
    n = 1 << 20  # an attached instance that runs on its own: hand-off entries of 64 bytes
    c = Calls(sc)
    lib = c.lib

    def step(cap, room=None):
        c.ctx.set_memory_cap(cap)
        b, tab = new_batch(lib), batch_of([c], n, 3, lt.ATTACHED)
        before = fake.fake_held()
        if room is not None:
            fake.fake_limit(before + room)
        st = lib.lt_batch_step(b, tab, 1, 0)
        held = fake.fake_held() - before
        fake.fake_limit(2 ** 64 - 1)
        lib.lt_batch_destroy(b)
        assert fake.fake_held() == before
        return st, held

    cells, scene = 64 * 257 * 257, c.ctx.workspace_bytes(c.args(1, 1)) - 512 - 51200 - 16
    st, free = step(0)
    assert st == lt.LT_OK and free >= 64 * n + (32 << 20)
    st, held = step(scene + 64 + cells)
    assert st == lt.LT_OK and held == free
    st, held = step(scene + 64 + cells - 1)
    assert st == lt.LT_OK and held < 64 * n + (2 << 20)
    st, held = step(0, room=64 * n + (2 << 20))  # room for the hand-off and the tables only
    assert st == lt.LT_OK and held < 64 * n + (2 << 20)


if __name__ == "__main__":
    launches()
    globals()[sys.argv[1]]()
    print("done")
