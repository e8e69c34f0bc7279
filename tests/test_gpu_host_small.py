"""GPU parity of small loads and stores against host memory (kv_host_kernel in csrc/kv_copy.hip), byte for byte: both sides of the
line to the copy engine's way, slices that end inside a page, host memory that the kernel may not touch itself, and replays."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B

pytestmark = pytest.mark.gpu


def _bytes(seed, *shape):
    return torch.from_numpy(np.random.default_rng(seed).integers(0, 256, size=shape, dtype=np.uint8))


def _host(t, pinned, n):
    """t behind `n` other bytes: the last bytes of an allocation"""
    flat = torch.zeros(n + t.numel(), dtype=torch.uint8, pin_memory=pinned)
    flat[n:] = t.reshape(-1)
    return flat[n:].view(t.shape)


class Layer:
    def __init__(self, page_bytes, n, pinned, seed=3):
        self.pb, self.n, self.N = page_bytes, n, n + 13
        self.k, self.v = (_host(_bytes(seed + i, n, page_bytes), pinned, 4096) for i in range(2))
        self.k_out, self.v_out = (_host(torch.zeros(n, page_bytes, dtype=torch.uint8), pinned, 256) for _ in range(2))
        # stages and pools between guard bytes that stay as they are
        self.guarded = [torch.full((512 + rows * page_bytes,), 0xA5, dtype=torch.uint8, device="cuda:0") for rows in (n, n, self.N, self.N)]
        self.ks, self.vs, self.kp, self.vp = (t[256:-256] for t in self.guarded)
        self.ids = torch.from_numpy(np.random.default_rng(seed).permutation(self.N)[:n].astype(np.int32)).cuda()

    def load(self, stream=None):
        B.mc_kv_load_layer(self.k, self.v, self.ks, self.vs, self.N, self.pb, self.ids, self.n, self.kp, self.vp, stream)

    def store(self, stream=None):
        B.mc_kv_store_layer(self.kp, self.vp, self.N, self.pb, self.ids, self.n, self.ks, self.vs, self.k_out, self.v_out, stream)

    def check_loaded(self):
        for host, stage, pool in ((self.k, self.ks, self.kp), (self.v, self.vs, self.vp)):
            want = torch.full((self.N, self.pb), 0xA5, dtype=torch.uint8)
            want[self.ids.cpu().long()] = host
            assert torch.equal(stage.cpu().view(self.n, self.pb), host) and torch.equal(pool.cpu().view(self.N, self.pb), want)
        for t in self.guarded:
            assert (t[:256] == 0xA5).all() and (t[-256:] == 0xA5).all()


# pinned memory: one vector, a page that ends inside a slice, 8 KiB + 16 bytes, 512 slices and 513 (the copy engine's)
@pytest.mark.parametrize("page_bytes,n", [(16, 1), (16, 512), (16, 513), (4080, 33), (4112, 33), (8208, 5), (32768, 64), (32784, 57), (32768, 65),
                                          (2048, 300), (24576, 7)])
@pytest.mark.parametrize("pinned", [True, False])
def test_small_load_and_store(page_bytes, n, pinned):
    print(f"small host case page_bytes={page_bytes} n={n} pinned={pinned}", flush=True)
    layer = Layer(page_bytes, n, pinned)
    layer.load()
    torch.cuda.synchronize()
    layer.check_loaded()
    layer.ks.zero_()
    layer.vs.zero_()
    layer.store()
    torch.cuda.synchronize()
    assert torch.equal(layer.k_out, layer.k) and torch.equal(layer.v_out, layer.v)
    layer.check_loaded()                                  # the stages hold the packed form again


def test_streams_and_replays():
    """Loads and stores of several layers on two streams, then the same from a graph, replayed over other host bytes."""
    layers = [Layer(4096, 24, True, seed) for seed in (11, 21, 31)]
    loads, stores = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(3):
        for layer in layers:
            layer.load(loads)
            stores.wait_stream(loads)
            layer.store(stores)
    torch.cuda.synchronize()
    for layer in layers:
        layer.check_loaded()
        assert torch.equal(layer.k_out, layer.k) and torch.equal(layer.v_out, layer.v)
    layer = layers[0]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer.load()
        layer.store()
    for seed in range(3):
        layer.k.copy_(_bytes(100 + seed, layer.n, layer.pb))
        layer.v.copy_(_bytes(200 + seed, layer.n, layer.pb))
        layer.k_out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        layer.check_loaded()
        assert torch.equal(layer.k_out, layer.k) and torch.equal(layer.v_out, layer.v)


def _hip():
    torch.cuda.init()
    with open("/proc/self/maps") as maps:
        return ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))


def _recorded(call):
    """What a call enqueues, by the kinds of the nodes of a graph that records it (0: kernel, 1: copy).  The graph is never run."""
    hip = _hip()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    handle, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(handle, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(handle, nodes, ctypes.byref(n)) == 0
    kinds = []
    for node in nodes:
        kind = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        kinds.append(kind.value)
    return sorted(kinds)


def _allocated(flags, n, page_bytes):
    """Host memory of hipHostMalloc with these flags, freed at the end of the process"""
    at = ctypes.c_void_p()
    assert _hip().hipHostMalloc(ctypes.byref(at), ctypes.c_size_t(n * page_bytes), ctypes.c_uint(flags)) == 0
    array = np.ctypeslib.as_array(ctypes.cast(at, ctypes.POINTER(ctypes.c_uint8)), (n, page_bytes))
    return torch.from_numpy(array)


@pytest.mark.parametrize("page_bytes,n,by_kernel", [(16, 1, True), (16, 512, True), (16, 513, False), (4112, 256, True), (4112, 257, False),
                                                    (32768, 64, True), (32768, 65, False)])
def test_which_way_a_call_goes(page_bytes, n, by_kernel):
    layer = Layer(page_bytes, n, True)
    for call in (layer.load, layer.store):
        assert _recorded(call) == ([0] if by_kernel else [0, 1, 1])


# plain, portable and mapped, NUMA-local, coherent; not coherent, write-combined
@pytest.mark.parametrize("flags,by_kernel", [(0, True), (0x3, True), (0x20000000, True), (0x40000000, True), (0x80000000, False), (0x4, False)])
def test_memory_that_a_kernel_may_not_touch_goes_by_the_copy_engine(flags, by_kernel):
    layer = Layer(4096, 24, True)
    want = layer.k.clone(), layer.v.clone()
    layer.k, layer.v, layer.k_out, layer.v_out = (_allocated(flags, 24, 4096) for _ in range(4))
    layer.k.copy_(want[0])
    layer.v.copy_(want[1])
    for call in (layer.load, layer.store):
        assert _recorded(call) == ([0] if by_kernel else [0, 1, 1])
    layer.load()
    layer.store()
    torch.cuda.synchronize()
    layer.check_loaded()
    assert torch.equal(layer.k_out, want[0]) and torch.equal(layer.v_out, want[1])
