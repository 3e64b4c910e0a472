"""The built library on the stand-in runtime of fake_hip.cpp, in a process of its own that never loads
torch:  python driver.py <stand-in .so> <libepd_encode.so> <function of this file> [<gemm_shim .so>]."""

import ctypes as C
import os
import re
import sys
import types

import numpy as np

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__)))))
from oracle import mm_store as S                                        # noqa: E402
from paper_2601_11590_amd import build, workloads as W                  # noqa: E402

OK, MISS, ERR_HIP = 0, 1, -5
LAST_ERROR, CAPTURE, LATE, LAUNCH_STATUS, SYNC_STATUS, HOST_FLAGS = range(6)
POOL = 0x7F0000000000                                                   # never dereferenced
U64P = C.POINTER(C.c_uint64)


def load(fake_path, lib_path):
    fake = C.CDLL(fake_path, mode=C.RTLD_GLOBAL)
    fake.fake_set.argtypes = [C.c_int, C.c_longlong]
    fake.fake_get.restype = C.c_longlong
    fake.fake_calls.restype = C.c_longlong
    fake.fake_calls.argtypes = [C.c_char_p]
    fake.fake_args.restype = C.c_void_p
    fake.fake_keep_args.argtypes = [C.c_char_p, C.c_size_t]
    fake.fake_launch.restype = C.c_char_p
    fake.fake_launch.argtypes = [C.c_int, C.POINTER(C.c_uint32)]
    # the package's own binding, with a torch that holds names only: the real one would load the real runtime
    torch = types.ModuleType("torch")
    torch.__getattr__ = lambda name: type(name, (), {})
    sys.modules["torch"] = torch
    build.library_path = lambda: lib_path
    from paper_2601_11590_amd import binding
    return fake, binding.lib


def binding():
    return sys.modules["paper_2601_11590_amd.binding"]


def encoder(cfg, max_tokens, max_segments, max_items):
    """An encoder handle over made-up device addresses."""
    B = binding()
    c, w = B.make_cfg(cfg, max_tokens, max_segments, max_items), B.epd_weights()
    layers = (B.epd_layer_weights * max(1, cfg.num_layers))()
    for f, _ in B.epd_layer_weights._fields_:
        for l in layers:
            setattr(l, f, 0x1000)
    for f in ("patch_w", "patch_b", "final_norm_g", "final_norm_b", "merge_w", "merge_b"):
        setattr(w, f, 0x1000)
    w.layers = C.cast(layers, C.POINTER(B.epd_layer_weights))
    c.weights, c.workspace, c.workspace_bytes = C.pointer(w), 0x100000, 1 << 60
    return B.epd_encode_create(c)


def launches(fake):
    out = []
    for i in range(fake.fake_launches()):
        v = (C.c_uint32 * 6)()
        out.append((fake.fake_launch(i, v).decode(), tuple(v[:3]), tuple(v[3:])))
    return out


class Store:
    def __init__(self, lib):
        self.lib, self.h = lib, C.c_void_p()
        assert lib.epd_store_create(POOL, 2 << 20, C.byref(self.h)) == OK

    def hash(self, *buffers):
        """(status, keys) of the buffers, hashed in one call."""
        data = np.frombuffer(b"".join(buffers), np.uint8)
        off = np.cumsum([0] + [len(b) for b in buffers]).astype(np.uint64)
        salt = np.arange(len(buffers), dtype=np.uint64)
        keys = np.zeros((len(buffers), 2), np.uint64)
        p = lambda a: a.ctypes.data_as(U64P)
        st = self.lib.epd_store_hash(self.h, data.ctypes.data, p(off), p(salt), len(buffers), p(keys), None)
        return st, [tuple(int(v) for v in k) for k in keys]

    def close(self):
        assert self.lib.epd_store_destroy(self.h) == OK


def buffers(seed, n=3):
    rng = np.random.default_rng(seed)
    return [rng.integers(0, 256, size=int(rng.integers(1, 40000)), dtype=np.uint8).tobytes() for _ in range(n)]


def keys_of(bufs):
    return [S.hash128(b, i) for i, b in enumerate(bufs)]


def hash_right(store, seed, n=3):
    b = buffers(seed, n)
    st, keys = store.hash(*b)
    assert st == OK and keys == keys_of(b), (st, keys, keys_of(b))


# ------------------------------------------------------------------ the tests

def hash_plain(fake, lib):
    s = Store(lib)
    for late in (0, 1):
        fake.fake_set(LATE, late)
        for seed in range(3):
            hash_right(s, seed)
        hash_right(s, 9, n=70)                                          # three launches
    s.close()


def hash_with_an_uncollected_error(fake, lib):
    s = Store(lib)
    for late in (0, 1):
        fake.fake_set(LATE, late)
        for seed in range(4):
            fake.fake_set(LAST_ERROR, 1)                                # left by some earlier call of the program
            hash_right(s, seed)
    s.close()


def partial_hashes_lie_in_coherent_memory(fake, lib):
    s = Store(lib)
    hash_right(s, 0)
    portable, coherent, non_coherent = 0x1, 0x40000000, 0x80000000      # hipHostMalloc flags
    assert fake.fake_get(HOST_FLAGS) & (portable | coherent | non_coherent) == portable | coherent
    s.close()


def pinned_memory_is_taken_at_create_and_the_bookkeeping_calls_nothing(fake, lib):
    key, where = (C.c_uint64 * 2)(1, 2), C.c_void_p()
    s = Store(lib)
    assert fake.fake_calls(b"hipHostMalloc") == 1                        # not by a hash: see epd_store_create in the header
    fake.fake_forget()
    assert lib.epd_store_lookup(s.h, key, C.byref(where), None) == MISS
    assert lib.epd_store_insert(s.h, key, 1000, C.byref(where)) == OK and where.value == POOL + (1 << 20)
    assert lib.epd_store_lookup(s.h, key, C.byref(where), None) == OK
    assert fake.fake_all_calls() == 0
    hash_right(s, 0)
    hash_right(s, 1)
    assert fake.fake_calls(b"hipHostMalloc") == 0
    s.close()
    assert fake.fake_calls(b"hipHostFree") == 1


def hash_after_a_failed_launch(fake, lib):
    s = Store(lib)
    hash_right(s, 0)
    fake.fake_set(LAUNCH_STATUS, 98)
    assert s.hash(*buffers(1))[0] == ERR_HIP
    fake.fake_set(LAUNCH_STATUS, 0)
    hash_right(s, 2)
    s.close()


def hash_after_a_failed_wait(fake, lib):
    s = Store(lib)
    fake.fake_set(LATE, 1)
    for seed in range(3):
        hash_right(s, seed)
        fake.fake_set(SYNC_STATUS, 719)
        assert s.hash(*buffers(seed + 10))[0] == ERR_HIP
        fake.fake_set(SYNC_STATUS, 0)
        fake.fake_drain()                                               # the kernel of the failed call ends only now
    hash_right(s, 5)
    s.close()


def hash_on_a_capturing_stream(fake, lib):
    s = Store(lib)
    hash_right(s, 0)
    fake.fake_forget()
    fake.fake_set(CAPTURE, 1)
    assert s.hash(*buffers(1))[0] == ERR_HIP
    assert launches(fake) == []                                         # a captured launch would run again with every replay
    fake.fake_set(CAPTURE, 0)
    hash_right(s, 2)
    s.close()


def cached_hits_beside_an_uncollected_error(fake, lib):
    B = binding()
    cfg = W.C2.replace(num_layers=1)
    grids, src = [(1, 2, 2), (1, 4, 2)], [(40, 30), (64, 32)]
    h, s = encoder(cfg, 64, 8, 8), Store(lib)
    px = np.random.default_rng(0).integers(0, 256, size=3 * (40 * 30 + 64 * 32), dtype=np.uint8)
    call = lambda: B.epd_encode_cached(h, s.h, 7, px.ctypes.data, src, grids, [0.5] * 3, [0.25] * 3, POOL, POOL, POOL, None)
    hit, keys = call()
    assert hit.tolist() == [0, 0]
    for status, want in ((0, None), (1, None), (98, ERR_HIP)):
        fake.fake_forget()
        fake.fake_set(LAST_ERROR, 1 if status == 1 else 0)              # left by some earlier call of the program
        if status == 98:
            fake.fake_refuse(b"copies_kernel", 98)
        try:
            hit, again = call()
            assert want is None and hit.tolist() == [1, 1] and (keys == again).all()
            assert sum("copies_kernel" in l[0] for l in launches(fake)) == 1
        except B.EpdError as e:
            assert e.status == want, e


def launches_stay_within_the_thread_limit(fake, lib):
    B = binding()

    def check(what, names):
        seen = set()
        for name, grid, block in launches(fake):
            seen |= {n for n in names if n in name}
            assert all(g * b < 2 ** 32 for g, b in zip(grid, block)), (what, name, grid, block)
        assert seen == set(names), (what, seen)

    one = dict(name="x", num_layers=1, mlp_dim=64, patch=4, temporal_patch=1, out_dim=64, merge=1, norm="rmsnorm")
    # fp32, 2^26 - 256 tokens with 64 rotary pairs each
    cfg = W.EncoderConfig(dtype="f32", hidden=128, num_heads=1, head_dim=128, rope="2d", rope_pairs=(0, 32, 32), **one)
    T = 2 ** 26 - 256
    h = encoder(cfg, T, 1024, 1)
    fake.fake_forget()
    B.epd_encode(h, POOL, np.linspace(0, T, 1025).astype(np.int32), [(T // 2 ** 8, 2 ** 4, 2 ** 4)], POOL, None)
    check("rotary table", ["plan_kernel", "attn_f32_kernel", "norm_kernel"])
    # fp32, 4.5 million segments of two tokens
    cfg = W.EncoderConfig(dtype="f32", hidden=8, num_heads=1, head_dim=8, rope="2d", rope_pairs=(0, 2, 2), **one)
    S = 4500000
    h = encoder(cfg, 2 * S, S, 1)
    fake.fake_forget()
    B.epd_encode(h, POOL, np.arange(S + 1, dtype=np.int32) * 2, [(S, 1, 2)], POOL, None)
    check("segments", ["plan_kernel", "attn_f32_kernel"])
    assert sum(g[0] for n, g, _ in launches(fake) if "attn_f32" in n) == S
    # bf16, 65 536 segments of two tokens at hidden 1024: as many (segment, four channels) pairs as blocks of 256 threads may be
    cfg = W.EncoderConfig(dtype="bf16", hidden=1024, num_heads=16, head_dim=64, rope="2d", rope_pairs=(0, 16, 16), **one)
    S = 65536
    h = encoder(cfg, 2 * S, S, 1)
    fake.fake_forget()
    B.epd_encode(h, POOL, np.arange(S + 1, dtype=np.int32) * 2, [(S, 1, 2)], POOL, None)
    check("pads", ["plan_kernel", "attn_bf16", "gemm_bf16"])
    # preprocessing: 33 slices of 512 x 512 patches of 32 x 32 pixels, a block of 512 threads each
    cfg = W.EncoderConfig(dtype="bf16", hidden=64, num_heads=1, head_dim=64, rope="2d", rope_pairs=(0, 16, 16), in_channels=1,
                          **dict(one, patch=32))
    T = 33 * 512 * 512
    h = encoder(cfg, T, 1, 2)
    fake.fake_forget()
    B.epd_preprocess(h, POOL, [(16384, 16384)], [(33, 512, 512)], [0.5], [0.25], POOL, None)
    check("patches", ["preprocess_kernel"])
    assert sum(g[0] for n, g, _ in launches(fake)) == T
    fake.fake_forget()
    B.epd_preprocess(h, POOL, [(50, 60), (64, 64)], [(1, 3, 5), (1, 2, 2)], [0.5], [0.25], POOL, None)
    assert [l[1:] for l in launches(fake)] == [((19, 1, 1), (512, 1, 1))]


# ------------------------------------------------------------------ launches of the bf16 GEMMs

def gemm_shim():
    C.CDLL(sys.argv[2], mode=C.RTLD_GLOBAL)                              # its names are for the shim
    shim = C.CDLL(sys.argv[4])
    shim.shim_gemm.argtypes = [C.c_int] * 8
    shim.shim_rot_lds.argtypes = [C.c_void_p]
    return shim


def gemm_launches(fake):
    """(tile rows, tile columns, gathered, whole tiles without clamping, blocks) of every bf16 GEMM launch."""
    out = []
    for name, grid, _ in launches(fake):
        m = re.search(r"gemm_bf16_kernelINS_4TileILi(\d+)ELi(\d+)E.*?EELi\d+ELi\d+ELb([01])ELb([01])E", name)
        if m:
            out.append((int(m[1]), int(m[2]), m[3] == "1", m[4] == "1", grid[0]))
    return out


def gathered_gemm_reads_past_its_weights_only_where_allowed(fake, lib):
    """Loads that take whole tiles read W past its last row, and A past its last row where its rows are not gathered."""
    shim = gemm_shim()
    for tile in (0, 2, 4, 5, 7, 8):
        for gather_n in (0, 4):
            for may_read in range(4):
                fake.fake_forget()
                shim.shim_gemm(300, 200, 512, 0, gather_n, may_read, tile, 256)
                (l,) = gemm_launches(fake)
                assert l[2] == (gather_n > 0)
                needs = 2 if gather_n else 3
                assert not l[3] or may_read & needs == needs, (tile, gather_n, may_read, l)
                # ... and where they are allowed they are taken (gathered rows: the large tiles)
                assert l[3] or may_read & needs != needs or (gather_n and tile in (4, 7, 8)), (tile, gather_n, may_read, l)


def rotary_table_rule_counts_the_units_of_the_stream(fake, lib):
    """The rotary table goes through LDS in launches of up to two rounds -- of the units the call runs on, not of a whole chip."""
    shim = gemm_shim()
    fake.fake_keep_args(b"gemm_bf16_kernel", shim.shim_args_size())
    seen = set()
    for tile, cols in ((0, 256), (5, 256), (2, 128)):
        for units in (0, 64, 128, 208, 256):
            for M in (2000, 7000, 12000, 16640, 30000, 60000):
                fake.fake_forget()
                shim.shim_gemm(M, 3072, 1024, 3, 0, 3, tile, units)
                (l,) = gemm_launches(fake)
                assert l[1] == cols
                two_rounds = l[4] <= 2 * (units or 256)
                assert shim.shim_rot_lds(fake.fake_args(0)) == two_rounds, (tile, units, M, l)
                seen.add((units, two_rounds))
    assert len(seen) == 10                                              # both answers for every number of units


def rows_behind_the_last_full_round(fake, lib):
    """Launches that are cut: the tile and the number of blocks of both parts on 256 units."""
    shim = gemm_shim()

    def plan(M, N, K, epilogue):
        fake.fake_forget()
        shim.shim_gemm(M, N, K, epilogue, 0, 3, -1, 256)
        return [(l[0], l[1], l[4]) for l in gemm_launches(fake)]

    G, R, Q = 1, 2, 3
    # against a long K the rest is one round of 256 x 128 tiles
    assert plan(32768, 3200, 12800, R) == [(256, 256, 118 * 13), (256, 128, 10 * 25)]
    assert plan(32768, 3200, 3200, R) == [(256, 256, 118 * 13), (256, 128, 10 * 25)]
    # ... and 128 x 128 tiles against a short one, with another epilogue, or where it would be more than one round
    assert plan(6272, 4096, 1024, G) == [(320, 256, 16 * 16), (128, 128, 9 * 32)]
    assert plan(9124, 2304, 768, Q) == [(256, 256, 28 * 9), (128, 128, 16 * 18)]
    for M in range(9000, 60000, 1111):
        for N in (1024, 1152, 3200):
            for K in (1024, 2048, 4352):
                l = plan(M, N, K, R)
                if len(l) == 2:
                    rest = M - l[0][2] // -(-N // 256) * l[0][0]
                    assert 0 < rest < M
                    assert l[1] in ((128, 128, -(-rest // 128) * -(-N // 128)), (256, 128, -(-rest // 256) * -(-N // 128))), (M, N, K, l)
                    assert l[1][1] == 128 and (l[1][0] == 128 or (K >= 2048 and l[1][2] <= 256)), (M, N, K, l)


if __name__ == "__main__":
    globals()[sys.argv[3]](*load(sys.argv[1], sys.argv[2]))
    print("passed", sys.argv[3])
