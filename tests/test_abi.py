"""The C-ABI library loads without a GPU, exports every function the header declares, and
rejects bad arguments on the host before anything is launched."""
import ctypes as C
import os
import re

import pytest

import paper_2508_06526_amd as pk
from paper_2508_06526_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "pikv.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(pikv_[a-z_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(pk.library_path()):
        from paper_2508_06526_amd import build
        build.build()
    return pk.load_library()


def test_every_declared_symbol_is_exported(lib):
    names = declared_functions()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_version_and_strerror(lib):
    assert pk.pikv_version() >= 100
    assert pk.pikv_strerror(0) == "ok"
    for code in (-1, -2, -3, -4, 77):
        assert pk.pikv_strerror(code)


def test_desc_struct_matches_header_layout():
    assert C.sizeof(pk.PikvDesc) == 64
    assert pk.PikvDesc.stride_h.offset == 32 and pk.PikvDesc.route_rows_per_seq.offset == 48
    assert pk.PikvDesc.flags.offset == 52 and pk.PikvDesc.tq.offset == 56


def test_workspace_size_is_zero_for_bad_geometry_and_positive_otherwise(lib):
    good = pk.make_desc(1, 32, 8, 128, 16, 8192)
    assert pk.pikv_attn_workspace_bytes(good, 4) > 0
    assert pk.pikv_attn_workspace_bytes(good, 0) == 0
    assert pk.pikv_attn_workspace_bytes(good, 17) == 0
    assert pk.pikv_attn_workspace_bytes(pk.make_desc(1, 32, 5, 128, 16, 8192), 4) == 0   # Hq % Hkv
    assert pk.pikv_attn_workspace_bytes(pk.make_desc(1, 32, 8, 96, 16, 8192), 4) == 0    # D
    assert pk.pikv_attn_workspace_bytes(pk.make_desc(1, 32, 8, 128, 65, 8192), 4) == 0   # E > 64
    assert pk.pikv_attn_workspace_bytes(pk.make_desc(1, 32, 8, 128, 16, 8192, rank=24), 4) == 0


def test_multi_query_steps_reach_to_the_32_bit_limit_of_a_kv_head(lib):
    """Draft queries are taken as long as the rows of a kv head span less than 4 GiB, whatever the row
    stride; from there on no kernel takes them."""
    for S in (1, 8, 40, 8192):
        below, at = ((1 << 31) - 8) // S // 8 * 8, -(-(1 << 31) // S // 8) * 8
        assert S * below * 2 < 1 << 32 <= S * at * 2
        for G in (2, 16, 32, 64):
            assert pk.pikv_attn_workspace_bytes(pk.make_desc(1, G, 1, 128, 4, S, stride_s=below, dtype=1, tq=2), 2) > 0
            assert pk.pikv_attn_workspace_bytes(pk.make_desc(1, G, 1, 128, 4, S, stride_s=at, dtype=1, tq=2), 2) == 0


def splits_of(desc, k):
    """Splits of the attention plan, from the workspace it asks for."""
    w = desc.rank or desc.D
    acc = lambda n: -(-desc.B * desc.Hq * k * n * w * 4 // 256) * 256 + -(-desc.B * desc.Hq * k * n * 2 * 4 // 256) * 256 + 256
    return next(n for n in range(1, 2049) if acc(n) == pk.pikv_attn_workspace_bytes(desc, k))


@pytest.mark.parametrize("rank", [0, 64])
def test_small_groups_of_narrow_rows_are_planned_one_head_per_block(lib, rank):
    """A few blocks of whole groups leave the chip empty: small calls with groups of other than 2, 4 or 8
    heads are cut as the one-head kernel cuts them (256 rows a split at the least; whole groups
    take 512), calls with blocks enough are not."""
    few = pk.make_desc(1, 48, 4, 64, 4, 847, rank=rank, dtype=1)
    assert splits_of(few, 3) == 3
    many = pk.make_desc(16, 48, 4, 64, 4, 847, rank=rank, dtype=1)
    assert splits_of(many, 3) == 1
    assert splits_of(pk.make_desc(1, 32, 4, 64, 4, 1100, rank=rank, dtype=1), 3) == 2      # 8 heads: always whole groups


def test_long_narrow_shards_are_cut_until_their_scores_fit_beside_the_tiles(lib):
    """More units than a round of blocks and shards whose scores of one split do not fit the LDS: the splits
    go up until they do, for groups of up to 4 rows, down to 4 rounds of tiles per block."""
    assert splits_of(pk.make_desc(32, 64, 16, 32, 8, 8832, dtype=1), 4) == 3               # 4 heads: 47 KiB for 2944 rows
    assert splits_of(pk.make_desc(32, 128, 16, 32, 8, 8832, dtype=1), 4) == 1              # 8 heads


@pytest.mark.parametrize("B,Hkv,k,S,group,splits", [
    (16, 4, 2, 4096, dict(D=64, G=8), 2), (16, 4, 2, 4097, dict(D=64, G=8), 4),          # 512 KiB of a block, 128 units
    (16, 8, 2, 4096, dict(D=128, G=4, rank=32), 1), (16, 8, 2, 4097, dict(D=128, G=4, rank=32), 4),
    (16, 8, 2, 2048, dict(D=128, G=4, rank=16), 1), (16, 8, 2, 2049, dict(D=128, G=4, rank=16), 2),   # 128 KiB
    (4, 8, 2, 4096, dict(D=128, G=4), 4), (4, 8, 2, 4097, dict(D=128, G=4), 12),
    (17, 4, 1, 4096, dict(D=64, G=8), 3), (8, 8, 3, 1024, dict(D=64, G=8), 1), (8, 8, 3, 1025, dict(D=64, G=8), 2),   # 204 blocks, 192
    (1, 8, 3, 8192, dict(D=128, G=4), 32), (3, 8, 1, 8192, dict(D=128, G=4), 10),        # 30 and 10 partials of a head
    (1, 8, 8, 4096, dict(D=64, G=8), 8), (1, 8, 8, 1024, dict(D=64, G=8), 4),            # 32 partials, short blocks
    (4, 8, 2, 1024, dict(D=128, G=4), 4), (4, 8, 2, 4096, dict(D=128, G=16), 8),         # two rounds; 16 rows
])
def test_groups_whose_units_make_a_block_per_cu(lib, B, Hkv, k, S, group, splits):
    """256 / units splits on one side of each line of the rule, the plan of several blocks per CU on the other."""
    desc = pk.make_desc(B, Hkv * group["G"], Hkv, group["D"], 16, S, rank=group.get("rank", 0), dtype=1)
    assert splits_of(desc, k) == splits


def test_host_side_argument_errors(lib):
    """NULL pointers / out-of-range sizes return PIKV_ERR_INVALID with no GPU present."""
    vp = C.c_void_p
    fake = vp(0x1000)        # never dereferenced: every call below fails validation first
    INVALID, UNSUPPORTED, WORKSPACE = -1, -2, -3
    r = lib.pikv_route
    assert r(None, fake, None, 1, 8, 4, 2, 0, fake, fake, None, None) == INVALID
    assert r(fake, fake, None, 1, 8, 4, 5, 0, fake, fake, None, None) == INVALID      # k > E
    assert r(fake, fake, None, 1, 8, 65, 2, 0, fake, fake, None, None) == INVALID     # E > 64
    assert r(fake, fake, None, 1, 0, 4, 2, 0, fake, fake, None, None) == INVALID      # d_r
    assert r(fake, fake, None, 1, 8, 4, 2, 9, fake, fake, None, None) == INVALID      # dtype
    assert r(fake, fake, None, 0, 8, 4, 2, 0, fake, fake, None, None) == 0            # no rows

    d = pk.make_desc(1, 4, 4, 64, 4, 256)
    a = lib.pikv_sharded_attn

    def attn(desc, q=fake, k=2, combine=0, ws=fake, ws_bytes=1 << 30, y=fake, uk=None):
        return a(C.byref(desc), q, fake, fake, uk, uk, fake, fake, None, k, combine, 0.0, y, None,
                 None, None, None, ws, ws_bytes, None)
    assert attn(d, q=None) == INVALID
    assert attn(d, y=None) == INVALID
    assert attn(d, k=0) == INVALID
    assert attn(d, combine=3) == INVALID
    assert attn(d, ws_bytes=16) == WORKSPACE
    assert attn(d, ws=None) == WORKSPACE
    assert attn(pk.make_desc(1, 4, 4, 64, 4, 256, rank=32)) == INVALID                 # U_K missing
    assert attn(pk.make_desc(1, 4, 4, 48, 4, 256)) == UNSUPPORTED
    assert attn(pk.make_desc(1, 4, 4, 64, 4, 256, stride_s=60)) == INVALID
    assert attn(pk.make_desc(1, 4, 4, 64, 4, 256, route_rows_per_seq=2)) == INVALID
    assert attn(pk.make_desc(0, 4, 4, 64, 4, 256)) == 0                                # B == 0

    u = lib.pikv_update_utility
    assert u(C.byref(d), None, fake, fake, fake, 2, 1.0, fake, None) == INVALID
    assert u(C.byref(d), fake, fake, fake, fake, 2, -0.5, fake, None) == INVALID
    assert u(C.byref(d), fake, fake, fake, fake, 9, 1.0, fake, None) == INVALID
    assert u(C.byref(d), fake, fake, fake, fake, 2, float("nan"), fake, None) == INVALID

    e = lib.pikv_evict
    assert e(C.byref(d), None, fake, 10, None, 0, fake, fake, 4, 0, None, None, None) == INVALID
    assert e(C.byref(d), fake, fake, -1, None, 0, fake, fake, 4, 0, None, None, None) == INVALID
    assert e(C.byref(d), fake, fake, 10, None, 0, fake, fake, 0, 0, None, None, None) == INVALID
    assert e(C.byref(d), fake, fake, 10, fake, 0, fake, fake, 4, 0, None, None, None) == INVALID
    assert e(C.byref(d), fake, fake, 10, None, 0, fake, fake, 4, 1, None, None, None) == INVALID

    ap = lib.pikv_append
    assert ap(C.byref(d), None, fake, fake, 2, None, None, 0, fake, fake, fake, fake, None) == INVALID
    assert ap(C.byref(d), fake, fake, fake, 5, None, None, 0, fake, fake, fake, fake, None) == INVALID
    assert ap(C.byref(d), fake, fake, fake, 2, fake, None, 1, fake, fake, fake, fake, None) == INVALID


def test_host_side_argument_errors_of_the_widened_entry_points(lib):
    vp = C.c_void_p
    fake = vp(0x1000)        # never dereferenced
    INVALID, UNSUPPORTED, WORKSPACE = -1, -2, -3
    d = pk.make_desc(2, 4, 4, 64, 8, 256, dtype=1)

    def step(desc=d, q=fake, K_new=fake, V_new=fake, eidx=fake, k=2, decay=1.0, combine=0, ws=fake,
             ws_bytes=1 << 30, scores=fake, scale=0.0, U=None):
        return lib.pikv_decode_step(C.byref(desc), q, fake, None, K_new, V_new, fake, fake, U, U, fake,
                                    fake, k, combine, scale, decay, fake, fake, eidx, fake, fake, None, None,
                                    scores, fake, ws, ws_bytes, None)
    assert step(q=None) == INVALID
    assert step(V_new=None) == INVALID                     # K_new without V_new
    assert step(eidx=None) == INVALID                      # insert without the eviction outputs
    assert step(k=0) == INVALID and step(k=9) == INVALID
    assert step(decay=-1.0) == INVALID and step(combine=2) == INVALID
    assert step(scores=None) == INVALID
    assert step(ws_bytes=8) == WORKSPACE
    # the checks of the attention pass are made before the step's first launch as well
    assert step(ws=vp(0x1010)) == INVALID                  # workspace not 256-byte aligned
    assert step(scale=float("nan")) == INVALID
    assert step(desc=pk.make_desc(2, 4, 4, 64, 8, 256, rank=32, dtype=1)) == INVALID   # codes without decoders
    assert step(desc=pk.make_desc(2, 4, 4, 64, 8, 256, dtype=1, route_rows_per_seq=4)) == UNSUPPORTED
    assert step(desc=pk.make_desc(0, 4, 4, 64, 4, 256, dtype=1)) == 0   # W_r rows of 8 bytes: accepted (nothing to launch)
    assert step(desc=pk.make_desc(0, 4, 4, 64, 8, 256, dtype=1)) == 0

    rr = lib.pikv_route_round_robin
    rr.argtypes = [C.c_int32, C.c_int32, C.c_int32, C.c_int64, vp, vp, vp]
    assert rr(2, 8, 9, 0, fake, fake, None) == INVALID
    assert rr(2, 65, 2, 0, fake, fake, None) == INVALID
    assert rr(2, 8, 2, -1, fake, fake, None) == INVALID
    assert rr(2, 8, 2, 0, None, fake, None) == INVALID
    assert rr(0, 8, 2, 0, fake, fake, None) == 0

    rp = lib.pikv_router_penalty
    assert rp(7, fake, 1, 2, 8, fake, None, 0.1, fake, None) == INVALID
    assert rp(3, fake, 1, 2, 8, fake, None, 0.1, fake, None) == INVALID           # modes are 0, 1, 2
    assert rp(0, fake, 1, 2, 8, None, None, 0.1, fake, None) == INVALID
    assert rp(0, fake, 1, 2, 65, fake, None, 0.1, fake, None) == INVALID
    assert rp(1, fake, 1, 2, 8, fake, None, 0.1, fake, None) == INVALID           # cache-aware needs miss
    assert rp(0, fake, 1, 2, 8, fake, None, float("nan"), fake, None) == INVALID

    cp = lib.pikv_compress
    dr = pk.make_desc(2, 4, 4, 64, 8, 256, rank=32, dtype=1)
    assert cp(C.byref(d), fake, fake, fake, None, None, None, None) == INVALID    # rank == 0
    assert cp(C.byref(dr), None, fake, fake, None, None, None, None) == INVALID
    assert cp(C.byref(dr), fake, fake, fake, fake, None, None, None) == INVALID   # partly given V

    st = lib.pikv_policy_stamp
    assert st(C.byref(d), None, 2, None, None, 0, fake, 5, fake, fake, fake, None) == INVALID
    assert st(C.byref(d), fake, 9, None, None, 0, fake, 5, fake, fake, fake, None) == INVALID
    assert st(C.byref(d), fake, 2, fake, None, 1, fake, 5, fake, fake, fake, None) == INVALID
    assert st(C.byref(d), fake, 2, fake, fake, 0, fake, 5, fake, fake, fake, None) == INVALID
    assert st(C.byref(pk.make_desc(2, 4, 4, 64, 8, 256, dtype=1, route_rows_per_seq=4)), fake, 2, None, None, 0,
              fake, 5, fake, fake, fake, None) == UNSUPPORTED

    tr = lib.pikv_update_utility_tracked
    assert tr(C.byref(d), fake, fake, fake, fake, 2, 1.0, None, 0.1, 5, None, fake, None) == INVALID
    assert tr(C.byref(d), fake, fake, fake, fake, 2, 1.0, None, -0.1, 5, fake, fake, None) == INVALID
    assert tr(C.byref(d), fake, fake, fake, fake, 2, -1.0, fake, 0.1, 5, fake, fake, None) == INVALID
    assert tr(C.byref(pk.make_desc(0, 4, 4, 64, 8, 256, dtype=1)), fake, fake, fake, fake, 2, 1.0, None, 0.1, 5,
              fake, fake, None) == 0

    lib.pikv_decode_step_policy.argtypes = list(lib.pikv_decode_step.argtypes) + [vp, vp]
    lib.pikv_decode_step_policy.restype = C.c_int

    def pstep(args):
        return lib.pikv_decode_step_policy(C.byref(d), fake, fake, None, fake, fake, fake, fake, None, None, fake,
                                           fake, 2, 0, 0.0, 1.0, fake, fake, fake, fake, fake, None, None, fake,
                                           fake, fake, 1 << 30, None, C.cast(C.pointer(args), vp), None)
    fakeptr = 0x1000
    bad = pk.PikvPolicyArgs(policy=9, now=1)
    assert pstep(bad) == INVALID
    assert pstep(pk.PikvPolicyArgs(policy=pk.POLICY_LRU, now=1)) == INVALID                     # needs last_access
    assert pstep(pk.PikvPolicyArgs(policy=pk.POLICY_SL, now=1, window=4)) == INVALID             # needs birth
    assert pstep(pk.PikvPolicyArgs(policy=pk.POLICY_LRU, now=1, last_access=fakeptr, freq=fakeptr,
                                   threshold=-1.0)) == INVALID                                   # tracking threshold
    assert pstep(pk.PikvPolicyArgs(policy=pk.POLICY_LRU_PLUS, now=1, lam=float("nan"), last_access=fakeptr,
                                   freq=fakeptr)) == INVALID
    def fstep(fb):
        return lib.pikv_decode_step_policy(C.byref(d), fake, fake, None, fake, fake, fake, fake, None, None, fake,
                                           fake, 2, 0, 0.0, 1.0, fake, fake, fake, fake, fake, None, None, fake,
                                           fake, fake, 1 << 30, None, None, C.cast(C.pointer(fb), vp))
    assert fstep(pk.PikvRouterFeedback(mode=5, coef=0.1, load=fakeptr, bias=fakeptr)) == INVALID
    assert fstep(pk.PikvRouterFeedback(mode=0, coef=0.1, load=None, bias=fakeptr)) == INVALID
    assert fstep(pk.PikvRouterFeedback(mode=1, coef=0.1, load=fakeptr, bias=fakeptr)) == INVALID   # needs miss
    assert fstep(pk.PikvRouterFeedback(mode=2, coef=float("nan"), load=fakeptr, bias=fakeptr)) == INVALID
    # descriptor flags: only the value-bias bit, and only with codes
    assert step(desc=pk.make_desc(2, 4, 4, 64, 8, 256, dtype=1, flags=1)) == INVALID
    assert step(desc=pk.make_desc(2, 4, 4, 64, 8, 256, dtype=1, flags=2)) == INVALID
    pc = lib.pikv_policy_compact
    assert pc(C.byref(d), None, fake, 4, fake, fake, fake, fake, None) == INVALID
    assert pc(C.byref(d), fake, fake, 0, fake, fake, fake, fake, None) == INVALID
    assert pc(C.byref(pk.make_desc(0, 4, 4, 64, 8, 256, dtype=1)), fake, fake, 4, fake, fake, fake, fake, None) == 0

    pu = lib.pikv_policy_utility
    assert pu(C.byref(d), 4, fake, 5, 0.0, 0, 0, fake, fake, fake, fake, fake, None) == INVALID
    assert pu(C.byref(d), 0, fake, 5, 0.0, 0, 0, fake, fake, fake, None, fake, None) == INVALID   # H2O needs h2o
    assert pu(C.byref(d), 1, fake, 5, 0.0, 3, 0, None, fake, fake, None, fake, None) == INVALID   # SL needs birth
    assert pu(C.byref(d), 2, fake, 5, 0.0, 0, 0, fake, None, fake, None, fake, None) == INVALID   # LRU needs last
    assert pu(C.byref(d), 3, fake, 5, float("nan"), 0, 0, fake, fake, fake, None, fake, None) == INVALID
    assert pu(C.byref(d), 2, fake, 5, 0.0, -1, 0, fake, fake, fake, None, fake, None) == INVALID
    assert pu(C.byref(d), 2, fake, 5, 0.0, 0, 2, None, fake, fake, None, fake, None) == INVALID   # protect needs birth
    assert pu(C.byref(d), 2, fake, 5, 0.0, 0, 0, None, fake, None, None, None, None) == INVALID   # out


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(OSError):
        binding.load_library()


@pytest.mark.parametrize("kind", ["absent", "unloadable"])
def test_binding_without_its_extension_takes_the_ctypes_path(tmp_path, monkeypatch, kind):
    """The extension belongs to one Python and one torch; where it is not there or does not load, libpikv.so alone is enough: every
    call goes through ctypes, which refuses host memory here as it always has."""
    import torch

    from paper_2508_06526_amd import binding
    path = tmp_path / "_pikv_native.so"
    if kind == "unloadable":
        path.write_bytes(b"built for another Python")
    monkeypatch.setattr(binding, "_NATIVE_PATH", str(path))
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    with pytest.warns(RuntimeWarning, match="_pikv_native"):
        lib = binding.load_library()
    assert lib.pikv_version() >= 100
    x = torch.zeros((2, 8))
    with pytest.raises(ValueError, match="device memory"):
        binding.pikv_route(x, x, None, 2, 8, 4, 2, x, x)
    desc = binding.make_desc(0, 4, 4, 64, 4, 16)             # no sequences: a checked call that launches nothing
    binding._check(lib.pikv_append(desc, 16, 16, 16, 2, None, None, 0, 16, 16, 16, 16, None), "pikv_append")
    for name in binding.EXPORTS:
        assert getattr(binding._calls(), name)(1, 2, 3) is None


def test_a_call_the_extension_leaves_to_ctypes_is_left_at_once():
    """Numbers of other types and tensor subclasses take the ctypes path, as they did before there was an extension: finding that
    out may not cost a C++ exception (4 us, as much as the whole call).  Against a call with the wrong number of arguments,
    which is turned down before any is looked at: 1.5 to 4 times as long, 23 with exceptions."""
    import time

    import torch
    native = binding._calls()
    x, many = torch.zeros((2, 8)), 20000

    def best(*args):
        times = []
        for _ in range(7):
            start = time.perf_counter()
            for _ in range(many):
                assert native.pikv_route(*args) is None
            times.append(time.perf_counter() - start)
        return min(times)

    nothing = best()
    assert best(x, x, None, 2, 8, 4, 2, x, x, None, None) < 10 * nothing            # on the host
    assert best(None, None, None, 2.0, 8, 4, 2, None, None, None, None) < 10 * nothing
