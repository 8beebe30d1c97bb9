"""No-GPU checks of the boundary: the library loads, exports every function include/dream.h declares,
and rejects bad arguments on the host before anything is launched."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import paper_2505_19201_amd as dream
from paper_2505_19201_amd import build as dream_build


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(dream.library_path()):
        dream_build.build(verbose=False)
    return dream.load()


def _declared_functions():
    """Every function any header under include/ declares (the boundary in dream.h, the test switches in dream_tuning.h)."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    names = set()
    for header in sorted(os.listdir(os.path.join(root, "include"))):
        text = open(os.path.join(root, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(dream_[a-z_]+)\s*\(", text))
    return sorted(names)


def test_every_declared_function_is_exported(lib):
    names = _declared_functions()
    assert {"dream_tree_verify_attn", "dream_draft_xattn", "dream_visual_compress", "dream_accept_path"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(dream.EXPORTED_SYMBOLS) == names


def test_binding_never_imports_the_oracle():
    import sys
    src = open(dream.binding.__file__).read() + open(dream.__file__).read()
    assert "oracle" not in src.replace("no CPU fallback", "")
    assert "oracle" not in [m.split(".")[0] for m in sys.modules if m.startswith("paper_2505_19201_amd")]


def test_tree_validation_on_host(lib):
    assert dream.dream_tree_validate_host(np.array([-1, 0, 0, 1, 3, 4])) == 4
    assert dream.dream_tree_validate_host(np.array([-1])) == 0
    for bad in ([0, 0], [-1, 1], [-1, 0, 3], [-1, -1]):
        with pytest.raises(dream.DreamError) as e:
            dream.dream_tree_validate_host(np.array(bad))
        assert e.value.status == -1


def test_host_side_argument_errors(lib):
    d = dream.attn_desc(1, 4, 4, 64, dream.BF16, 128)
    one = C.c_void_p(16)      # never dereferenced: every call below fails validation first
    f = lib.dream_tree_verify_attn
    args = lambda desc, n_tree=8, maxkv=100, ws=one, wsb=1 << 30, q=one: (  # noqa: E731
        C.byref(desc), q, one, one, one, C.c_int32(n_tree), one, None, C.c_int64(maxkv), one, None, ws, C.c_size_t(wsb), None)
    assert f(*args(d, q=None)) == -1
    assert f(*args(dream.attn_desc(1, 6, 4, 64, dream.BF16, 128))) == -1          # Hq % Hkv
    assert f(*args(dream.attn_desc(1, 4, 4, 96, dream.BF16, 128))) == -2          # head_dim
    assert f(*args(d, n_tree=257)) == -2
    assert f(*args(d, n_tree=0)) == -2
    assert f(*args(d, maxkv=129)) == -1                                           # beyond s_max
    big = dream.attn_desc(1, 32, 8, 128, dream.BF16, 4200)                        # a long cache with few KV heads: key splits need a workspace
    assert dream.dream_tree_verify_attn_workspace(big, 60, 4156) > 65536
    assert f(*args(big, n_tree=60, maxkv=4156, wsb=65536)) == -3                   # workspace too small
    assert "workspace" in dream.dream_last_error()
    g = lib.dream_accept_path
    assert g(one, C.c_int32(1), C.c_int32(1), C.c_int32(2000), C.c_int32(100), one, one, C.c_int32(6), one, one, one, one,
             one, C.c_size_t(1 << 30), None) == -2
    assert g(one, C.c_int32(5), C.c_int32(1), C.c_int32(8), C.c_int32(100), one, one, C.c_int32(6), one, one, one, one,
             one, C.c_size_t(1 << 30), None) == -1
    h = lib.dream_visual_compress
    base = [C.byref(d), one, None, C.c_int32(64), one, C.c_int32(64), C.c_int32(0), C.c_int32(32), C.c_int32(1), C.c_int32(2),
            None, None, None, one, None, None, C.c_int64(0), None, C.c_int64(0), one, C.c_size_t(1 << 30), None]
    bad = list(base); bad[9] = C.c_int32(0)
    assert h(*bad) == -1                                                          # keep_den
    bad = list(base); bad[8] = C.c_int32(3)
    assert h(*bad) == -1                                                          # keep_num > keep_den
    bad = list(base); bad[6] = C.c_int32(40)
    assert h(*bad) == -1                                                          # span beyond keys
    bad = list(base); bad[20] = C.c_size_t(16)
    assert h(*bad) == -3


def test_workspace_sizes_are_monotone(lib):
    d = dream.attn_desc(1, 32, 32, 128, dream.BF16, 800)
    a = dream.dream_tree_verify_attn_workspace(d, 60, 764)
    assert a >= 256
    dream.dream_set_kv_splits(4)
    try:
        assert dream.dream_tree_verify_attn_workspace(d, 60, 764) > a            # forced splits need room for their states
    finally:
        dream.dream_set_kv_splits(0)
    assert dream.dream_accept_path_workspace(1, 60, 32000) >= 2 * 60 * 4 * 4
    assert dream.dream_visual_compress_workspace(d, 704, 576) >= 32 * 704 * 4 + 32 * 576 * 4


def test_launch_plans_of_the_paper_shapes(lib):
    """The plan is host logic: one sequence with a short cache takes the single-launch wave kernel with its output
    columns split over workgroups (MHA, and GQA groups of up to 4 heads), a long cache or a batch of sequences the
    shared-tile kernel, with key splits and a merge launch where the streams are few."""
    def plan(B, hq, hkv, d, n_q, s):
        return dream.dream_attn_plan_describe(dream.attn_desc(B, hq, hkv, d, dream.BF16, s), n_q, s)
    llava = plan(1, 32, 32, 128, 60, 764)
    assert llava.startswith("attn_wave_kernel<128,8,2,1>") and "workgroups=256" in llava and "merge_launch=0" in llava
    level = plan(1, 32, 32, 128, 16, 764)            # one drafted tree level: a single query tile per head
    assert level.startswith("attn_wave_kernel<128,8,4,1>") and "workgroups=128" in level
    pixtral = plan(1, 32, 8, 128, 60, 1340)
    assert pixtral.startswith("attn_wave_kernel<128,8,2,1>") and "workgroups=256" in pixtral and "merge_launch=0" in pixtral
    gemma3 = plan(1, 16, 8, 256, 60, 1340)
    assert gemma3.startswith("attn_wave_kernel<256,4,4,1>") and "workgroups=256" in gemma3
    long_cache = plan(1, 32, 8, 128, 60, 4156)        # more than 64 key tiles
    assert long_cache.startswith("attn_bf16_kernel<128,1,") and "splits=8" in long_cache and "merge_launch=1" in long_cache
    batch = plan(32, 32, 32, 64, 60, 1660)
    assert batch.startswith("attn_bf16_kernel<64,1,") and "splits=1 " in batch and "merge_launch=0" in batch
    f32 = dream.dream_attn_plan_describe(dream.attn_desc(1, 4, 4, 64, dream.F32, 104), 8, 104)
    assert f32.startswith("attn_f32_kernel")
    with pytest.raises(dream.DreamError):
        dream.dream_attn_plan_describe(dream.attn_desc(1, 32, 32, 96, dream.BF16, 764), 60, 764)


def test_every_attention_kernel_variant_has_a_parity_case(lib):
    """The GPU suite runs tests/attn_cases.VARIANT_CASES all elements against the oracle; here, without a GPU: the
    list names every variant the library can dispatch to, and each case's shape really plans its variant."""
    import dream_inputs as di
    from tests.attn_cases import (EXTRA_W8_CASES, FULL_VERIFY_PLANS, FULL_XATTN_PLANS, STREAMING_PLANS, VARIANT_CASES, variant_config,
                                  variant_prefix_lens)
    built = dream.dream_attn_variants()
    assert len(built) == len(set(built))
    assert sorted(c.variant for c in VARIANT_CASES) == sorted(built)
    for case in VARIANT_CASES + EXTRA_W8_CASES:
        cfg = variant_config(case)
        pl = variant_prefix_lens(case)
        assert max(pl) == pl[0] == case.kv_len - case.n_tree and min(pl) >= 0
        dream.dream_set_kv_splits(case.splits)
        dream.dream_set_q_tiles(case.q_tiles)
        dream.dream_set_tile_waves(case.waves)
        try:
            desc = dream.attn_desc(cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, dream.BF16, case.kv_len + 5)
            plan = dream.dream_attn_plan_describe(desc, case.n_tree, case.kv_len)
        finally:
            dream.dream_set_kv_splits(0)
            dream.dream_set_q_tiles(0)
            dream.dream_set_tile_waves(0)
        assert plan.startswith(case.variant + " "), (case, plan)
    for name, want in FULL_VERIFY_PLANS.items():
        cfg = di.CONFIGS[name]
        S = cfg.prefix + cfg.n_tree
        desc = dream.attn_desc(cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, dream.BF16, S + 5)
        assert dream.dream_attn_plan_describe(desc, cfg.n_tree, S) == want, name
        for n_q, want_x in zip((1, 10), FULL_XATTN_PLANS[name]):
            assert dream.dream_attn_plan_describe(desc, n_q, S) == want_x, (name, n_q)
        assert want.split(" ")[0] in built
    for name, want in STREAMING_PLANS.items():
        cfg = di.CONFIGS[name].with_batch(32)
        S = cfg.prefix + cfg.n_tree
        desc = dream.attn_desc(cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, dream.BF16, S)
        assert dream.dream_attn_plan_describe(desc, cfg.n_tree, S) == want, name


def test_kv_commit_argument_errors(lib):
    """Host-side checks of dream_kv_commit return before any launch."""
    import ctypes as C
    desc = dream.attn_desc(1, 4, 4, 128, dream.BF16, 100)
    ptrs = (C.c_void_p * 1)(0x1000)
    fake = C.c_void_p(0x2000)

    def call(d=desc, caches=ptrs, n=1, pl=fake, n_tree=8, path=fake, stride=7, alen=fake, out=None):
        return lib.dream_kv_commit(C.byref(d), caches, C.c_int32(n), pl, C.c_int32(n_tree), path, C.c_int32(stride), alen,
                                   out, None)
    assert call(caches=None) == -1
    assert call(n=0) == -1
    assert call(n_tree=0) == -1
    assert call(n_tree=101) == -1                  # the tree rows must fit the cache
    assert call(stride=0) == -1
    assert call(out=fake) == -1                    # aliases prefix_len
    assert "alias" in dream.dream_last_error()
    assert call(caches=(C.c_void_p * 1)(0x1008)) == -1   # not 16-byte aligned
    assert call(caches=(C.c_void_p * 1)(None)) == -1
    wide = dream.attn_desc(1, 4, 4, 1024, dream.F32, 1000)   # 4 KB rows: 64 of them exceed 64 KB
    assert call(d=wide, n_tree=64, stride=64) == -2
    odd = dream.attn_desc(1, 4, 4, 60, dream.BF16, 100)      # 120-byte rows
    assert call(d=odd) == -2


def test_tree_build_argument_errors(lib):
    """Host-side checks of the tree-construction entry points return before any launch."""
    import ctypes as C
    fake = C.c_void_p(0x1000)

    def expand(logits=fake, dt=dream.BF16, B=1, F=4, V=32000, cum=fake, k=4, tok=fake, sc=fake, nxt=fake, ws=fake, nb=1 << 30):
        return lib.dream_tree_expand_level(logits, C.c_int32(dt), C.c_int32(B), C.c_int32(F), C.c_int32(V), cum, C.c_int32(k), tok, sc,
                                           nxt, ws, C.c_size_t(nb), None)
    assert expand(logits=None) == -1 and expand(cum=None) == -1 and expand(nxt=None) == -1
    assert expand(dt=7) == -1
    assert expand(F=0) == -1 and expand(F=17) == -1
    assert expand(k=0) == -1 and expand(k=17) == -1 and expand(V=3, k=4) == -1
    assert expand(B=0) == -1 and expand(B=5000, F=16) == -1
    need = dream.dream_tree_expand_workspace(1, 4, 32000, 4)
    assert need > 256 and expand(nb=need - 1) == -3 and expand(ws=None) == -3
    assert dream.dream_tree_expand_workspace(1, 4, 262144, 4) > need
    assert dream.dream_tree_expand_workspace(2, 4, 32000, 4) > need

    def finalize(score=fake, parent=fake, token=fake, B=1, N=85, budget=32, tp=fake, tt=fake, ti=fake):
        n = C.c_int32(-1)
        return lib.dream_tree_finalize(score, parent, token, C.c_int32(B), C.c_int32(N), C.c_int32(budget), tp, tt, ti, C.byref(n), None), n.value
    assert finalize(score=None)[0] == -1 and finalize(ti=None)[0] == -1
    assert finalize(N=0)[0] == -1 and finalize(N=1025)[0] == -1 and finalize(budget=-1)[0] == -1 and finalize(B=0)[0] == -1


def test_attention_entropy_argument_errors(lib):
    import ctypes as C
    fake = C.c_void_p(0x1000)
    desc = dream.attn_desc(1, 32, 32, 128, dream.BF16, 764)

    def call(d=desc, q=fake, n_q=704, k=fake, n_keys=704, ae=fake, ws=fake, nb=1 << 30):
        return lib.dream_attention_entropy(C.byref(d), q, None, C.c_int32(n_q), k, C.c_int32(n_keys), None, ae, ws, C.c_size_t(nb), None)
    assert call(q=None) == -1 and call(k=None) == -1 and call(ae=None) == -1
    assert call(n_q=0) == -1 and call(n_keys=0) == -1 and call(n_keys=765) == -1
    assert call(n_q=705) == -1                       # rows at positions 0..704 but 704 keys
    assert call(d=dream.attn_desc(1, 32, 32, 96, dream.BF16, 764)) == -2
    assert call(d=dream.attn_desc(1, 32, 5, 128, dream.BF16, 764)) == -1
    need = dream.dream_attention_entropy_workspace(desc, 704)
    assert need > 256 and call(nb=need - 1) == -3 and call(ws=None) == -3


def test_spec_accept_argument_errors(lib):
    import ctypes as C
    fake = C.c_void_p(0x1000)

    def call(tl=fake, dl=fake, dt=dream.BF16, B=1, T=60, V=32000, tok=fake, par=fake, ua=fake, ub=fake, depth=6, temp=1.0, al=fake,
             ap=fake, bt=fake, ws=fake, nb=1 << 30):
        return lib.dream_spec_accept(tl, dl, C.c_int32(dt), C.c_int32(B), C.c_int32(T), C.c_int32(V), tok, par, ua, ub, C.c_int32(depth),
                                     C.c_float(temp), al, ap, bt, ws, C.c_size_t(nb), None)
    assert call(tl=None) == -1 and call(dl=None) == -1 and call(ua=None) == -1 and call(ub=None) == -1 and call(bt=None) == -1
    assert call(dt=9) == -1 and call(B=0) == -1 and call(V=0) == -1 and call(depth=-1) == -1 and call(depth=1024) == -1
    assert call(T=0) == -2 and call(T=1025) == -2
    assert call(temp=0.0) == -1 and call(temp=-1.0) == -1
    assert "greedy" in dream.dream_last_error()
    need = dream.dream_spec_accept_workspace(1, 60, 32000)
    assert need == 256 + 3 * 32000 * 4 + 3 * 2048 + 1024 and call(nb=need - 1) == -3 and call(ws=None) == -3
    assert call(B=1100, T=60) == -2                  # more than 65535 rows


def test_project_rows_argument_errors(lib):
    import ctypes as C
    fake = C.c_void_p(0x1000)
    desc = dream.attn_desc(1, 32, 32, 128, dream.BF16, 764)

    def call(d=desc, x=fake, R=10, hid=4096, w=fake, H=32, rb=None, ri=None, out=fake):
        return lib.dream_project_rows(C.byref(d), x, C.c_int32(R), C.c_int32(hid), w, C.c_int32(H), rb, ri, out, None)
    assert call(x=None) == -1 and call(w=None) == -1 and call(out=None) == -1
    assert call(R=0) == -1 and call(H=0) == -1 and call(R=(1 << 20) + 1) == -1
    assert call(hid=0) == -2 and call(hid=4000) == -2
    assert call(d=dream.attn_desc(1, 32, 32, 72, dream.BF16, 764)) == -2
    assert call(d=dream.attn_desc(1, 32, 32, 128, dream.F32, 764)) == -2
    assert call(ri=fake) == -1                        # a row index needs a row base
    assert call(x=C.c_void_p(0x1008)) == -1 and "aligned" in dream.dream_last_error()

    from paper_2505_19201_amd.binding import ProjJob

    def multi(n=1, job=None):
        arr = (ProjJob * 5)(*[job or ProjJob(0x1000, 0x2000, 8, None, None, 0x3000)] * 5)
        return lib.dream_project_rows_multi(C.byref(desc), arr, C.c_int32(n), C.c_int32(10), C.c_int32(4096), None)
    assert multi(0) == -1 and multi(5) == -1
    assert multi(2, ProjJob(0x1000, None, 8, None, None, 0x3000)) == -1
    assert multi(1, ProjJob(0x1000, 0x2000, 0, None, None, 0x3000)) == -1
    assert lib.dream_project_rows_multi(C.byref(desc), None, C.c_int32(1), C.c_int32(10), C.c_int32(4096), None) == -1


def test_header_compiles_as_c_and_host_calls_work(lib, tmp_path):
    """include/dream.h is a C header: a C99 program built against it with gcc calls the host-only entry points."""
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no gcc")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    libdir = os.path.dirname(dream.library_path())
    exe = str(tmp_path / "abi_check")
    subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-Werror", "-I", os.path.join(root, "include"),
                    os.path.join(root, "tests", "c", "abi_check.c"), "-o", exe, "-L", libdir, "-ldream", "-Wl,-rpath," + libdir],
                   check=True, capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    assert out.startswith("attn_wave_kernel<128,8,2,1>")


def test_every_plan_names_a_built_variant(lib):
    """Host-only sweep of shapes (batch, heads, grouping, head_dim, rows, key range): whatever the launch plan chooses,
    the variant exists (dream_attn_plan_describe fails with 'not built' otherwise) and its name is in the variant list."""
    built = set(dream.dream_attn_variants())
    seen = set()
    for D in (64, 128, 256):
        for hkv, g in ((1, 1), (2, 4), (8, 1), (8, 2), (8, 4), (32, 1), (4, 8)):
            for B in (1, 2, 3, 4, 7, 8, 16, 32, 64, 100):
                for n_q in (1, 10, 16, 17, 33, 60, 64, 65, 130, 256):
                    for kv in (n_q, 40, 150, 700, 1340, 2600, 9000):
                        if kv < n_q:
                            continue
                        desc = dream.attn_desc(B, hkv * g, hkv, D, dream.BF16, kv + 3)
                        plan = dream.dream_attn_plan_describe(desc, n_q, kv)
                        name = plan.split(" ")[0]
                        assert name in built, (D, hkv, g, B, n_q, kv, plan)
                        assert dream.dream_tree_verify_attn_workspace(desc, n_q, kv) >= 256
                        seen.add(name)
    assert len(seen) >= 25, sorted(built - seen)   # the sweep reaches most of the table without any override


def test_few_stream_kernels_launch_at_most_one_workgroup_per_cu(lib):
    """The kernels without a key split are chosen for shapes whose workgroups all run at once; a second one on a CU would double the time."""
    seen = set()
    for D in (64, 128, 256):
        for hkv, g in ((8, 1), (8, 2), (8, 3), (8, 4), (16, 2), (32, 1), (5, 4)):
            for B in list(range(1, 25)) + [32, 40]:
                for n_q in (1, 8, 10, 12, 16, 17, 24, 33, 48, 49, 64):
                    plan = dream.dream_attn_plan_describe(dream.attn_desc(B, hkv * g, hkv, D, dream.BF16, 400), n_q, 400)
                    if re.match("attn_(wave|pair|quad)_kernel", plan):
                        assert int(re.search(r"workgroups=(\d+)", plan).group(1)) <= 256, (D, hkv, g, B, n_q, plan)
                        seen.add(plan.split(" ")[0])
    assert len(seen) >= 15


def test_few_stream_kernels_fit_the_cus_of_every_xcd(lib):
    """A KV head's workgroups share an XCD, so it is the XCD with most KV heads whose 32 CUs have to hold them, whatever the number of heads."""
    seen = set()
    for D in (64, 128, 256):
        for hkv, g in ((1, 4), (2, 3), (3, 1), (4, 4), (5, 3), (5, 4), (7, 2), (12, 1), (20, 1)):
            for B in list(range(1, 25)) + [32, 40, 48]:
                for n_q in (1, 8, 16, 17, 33, 60):
                    plan = dream.dream_attn_plan_describe(dream.attn_desc(B, hkv * g, hkv, D, dream.BF16, 400), n_q, 400)
                    if re.match("attn_(wave|pair|quad)_kernel", plan):
                        per_head = int(re.search(r"workgroups=(\d+)", plan).group(1)) // (B * hkv)
                        assert -(-B * hkv // 8) * per_head <= 32, (D, hkv, g, B, n_q, plan)
                        seen.add(plan.split(" ")[0])
    assert len(seen) >= 15


def _signature(name):
    """Parameters of an entry point as include/dream.h declares them: [(type, name)]."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    text = re.sub(r"/\*.*?\*/", "", open(os.path.join(root, "include", "dream.h")).read(), flags=re.S)
    params = re.search(r"\bint %s\((.*?)\);" % name, text, flags=re.S).group(1)
    return [tuple(re.match(r"(.*?)(\w+)$", " ".join(p.split())).groups()) for p in params.split(",")]


ENTRY_POINTS = ("dream_tree_verify_attn", "dream_draft_xattn", "dream_visual_compress", "dream_accept_path", "dream_accept_path_static",
                "dream_kv_commit", "dream_project_rows", "dream_project_rows_multi", "dream_spec_accept", "dream_attention_entropy",
                "dream_tree_expand_level", "dream_tree_finalize")


def _plain_arguments(name):
    """One argument per parameter that converts, every device pointer NULL: the library refuses the call without a launch."""
    args = []
    for kind, param in _signature(name):
        if "dream_attn_desc" in kind:
            args.append(dream.attn_desc(1, 4, 4, 64, dream.BF16, 128))
        elif "*const *" in kind or "dream_proj_job" in kind:
            args.append([])
        elif param == "stream":
            args.append(0)
        else:
            args.append(None if "*" in kind else 1)
    return args


@pytest.mark.parametrize("name", ENTRY_POINTS)
def test_device_pointers_take_device_tensors_only(lib, name):
    """Host memory in any form, and plain addresses, are refused in every device slot; a tensor on the host as before."""
    import torch
    from paper_2505_19201_amd.binding import _native
    call = getattr(_native(), name)
    assert call(*_plain_arguments(name)) < 0
    device = [i for i, (kind, param) in enumerate(_signature(name))
              if "*" in kind and not param.endswith("_host") and param not in ("desc", "jobs", "stream")]
    assert device or name == "dream_project_rows_multi"
    for i in device:
        for bad, error in ((np.zeros(64), TypeError), (b"0" * 64, TypeError), (bytearray(64), TypeError), (0x1000, TypeError),
                           (C.c_int32(0), TypeError), (torch.zeros(64), ValueError)):
            args = _plain_arguments(name)
            args[i] = bad
            with pytest.raises(error):
                call(*args)
    for i, (kind, param) in enumerate(_signature(name)):
        args = _plain_arguments(name)
        if param == "desc":
            for bad in (None, b"0" * C.sizeof(dream.AttnDesc), bytearray(8), C.c_int32(0), 0x1000):
                args[i] = bad
                with pytest.raises((TypeError, BufferError)):
                    call(*args)
        elif kind.strip() == "int32_t *" and param.endswith("_host"):
            for bad in (b"0000", bytearray(8), 0x1000):
                args[i] = bad
                with pytest.raises((TypeError, BufferError)):
                    call(*args)
            args[i] = C.c_int32(7)
            assert call(*args) < 0
        elif param == "jobs":
            for field in (0, 1, 3, 4, 5):
                job = [None, None, 1, None, None, None]
                job[field] = np.zeros(64)
                args[i] = [tuple(job)]
                with pytest.raises(TypeError):
                    call(*args)
        elif param == "caches_host":
            args[i] = [np.zeros(64)]
            with pytest.raises(TypeError):
                call(*args)


def test_torch_errors_become_python_errors(lib):
    """A tensor that cannot name its bytes (a sparse one) raises; in a process of its own, since an exception that leaves the
    extension's C functions would end Python."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = ("import torch\n"
            "from tests.test_abi import ENTRY_POINTS, _plain_arguments, _signature\n"
            "from paper_2505_19201_amd.binding import _native\n"
            "sparse = torch.zeros(4, 4).to_sparse()\n"
            "tried = 0\n"
            "for name in ENTRY_POINTS:\n"
            "    for i, (kind, param) in enumerate(_signature(name)):\n"
            "        if kind.strip() == 'size_t':\n"
            "            args = _plain_arguments(name)\n"
            "            args[i] = sparse\n"
            "            try:\n"
            "                getattr(_native(), name)(*args)\n"
            "            except RuntimeError:\n"
            "                tried += 1\n"
            "print('refused', tried)\n")
    p = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    assert p.stdout.strip() == "refused 7"


def test_a_projection_job_is_any_sequence_of_six(lib):
    """Jobs given as lists, tuples or iterators reach the library (which refuses the NULL tensors in them); five fields do not."""
    desc = dream.attn_desc(1, 4, 4, 64, dream.BF16, 128)
    job = (None, None, 4, None, None, None)
    for form in (tuple, list, iter):
        with pytest.raises(dream.DreamError, match="NULL tensor in job 0"):
            dream.dream_project_rows_multi(desc, [form(job)], 1, 256, stream=_NoStream())
    with pytest.raises(ValueError):
        dream.dream_project_rows_multi(desc, [job[:5]], 1, 256, stream=_NoStream())


class _NoStream:
    cuda_stream = 0


def test_dream_init_raises_every_limit_and_launches_stay_within_it(lib, tmp_path):
    """tests/c/launch_check.c stands in for HIP's launch functions: after dream_init no entry point sets a kernel attribute, and every
    launch of a sweep over all entry points fits its kernel's LDS limit and the grid limits."""
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no gcc")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    libdir = os.path.dirname(dream.library_path())
    exe = str(tmp_path / "launch_check")
    subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-Werror", "-rdynamic", "-I", os.path.join(root, "include"),
                    os.path.join(root, "tests", "c", "launch_check.c"), "-o", exe, "-L", libdir, "-ldream", "-Wl,-rpath," + libdir],
                   check=True, capture_output=True, text=True)
    p = subprocess.run([exe], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout[-3000:] + p.stderr[-1000:]


@pytest.mark.parametrize("B,hq,hkv,D,n_tree,line,short,long", [
    # three splits or two against one workgroup with two key groups, at the key tile where the measurements cross
    (9, 8, 1, 128, 60, 32, "attn_bf16_kernel<128,1,1,2,8,1,0,2> workgroups=72 splits=1", "attn_bf16_kernel<128,1,1,2> workgroups=216 splits=3"),
    (3, 28, 4, 64, 60, 32, "attn_bf16_kernel<64,1,2,2,8,1,0,2> workgroups=84 splits=1", "attn_bf16_kernel<64,1,2,2> workgroups=252 splits=3"),
    (11, 16, 2, 128, 30, 52, "attn_bf16_kernel<128,1,1,2,8,1,0,2> workgroups=88 splits=1", "attn_bf16_kernel<128,1,1,2> workgroups=176 splits=2"),
    (3, 32, 32, 128, 60, 52, "attn_bf16_kernel<128,1,1,2,8,1,1,2> workgroups=96 splits=1", "attn_bf16_kernel<128,1,1,2,4,1,1> workgroups=192 splits=2"),
    (2, 64, 8, 128, 60, 64, "attn_bf16_kernel<128,1,1,2,8,1,0,2> workgroups=128 splits=1", "attn_bf16_kernel<128,1,1,2> workgroups=256 splits=2"),
    # head_dim 256, up to 4 query tiles: the 8-wave form against three splits and two
    (9, 8, 8, 256, 60, 24, "attn_bf16_kernel<256,1,1,2,8> workgroups=72 splits=1", "attn_bf16_kernel<256,1,1,2,4,1,1> workgroups=216 splits=3"),
    (12, 8, 8, 256, 60, 32, "attn_bf16_kernel<256,1,1,2,8> workgroups=96 splits=1", "attn_bf16_kernel<256,1,1,2,4,1,1> workgroups=192 splits=2"),
])
def test_launch_plans_on_both_sides_of_a_length_line(lib, B, hq, hkv, D, n_tree, line, short, long):
    """The lengths at which a plan changes (attn.hip names the times on both sides), one key tile of 32 before and after."""
    desc = dream.attn_desc(B, hq, hkv, D, dream.BF16, 4200)
    assert dream.dream_attn_plan_describe(desc, n_tree, line * 32).startswith(short)
    assert dream.dream_attn_plan_describe(desc, n_tree, line * 32 + 1).startswith(long)


@pytest.mark.parametrize("B,hq,hkv,D,n_q,line,upto,beyond", [
    # one launch without key splits against eight splits: fewer workgroups, an earlier line
    (1, 32, 32, 128, 8, 41, "attn_wave_kernel<128,8,4,1>", "attn_bf16_kernel<128,1,1,2,4,1,1> workgroups=256 splits=8"),
    (1, 32, 32, 64, 8, 63, "attn_wave_kernel<64,8,2,1>", "attn_bf16_kernel<64,1,2,2,4,1,1> workgroups=256 splits=8"),
    (1, 32, 32, 64, 64, 90, "attn_wave_kernel<64,8,2,1>", "attn_bf16_kernel<64,1,2,2,4,1,1> workgroups=256 splits=8"),
    (1, 32, 8, 128, 64, 84, "attn_wave_kernel<128,8,2,1>", "attn_bf16_kernel<128,1,1,2> workgroups=256 splits=8"),
    (2, 16, 8, 256, 8, 40, "attn_wave_kernel<256,4,4,1>", "attn_bf16_kernel<256,1,1,2,4,1,1> workgroups=128 splits=8"),
    (2, 24, 8, 128, 33, 49, "attn_wave_kernel<128,8,1,1>", "attn_bf16_kernel<128,1,1,2> workgroups=240 splits=5"),
    # against four, three and two
    (2, 32, 32, 128, 8, 62, "attn_wave_kernel<128,8,4,1>", "attn_bf16_kernel<128,1,1,2,4,1,1> workgroups=256 splits=4"),
    (3, 24, 8, 128, 33, 88, "attn_wave_kernel<128,8,1,1>", "attn_bf16_kernel<128,1,1,2> workgroups=216 splits=3"),
    (3, 32, 32, 64, 8, 120, "attn_wave_kernel<64,8,2,1>", "attn_bf16_kernel<64,1,2,2,4,1,1> workgroups=192 splits=2"),
    # four slots for all rows of a KV head, from a length on
    (24, 32, 8, 128, 17, 23, "attn_bf16_kernel<128,1,1,2,8>", "attn_quad_kernel<128,1,2>"),
])
def test_single_launches_on_both_sides_of_their_line(lib, B, hq, hkv, D, n_q, line, upto, beyond):
    """The lengths at which the kernels without key splits begin and end, in key tiles; each depends on the splits replaced and on the workgroups."""
    desc = dream.attn_desc(B, hq, hkv, D, dream.BF16, 4200)
    plans = [dream.dream_attn_plan_describe(desc, n_q, n) for n in (line * 32, line * 32 + 1)]
    assert plans[0].startswith(upto) and plans[1].startswith(beyond), plans


@pytest.mark.parametrize("B,hq,hkv,D,n_q,keys", [(1, 8, 8, 128, 60, 2047), (1, 8, 4, 256, 60, 2047), (1, 8, 8, 64, 60, 3584), (1, 32, 8, 128, 8, 2047), (1, 24, 8, 64, 33, 4095)])
def test_single_launches_over_small_caches(lib, B, hq, hkv, D, n_q, keys):
    """Up to 8 MB of keys and values a layer, which the memory-side cache holds for all layers, one launch without key splits is taken for longer."""
    desc = dream.attn_desc(B, hq, hkv, D, dream.BF16, 4200)
    plans = [dream.dream_attn_plan_describe(desc, n_q, n) for n in (keys, keys + 1)]
    assert plans[0].startswith("attn_wave_kernel") and plans[1].startswith("attn_bf16_kernel"), plans
    for n in (keys // 2, keys):
        assert dream.dream_tree_verify_attn_workspace(desc, n_q, n) <= dream.dream_tree_verify_attn_workspace(desc, n_q, keys + 1)


def test_a_workspace_for_the_longest_range_fits_every_shorter_call(lib):
    """Programs query once, for the longest key range; the plans of shorter ranges (other splits, other kernels) never need more."""
    for D in (64, 128, 256):
        for hq, hkv in ((8, 8), (32, 8), (28, 4), (16, 8), (8, 1), (16, 2)):
            for B in (1, 2, 3, 4, 6, 9, 11, 12, 16, 24):
                desc = dream.attn_desc(B, hq, hkv, D, dream.BF16, 4200)
                for n_q in (1, 10, 33, 60):
                    need = [dream.dream_tree_verify_attn_workspace(desc, n_q, tiles * 32) for tiles in range(2, 131, 3)]
                    assert need == sorted(need), (D, hq, hkv, B, n_q)
