"""The C-ABI library loads and exports every symbol include/pit.h declares (no GPU needed)."""
import ctypes
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "pit.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(pit_[a-z_0-9]+)\s*\(", text)))


def test_header_symbols_are_exported():
    lib_path = os.path.join(ROOT, "paper_2301_10936_amd", "libpit_hip.so")
    if not os.path.exists(lib_path):
        from paper_2301_10936_amd import build
        build.build()
    lib = ctypes.CDLL(lib_path)
    names = _declared()
    assert {"pit_build_index", "pit_sread_gemm", "pit_moe_dispatch_gemm", "pit_sparse_attn"} <= set(names)
    missing = [n for n in names if not hasattr(lib, n)]
    assert not missing, missing
    assert lib.pit_version() >= 100


def test_binding_names_match_header():
    from paper_2301_10936_amd import pit
    assert sorted(pit.EXPORTS) == _declared()
    for n in pit.EXPORTS:
        if n not in ("pit_last_hip_error", "pit_version"):
            assert hasattr(pit, n), n


def test_host_side_argument_checks_need_no_gpu():
    """Validation that happens before any HIP call works on a machine without a GPU."""
    from paper_2301_10936_amd import pit
    lib, CIndex = pit.raw()
    assert lib.pit_build_index_workspace(64, 64, 1, 24, 0, 0) == 0          # 64 % 24 != 0
    assert lib.pit_build_index_workspace(8192, 2048, 1, 128, 0, 0) >= 16 * 128 * 8
    assert lib.pit_build_index(None, pit.PIT_F16, 64, 64, 64, 1, 32, 0, None, None, 0, None) == pit.PIT_EINVAL
    ci = CIndex(None, None, None, 2, 128)
    assert lib.pit_build_index(None, pit.PIT_F16, 64, 64, 64, 1, 32, 0, ctypes.byref(ci), None, 0, None) == pit.PIT_EINVAL
    assert lib.pit_sread_gemm(0, None, 0, None, 0, None, 0, 128, 100, 64, pit.PIT_BF16, pit.PIT_F32, None, 64, 1, None) == pit.PIT_EINVAL
    ci2 = CIndex(1, 1, None, 1, 128)   # non-null dummies; rejected before being dereferenced
    assert lib.pit_sread_gemm(0, None, 0, None, 0, None, 0, 128, 100, 64, pit.PIT_BF16, pit.PIT_F32, ctypes.byref(ci2), 64, 1, None) == pit.PIT_ESHAPE
    assert lib.pit_moe_workspace(4096, 768, 3072, 64) > 4096 * 3072 * 2
    assert lib.pit_moe_dispatch_gemm(None, None, None, None, None, None, pit.PIT_F32, 16, 100, 128, 2, pit.PIT_BF16, 0, None, None, 0, None) == pit.PIT_ESHAPE


def test_select_kernel_on_the_host_matches_the_oracle():
    """pit_select_kernel is host-only: check it here against the oracle's Algorithm 1 on counts the
    oracle's CoverAlgo produced (so the comparison covers the cost sum, the dense rule and the tie rule)."""
    import numpy as np
    from oracle import pit_oracle as orc
    from paper_2301_10936_amd import pit, workloads as wl
    cands = [{"mt_rows": 2, "mt_cols": 1, "tile_cost": 2.0},
             {"mt_rows": 8, "mt_cols": 1, "tile_cost": 3.5},
             {"mt_rows": 32, "mt_cols": 1, "tile_cost": 9.0},
             {"mt_rows": 32, "mt_cols": 1, "tile_cost": 8.0, "dense": True},
             {"mt_rows": 8, "mt_cols": 1, "tile_cost": 3.5}]          # equal to candidate 1: the first one wins
    for s in (0.999, 0.97, 0.8, 0.3):
        samples = [wl.iid_block_mask(256, 128, 2, 1, s, seed=k) for k in range(3)]
        num = [[orc.cover_count(D, c["mt_rows"], c["mt_cols"]) for c in cands] for D in samples]
        grid = [[(D.shape[0] // c["mt_rows"]) * (D.shape[1] // c["mt_cols"]) for c in cands] for D in samples]
        best, costs = pit.pit_select_kernel(cands, num, grid)
        want_best, want_costs = orc.select_kernel(samples, cands)
        assert best == want_best and best != 4
        assert np.allclose(costs, want_costs, rtol=1e-12)
    assert pit.pit_select_kernel(cands, [], []) == (0, [0.0] * 5)
    import pytest
    with pytest.raises(pit.PitError):
        pit.pit_select_kernel([{"mt_rows": 0, "mt_cols": 1, "tile_cost": 1.0}], [[1]], [[1]])
    with pytest.raises(pit.PitError):
        pit.pit_select_kernel(cands, [[-1] * 5], [[1] * 5])


def test_selection_with_the_profiled_tile_costs():
    """The committed offline profile (paper_2301_10936_amd/tile_cost.py, one MI355X) drives Algorithm 1 as
    the paper describes: with iid ReLU zeros nearly every 128 x 1 micro-tile is live and the dense kernel wins;
    with zeros correlated across tokens the sparse kernel wins."""
    import json
    import os
    import numpy as np
    from oracle import pit_oracle as orc
    from paper_2301_10936_amd import pit, workloads as wl
    here = os.path.dirname(os.path.abspath(pit.__file__))
    prof = json.load(open(os.path.join(here, "tile_cost_mi355x.json")))["candidates"]["gather_k"]
    cands = [{"mt_rows": 1, "mt_cols": 128, "tile_cost": prof["sparse_ns_per_tile"]},
             {"mt_rows": 1, "mt_cols": 128, "tile_cost": prof["dense_ns_per_tile"], "dense": True}]
    picks = {}
    for name, prob in (("iid", None), ("correlated", 0.25)):
        w = wl.relu_ffn(M=512, K=1024, N=128, seed=1, channel_live_prob=prob)     # Xt is [K, M]: micro-tile 1 x 128
        num = [[orc.cover_count(w.Xt, 1, 128)] * 2]
        grid = [[w.Xt.shape[0] * (w.Xt.shape[1] // 128)] * 2]
        picks[name] = pit.pit_select_kernel(cands, num, grid)[0]
        assert picks[name] == orc.select_kernel([orc.to_f64(w.Xt)], cands)[0]
    assert picks == {"iid": 1, "correlated": 0}


def test_build_leaves_out_an_option_the_compiler_does_not_know(tmp_path, monkeypatch):
    """An option that one source asks for is an optimisation: a compiler without it still builds the library."""
    import shutil
    import pytest
    from paper_2301_10936_amd import build
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    monkeypatch.setattr(build, "OPTIONAL", {"pit_api.hip": ["-mllvm", "-no-such-option-of-the-compiler"]})
    obj = tmp_path / "pit_api.o"
    build._compile(os.path.join(build.CSRC, "pit_api.hip"), str(obj), False)
    assert obj.stat().st_size > 0


def test_index_calls_refuse_a_tensor_that_is_not_a_matrix_in_the_same_way():
    """Checked before anything else is done with the tensor: no GPU needed."""
    import pytest
    import torch
    from paper_2301_10936_amd import pit
    for shape in ((8,), (2, 4, 8)):
        for call in (lambda t: pit.pit_build_index(t, 1, 1, 0), lambda t: pit.pit_build_index_static(t, 1, 1, 0, None),
                     lambda t: pit.pit_cover_count(t, 1, 1)):
            with pytest.raises(AssertionError):
                call(torch.zeros(shape))
    with pytest.raises(AssertionError):
        pit.pit_build_index(torch.zeros((4, 8)).t(), 1, 1, 0)
