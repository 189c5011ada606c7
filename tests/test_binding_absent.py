"""The package without its marshalling module (not built, or built for another Python or
torch): one warning, and every call goes through ctypes.  The build without a host
compiler or torch's headers still makes the library."""
import os

import pytest
import torch

import paper_2609_29364_amd as nsd
from paper_2609_29364_amd import build


@pytest.fixture(params=["missing", "unloadable"])
def no_binding(request, tmp_path, monkeypatch):
    if not os.path.exists(nsd.LIB_PATH):
        build.build()
    path = tmp_path / "_nsd_torch.so"
    if request.param == "unloadable":
        path.write_bytes(b"not a shared object")
    monkeypatch.setattr(nsd, "BINDING_PATH", str(path))
    monkeypatch.setattr(nsd, "_native_module", None)


def test_calls_reach_the_ctypes_path(no_binding):
    k = torch.zeros((2, 2, 8, 16, 8), dtype=torch.bfloat16)
    v = torch.zeros((2, 2, 64, 16), dtype=torch.bfloat16)
    ids = torch.zeros(1, dtype=torch.int32)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        with pytest.raises(ValueError, match="must be on a GPU"):    # the Python path's check
            nsd.kv_gather(k, v, k, v, ids, ids)
    with pytest.raises(ValueError, match="must be on a GPU"):        # and no second warning
        nsd.commit_lengths(ids, ids, ids)


@pytest.mark.gpu
def test_results_without_the_module(no_binding, device):
    from test_gpu_native_binding import setup
    from paper_2609_29364_amd.round import verify_round
    from workload import make_accept
    from parity import i32
    cfg, meta, planes = setup(device)
    a = make_accept(cfg, meta, device)

    def call():
        k, v, ks, vs, q = (t.clone() for t in planes)
        ws = nsd.new_workspace(nsd.verify_attention_workspace_size(
            cfg.bs, 8, 2, 128, meta.max_q, meta.max_seq_len), device)
        out = torch.zeros_like(q)
        r = verify_round(k, v, ks, vs, i32(meta.src_ids, device), i32(meta.dst_ids, device), q,
                         i32(meta.block_table, device), i32(meta.seq_lens, device),
                         i32(meta.q_indptr, device), meta.max_q, meta.max_seq_len, out=out,
                         workspace=ws, accept=(a.p_target, a.q_draft, a.draft_tokens, a.uniforms,
                                               meta.max_q - 1))
        torch.cuda.synchronize()
        return [*r, k, v]

    with pytest.warns(RuntimeWarning, match="ctypes"):
        without = call()
    nsd._native_module, nsd.BINDING_PATH = None, build.BINDING_PATH   # (the fixture puts them back)
    for x, y in zip(call(), without, strict=True):
        assert torch.equal(x, y)
    assert not isinstance(nsd._native(), nsd._NoBinding)


def test_build_without_a_host_compiler(tmp_path, monkeypatch, capsys):
    path = tmp_path / "_nsd_torch.so"
    path.write_bytes(b"of older sources")
    monkeypatch.setattr(build, "BINDING_PATH", str(path))
    monkeypatch.setenv("CXX", str(tmp_path / "none"))
    build._build_binding()
    assert not path.exists() and "no torch_binding.cpp built" in capsys.readouterr().err


@pytest.mark.parametrize("how", ["path", "name", "link"])
def test_hip_headers_are_found(how, tmp_path, monkeypatch):
    """HIPCC as a path, as a name to look up in PATH, and behind a link."""
    (tmp_path / "rocm" / "bin").mkdir(parents=True)
    (tmp_path / "rocm" / "include" / "hip").mkdir(parents=True)
    (tmp_path / "rocm" / "include" / "hip" / "hip_runtime_api.h").write_text("")
    hipcc = tmp_path / "rocm" / "bin" / "hipcc"
    hipcc.write_text("")
    hipcc.chmod(0o755)
    (tmp_path / "link").mkdir()
    (tmp_path / "link" / "hipcc").symlink_to(hipcc)
    at = {"path": str(hipcc), "name": "hipcc", "link": str(tmp_path / "link" / "hipcc")}[how]
    monkeypatch.delenv("ROCM_PATH", raising=False)
    monkeypatch.setenv("PATH", str(hipcc.parent), prepend=os.pathsep)
    monkeypatch.setattr(build, "HIPCC", at)
    assert build._rocm_include() == str(tmp_path / "rocm" / "include")
