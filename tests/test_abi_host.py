"""Host-only checks of the C-ABI library: it loads, exports every entry point the header declares,
sizes workspaces consistently, and rejects bad arguments before anything is launched."""
import ctypes as C
import os
import re

import pytest

import paper_2106_10715_amd as M

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "moe355.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(moe_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = _declared()
    assert {"moe_route", "moe_permute", "moe_expert_ffn", "moe_combine", "moe_layer_forward"} <= set(names)
    L = M.lib()
    for n in names:
        assert hasattr(L, n), f"{n} declared in moe355.h but not exported"


def test_binding_has_the_same_names():
    for n in ("moe_route", "moe_permute", "moe_expert_ffn", "moe_combine", "moe_layer_forward", "moe_pack_weights",
              "moe_workspace_bytes", "moe_expert_bytes", "moe_gate_bytes", "moe_pack_gate", "moe_layer_forward_timed"):
        assert callable(getattr(M, n))


def test_sizes():
    c = M.MoeCfg.make(4096, 4096, 10240, 32)
    assert M.moe_expert_bytes(c) == 240 * 2 ** 20          # one bf16 expert of the Table 1 shape
    ws = M.moe_workspace_bytes(c)
    A = 4096
    need = A * 10240 * 2 + 2 * A * 4096 * 2 + 4 * A * 4
    assert need <= ws < need + (1 << 20)
    c32 = M.MoeCfg.make(64, 256, 512, 4, dtype="f32")
    assert M.moe_expert_bytes(c32) == 3 * 256 * 512 * 4
    assert M.moe_workspace_bytes(M.MoeCfg.make(0, 64, 64, 1)) >= 256


@pytest.mark.parametrize("kw,frag", [
    (dict(T=-1, d=64, f=64, E=2), "T must be"),
    (dict(T=1, d=96, f=64, E=2), "d must be"),
    (dict(T=1, d=64, f=100, E=2), "f must be"),
    (dict(T=1, d=64, f=64, E=0), "E must be"),
    (dict(T=1, d=64, f=64, E=257), "E must be"),
    (dict(T=1, d=64, f=64, E=4, k=5), "k must be"),
    (dict(T=1, d=64, f=64, E=16, k=9), "k must be"),
    (dict(T=1, d=64, f=64, E=2, renorm=2), "renorm"),
    (dict(T=1, d=64, f=64, E=2, act=3), "act"),
    (dict(T=1, d=64, f=64, E=2, gate_packed=2), "gate_packed"),
    (dict(T=1 << 20, d=4096, f=10240, E=2), "2^31"),
])
def test_bad_cfg_is_rejected(kw, frag):
    cfg = M.MoeCfg.make(**kw)
    with pytest.raises(M.MoeError, match=re.escape(frag)):
        M.moe_workspace_bytes(cfg)
    L = M.lib()
    n = C.c_size_t(0)
    assert L.moe_expert_bytes(C.byref(cfg), C.byref(n)) == -1
    assert L.moe_route(C.byref(cfg), None, None, None, None, None, None, None) == -1
    assert L.moe_layer_forward(C.byref(cfg), None, None, None, None, None, None, None, None) == -1
    assert frag.encode() in L.moe_last_error()


def test_null_pointers_are_rejected_before_launch():
    L = M.lib()
    cfg = M.MoeCfg.make(8, 64, 64, 2)
    assert L.moe_route(None, None, None, None, None, None, None, None) == -1
    assert L.moe_route(C.byref(cfg), None, None, None, None, None, None, None) == -1
    assert b"W_g is NULL" in L.moe_last_error()
    assert L.moe_permute(C.byref(cfg), None, None, None, None, None, None, None, None, None) == -1
    assert L.moe_expert_ffn(C.byref(cfg), None, None, None, None, None, None) == -1
    assert L.moe_combine(C.byref(cfg), None, None, None, None, None) == -1
    assert L.moe_layer_forward(C.byref(cfg), None, None, None, None, None, None, None, None) == -1
    h = C.c_void_p(None)
    assert L.moe_stream_ctx_create(C.byref(cfg), None, 0, None, 2, C.byref(h)) == -1
    assert L.moe_stream_ctx_destroy(None) == 0
    # misaligned buffers
    buf = C.create_string_buffer(4096)
    base = C.addressof(buf)
    al = (base + 255) & ~255
    assert L.moe_combine(C.byref(cfg), C.c_void_p(al + 2), C.c_void_p(al), C.c_void_p(al), C.c_void_p(al), None) == -1
    assert b"aligned" in L.moe_last_error()
    # wrong expert size / slot count for the streamed mode
    assert L.moe_stream_ctx_create(C.byref(cfg), C.c_void_p(al), 123, C.c_void_p(al), 2, C.byref(h)) == -1
    assert b"expert_bytes" in L.moe_last_error()
    assert L.moe_stream_ctx_create(C.byref(cfg), C.c_void_p(al), 3 * 64 * 64 * 2, C.c_void_p(al), 0, C.byref(h)) == -1
    assert b"K must be" in L.moe_last_error()


def test_build_refuses_spill_code_inside_a_load_pipeline():
    """The build's assembly check: scratch accesses are tolerated outside the bracketed regions and outside
    nested loops of the named kernels, and refused inside them."""
    from paper_2106_10715_amd.build import check_no_spill
    ok = "\n".join([
        "_ZN3moe8ffn_mfma_kernelEv: ; @x",
        "\tscratch_store_dword off, v1, off",
        "\t; pipeline begin",
        "\tglobal_load_dwordx4 v[0:3], v4, s[0:1]",
        "\t; pipeline end",
        "\tscratch_load_dword v1, off, off",
        ".LBB0_1:                                ; =>This Inner Loop Header: Depth=1",
        "\tscratch_load_dword v1, off, off",
        ".LBB0_2:                                ;   Parent Loop BB0_1 Depth=1",
        "                                        ; =>  This Inner Loop Header: Depth=2",
        "\ts_nop 0",
        "; %bb.3:                                ;   in Loop: Header=BB0_1 Depth=1",
        "\tscratch_load_dword v1, off, off",
        "\t.end_amdhsa_kernel",
        "_ZN3moe5otherEv: ; @y",
        ".LBB1_1:                                ;   Parent Loop BB1_0 Depth=1",
        "                                        ; =>  This Inner Loop Header: Depth=2",
        "\tscratch_load_dword v1, off, off",
    ])
    check_no_spill(ok, "ffn_mfma")
    bracketed = ok.replace("\tglobal_load_dwordx4 v[0:3], v4, s[0:1]", "\tscratch_store_dword off, v9, off")
    with pytest.raises(RuntimeError, match="spill code"):
        check_no_spill(bracketed, "ffn_mfma")
    nested = "\n".join([
        "_ZN3moe8ffn_mfma_kernelEv: ; @x",
        ".LBB0_5:                                ;   Parent Loop BB0_1 Depth=1",
        "                                        ; =>  This Inner Loop Header: Depth=2",
        "\tscratch_load_dword v1, off, off",
    ])
    with pytest.raises(RuntimeError, match="spill code"):
        check_no_spill(nested, "ffn_mfma")


def test_build_refuses_a_loop_that_touches_a_register_with_a_load_in_flight():
    """The build's second assembly check walks the pipelined loops twice with the loads in issue order."""
    from paper_2106_10715_amd.build import check_loads_in_flight

    def kernel(body):
        return "\n".join(["_ZN3moe8ffn_mfma_kernelEv: ; @x", "\t; pipeline begin",
                          ".LBB0_2:                                ;   Parent Loop BB0_1 Depth=1",
                          "                                        ; =>  This Inner Loop Header: Depth=2"]
                         + ["\t" + l for l in body] + ["\ts_cbranch_scc1 .LBB0_2", "\t; pipeline end", "\t.end_amdhsa_kernel"])

    good = ["global_load_dwordx4 v[8:11], v40, s[2:3] offset:0 nt",       # prefetch for the next round
            "s_waitcnt vmcnt(1)",                                          # the previous round's load has landed
            "v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], v[12:15], v[16:31]",
            "global_load_dwordx4 v[12:15], v40, s[2:3] offset:1024 nt",    # refilled right after its last use
            "s_waitcnt vmcnt(1)",
            "v_mfma_f32_32x32x16_bf16 v[16:31], v[4:7], v[8:11], v[16:31]"]
    assert check_loads_in_flight(kernel(good), "ffn_mfma") == 1
    # the consumer moved above its wait
    early = [good[0], good[2], good[1]] + good[3:]
    with pytest.raises(RuntimeError, match="has not been waited for"):
        check_loads_in_flight(kernel(early), "ffn_mfma")
    # a copy of a register that was loaded in the previous round and is still in flight at the loop end
    copied = good + ["v_mov_b64_e32 v[50:51], v[12:13]"]
    with pytest.raises(RuntimeError, match="has not been waited for"):
        check_loads_in_flight(kernel(copied), "ffn_mfma")
    # other kernels are not looked at; a loop of several blocks cannot be verified and is refused
    assert check_loads_in_flight(kernel(copied).replace("ffn_mfma", "other"), "ffn_mfma") == 0
    with pytest.raises(RuntimeError, match="not a single block"):
        check_loads_in_flight(kernel(good[:2] + [".LBB0_3:"] + good[2:]).replace("\t.LBB0_3:", ".LBB0_3:"), "ffn_mfma")


def test_build_refuses_a_touch_of_a_register_in_flight_before_the_loop():
    """The third assembly check covers the code between the start of a pipeline region and its loop: loads
    issued as inline assembly are in flight until a wait retires them; loads the compiler generated are
    not counted (a wave that does not execute them would otherwise look further along than it is)."""
    from paper_2106_10715_amd.build import check_prologue_in_flight

    def kernel(body):
        return "\n".join(["_ZN3moe8ffn_mfma_kernelEv: ; @x", "\t;;#ASMSTART", "\t; pipeline begin", "\t;;#ASMEND"]
                         + ["\t" + l for l in body] +
                         [".LBB0_2:                                ;   Parent Loop BB0_1 Depth=1",
                          "                                        ; =>  This Inner Loop Header: Depth=2",
                          "\ts_cbranch_scc1 .LBB0_2", "\t; pipeline end", "\t.end_amdhsa_kernel"])

    asm_load = lambda dst, off: [";;#ASMSTART", f"global_load_dwordx4 {dst}, v40, s[2:3] offset:{off}", ";;#ASMEND"]
    good = (asm_load("v[4:7]", 0) + asm_load("v[8:11]", 1024) + ["s_waitcnt vmcnt(1)", "ds_write_b128 v50, v[4:7]"])
    assert check_prologue_in_flight(kernel(good), "ffn_mfma") == 1
    with pytest.raises(RuntimeError, match="has not been waited for"):
        check_prologue_in_flight(kernel(good + ["v_mov_b32_e32 v60, v9"]), "ffn_mfma")
    # a load of the compiler's own between the two does not make the wait look stricter than it is:
    # counted, vmcnt(2) would seem to retire v[4:7]; for a wave that skips the branch it does not
    own = (asm_load("v[4:7]", 0) + asm_load("v[8:11]", 1024) + [".LBB0_1:", "global_load_dword v70, v71, s[4:5]",
           "s_waitcnt vmcnt(2)", "ds_write_b128 v50, v[4:7]"])
    with pytest.raises(RuntimeError, match="has not been waited for"):
        check_prologue_in_flight(kernel(own).replace("\t.LBB0_1:", ".LBB0_1:"), "ffn_mfma")
    assert check_prologue_in_flight(kernel(good).replace("ffn_mfma", "other"), "ffn_mfma") == 0


def test_gelu_tail_polynomial_of_the_ffn_kernel_is_accurate():
    """The bf16 FFN epilogue evaluates exact GELU as max(z, 0) - a 2^P(a), a = min(|z|, 8), with the seven
    coefficients of P written in ffn.hip.  Evaluated here in float32 steps like the kernel's fused
    multiply-adds, the result must agree with z Phi(z) from the error function to 1.5e-7 absolute over
    the whole range, and 2^P(a) with the normal tail 0.5 erfc(a / sqrt 2) to 1e-3 relative up to a = 4 (the fit levels the
    absolute error of GELU, so the relative error of the tail grows as the tail vanishes)."""
    import numpy as np
    from scipy.special import erfc
    src = open(os.path.join(os.path.dirname(M.__file__), "csrc", "ffn.hip")).read()
    body = re.search(r"kGeluTail\[7\]\s*=\s*\{([^}]*)\}", src).group(1)
    coef = [np.float32(float(t.strip().rstrip("f"))) for t in body.split(",")]
    assert len(coef) == 7
    z = np.linspace(-12.0, 12.0, 1_200_001).astype(np.float32)
    a = np.minimum(np.abs(z), np.float32(8.0))
    p = np.full_like(a, coef[6])
    for c in coef[5::-1]:
        p = (p.astype(np.float64) * a.astype(np.float64) + np.float64(c)).astype(np.float32)   # one rounding, as an fma
    q = np.exp2(p.astype(np.float64))
    gelu = np.maximum(z, 0).astype(np.float64) - a.astype(np.float64) * q
    z64 = z.astype(np.float64)
    exact = z64 * 0.5 * erfc(-z64 / np.sqrt(2.0))
    assert np.abs(gelu - exact).max() <= 1.5e-7
    near = a <= 4.0
    tail = 0.5 * erfc(a[near].astype(np.float64) / np.sqrt(2.0))
    assert np.abs(q[near] / tail - 1.0).max() <= 1e-3


def test_bench_refuses_more_than_one_gpu():
    """The layer is built and measured on one GPU; asked for more, the bench says so and exits without touching a device."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0 and "one GPU" in r.stderr and r.stdout.strip() == ""


def test_gate_and_timer_arguments_are_checked_on_the_host():
    cfg = M.MoeCfg.make(8, 64, 64, 4)
    assert M.moe_gate_bytes(cfg) >= 64 * 32 * 2                  # columns padded to 32, plus the per-group sums of squares
    assert M.moe_gate_bytes(M.MoeCfg.make(8, 64, 64, 4, dtype="f32")) >= 64 * 4 * 4
    L = M.lib()
    assert L.moe_pack_gate(C.byref(cfg), None, None, None) == -1 and b"W_g" in L.moe_last_error()
    h = C.c_void_p(None)
    assert L.moe_timer_create(0, 0, C.byref(h)) == -1 and b"max_calls" in L.moe_last_error()
    assert L.moe_timer_create(4, 9, C.byref(h)) == -1 and b"mode" in L.moe_last_error()
    assert L.moe_timer_destroy(None) == 0
    assert L.moe_layer_forward_timed(C.byref(cfg), None, None, None, None, None, None, None, None) == -1
    assert L.moe_stream_ctx_share_loader(None, None) == -1
    # the batching entry point without a workspace refuses what its fixed array cannot hold, before touching anything
    big = M.MoeCfg.make(262145, 64, 64, 4)
    assert L.moe_permute_static(C.byref(big), None, C.c_void_p(8), C.c_void_p(8), C.c_void_p(8), C.c_void_p(8), C.c_void_p(8), None, None) == -3
    assert b"262144" in L.moe_last_error()


def test_build_refuses_m0_outside_of_the_loads_into_lds():
    from paper_2106_10715_amd import build as B
    load = "\t;;#ASMSTART\n\ts_add_u32 m0, s92, 0x1000\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v1, s[60:61]\n\t;;#ASMEND\n"
    kernel = "_Zk_ffn_mfma: ; @k\n" + load + "{}" + load + ".Lfunc_end0:\n"
    assert B.check_m0_free(kernel.format("\ts_mov_b32 s0, s1 ; m0 is free\n"), "ffn_mfma") == 2
    for use in ("\ts_mov_b32 m0, s1\n", "\tv_readlane_b32 s3, v0, m0\n"):
        with pytest.raises(RuntimeError, match="m0"):
            B.check_m0_free(kernel.format(use), "ffn_mfma")
    assert B.check_m0_free("_Zother:\n\ts_mov_b32 m0, s1\n.Lfunc_end0:\n", "ffn_mfma") == 0


def test_build_refuses_sums_of_matrix_instructions_in_assembly_touched_early():
    from paper_2106_10715_amd import build as B
    mfma = "\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[12:15], v[4:7]\n\t;;#ASMEND\n"
    def kernel(*body):
        return "_Zk_ffn_mfma: ; @k\n.LBB0_1:\n" + "".join(body) + "\ts_endpgm\n.Lfunc_end0:\n"
    use, wait = "\tv_mov_b32_e32 v1, v6\n", "\ts_nop 15\n\ts_nop 15\n"
    assert B.check_sums_settle(kernel(mfma, mfma, wait, use), "ffn_mfma") == 2          # the same sum again, and the use in time
    jumps = (mfma, "\ts_cbranch_scc1 .LBB0_2\n", wait, "\ts_endpgm\n.LBB0_2:\n\ts_branch .LBB0_3\n.LBB0_4:\n", wait, "\ts_endpgm\n.LBB0_3:\n")      # two jumps to the use
    for bad in (kernel(mfma, use), kernel(mfma, "\ts_nop 15\n", use), kernel(use, mfma, "\ts_cbranch_scc1 .LBB0_1\n"),
                kernel(mfma, mfma.replace("v[4:7], v[8:11]", "v[20:23], v[4:7]").replace(", v[4:7]\n", ", v[20:23]\n")),
                kernel(mfma, mfma.replace("v[4:7]", "v[6:9]")), kernel(*jumps, use), kernel("\tv_mov_b32_e32 v9, v1\n", mfma, wait), kernel("\tv_mov_b32_e32 v5, 0\n\ts_nop 0\n", mfma)):
        with pytest.raises(RuntimeError, match="wait states"):
            B.check_sums_settle(bad, "ffn_mfma")
    assert B.check_sums_settle(kernel(*jumps, wait, use), "ffn_mfma") == 1
    assert B.check_sums_settle(kernel("\tv_mov_b32_e32 v9, v1\n\ts_nop 1\n", mfma, wait), "ffn_mfma") == 1
    for lost in ("\ts_cbranch_scc1 .LBB0_9\n", "\ts_setpc_b64 s[2:3]\n"):
        with pytest.raises(RuntimeError, match="unknown place"):
            B.check_sums_settle(kernel(mfma, lost, wait), "ffn_mfma")
    assert B.check_sums_settle(kernel(mfma, use).replace("ffn_mfma", "other"), "ffn_mfma") == 0


def test_build_wants_matrix_instructions_in_assembly_where_tiles_are_tall(monkeypatch, tmp_path):
    """An assembly that the check finds none in (printed in another way, say) is no proof that they are used in time."""
    from paper_2106_10715_amd import build as B
    monkeypatch.setattr(B, "_built", lambda *a: str(tmp_path / "x.s"))
    (tmp_path / "x.s").write_text("")
    monkeypatch.setattr(B.subprocess, "run", lambda *a, **k: type("Done", (), {"returncode": 0, "stderr": ""}))
    for name in ("check_loads_in_flight", "check_prologue_in_flight", "check_m0_free"):
        monkeypatch.setattr(B, name, lambda *a: 1)
    B._check("ffn.hip", 2)
    for part in B.TALL:
        with pytest.raises(RuntimeError, match="in assembly found"):
            B._check("ffn.hip", part)
