"""Host-side checks of the C ABI that need no GPU: the library loads, exports every declared symbol,
sizes workspaces, and rejects bad arguments before anything is launched."""
import ctypes
import os
import re

import pytest

from paper_1811_12019_amd import binding as kb
from paper_1811_12019_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "kfac.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(kfac_[a-z_A-Z]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = kb.load_library()
    names = declared_symbols()
    assert set(names) == set(kb.EXPORTED_SYMBOLS)
    for n in names:
        assert getattr(lib, n) is not None


def test_status_strings():
    assert kb.status_string(0) == "ok"
    assert "argument" in kb.status_string(kb.KFAC_ERR_INVALID_ARG)
    assert "workspace" in kb.status_string(kb.KFAC_ERR_WORKSPACE)


def test_struct_sizes_match_header():
    assert ctypes.sizeof(kb.kfac_layer_desc) == 13 * 4
    assert ctypes.sizeof(kb.kfac_inverse_item) == 4 * 8 + 8 + 8 + 8
    assert ctypes.sizeof(kb.kfac_precond_item) == 5 * 8 + 8 + 2 * 8
    assert ctypes.sizeof(kb.kfac_factor_item) == 56 + 4 * 8 + 8 + 16


def test_workspace_sizes():
    d = kb.make_desc(synth.config1(), kb.KFAC_NHWC, kb.KFAC_BF16, kb.KFAC_ORDER_KH_KW_C)
    for op in (kb.KFAC_OP_FACTOR_A, kb.KFAC_OP_FACTOR_G):
        assert kb.kfac_factor_workspace_bytes(op, d) % 256 == 0
    assert kb.kfac_factor_workspace_bytes(7, d) == 0
    bad = kb.make_desc(synth.config1(), kb.KFAC_NHWC, kb.KFAC_BF16, kb.KFAC_ORDER_KH_KW_C)
    bad.stride = 0
    assert kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_A, bad) == 0
    assert kb.kfac_inverse_workspace_bytes(0) == 0
    assert kb.kfac_inverse_workspace_bytes(64) > 0
    assert kb.kfac_inverse_workspace_bytes(4609) >= (2 * 4609 * 128 + 128 * 128) * 4
    assert kb.kfac_precondition_workspace_bytes(512, 4609) >= 512 * 4609 * 4
    assert kb.kfac_precondition_workspace_bytes(-1, 5) == 0


def test_bad_arguments_are_rejected_on_the_host():
    lib = kb.load_library()
    d = kb.make_desc(synth.config0(), kb.KFAC_NCHW, kb.KFAC_F32, kb.KFAC_ORDER_C_KH_KW)
    fake = ctypes.c_void_p(0x1000)     # never dereferenced: every call below must fail validation first
    assert lib.kfac_factor_A(ctypes.byref(d), None, 0.0, fake, None, 0, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_factor_A(None, fake, 0.0, fake, None, 0, None) == kb.KFAC_ERR_INVALID_ARG
    bad = kb.make_desc(synth.config0(), kb.KFAC_NCHW, kb.KFAC_F32, kb.KFAC_ORDER_C_KH_KW)
    bad.layout = 5
    assert lib.kfac_factor_G(ctypes.byref(bad), fake, 0.0, fake, None, 0, None) == kb.KFAC_ERR_INVALID_ARG
    bad = kb.make_desc(synth.config0(), kb.KFAC_NCHW, kb.KFAC_F32, kb.KFAC_ORDER_C_KH_KW)
    bad.kh = 30                        # kernel larger than the padded image
    assert lib.kfac_factor_A(ctypes.byref(bad), fake, 0.0, fake, None, 0, None) == kb.KFAC_ERR_INVALID_ARG
    # a build that needs scratch but gets none
    big = kb.make_desc(synth.config2(), kb.KFAC_NHWC, kb.KFAC_BF16, kb.KFAC_ORDER_KH_KW_C)
    assert kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_G, big) > 0
    assert lib.kfac_factor_G(ctypes.byref(big), fake, 0.0, fake, None, 0, None) == kb.KFAC_ERR_WORKSPACE
    assert lib.kfac_factor_G(ctypes.byref(big), fake, 0.0, fake, ctypes.c_void_p(0x1010), 1 << 40, None) == kb.KFAC_ERR_WORKSPACE

    fit = (kb.kfac_factor_item * 1)()
    fit[0] = kb.kfac_factor_item(big, 0x1000, 0x2000, None, 0, 0.0, kb.KFAC_OP_FACTOR_G, None, 0.0, 0)       # needs scratch, has none
    assert lib.kfac_factor_batched(fit, fake, 1, None) == kb.KFAC_ERR_WORKSPACE
    fit[0] = kb.kfac_factor_item(big, 0x1000, 0x2000, None, 0, 0.0, 9, None, 0.0, 0)                          # unknown op
    assert lib.kfac_factor_batched(fit, fake, 1, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_factor_batched(fit, None, 1, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_factor_batched(fit, fake, 0, None) == kb.KFAC_OK                    # nothing to do, no launch
    assert lib.kfac_factor_batched(fit, fake, -1, None) == kb.KFAC_ERR_INVALID_ARG

    assert lib.kfac_ema(None, fake, 4, 0.95, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_ema(fake, fake, 4, 0.95, None) == kb.KFAC_ERR_INVALID_ARG          # overlap
    assert lib.kfac_ema(fake, ctypes.c_void_p(0x9000), 4, 1.5, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_ema(fake, ctypes.c_void_p(0x9000), 0, 0.5, None) == kb.KFAC_ERR_INVALID_ARG
    items = (kb.kfac_ema_item * 2)(kb.kfac_ema_item(0x1000, 0x9000, 4), kb.kfac_ema_item(0x1000, 0x1000, 4))
    assert lib.kfac_ema_batched(items, 2, 0.95, None) == kb.KFAC_ERR_INVALID_ARG        # second item overlaps
    assert lib.kfac_ema_batched(None, 1, 0.95, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_ema_batched(items, 1, -0.1, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_ema_batched(items, 0, 0.95, None) == kb.KFAC_OK                     # nothing to do, no launch
    pk = (kb.kfac_pack_item * 1)(kb.kfac_pack_item(0x10000, 0x10010, 4))                 # packed inside full
    assert lib.kfac_pack_upper_batched(pk, 1, None) == kb.KFAC_ERR_INVALID_ARG
    pk[0] = kb.kfac_pack_item(0x10000, 0x90000, 0)
    assert lib.kfac_pack_upper_batched(pk, 1, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_pack_upper_batched(None, 1, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_pack_upper_batched(pk, 0, None) == kb.KFAC_OK
    ep = (kb.kfac_ema_packed_item * 1)(kb.kfac_ema_packed_item(0x10000, 0x90000, 4))
    assert lib.kfac_ema_packed_batched(ep, 1, 1.5, None) == kb.KFAC_ERR_INVALID_ARG
    ep[0] = kb.kfac_ema_packed_item(0x10000, None, 4)
    assert lib.kfac_ema_packed_batched(ep, 1, 0.95, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_ema_packed_batched(ep, 0, 0.95, None) == kb.KFAC_OK
    di = (kb.kfac_diff_item * 2)(kb.kfac_diff_item(0x10000, 0x90000, 100), kb.kfac_diff_item(0x10000, 0x90000, 91))
    need = lib.kfac_factor_diff_workspace_bytes(di, 2)
    assert need == 256 * -(-((2 + 2) * 16) // 256)                                      # 2 + 2 chunks of 8192, two doubles each
    assert lib.kfac_factor_diff_workspace_bytes(di, 0) == 0
    assert lib.kfac_factor_diff_batched(di, 2, fake, None, 0, None) == kb.KFAC_ERR_WORKSPACE
    assert lib.kfac_factor_diff_batched(di, 2, None, fake, 1 << 20, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_factor_diff_batched(di, 0, None, None, 0, None) == kb.KFAC_OK
    di[1] = kb.kfac_diff_item(0x10000, None, 91)
    assert lib.kfac_factor_diff_batched(di, 2, fake, fake, 1 << 20, None) == kb.KFAC_ERR_INVALID_ARG
    ui = (kb.kfac_update_item * 1)(kb.kfac_update_item(0x10000, 0x20000, 0x30000, 5000, 64))
    assert lib.kfac_weight_update_workspace_bytes(ui, 1) == 256                          # 2 chunks, one double each
    assert lib.kfac_weight_update_batched(ui, 1, 0.1, 0.9, 1e-9, None, 0, None) == kb.KFAC_ERR_WORKSPACE
    assert lib.kfac_weight_update_batched(ui, 1, 0.1, 0.9, -1.0, fake, 1 << 20, None) == kb.KFAC_ERR_INVALID_ARG
    ui[0] = kb.kfac_update_item(0x10000, 0x10010, 0x30000, 5000, 64)                     # w and w_prev overlap
    assert lib.kfac_weight_update_batched(ui, 1, 0.1, 0.9, 1e-9, fake, 1 << 20, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_weight_update_batched(ui, 0, 0.1, 0.9, 1e-9, None, 0, None) == kb.KFAC_OK
    assert lib.kfac_bn_sample_grads_workspace_bytes(2, 64, 552) == 2 * 2 * 128 * 4         # two chunks of 512 positions
    assert lib.kfac_bn_sample_grads(fake, fake, 2, 64, 552, kb.KFAC_BF16, fake, None, 0, None) == kb.KFAC_ERR_WORKSPACE
    assert lib.kfac_bn_sample_grads(None, fake, 2, 64, 552, kb.KFAC_BF16, fake, fake, 1 << 20, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_bn_sample_grads(fake, fake, 2, 64, 552, 7, fake, fake, 1 << 20, None) == kb.KFAC_ERR_INVALID_ARG
    bi = (kb.kfac_bn_item * 2)(kb.kfac_bn_item(0x1000, 0x1000, 0x1000, 2, 64, 552, kb.KFAC_BF16),
                               kb.kfac_bn_item(0x1000, 0x1000, 0x1000, 2, 2048, 49, kb.KFAC_BF16))
    assert lib.kfac_bn_sample_grads_batched_workspace_bytes(bi, 2) == 2048                  # the second layer is one chunk
    assert lib.kfac_bn_sample_grads_batched(bi, 2, None, 0, None) == kb.KFAC_ERR_WORKSPACE
    assert lib.kfac_bn_sample_grads_batched(bi, 0, None, 0, None) == kb.KFAC_OK
    bi[1].C = 0
    assert lib.kfac_bn_sample_grads_batched(bi, 2, fake, 1 << 20, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_bn_diag_precondition(fake, 2, 128, None, 0.1, None, fake, None) == kb.KFAC_ERR_INVALID_ARG   # out without grad
    assert lib.kfac_bn_diag_precondition(fake, 2, 128, fake, -0.1, fake, fake, None) == kb.KFAC_ERR_INVALID_ARG


    assert lib.kfac_damped_inverse(fake, 0, 0.1, ctypes.c_void_p(0x9000), None, None, 0, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_damped_inverse(fake, 8, 0.1, fake, None, None, 0, None) == kb.KFAC_ERR_INVALID_ARG   # in place
    assert lib.kfac_damped_inverse(fake, 300, 0.1, ctypes.c_void_p(0x90000), None, None, 0, None) == kb.KFAC_ERR_WORKSPACE

    items = (kb.kfac_inverse_item * 2)()
    items[0] = kb.kfac_inverse_item(0x1000, 0x90000, 0x200000, None, 64, 0.1, None)
    items[1] = kb.kfac_inverse_item(0x1000, 0x90000, 0x200000, None, 300, 0.1, None)       # not sorted largest-first
    assert lib.kfac_damped_inverse_batched(items, 2, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_damped_inverse_batched(items, 0, None) == kb.KFAC_OK                # nothing to do, no launch
    assert lib.kfac_damped_inverse_batched(items, -1, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_damped_inverse_batched(None, 1, None) == kb.KFAC_ERR_INVALID_ARG

    pit = (kb.kfac_precond_item * 1)()
    pit[0] = kb.kfac_precond_item(0x1000, 0x2000, 0x3000, 0x3000, 0x4000, 4, 5)      # out aliases gradW
    assert lib.kfac_precondition_batched(pit, fake, 1, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_precondition_batched(pit, None, 1, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_precondition_batched(pit, fake, 0, None) == kb.KFAC_OK              # nothing to do, no launch
    assert lib.kfac_precondition_batched(pit, fake, -1, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_precondition(fake, fake, fake, 4, 5, None, fake, 1 << 20, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_precondition(fake, fake, fake, 4, 5, ctypes.c_void_p(0x9000), None, 0, None) == kb.KFAC_ERR_WORKSPACE
    assert lib.kfac_precondition(fake, fake, fake, 4, 5, fake, ctypes.c_void_p(0x9000), 1 << 20, None) == kb.KFAC_ERR_INVALID_ARG


@pytest.mark.parametrize("batch,layout,dtype,most", [(32, kb.KFAC_NHWC, kb.KFAC_BF16, 3.0e9), (128, kb.KFAC_NHWC, kb.KFAC_BF16, 4.0e9),
                                                     (32, kb.KFAC_NCHW, kb.KFAC_BF16, 3.5e9)])
def test_factor_scratch_of_a_whole_network(batch, layout, dtype, most):
    """Every build's scratch covers the partial sums of the most row ranges its rows can be cut into, and no more."""
    total = 0
    for s in synth.resnet50_layers(batch):
        desc = kb.make_desc(s, layout, dtype, kb.KFAC_ORDER_KH_KW_C)
        total += sum(kb.kfac_factor_workspace_bytes(op, desc) for op in (kb.KFAC_OP_FACTOR_A, kb.KFAC_OP_FACTOR_G))
    assert 1.0e9 < total < most


@pytest.mark.parametrize("C,HW", [(8, 4097), (64, 552), (64, 12544), (256, 3136), (264, 513), (512, 784), (2048, 49)])
def test_bn_scratch_does_not_depend_on_the_dtype(C, HW):
    """An fp32 layer whose channels are whole vectors in every dtype needs no more scratch than a 16-bit one, so that the
    single-layer size, which is asked for by shape alone, is the 16-bit one."""
    lib = kb.load_library()
    size = {dt: lib.kfac_bn_sample_grads_batched_workspace_bytes((kb.kfac_bn_item * 1)(kb.kfac_bn_item(0x1000, 0x1000, 0x1000, 3, C, HW, dt)), 1)
            for dt in (kb.KFAC_F32, kb.KFAC_BF16, kb.KFAC_F16)}
    assert size[kb.KFAC_F32] <= size[kb.KFAC_BF16] == size[kb.KFAC_F16]
    assert lib.kfac_bn_sample_grads_workspace_bytes(3, C, HW) == size[kb.KFAC_BF16]


@pytest.mark.parametrize("missing", [(), ("_cuda_getDevice",), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice", "_cuda_getCurrentRawStream")])
def test_current_stream_with_and_without_torchs_private_functions(monkeypatch, missing):
    import types
    import torch
    private = types.SimpleNamespace(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda device: 1000 + device)
    for name in missing:
        delattr(private, name)
    monkeypatch.setattr(torch, "_C", private)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert kb._stream(None) == (77 if missing else 1003)
    assert kb._stream(5) == 5 and kb._stream(types.SimpleNamespace(cuda_stream=6)) == 6
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)          # (current_stream() initialises)
    assert kb._stream(None) == 77


def test_profiled_traffic_is_used_only_for_the_code_it_was_counted_on(monkeypatch):
    """bench.py's roofline takes a kernel's HBM bytes from the profile summary, which names the code it was counted on; the
    summaries name no kernel that the sources do not have."""
    import bench
    assert re.fullmatch("[0-9a-f]{16}", bench.kernel_code_digest())
    text = open(os.path.join(ROOT, "profiles", "hbm_traffic_resnet50_b32_step.md")).read()
    counted = re.search("Kernel code ([0-9a-f]{16})", text).group(1)
    monkeypatch.setattr(bench, "kernel_code_digest", lambda: counted)
    assert bench.measured_traffic("inv_update_kernel", 32)["bytes_per_launch"] > 0
    assert bench.measured_traffic("inv_update_kernel", 128) is None and bench.measured_traffic("no_such_kernel", 32) is None
    monkeypatch.setattr(bench, "kernel_code_digest", lambda: "0" * 16)
    assert bench.measured_traffic("inv_update_kernel", 32) is None
    csrc = os.path.join(ROOT, "paper_1811_12019_amd", "csrc")
    sources = "".join(open(os.path.join(csrc, f)).read() for f in os.listdir(csrc))
    for name in os.listdir(os.path.join(ROOT, "profiles")):
        for kernel in re.findall(r"^\| `(\w+_kernel)\b", open(os.path.join(ROOT, "profiles", name)).read(), flags=re.M):
            assert re.search(rf"\b{kernel}\(", sources), (name, kernel)


def test_product_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_1811_12019_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith(".py"):
                text = open(os.path.join(dirpath, f)).read()
                assert not re.search(r"^\s*(from|import)\s+oracle\b|import_module\(.oracle|kfac_oracle", text, flags=re.M), \
                    f"{f} reaches into the oracle"
    ora = open(os.path.join(ROOT, "oracle", "kfac_oracle.py")).read()
    assert "paper_1811_12019_amd" not in ora and "ctypes" not in ora


def test_schedule_host_functions_against_hand_worked_values():
    """The host functions of Sec. 4.2 (warm-up damping) and Sec. 5.4 (refresh intervals) against values worked by hand
    from the paper's formulas and its Table 3 (not against the oracle's text)."""
    # interval(e) = min(20, 5 floor(e / 5) + 1): 1 for epochs 0-4, 6 for 5-9, 11, 16, then 20 from epoch 20 on
    want = {0: 1, 4: 1, 5: 6, 9: 6, 10: 11, 14: 11, 15: 16, 19: 16, 20: 20, 21: 20, 44: 20}
    for e, v in want.items():
        assert kb.kfac_refresh_interval(e, kb.KFAC_REFRESH_GROWING) == v
    # second heuristic: every step before epoch 13, every 20th afterwards
    for e, v in {0: 1, 12: 1, 13: 20, 40: 20}.items():
        assert kb.kfac_refresh_interval(e, kb.KFAC_REFRESH_LATE) == v
    assert kb.kfac_refresh_interval(-1, 0) == -1 and kb.kfac_refresh_interval(3, 7) == -1
    # Table 3, BS 4,096: gamma0 = 2.5e-2 = 100 gamma_target, t_warmup = 313 -> alpha = 2 * 2 / 313
    alpha = kb.kfac_warmup_damping_alpha(2.5e-2, 2.5e-4, 313)
    assert alpha == pytest.approx(4.0 / 313.0, rel=1e-14)
    assert kb.kfac_warmup_damping_next(2.5e-2, 2.5e-4, alpha) == pytest.approx(0.025 - 0.02475 * 4.0 / 313.0, rel=1e-14)
    assert kb.kfac_warmup_damping_next(2.5e-4, 2.5e-4, alpha) == pytest.approx(2.5e-4, rel=1e-14)
    assert kb.kfac_warmup_damping_alpha(0.0, 1.0, 10) != kb.kfac_warmup_damping_alpha(0.0, 1.0, 10)     # NaN
    assert kb.kfac_bn_damping(2.5e-4, 16.0) == pytest.approx(4.0e-3)


def test_pi_damping_arguments():
    lib = kb.load_library()
    fake = ctypes.c_void_p(0x1000)
    items = (kb.kfac_pi_item * 1)(kb.kfac_pi_item(0x1000, 0x2000, 5, 0))          # dG = 0
    assert lib.kfac_pi_damping_batched(items, 1, 1e-3, fake, None) == kb.KFAC_ERR_INVALID_ARG
    items[0] = kb.kfac_pi_item(0x1000, 0x2000, 5, 3)
    assert lib.kfac_pi_damping_batched(items, 1, -1.0, fake, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_pi_damping_batched(items, 1, 1e-3, None, None) == kb.KFAC_ERR_INVALID_ARG
    assert lib.kfac_pi_damping_batched(items, 0, 1e-3, None, None) == kb.KFAC_OK
