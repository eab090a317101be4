"""The native argument marshalling of the binding, on the CPU: what it takes for tensors, integers and lists, and what it refuses."""
import ctypes as ct

import numpy as np
import pytest

from paper_2011_10170_amd import binding as B


class Tensor:
    def data_ptr(self):
        return 1 << 63 | 4096


class Broken:
    def data_ptr(self):
        raise RuntimeError("no storage")


DESC = B.make_desc(1, 4, 4, 8, 8, 1, B.PC_BF16)
MASKS = [0x1B0, 0x0D8]


def refused(call):
    """The library is reached and refuses the null context."""
    with pytest.raises(B.PcError) as e:
        call()
    assert e.value.status == B.PC_ERR_INVALID_ARG


def test_arguments_reach_the_library():
    t = Tensor()
    refused(lambda: B.pc_conv_fwd(None, DESC, None, t, 64))
    refused(lambda: B.pc_conv_bwd_weight(None, DESC, 0, t, np.int64(64), t))
    refused(lambda: B.pc_act_pool_fwd(None, t, np.int32(1), 2.0, 2, 8, B.PC_BF16, 2, t, t))
    refused(lambda: B.pc_pattern_select(None, t, None, 8, 8, MASKS, 0, 4, 0, t, t))
    refused(lambda: B.pc_pattern_select_batch(None, [t, 64], None, [8, 8], (8, np.int64(8)), MASKS, 0, [4, 4], 0, [t, t], [t, t]))
    refused(lambda: B.pc_pack_batch(None, [t], [t], [t], MASKS, [64]))
    refused(lambda: B.pc_conv_bwd_weight_batch(None, [DESC, DESC], [64, 64], [t, t], [t, t], [t, t]))
    refused(lambda: B.pc_group_lasso_grad_batch(None, [t], [t], [t], [8], [8], MASKS, 1, 1e-4, [t], penalty=None))
    refused(lambda: B.pc_finalize_pick_batch(None, [t, t], [8], [8], 4, [t]))      # (one layer: what goes beyond is not read)


def test_what_is_no_argument():
    t = Tensor()
    with pytest.raises(RuntimeError, match="no storage"):
        B.pc_conv_fwd(None, DESC, None, Broken(), t)
    for bad in (object(), "x"):
        with pytest.raises((TypeError, ValueError)):
            B.pc_conv_fwd(None, DESC, None, bad, t)
    with pytest.raises(TypeError):
        B.pc_conv_fwd(None, None, None, t, t)
    with pytest.raises(TypeError):
        B.pc_conv_fwd(None, np.zeros(3, np.int32), None, t, t)
    with pytest.raises(TypeError):
        B.pc_update_values_batch(None, 5, [t])
    with pytest.raises(OverflowError):
        B.pc_conv_fwd(None, DESC, 1 << 70, t, t)


@pytest.mark.parametrize("call", [
    lambda t: B.pc_pattern_select_batch(None, [t, t], [t], [8, 8], [8, 8], MASKS, 0, [4, 4], 0, [t, t], [t, t]),
    lambda t: B.pc_pattern_select_batch(None, [t, t], [t, t], [8], [8, 8], MASKS, 0, [4, 4], 0, [t, t], [t, t]),
    lambda t: B.pc_pattern_select_batch(None, [t, t], [t, t], [8, 8], [8, 8], MASKS, 0, [4, 4, 4], 0, [t, t], [t, t]),
    lambda t: B.pc_pack_batch(None, [t], [t], [t], MASKS, [64, 64]),
    lambda t: B.pc_update_values_batch(None, [64, 64], [t]),
    lambda t: B.pc_conv_bwd_weight_batch(None, [DESC, DESC], [64, 64], [t, t], [t], [t, t]),
    lambda t: B.pc_finalize_count_batch(None, [t, t], [8, 8], [8], 4, [t, t]),
    lambda t: B.pc_finalize_pick_batch(None, [t], [8, 8], [8, 8], 4, [t, t]),
    lambda t: B.pc_dppg_accumulate_batch(None, [t, t], [t, t], [8, 8], [8, 8], t, [t]),
    lambda t: B.pc_group_lasso_grad_batch(None, [t], [t], [], [8], [8], MASKS, 1e-4, 1e-4, [t])])
def test_lists_of_different_lengths(call):
    with pytest.raises(ValueError):
        call(Tensor())


class Copy(ct.Structure):          # of the descriptor's size
    _fields_ = [("v", ct.c_int32 * 7)]


def every_handle():
    """Calls with the context's and the pack's place left open."""
    t = Tensor()
    return [lambda c, k: B.pc_conv_fwd(c, DESC, k, t, t), lambda c, k: B.pc_conv_fwd_relu(c, DESC, k, t, t), lambda c, k: B.pc_conv_bwd_data(c, DESC, k, t, t),
            lambda c, k: B.pc_conv_bwd_data_relu(c, DESC, k, t, t, t), lambda c, k: B.pc_conv_bwd_weight(c, DESC, k, t, t, t), lambda c, k: B.pc_scatter_dense(c, k, t, t),
            lambda c, k: B.pc_unpack_dense(c, k, t), lambda c, k: B.pc_update_values(c, k, t), lambda c, k: B.pc_pack(c, t, t, t, 8, 8, MASKS, B.PC_BF16, reuse=k)]


@pytest.mark.parametrize("i", range(9))
def test_handles_are_what_ctypes_takes(i):
    call = every_handle()[i]
    refused(lambda: call(None, ct.c_void_p(64)))
    refused(lambda: call(ct.c_void_p(None), 64))
    for bad in (Tensor(), 64.0, np.int64(64), np.zeros(4), object()):      # none of these is an address of the library's
        with pytest.raises((TypeError, ValueError, ct.ArgumentError)):
            call(None, bad)
        with pytest.raises((TypeError, ct.ArgumentError)):
            call(bad, 64)


def test_handles_in_lists():
    t = Tensor()
    refused(lambda: B.pc_pack_batch(None, [t], [t], [t], MASKS, [np.int64(64)]))
    refused(lambda: B.pc_update_values_batch(ct.c_void_p(None), [64.0], [t]))
    for bad in (t, None, np.zeros(4), object(), "pack"):
        with pytest.raises((TypeError, ValueError)):
            B.pc_pack_batch(None, [t], [t], [t], MASKS, [bad])
        with pytest.raises((TypeError, ValueError)):
            B.pc_update_values_batch(None, [bad], [t])
        with pytest.raises((TypeError, ValueError)):
            B.pc_conv_bwd_weight_batch(None, [DESC], [bad], [t], [t], [t])


def test_descriptors_are_of_their_type():
    t = Tensor()

    class Sub(B.pc_conv_desc):
        pass

    for call in (lambda d: B.pc_conv_fwd(None, d, 64, t, t), lambda d: B.pc_conv_fwd_relu(None, d, 64, t, t), lambda d: B.pc_conv_bwd_data(None, d, 64, t, t),
                 lambda d: B.pc_conv_bwd_data_relu(None, d, 64, t, t, t), lambda d: B.pc_conv_bwd_weight(None, d, 64, t, t, t),
                 lambda d: B.pc_conv_bwd_weight_batch(None, [d], [64], [t], [t], [t])):
        refused(lambda: call(Sub(1, 4, 4, 8, 8, 1, B.PC_BF16)))
        for bad in (Copy(), bytes(28), np.zeros(7, np.int32), None, 64):
            with pytest.raises(TypeError):
                call(bad)
    refused(lambda: B.pc_conv_bwd_weight_batch(None, [(1, 4, 4, 8, 8, 1, B.PC_BF16)], [64], [t], [t], [t]))      # (a ctypes array takes tuples)


def test_numbers_are_what_float_takes():
    t = Tensor()
    refused(lambda: B.pc_group_lasso_grad_batch(None, [t], [t], [t], [8], [8], MASKS, "1e-4", np.float32(1e-4), [t]))


def test_a_list_that_shrinks_while_it_is_read():
    items = []

    class Shrinks:
        def data_ptr(self):
            items.clear()
            return 64

    items += [Shrinks() for _ in range(1000)]
    with pytest.raises((ValueError, RuntimeError)):
        B.pc_update_values_batch(None, [64] * 1000, items)
