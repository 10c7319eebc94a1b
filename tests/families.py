"""Handles bound to one kernel family.

Teacher forcing on a default handle takes all steps of a call at once, whichever family generates; bound to a
family (WN_KERNEL) a handle forces step by step on that family's own kernel, so a test that means its logits
forces on such a handle."""


def bound(monkeypatch, variant, make):
    """make()'s handle, bound to the family that wn_kernel_variant calls `variant`."""
    with monkeypatch.context() as m:
        m.setenv("WN_KERNEL", "stream" if variant == "stream_l2" else variant)
        return make()
