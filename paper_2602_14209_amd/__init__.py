"""MI355X-native hot path of MAGE ([MASK]-Guided Sparse Attention, arxiv 2602.14209).

``binding``   Python front end of the C-ABI HIP library (libmage.so)
``workloads`` seeded synthetic inputs
``build``     in-tree build of the library and of the binding's marshalling module
"""
__all__ = ["binding", "workloads", "build"]
