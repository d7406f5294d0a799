/*
 * Between pycall.c, which knows only the interpreter, and tensor_reader.cpp, which knows one torch: how a tensor's
 * properties are read without the interpreter.  While overridden() returns 1, a torch-function mode is active, whose answers count:
 * none of the others is to be called.  They return 1 if they could say, else 0; then the caller asks the
 * tensor's methods, which also say what is wrong.  None raises, none keeps the tensor.
 */
#ifndef DT_TENSOR_READER_H
#define DT_TENSOR_READER_H
#include <Python.h>

#define DT_TENSOR_READER "paper_2601_12212_amd.tensor_reader" /* the capsule's name */

typedef struct {
    int (*overridden)(void);
    int (*data_ptr)(PyObject *t, void **out);
    int (*sizes)(PyObject *t, int n, int exact, long long *out); /* the first n, of at least (exactly, if `exact`) n */
    int (*stride)(PyObject *t, long dim, long long *out);
    int (*dtype)(PyObject *t, int *bf16);                        /* float32 or bfloat16, no other */
    int (*nbytes)(PyObject *t, size_t *out);
} dt_tensor_reader;
#endif
