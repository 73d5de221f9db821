#include "jz_stage_kernel.h"
namespace jz {
#define K(R,I,O,M,X,Y,MODE) template __global__ void stage_kernel<R,I,O,M,X,Y,MODE,true>(StageArgs,const int*);
K(double,double,double,false,20,16,0) K(double,double,double,false,20,16,1) K(double,double,double,false,20,16,2)
K(float,float,float,true,36,20,0) K(float,double,float,true,36,20,1) K(float,float,double,true,36,20,2)
}
